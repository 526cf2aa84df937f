"""Launch shapes chosen by size: every variant of a kernel whose tile, split or
segment count depends on the problem, at the sizes where it can go wrong
(one tile and less, tile edges, ragged remainders), against the FP64 oracle."""
import numpy as np
import pytest

from oracle import factorised
from paper_2304_07006_amd import inputs

pytestmark = pytest.mark.gpu

# FP64 outputs are O(1) sums of at most 4000 terms of at most 1e-2: 1e-11 covers
# every summation order (4000 terms x 1e-2 x 1.1e-16 = 5e-15 per entry of K, then
# products of two such sums)
TOL = 1e-11


@pytest.fixture(scope="module")
def torch_cuda():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no HIP device")
    return torch


# one orbital pair; one 64-tile and one more pair than it (N=11: 66); the 128 edge
# (N=15: 120, N=16: 136); grids of one row tile, one row more, ragged chunks
# (the sizes below are whole centres of four functions; one pair, N=11, N=15 and
# other N between them run in test_gpu_odd_sizes.py)
@pytest.mark.parametrize("N,nocc,Ng,chunk,centres", [
    (4, 1, 17, 17, 1), (8, 2, 64, 64, 2), (8, 2, 65, 33, 2), (8, 3, 1999, 1999, 2), (12, 3, 129, 97, 3),
    (16, 4, 1025, 1025, 4), (20, 5, 2047, 700, 5), (32, 6, 1500, 1500, 4), (40, 8, 4000, 4000, 5)])
def test_fp64_forward_at_split_and_tile_edges(torch_cuda, N, nocc, Ng, chunk, centres):
    from paper_2304_07006_amd import xtc
    print(f"case: FP64 forward N={N} nocc={nocc} Ng={Ng} chunk={chunk}", flush=True)
    p = inputs.make_problem(N, nocc, Ng, centres, "chain", "pade", seed=900 + N + Ng)
    V2o, h1o, E0o = factorised.closed_shell(p.xyz, p.w, p.phi, p.occ, p.jastrow)
    V2, h1, E0 = xtc.forward(p, prec="fp64", chunk_rows=chunk)
    scale = max(1.0, np.abs(V2o).max())
    assert np.abs(V2.cpu().numpy() - V2o).max() < TOL * scale
    assert np.abs(h1.cpu().numpy() - h1o).max() < TOL * max(1.0, np.abs(h1o).max())
    assert abs(float(E0.cpu()[0]) - E0o) < TOL * max(1.0, abs(E0o))
    again = xtc.forward(p, prec="fp64", chunk_rows=chunk)
    assert torch_cuda.equal(V2, again[0]) and torch_cuda.equal(h1, again[1]) and torch_cuda.equal(E0, again[2])


# matrix in LDS (N <= 140) and beyond, odd N (dummy partner), one function,
# one 64-row tile and one row more, fewer points than a wave's 64
@pytest.mark.parametrize("N,Ng", [(1, 40), (3, 50), (37, 1500), (64, 700), (65, 2100), (140, 3000), (141, 3000),
                                  (160, 4133)])
def test_lowdin_at_matrix_and_tile_edges(torch_cuda, N, Ng):
    from oracle import lowdin as ol
    from paper_2304_07006_amd import xtc
    print(f"case: lowdin N={N} Ng={Ng}", flush=True)
    nc = max(1, (N + 3) // 4)
    rng = np.random.default_rng(70 + N)
    centres = inputs.chain_centres(nc, rng)
    xyz, w = inputs.sample_grid(centres, Ng, rng)
    chi = np.ascontiguousarray(inputs.basis_values(xyz, centres, 4, rng)[0][:N])
    phi_o, _, lam_o = ol.lowdin(chi, w)
    phi, lam = xtc.lowdin(chi, w)
    # S is formed to a few ulp of its largest entry, S^{-1/2} to cond(S) times that
    tol = 50 * np.finfo(float).eps * lam_o.max() / lam_o.min() * max(1, N / 8)
    assert np.abs(np.sort(lam.cpu().numpy()) - np.sort(lam_o)).max() < 50 * N * np.finfo(float).eps * lam_o.max()
    assert np.abs(phi.cpu().numpy() - phi_o).max() < tol * max(1.0, np.abs(phi_o).max())
    again = xtc.lowdin(chi, w)
    assert torch_cuda.equal(phi, again[0]) and torch_cuda.equal(lam, again[1])


# the reduced forms' small K-build tiles and small transposed products, and the
# sizes around them (one row tile, one column tile, one k-step; many tiles)
@pytest.mark.parametrize("prec", ["fp32", "bf16x3", "bf16x6"])
@pytest.mark.parametrize("N,nocc,Ng,chunk,centres", [
    (4, 1, 33, 33, 1), (8, 2, 2000, 2000, 2), (20, 5, 1501, 700, 5), (28, 6, 1024, 1024, 7), (40, 6, 3000, 1500, 5)])
def test_reduced_forward_at_tile_edges(torch_cuda, prec, N, nocc, Ng, chunk, centres):
    from paper_2304_07006_amd import xtc
    print(f"case: {prec} forward N={N} nocc={nocc} Ng={Ng} chunk={chunk}", flush=True)
    p = inputs.make_problem(N, nocc, Ng, centres, "chain", "power16", seed=300 + N + Ng)
    V2o, h1o, E0o = factorised.closed_shell(p.xyz, p.w, p.phi, p.occ, p.jastrow)
    V2, h1, E0 = xtc.forward(p, prec=prec, chunk_rows=chunk)
    # 1e-6 is the bar of the forms on outputs of order one; it scales with the output
    assert np.abs(V2.cpu().numpy() - V2o).max() < 1e-6 * max(1.0, np.abs(V2o).max())
    assert np.abs(h1.cpu().numpy() - h1o).max() < 1e-6 * max(1.0, np.abs(h1o).max())
    assert abs(float(E0.cpu()[0]) - E0o) < 1e-8 * max(1.0, abs(E0o))
    again = xtc.forward(p, prec=prec, chunk_rows=chunk)
    assert torch_cuda.equal(V2, again[0]) and torch_cuda.equal(h1, again[1]) and torch_cuda.equal(E0, again[2])
