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
