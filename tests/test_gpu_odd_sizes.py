"""Orbital counts that are not multiples of 4 (every remainder of the kernels'
2 x 2, 16- and 32-wide blocks, odd numbers of orbital pairs), and every shape of
the FP64 K build, against the FP64 oracles; and the reduced K build's tile
variants against each other.

Problems take the first N functions of whole centres, orthonormalised."""
import ctypes
import functools

import numpy as np
import pytest

from paper_2304_07006_amd import inputs, xtc

gpu = pytest.mark.gpu
FORMS = ["fp64", "fp32", "bf16x3", "bf16x6"]
# N, nocc, Ng, chunk: 3 pairs; 6; 66 (one 64-tile and two more); 120 (the 128
# edge); 231; 561 (above 512); ragged chunks of odd length
SIZES = [(2, 1, 300, 130), (3, 2, 500, 500), (11, 3, 700, 299), (15, 4, 641, 641), (21, 5, 900, 451), (33, 7, 1100, 555)]
GRADIENT_SIZES = SIZES[:-1] + [(33, 7, 450, 231)]        # (the oracle's gradient is 32 forward passes)
# FP64 outputs are sums of at most 1100 terms of at most 1e-2, squared at most
TOL = 1e-11


@pytest.fixture(scope="module")
def torch_cuda():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no HIP device")
    return torch


@functools.lru_cache(maxsize=None)
def _problem(N, nocc, Ng, open_shell=False):
    nc = (N + 3) // 4
    p = inputs.make_problem(4 * nc, 1, Ng, nc, "chain", "power16", seed=700 + N)
    chi = p.chi[:N]
    X = inputs.lowdin_matrix(chi, p.w)
    dphi = np.einsum("ij,xjg->xig", X, inputs.basis_gradients(p.xyz, p.centres, p.meta["shells"])[:, :N])
    q = inputs.Problem(p.xyz, p.w, chi, np.ascontiguousarray(X @ chi), np.arange(nocc, dtype=np.int32), p.centres,
                       p.jastrow)
    if open_shell:
        q.occ_n, q.occ_n_beta = np.ones(nocc), np.where(np.arange(nocc) < nocc // 2, 1.0, 0.0)
    return q, np.ascontiguousarray(dphi)


def _gammas(p):
    out = []
    for n in (p.occ_n, p.occ_n_beta):
        g = np.zeros((p.N, p.N))
        g[p.occ, p.occ] = n
        out.append(g)
    return out


@functools.lru_cache(maxsize=None)
def _forward_oracle(N, nocc, Ng, open_shell):
    from oracle import factorised as fb
    p, _ = _problem(N, nocc, Ng, open_shell)
    if not open_shell:
        return fb.closed_shell(p.xyz, p.w, p.phi, p.occ, p.jastrow)
    V2, h1, E0 = fb.open_shell(p.xyz, p.w, p.phi, *_gammas(p), p.jastrow)
    return np.stack([V2[0][0], V2[0][1], V2[1][1]]), np.stack(h1), E0


@gpu
@pytest.mark.parametrize("prec", FORMS)
@pytest.mark.parametrize("open_shell", [False, True], ids=["closed", "open"])
@pytest.mark.parametrize("N,nocc,Ng,chunk", SIZES)
def test_forward(torch_cuda, N, nocc, Ng, chunk, open_shell, prec):
    print(f"case: forward N={N} nocc={nocc} Ng={Ng} chunk={chunk} open={open_shell} {prec}", flush=True)
    V2o, h1o, E0o = _forward_oracle(N, nocc, Ng, open_shell)
    V2, h1, E0 = xtc.forward(_problem(N, nocc, Ng, open_shell)[0], prec=prec, chunk_rows=chunk)
    tol = (TOL, TOL, TOL) if prec == "fp64" else (1e-6, 1e-6, 1e-8)
    assert np.abs(V2.cpu().numpy() - V2o).max() < tol[0] * max(1.0, np.abs(V2o).max())
    assert np.abs(h1.cpu().numpy() - h1o).max() < tol[1] * max(1.0, np.abs(h1o).max())
    assert abs(float(E0.cpu()[0]) - E0o) < tol[2] * max(1.0, abs(E0o))


@functools.lru_cache(maxsize=None)
def _gradient_oracle(N, nocc, Ng, open_shell):
    from oracle import gradient as og
    p, _ = _problem(N, nocc, Ng, open_shell)
    coef = np.array(p.jastrow.coef)
    w = [inputs.loss_weights(N, 40 + i) for i in range(3)]
    if not open_shell:
        return og.exact_gradient(p.xyz, p.w, p.phi, p.occ, coef, *w[0]), w[0][0], w[0][1]
    D, G = (w[0][0], w[1][0]), tuple(x[1] for x in w)
    return og.exact_gradient_open(p.xyz, p.w, p.phi, *_gammas(p), coef, D, G), np.stack(D), np.stack(G)


@gpu
@pytest.mark.parametrize("prec", FORMS)
@pytest.mark.parametrize("open_shell", [False, True], ids=["closed", "open"])
@pytest.mark.parametrize("N,nocc,Ng,chunk", GRADIENT_SIZES)
def test_gradient(torch_cuda, N, nocc, Ng, chunk, open_shell, prec):
    print(f"case: gradient N={N} nocc={nocc} Ng={Ng} chunk={chunk} open={open_shell} {prec}", flush=True)
    go, D, G = _gradient_oracle(N, nocc, Ng, open_shell)
    p, _ = _problem(N, nocc, Ng, open_shell)
    dp = xtc.device_problem(p.xyz, p.w, p.phi, p.occ, occ_n=p.occ_n, occ_n_beta=p.occ_n_beta)
    t = lambda a: torch_cuda.as_tensor(np.ascontiguousarray(a)).cuda()
    g = xtc.backward(dp, list(p.jastrow.coef), t(G), t(D), 1.0, prec, chunk).cpu().numpy()
    # the split forms leave out up to 2^-16 of a product in each of two
    # contractions; a factor 4 for what cancels in their sums
    scale = np.abs(go).max()
    assert np.abs(g - go).max() < (1e-10 * max(1.0, scale) if prec == "fp64" else 2.0**-13 * scale)


@functools.lru_cache(maxsize=None)
def _tc_oracle(N, nocc, Ng):
    from oracle import tc2
    p, dphi = _problem(N, nocc, Ng)
    return tc2.tc_two_body(p.xyz, p.w, p.phi, dphi, p.jastrow)


@gpu
@pytest.mark.parametrize("prec", FORMS)
@pytest.mark.parametrize("N,nocc,Ng,chunk", SIZES)
def test_tc_integrals(torch_cuda, N, nocc, Ng, chunk, prec):
    print(f"case: TC integrals N={N} Ng={Ng} chunk={chunk} {prec}", flush=True)
    p, dphi = _problem(N, nocc, Ng)
    Ko = _tc_oracle(N, nocc, Ng)
    K = xtc.tc_two_body(p, dphi, prec, chunk).cpu().numpy()
    tol = {"fp64": TOL, "bf16x3": 2.0**-16, "bf16x6": 2.0**-19, "fp32": 2.0**-16}[prec]
    assert np.abs(K - Ko).max() < tol * max(1.0, np.abs(Ko).max())


@gpu
@pytest.mark.parametrize("N,ncore", [(2, 0), (2, 1), (3, 1), (11, 2), (15, 14), (21, 4), (33, 5)])
def test_frozen_core(torch_cuda, N, ncore):
    from oracle import factorised as fb
    print(f"case: frozen core N={N} core={ncore}", flush=True)
    rng = np.random.default_rng(N)
    V2, h1, E0 = rng.standard_normal((N,) * 4), rng.standard_normal((N, N)), rng.standard_normal(1)
    core, act = list(range(ncore)), list(range(ncore, N))
    Vo, ho, Eo = fb.frozen_core(V2, h1, float(E0[0]), core, act)
    V, h, E = xtc.frozen_core(*(torch_cuda.as_tensor(a).cuda() for a in (V2, h1, E0)), core, act)
    assert np.array_equal(V.cpu().numpy(), V2[np.ix_(act, act, act, act)])
    # sums of at most 2 N terms of order one
    assert np.abs(h.cpu().numpy() - ho).max() < 1e-12 and abs(float(E.cpu()[0]) - Eo) < 1e-12 * max(1.0, ncore**2)


# ------------------------------------------------ shapes of the FP64 K build --
class Plan(ctypes.Structure):
    _fields_ = [(n, ctypes.c_int) for n in ("nb", "cw", "ncol", "nseg", "seg_len")]


def _plan(N, rows, Ng):
    """kf64_plan as xtc_build_K calls it with room for every partial."""
    import torch  # noqa: F401  (its HIP runtime before the library's, so that the process has one)
    fn = xtc.load()._ZN3xtc9kf64_planEiiiiim
    fn.restype, fn.argtypes = Plan, [ctypes.c_int] * 5 + [ctypes.c_size_t]
    P = N * (N + 1) // 2
    ld, ngp = -(-P // 128) * 128, -(-Ng // 128) * 128
    return fn(P, ld, rows, ngp, min(16, (192 << 20) // (16 * 3 * ld * 8) * 16 // rows), 1 << 60)


# (blocks per wave, waves per row group, split over g') -> N, rows, Ng; rows are
# ragged against the 16 and 32 of a workgroup
SHAPES = {
    (1, 2, True): (1, 250, 500), (1, 4, False): (1, 9, 40), (1, 4, True): (1, 15, 300),
    (2, 2, True): (28, 751, 1501), (2, 4, False): (224, 20, 40), (2, 4, True): (64, 50, 1000),
    (3, 2, False): (144, 200, 1000), (3, 2, True): (11, 1000, 1000), (3, 4, False): (128, 60, 300),
    (3, 4, True): (16, 1000, 1000), (4, 2, False): (224, 60, 300), (4, 2, True): (57, 151, 3001),
    (4, 4, False): (144, 150, 300), (4, 4, True): (71, 100, 2000), (5, 2, False): (114, 150, 300),
    (5, 2, True): (16, 601, 3001), (5, 4, False): (115, 150, 300), (5, 4, True): (93, 50, 1000),
    (6, 2, False): (101, 500, 500), (6, 2, True): (51, 751, 1501), (6, 4, False): (102, 500, 500),
    (6, 4, True): (72, 151, 3001), (7, 2, False): (101, 300, 300), (7, 2, True): (20, 1501, 1501),
    (7, 4, False): (102, 300, 300), (7, 4, True): (111, 50, 1000),
}


def test_plans_cover_every_shape():
    """The sizes below take the shapes they stand for, and every shape of the
    kernel is among them."""
    for (nb, cw, split), size in SHAPES.items():
        p = _plan(*size)
        assert (p.nb, p.cw, p.nseg > 1) == (nb, cw, split), (size, p.nb, p.cw, p.nseg)
    assert {k[:2] for k in SHAPES} == {(nb, cw) for nb in range(1, 8) for cw in (2, 4)}


@gpu
@pytest.mark.parametrize("kind", ["pade", "power16"])
@pytest.mark.parametrize("shape", list(SHAPES), ids=lambda s: f"{s[0]}x{s[1]}{'-split' if s[2] else ''}")
def test_fp64_K_build_of_every_shape(torch_cuda, shape, kind):
    from oracle.jastrow import grad1
    N, rows, Ng = SHAPES[shape]
    print(f"case: FP64 K build N={N} rows={rows} Ng={Ng} {kind}", flush=True)
    rng = np.random.default_rng(N + Ng)
    xyz, w, phi = rng.standard_normal((Ng, 3)), rng.uniform(0.5, 1.5, Ng) / Ng, rng.standard_normal((N, Ng))
    jas = inputs.make_jastrow(kind, 5)
    dp = xtc.device_problem(xyz, w, phi, [0])
    ps = xtc.Pass(dp, xtc.XTC_FP64, rows)
    g0 = Ng - rows
    xtc.xtc_prepare(dp, ps.prec, ps.chunk, ps.ws)
    K = ps.K_view(g0, Ng)
    K.fill_(float("nan"))
    xtc.xtc_build_K(dp, xtc.make_jastrow(jas), g0, Ng, ps.prec, K, ps.ws)
    i, j = np.triu_indices(N)
    ref = grad1(xyz[g0:], xyz, jas) @ (w * phi[i] * phi[j]).T                 # [3][rows][pairs]
    got = K.cpu().numpy()
    # sums of Ng products: Ng x 2^-53 of the largest sum of magnitudes, times a few for d
    assert np.abs(got[:, :, :len(i)] - ref).max() < 4 * Ng * 2.0**-53 * max(1.0, np.abs(ref).max())
    assert np.all(got[:, :, len(i):] == 0.0)


# ------------------------------------------------- tiles of the reduced K build --
@gpu
@pytest.mark.parametrize("kind", ["pade", "power16"])
@pytest.mark.parametrize("prec", FORMS[1:])
@pytest.mark.parametrize("N,Ng", [(13, 9001), (24, 9001), (41, 9001), (32, 17001)])
def test_reduced_K_tiles_agree_bitwise(torch_cuda, N, Ng, prec, kind):
    """The tile variant follows the rows of the call; the sums do not.  91, 300
    and 861 pairs: part of a 512-column tile, one and a part; 528 on a grid long
    enough that the last 16 get a launch of small tiles of their own."""
    print(f"case: {prec} {kind} K tiles N={N} Ng={Ng}", flush=True)
    rng = np.random.default_rng(4)
    xyz, w, phi = rng.standard_normal((Ng, 3)), rng.uniform(0.5, 1.5, Ng) / Ng, rng.standard_normal((N, Ng))
    jas = xtc.make_jastrow(inputs.make_jastrow(kind, 6))
    dp = xtc.device_problem(xyz, w, phi, [0])
    ps = xtc.Pass(dp, xtc.PRECISIONS[prec], Ng)
    xtc.xtc_prepare(dp, ps.prec, ps.chunk, ps.ws)
    whole = torch_cuda.empty((3, Ng, ps.ldP), dtype=torch_cuda.float64, device="cuda")
    xtc.xtc_build_K(dp, jas, 0, Ng, ps.prec | xtc.XTC_K_REDUCED_OCC, whole, ps.ws)
    for rows in (1, 33, 250, 500, 1000, 2000, 4001):
        K = ps.K_view(0, rows)
        xtc.xtc_build_K(dp, jas, 32, 32 + rows, ps.prec | xtc.XTC_K_REDUCED_OCC, K, ps.ws)
        assert torch_cuda.equal(K, whole[:, 32:32 + rows]), rows
