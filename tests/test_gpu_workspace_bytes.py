"""Passes in the smallest workspace that holds their chunk (the byte counts of
test_workspace_bytes): the launch plans then have few or no segment partials,
and the outputs agree with those of a workspace of xtc_workspace_size bytes to
the rounding of the FP64 sums.  The workspace is filled with NaN first and a
guard behind it has to stay as it was."""
import ctypes

import numpy as np
import pytest

from paper_2304_07006_amd import inputs
from test_workspace_bytes import BWD, LOWDIN, TABLE, TC2

pytestmark = pytest.mark.gpu

# sums of at most 2000 terms in another order: 2000 x 1.1e-16 of the largest
# magnitude, with a factor 5 for the products of two such sums
TOL = 1e-12
GUARD = 1 << 16


@pytest.fixture(scope="module")
def torch_cuda():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no HIP device")
    return torch


def _problem(N, nocc, Ng, open_shell):
    """The first N functions of a problem of whole centres, orthonormalised."""
    nc = max(1, (N + 3) // 4)
    p = inputs.make_problem(4 * nc, min(4 * nc, nocc), Ng, nc, "chain", "power16", seed=500 + N + Ng)
    chi = p.chi[:N]
    lam, U = np.linalg.eigh((chi * p.w) @ chi.T)
    p.phi = np.ascontiguousarray((U * lam ** -0.5) @ U.T @ chi)
    occ = np.arange(nocc, dtype=np.int32)
    beta = np.where(occ < nocc - 1, 1.0, 0.0) if open_shell else None
    return p, occ, (np.ones(nocc) if open_shell else None), beta


def _guarded(torch, nbytes):
    buf = torch.empty(nbytes + GUARD, dtype=torch.uint8, device="cuda")
    buf.fill_(0xFF)
    return buf, buf[:nbytes]


def _close(a, b):
    a, b = a.cpu().numpy(), b.cpu().numpy()
    assert np.all(np.isfinite(b))
    assert np.abs(a - b).max() <= TOL * max(1.0, np.abs(a).max())


@pytest.mark.parametrize("N,nocc,Ng,chunk,prec,open_shell,nbytes", [t for t in TABLE if t[0] < 64])
def test_smallest_workspace_gives_the_same_outputs(torch_cuda, N, nocc, Ng, chunk, prec, open_shell, nbytes):
    from paper_2304_07006_amd import xtc
    torch = torch_cuda
    print(f"case: N={N} nocc={nocc} Ng={Ng} chunk={chunk} prec={prec:#x} open={open_shell} in {nbytes} bytes", flush=True)
    p, occ, occ_n, occ_b = _problem(N, nocc, Ng, open_shell)
    dp = xtc.device_problem(p.xyz, p.w, p.phi, occ, occ_n=occ_n, occ_n_beta=occ_b)
    jas = xtc.make_jastrow(p.jastrow)
    buf, ws = _guarded(torch, nbytes)
    ref = xtc.Pass(dp, prec, chunk)
    got = xtc.Pass(dp, prec, chunk)
    got.ws = ws
    for a, b in zip(ref.run(jas), got.run(jas)):
        _close(a, b)
    if prec & BWD:
        G = torch.as_tensor(inputs.loss_weights(N, 7)[1]).cuda()
        g = torch.empty(16, dtype=torch.float64, device="cuda")
        coef = list(p.jastrow.coef)
        xtc.xtc_prepare(dp, prec, chunk, ws)
        xtc.xtc_backward(dp, xtc.power_jastrow(coef), prec, G, None, 1.0, g, ws)
        _close(xtc.backward(dp, coef, G, None, 1.0, prec & ~BWD, chunk), g)
    if prec & TC2:
        rng = np.random.default_rng(3)
        dphi = torch.as_tensor(rng.standard_normal((3, N, Ng))).cuda()
        outs = []
        for w in (ref.ws, ws):
            K2 = torch.empty((N,) * 4, dtype=torch.float64, device="cuda")
            xtc.xtc_prepare(dp, prec, chunk, w)
            for g0 in range(0, Ng, chunk):
                g1 = min(Ng, g0 + chunk)
                K = got.K_view(g0, g1)
                xtc.xtc_build_K(dp, jas, g0, g1, prec | xtc.XTC_K_REDUCED_OCC, K, w)
                st = xtc.load().xtc_tc_2body(
                    ctypes.byref(dp.c), ctypes.byref(jas), ctypes.c_void_p(dphi.data_ptr()),
                    ctypes.c_void_p(K.data_ptr()), g0, g1, prec, xtc.XTC_FINALIZE if g1 == Ng else 0,
                    ctypes.c_void_p(K2.data_ptr()), ctypes.c_void_p(w.data_ptr()), w.numel(),
                    ctypes.c_void_p(torch.cuda.current_stream().cuda_stream))
                assert st == 0, xtc.last_error()
            outs.append(K2)
        _close(*outs)
    torch.cuda.synchronize()
    assert bool((buf[nbytes:] == 0xFF).all())


@pytest.mark.parametrize("N,Ng,nbytes", LOWDIN)
def test_smallest_lowdin_workspace(torch_cuda, N, Ng, nbytes):
    """Rotations of a few sweeps at a time (one for N=64 and 65: a pass per
    sweep): against the oracle with the tolerance of the solver's other tests."""
    from oracle import lowdin as ol
    from paper_2304_07006_amd import xtc
    torch = torch_cuda
    print(f"case: lowdin N={N} Ng={Ng} in {nbytes} bytes", flush=True)
    rng = np.random.default_rng(70 + N)
    centres = inputs.chain_centres(max(1, (N + 3) // 4), rng)
    xyz, w = inputs.sample_grid(centres, Ng, rng)
    chi = np.ascontiguousarray(inputs.basis_values(xyz, centres, 4, rng)[0][:N])
    phi_o, _, lam_o = ol.lowdin(chi, w)
    buf, ws = _guarded(torch, nbytes)
    chi_t, w_t = torch.as_tensor(chi).cuda(), torch.as_tensor(w).cuda()
    phi, lam = torch.empty_like(chi_t), torch.empty(N, dtype=torch.float64, device="cuda")
    xtc.xtc_lowdin(N, Ng, chi_t, w_t, phi, lam, ws)
    eps = np.finfo(float).eps
    tol = 50 * eps * lam_o.max() / lam_o.min() * max(1, N / 8)
    assert np.abs(np.sort(lam.cpu().numpy()) - np.sort(lam_o)).max() < 50 * N * eps * lam_o.max()
    assert np.abs(phi.cpu().numpy() - phi_o).max() < tol * max(1.0, np.abs(phi_o).max())
    assert bool((buf[nbytes:] == 0xFF).all())


@pytest.mark.parametrize("prec", ["fp64", "fp32", "bf16x3"])
@pytest.mark.parametrize("N,nocc,Ng,chunk", [(8, 2, 2000, 512), (24, 6, 3000, 800), (40, 17, 2600, 700)])
def test_next_K_build_beside_the_contraction(torch_cuda, N, nocc, Ng, chunk, prec):
    """K of chunk c + 1 built on a second stream while chunk c is contracted, on
    one workspace and two K buffers (ragged last chunk): the K build's partials
    have a part of the workspace of their own, so the outputs are those of the
    pass on one stream, bit for bit."""
    from paper_2304_07006_amd import xtc
    torch = torch_cuda
    print(f"case: K build beside the contraction N={N} Ng={Ng} chunk={chunk} {prec}", flush=True)
    p, occ, _, _ = _problem(N, nocc, Ng, False)
    dp = xtc.device_problem(p.xyz, p.w, p.phi, occ)
    jas = xtc.make_jastrow(p.jastrow)
    ref = [t.clone() for t in xtc.Pass(dp, xtc.PRECISIONS[prec], chunk).run(jas)]
    ps = xtc.Pass(dp, xtc.PRECISIONS[prec], chunk)
    K2 = torch.empty_like(ps.K)
    for _ in range(3):
        build, contract = torch.cuda.Stream(), torch.cuda.Stream()
        torch.cuda.synchronize()
        xtc.xtc_prepare(dp, ps.prec, ps.chunk, ps.ws, build)
        ch = ps.chunks()
        free = [None, None]
        for i, (g0, g1) in enumerate(ch):
            n = 3 * (g1 - g0) * ps.ldP
            K = (ps.K, K2)[i % 2].view(-1)[:n].view(3, g1 - g0, ps.ldP)
            if free[i % 2] is not None:
                build.wait_event(free[i % 2])
            xtc.xtc_build_K(dp, jas, g0, g1, ps.prec, K, ps.ws, build)
            contract.wait_event(build.record_event())
            flags = (xtc.XTC_RESET if i == 0 else 0) | (xtc.XTC_FINALIZE if i == len(ch) - 1 else 0)
            xtc.xtc_contract_2body(dp, K, g0, g1, ps.prec, flags, ps.V2, ps.ws, contract)
            xtc.xtc_contract_1body_0body(dp, K, g0, g1, ps.prec, flags, ps.h1, ps.E0, ps.ws, contract)
            free[i % 2] = contract.record_event()
        torch.cuda.synchronize()
        for a, b in zip(ref, (ps.V2, ps.h1, ps.E0)):
            assert torch.equal(a, b)
