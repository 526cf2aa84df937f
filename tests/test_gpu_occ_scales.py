"""The digit scale of the integer occupied block over the range of Jastrow
sizes: coincident points (every g = g') must contribute exactly nothing
whatever the size of u', and a |u'| too small for the integer scale gets the
FP64 block.  Reference and tolerance as for the block itself: the FP64 block
of the same call, 2^-30 of its largest entry."""
import numpy as np
import pytest

from paper_2304_07006_amd import inputs

pytestmark = pytest.mark.gpu

TOL_REL = 2.0**-30


@pytest.fixture(scope="module")
def torch_cuda():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no HIP device")
    return torch


def _K_occ(p, kflags=0):
    import torch
    from paper_2304_07006_amd import xtc
    dp = xtc.device_problem(p.xyz, p.w, p.phi, p.occ)
    ps = xtc.Pass(dp, xtc.XTC_BF16X3, p.Ng)
    xtc.xtc_prepare(dp, ps.prec, ps.chunk, ps.ws)
    K = ps.K_view(0, p.Ng)
    xtc.xtc_build_K(dp, xtc.make_jastrow(p.jastrow), 0, p.Ng, ps.prec | kflags, K, ps.ws)
    torch.cuda.synchronize()
    N, occ = p.N, sorted(int(k) for k in p.occ)
    cols = [a * N - a * (a - 1) // 2 + (b - a) for i, a in enumerate(occ) for b in occ[i:]]
    return K.cpu().numpy()[:, :, cols]


# 1e-150, 1e-160, 1e-240: integer block (at 1e-158 and below 1/r of the r^2
# floor times the reciprocal scale is past the FP64 range); 1e-300, 1e-305: the
# FP64 block; 1e+280: the large end
@pytest.mark.parametrize("size,fp64", [(1e-150, False), (1e-160, False), (1e-240, False), (1e-300, True),
                                       (1e-305, True), (1e280, False)])
def test_coincident_points_at_every_size_of_u(torch_cuda, size, fp64):
    from paper_2304_07006_amd import xtc
    print(f"case: power Jastrow of size {size:g}, integer occupied block", flush=True)
    p = inputs.make_problem(24, 6, 1200, 6, "chain", "power16", seed=65)
    p.jastrow = inputs.Jastrow("power", coef=tuple(size * c for c in p.jastrow.coef))
    Ki, Kf = _K_occ(p), _K_occ(p, xtc.XTC_K_OCC_FP64)
    assert np.all(np.isfinite(Kf)) and np.abs(Kf).max() > 0
    if fp64:
        assert np.array_equal(Ki, Kf)
    assert np.abs(Ki - Kf).max() < TOL_REL * np.abs(Kf).max()
