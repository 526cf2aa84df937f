"""How many bytes of workspace the library needs.  The table holds the byte
counts of the library's first release of each layout, which callers with a
fixed scratch budget have sized for: a chunk of that many rows must still be
accepted with them.  What xtc_workspace_size adds to them are segment partials
that only make launches faster, and only where a launch plan asks for them.

Calls pass fake device pointers: accepted ones end in a launch failure, so the
tests run only where no device exists (the kernel driver's /dev/kfd absent)."""
import ctypes
import os

import numpy as np
import pytest

from paper_2304_07006_amd import xtc

nodevice = pytest.mark.skipif(os.path.exists("/dev/kfd"), reason="a HIP device is present: fake pointers would be used")

BWD, TC2 = xtc.XTC_WITH_BACKWARD, xtc.XTC_WITH_TC2
# N, nocc, Ng, chunk rows, prec, open shell, bytes
TABLE = [
    (1, 1, 40, 40, xtc.XTC_FP64, False, 605184),
    (8, 2, 2000, 2000, xtc.XTC_FP64, False, 10882048),
    (8, 2, 2000, 700, xtc.XTC_FP64, False, 5424128),
    (24, 6, 1501, 1501, xtc.XTC_FP64, False, 25908224),
    (24, 6, 1501, 1501, xtc.XTC_FP64, True, 45668352),
    (24, 6, 1501, 500, xtc.XTC_FP64 | BWD, False, 31192832),
    (8, 2, 600, 256, xtc.XTC_FP64 | TC2, False, 3384320),
    (8, 2, 2000, 2000, xtc.XTC_BF16X3, False, 94178816),
    (21, 5, 1501, 700, xtc.XTC_BF16X3, False, 47010304),
    (21, 5, 1501, 700, xtc.XTC_FP32, True, 57674240),
    (21, 5, 1501, 700, xtc.XTC_BF16X6, False, 54350336),
    (12, 3, 900, 256, xtc.XTC_BF16X3 | BWD, False, 26670592),
    (12, 3, 900, 256, xtc.XTC_BF16X3 | TC2, False, 24532480),
    (24, 17, 1500, 800, xtc.XTC_BF16X3, False, 147040000),
    (64, 8, 20000, 20000, xtc.XTC_FP64, False, 1791798272),
    (128, 16, 150000, 7500, xtc.XTC_BF16X3, False, 38388347904),
]
# Loewdin: N, Ng, bytes
LOWDIN = [
    (1, 40, 34048), (3, 50, 34048), (8, 2000, 34816), (37, 1500, 66304),
    (64, 700, 131584), (65, 2100, 233728), (128, 9000, 786944), (140, 3000, 766208),
    (141, 3000, 773120), (256, 5000, 2621952),
]


@pytest.fixture(scope="module")
def lib():
    if not os.path.exists(xtc.LIB_PATH):
        pytest.skip("libxtc.so not built")
    return xtc.load()


def _problem(N, nocc, Ng, open_shell):
    occ, beta = np.arange(nocc, dtype=np.int32), np.ones(nocc)
    f = ctypes.c_void_p(0x10000)
    c = xtc.XtcProblem(N, Ng, nocc, 0, f, f, f, occ.ctypes.data_as(ctypes.POINTER(ctypes.c_int32)))
    if open_shell:
        c.occ_n_beta = beta.ctypes.data_as(ctypes.POINTER(ctypes.c_double))
    c.keep = (occ, beta)
    return c


@nodevice
@pytest.mark.parametrize("N,nocc,Ng,chunk,prec,open_shell,nbytes", TABLE)
def test_the_first_byte_counts_are_accepted(lib, N, nocc, Ng, chunk, prec, open_shell, nbytes):
    c = _problem(N, nocc, Ng, open_shell)
    ws, f, j = ctypes.c_void_p(0x100000), ctypes.c_void_p(0x20000), xtc.power_jastrow([0.5])
    assert lib.xtc_prepare(ctypes.byref(c), prec, chunk, ws, nbytes, None) == xtc.XTC_E_HIP
    assert lib.xtc_build_K(ctypes.byref(c), ctypes.byref(j), Ng - chunk, Ng, prec, f, ws, nbytes, None) == xtc.XTC_E_HIP
    assert lib.xtc_contract_2body(ctypes.byref(c), f, 0, chunk, prec, xtc.XTC_FINALIZE, f, ws, nbytes,
                                  None) == xtc.XTC_E_HIP
    assert lib.xtc_contract_1body_0body(ctypes.byref(c), f, 0, chunk, prec, 0, None, None, ws, nbytes,
                                        None) == xtc.XTC_E_HIP
    # and what is clearly too small is still refused
    assert lib.xtc_prepare(ctypes.byref(c), prec, chunk, ws, nbytes // 4, None) == xtc.XTC_E_WORKSPACE


@pytest.mark.parametrize("N,nocc,Ng,chunk,prec,open_shell,nbytes", TABLE)
def test_partials_are_reserved_where_a_plan_uses_them(lib, N, nocc, Ng, chunk, prec, open_shell, nbytes):
    """The reduced forms and the adjoint find room for their partials in the
    chunk's own buffers; FP64 passes add at most 192 MiB for the K build and 192
    for the products, and nothing where the matrix fills the chip by itself."""
    c = _problem(N, nocc, Ng, open_shell)
    n = lib.xtc_workspace_size(ctypes.byref(c), prec, chunk)
    assert 0 < n <= nbytes + ((384 << 20) if prec in (xtc.XTC_FP64, xtc.XTC_FP64 | TC2) else 0)
    big = _problem(128, 16, 150000, False)
    assert lib.xtc_workspace_size(ctypes.byref(big), xtc.XTC_FP64, 7500) <= 12584135680


@nodevice
@pytest.mark.parametrize("N,Ng,nbytes", LOWDIN)
def test_the_first_lowdin_byte_counts_are_accepted(lib, N, Ng, nbytes):
    f, ws = ctypes.c_void_p(0x10000), ctypes.c_void_p(0x100000)
    assert lib.xtc_lowdin(N, Ng, f, f, f, None, ws, nbytes, None) == xtc.XTC_E_HIP
    assert lib.xtc_lowdin(N, Ng, f, f, f, None, ws, nbytes - 1, None) == xtc.XTC_E_WORKSPACE
    assert nbytes <= lib.xtc_lowdin_workspace_size(N, Ng) <= nbytes + (32 << 20)
