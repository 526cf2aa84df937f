"""The digits of four values taken together, as the integer occupied block makes
them (one FP64 shifter that carries the +8256, byte selections of the packed
integers, the fields recentred a register at a time), transcribed in numpy and
compared with the digits of one value at a time (test_digit_scheme), at the
ends of every digit's range and with mixed signs in one register."""
import numpy as np

from test_digit_scheme import _samples, digits

SHIFT = 6755399441055744.0 + 8256.0      # 1.5 * 2^52 + 64 (2^7 + 1)
M32 = np.uint32(0xFFFFFFFF)


def _perm(a, b, sel):
    """Byte k of the result: byte sel_k of (a: 0..3, b: 4..7), 0 for 0x0c."""
    out = np.zeros_like(a)
    for k in range(4):
        c = (sel >> (8 * k)) & 255
        if c == 0x0C:
            continue
        src = a if c < 4 else b
        out |= ((src >> np.uint32(8 * (c & 3))) & np.uint32(255)) << np.uint32(8 * k)
    return out


def _center(x):
    y = (x & np.uint32(0x7F7F7F7F)) ^ np.uint32(0x40404040)
    return y | ((y & np.uint32(0x40404040)) << np.uint32(1))


def _fields(u):
    w01, w23 = _perm(u[0], u[1], 0x05040100), _perm(u[2], u[3], 0x05040100)
    l = _center(_perm(w01, w23, 0x06040200))
    m = _center(_perm(w01 >> np.uint32(7), w23 >> np.uint32(7), 0x06040200))
    s = [(x.view(np.int32) >> 14).view(np.uint32) for x in u]
    return _perm(s[0], s[1], 0x0C0C0400) | _perm(s[2], s[3], 0x04000C0C), m, l


def packed_digits(v):
    """[6][4][n] digits of v [4][n]."""
    h = np.asarray(v, np.float64) * 2.0**21
    th = h + SHIFT
    tl = (h - (th - SHIFT)) * 2.0**21 + SHIFT
    low = lambda x: (np.ascontiguousarray(x).view(np.uint64) & np.uint64(0xFFFFFFFF)).astype(np.uint32)
    regs = [*_fields(list(low(th))), *_fields(list(low(tl)))]
    byte = lambda r, b: ((r >> np.uint32(8 * b)) & np.uint32(255)).astype(np.uint8).view(np.int8).astype(np.int64)
    return np.stack([np.stack([byte(r, b) for b in range(4)]) for r in regs])


def _edges():
    """Values whose 21-bit halves sit at the ends of their digits: t = +-64,
    fields of 0 and 127 before centring, and one off each."""
    H = [s * (t * 16384 + m * 128 + l) for s in (1, -1) for t in (0, 1, 63, 64) for m in (-64, -63, 0, 62, 63)
         for l in (-64, -63, -1, 0, 1, 63)]
    H = np.array([h for h in H if abs(h) <= 1 << 20], np.float64)
    L = np.array([-(1 << 20), -(1 << 20) + 1, -8256, -8255, -1, 0, 1, 8127, 8128, (1 << 20) - 1], np.float64)
    v = (H[:, None] * 2.0**-21 + L[None, :] * 2.0**-42).ravel()
    return v[np.abs(v) <= 0.5]


def test_packed_digits_are_the_digits():
    for v in (_samples(5, 40000), _edges()):
        rng = np.random.default_rng(6)
        x = rng.permutation(np.concatenate([v, -v]))
        x = x[: len(x) // 4 * 4].reshape(4, -1)
        got = packed_digits(x)
        want = np.stack([digits(x[b]) for b in range(4)], axis=1)
        assert np.array_equal(got, want)


def test_a_wrong_byte_selection_is_seen():
    """The comparison notices a swapped pair of values in one register."""
    x = _edges()[:400].reshape(4, -1)
    assert not np.array_equal(packed_digits(x[[1, 0, 2, 3]]), np.stack([digits(x[b]) for b in range(4)], axis=1))
