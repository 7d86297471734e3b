"""The compositing's support test, emulated in FP32 on the CPU.

A wave skips a list entry whose support ellipse misses the rectangle of its
pixel centres (gs_render.hip, ellipse_mask and conic_min_rect).  That must never
skip a (pixel, entry) pair that the per-pixel evaluation keeps.  The emulation
rounds each operation as the kernel does, takes the hardware's reciprocal and
base-2 logarithm wrong by their largest error in either direction, and puts the
pixels where it matters: at the edge of the support ellipse."""
import numpy as np
import pytest

F = np.float32
LOG2E = F(1.4426950408889634)


def _fma(a, b, c):
    # the exact product of two FP32 values fits FP64
    return (a.astype(np.float64) * b.astype(np.float64) + c.astype(np.float64)).astype(F)


def _ulps(x, k):
    return (x.view(np.int32) + np.int32(k)).view(F)


def _conics(rng, n, cond_max):
    """FP32 conics (A, B, C) of random footprints: the smaller variance 0.3 and up."""
    small = 0.3 * np.exp(rng.uniform(0, np.log(1e4), n))
    big = small * np.exp(rng.uniform(0, np.log(cond_max), n))
    t = rng.uniform(0, np.pi, n)
    c, s = np.cos(t), np.sin(t)
    A, C = c * c / big + s * s / small, s * s / big + c * c / small
    B = c * s * (1 / big - 1 / small)
    return A.astype(F), B.astype(F), C.astype(F)


def _reaches(u, v, A, B, C, o, px, py):
    """The kernel's per-pixel test (eval_pair), with 2^-22 in favour of the pair
    for the hardware's base-2 exponential."""
    h = F(-0.5) * LOG2E
    pz, pw, qx = h * A, h * B, h * C
    dx, dy = u - px, v - py
    nx, ny = _fma(pz, dx, pw * dy), _fma(qx, dy, pw * dx)
    p2 = _fma(dx, nx, dy * ny)
    og = o.astype(np.float64) * np.exp2(p2.astype(np.float64)) * (1 + 2.0 ** -22)
    return (p2 <= 0) & (og >= float(F(1.0) / F(255.0)) * (1 - 2.0 ** -23))


def _clamp(x, lo, hi):
    return np.minimum(np.maximum(x, lo), hi)


def _conic_min(A, B2, C, mA, mC, xa, xb, ya, yb):
    z = F(0)
    X, Y = _clamp(z, xa, xb), _clamp(z, ya, yb)
    y, x = _clamp(mC * X, ya, yb), _clamp(mA * Y, xa, xb)
    q1 = _fma(_fma(A, X, B2 * y), X, C * y * y)
    q2 = _fma(_fma(C, Y, B2 * x), Y, A * x * x)
    return np.minimum(q1, q2)


def _kept(u, v, A, B, C, o, xa, xb, ya, yb, rcp_ulp, log_err):
    """The kernel's test of one rectangle of pixel centres."""
    mA, mC = -B * _ulps(F(1) / A, rcp_ulp), -B * _ulps(F(1) / C, rcp_ulp)
    lg = (np.log2((F(255) * o).astype(np.float64)) + log_err).astype(F)
    rho2 = F(2.0 * 1.04 * 0.6931471805599453) * lg + F(4e-4)
    dl = F(1e-3) + F(1e-6) * np.maximum(np.abs(u), np.abs(v))
    q = _conic_min(A, F(2) * B, C, mA, mC, xa - dl - u, xb + dl - u, ya - dl - v, yb + dl - v)
    return q <= rho2, q


def _exact_min(A, B, C, xa, xb, ya, yb):
    """The least value over the rectangle in FP64, from all four edges."""
    A, B, C, xa, xb, ya, yb = (t.astype(np.float64) for t in (A, B, C, xa, xb, ya, yb))
    best = np.where((xa <= 0) & (xb >= 0) & (ya <= 0) & (yb >= 0), 0.0, np.inf)
    q = lambda x, y: A * x * x + 2 * B * x * y + C * y * y
    for X in (xa, xb):
        best = np.minimum(best, q(X, _clamp(-B * X / C, ya, yb)))
    for Y in (ya, yb):
        best = np.minimum(best, q(_clamp(-B * Y / A, xa, xb), Y))
    return best


@pytest.mark.parametrize("cond_max", [1.5, 100.0, 1e5])
@pytest.mark.parametrize("size", [8, 4, 1])
def test_no_reached_pixel_is_skipped(cond_max, size):
    """8 x 8 quadrants, and the boxes of 4 x 4 blocks with some pixels stopped."""
    rng = np.random.default_rng(int(cond_max) * 10 + size)
    n = 400_000
    A, B, C = _conics(rng, n, cond_max)
    ok = A.astype(np.float64) * C.astype(np.float64) > B.astype(np.float64) ** 2 * (1 + 1e-5)
    A, B, C = A[ok], B[ok], C[ok]
    n = len(A)
    o = np.exp(rng.uniform(np.log(1.0 / 255), 0, n)).astype(F)
    o = np.where(F(255) * o > F(1), o, F(0.5))
    # the rectangle's first pixel, and (sizes below 8) how far it goes
    x0 = (np.floor(rng.uniform(-64, 4096, n)) + 0.5).astype(F)
    y0 = (np.floor(rng.uniform(-64, 2304, n)) + 0.5).astype(F)
    wx = (size - 1 if size == 8 else rng.integers(0, size, n)) * np.ones(n, F)
    wy = (size - 1 if size == 8 else rng.integers(0, size, n)) * np.ones(n, F)
    wx, wy = wx.astype(F), wy.astype(F)
    # one of its pixels, most often on the border, at the edge of the support: q(d) = rho^2 (1 - e)
    px = x0 + np.floor(rng.uniform(0, 1, n) * (wx + 1)).astype(F)
    py = y0 + np.floor(rng.uniform(0, 1, n) * (wy + 1)).astype(F)
    side = rng.integers(0, 6, n)
    px = np.where(side == 0, x0, np.where(side == 1, x0 + wx, px))
    py = np.where(side == 2, y0, np.where(side == 3, y0 + wy, py))
    rho = np.sqrt(2 * np.log(255 * o.astype(np.float64)) * (1 - np.exp(rng.uniform(np.log(1e-7), np.log(0.2), n))))
    t = rng.uniform(0, 2 * np.pi, n)
    a64, b64, c64 = A.astype(np.float64), B.astype(np.float64), C.astype(np.float64)
    l11 = np.sqrt(a64)                               # d = rho L^-T (cos, sin), Q = L L^T
    l21 = b64 / l11
    l22 = np.sqrt(c64 - l21 * l21)
    dy = rho * np.sin(t) / l22
    dx = (rho * np.cos(t) - l21 * dy) / l11
    u, v = (px.astype(np.float64) + dx).astype(F), (py.astype(np.float64) + dy).astype(F)
    reached = _reaches(u, v, A, B, C, o, px, py)
    assert reached.mean() > 0.5                      # the pairs are what they are meant to be
    for rcp_ulp in (-2, 2):
        for log_err in (-1e-6, 1e-6):
            kept, q = _kept(u, v, A, B, C, o, x0, x0 + wx, y0, y0 + wy, rcp_ulp, log_err)
            assert kept[reached].all(), (reached & ~kept).sum()
            # and the value itself, against all four edges in FP64 (2 eps cond, plus
            # the rounding of the rectangle's corners)
            dl = F(1e-3) + F(1e-6) * np.maximum(np.abs(u), np.abs(v))
            want = _exact_min(A, B, C, x0 - dl - u, x0 + wx + dl - u, y0 - dl - v, y0 + wy + dl - v)
            assert (q <= want * (1 + 0.02) + 2e-4).all()


def test_the_ellipse_skips_what_the_box_keeps():
    """The test is worth its cost: most rectangles that the box of a long footprint
    meets lie outside its ellipse."""
    rng = np.random.default_rng(3)
    n = 200_000
    A, B, C = _conics(rng, n, 1e3)
    o = np.full(n, 0.9, F)
    det = A.astype(np.float64) * C - B.astype(np.float64) ** 2
    rho2 = 2 * np.log(255 * 0.9)
    ex, ey = np.sqrt(rho2 * C / det), np.sqrt(rho2 * A / det)
    u, v = (rng.uniform(-1, 1, n) * (ex + 7)).astype(F), (rng.uniform(-1, 1, n) * (ey + 7)).astype(F)
    z = np.zeros(n, F)
    kept, _ = _kept(u, v, A, B, C, o, z + F(0.5), z + F(7.5), z + F(0.5), z + F(7.5), 0, 0.0)
    assert 0.2 < kept.mean() < 0.8
