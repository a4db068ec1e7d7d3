"""The FP32 screen of the lane-per-particle list build: its operations, step
by step in FP32, against the exact d^2 - r^2 of the same positions; the guard
band of the builder must cover the error (it is twice the derived bound of
the rounding of |x|^2 plus eight times that of the coordinates)."""
import numpy as np
import pytest

U = 1.0 / 16777216.0  # 2^-24


def _fma(a, b, c):
    return (a.astype(np.float64) * b.astype(np.float64) + c.astype(np.float64)).astype(np.float32)


@pytest.mark.parametrize("brick", [1, 2, 3])
@pytest.mark.parametrize("cell,radius", [(2.8, 2.8), (2.86, 2.8), (3.3, 3.3), (5.5, 4.0), (1.1, 1.0)])
def test_guard_band_covers_the_screen(brick, cell, radius):
    rng = np.random.default_rng(int(100 * cell) + brick)
    span = (brick + 2) * cell
    r2 = radius * radius
    err = 2.0 * np.sqrt(3.0) * radius * U * (2.0 * span + 2.0 * radius) + 3.0 * U * r2
    guard = 8.0 * err + 2.0 * 17.3 * span * span * U
    corner = rng.uniform(-50.0, 50.0, 3)
    n = 200_000
    p = corner + rng.uniform(0.0, span, (n, 3))
    d = rng.normal(size=(n, 3))
    d *= (radius * (1.0 + rng.uniform(-1e-3, 1e-3, n)) / np.linalg.norm(d, axis=1))[:, None]
    q = p + d
    inside = np.all((q >= corner) & (q <= corner + span), axis=1)
    p, q = p[inside], q[inside]
    centre = corner + 0.5 * span
    a, b = (p - centre).astype(np.float32), (q - centre).astype(np.float32)
    c = ((a.astype(np.float64) ** 2).sum(1) - r2).astype(np.float32)
    e = c
    for k in range(3):
        e = _fma(b[:, k], np.float32(-2.0) * a[:, k], e)
    sq = _fma(b[:, 2], b[:, 2], _fma(b[:, 1], b[:, 1], b[:, 0] * b[:, 0]))
    e = (e.astype(np.float64) + sq.astype(np.float64)).astype(np.float32)
    exact = ((p - q) ** 2).sum(1) - r2
    worst = np.abs(e - exact).max()
    print(f"{len(p)} pairs, worst error {worst:.2e}, band {guard:.2e}")
    assert len(p) > 100 and worst <= 0.5 * guard
