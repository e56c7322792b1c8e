"""CPU: the upper bound of a hypothesis's inlier count that decides which
hypotheses of a large cluster are counted (score_pruned in csrc/rv.hip).

The cluster's points lie in a table of direction bin x residual bin under a
reference velocity r.  Hypothesis h's bound is the sum, over the direction bins,
of the points whose residual bin lies between those of f - rad and f + rad,
where f = (h - r).u at the bin's centre direction u and rad = w |(h - r) x u| +
w^2/2 |h - r| + tau + 2^-18 (tau + M).  The bound holds if every float32 inlier
of h lies inside its bin's window.  This models the arithmetic in numpy float32
(the reciprocal of the direction key perturbed by an ulp either way) and checks
the containment point by point, on inputs built against it: points whose
residual under h is within 10^-7 tau of tau, directions on bin edges, hypotheses
near to and far from r, velocities to 10^6 m/s, tau from 10^-4 to 10^3, narrow,
wide and full-circle azimuth ranges.  No tolerance: one point outside fails.
"""
import numpy as np
import pytest

F32 = np.float32
BINS, RES = 8, 256


def fma(a, b, c):
    return (np.float64(a) * np.float64(b) + np.float64(c)).astype(F32)


def direction_key(c, s, rng):
    rcp = (1.0 / (np.abs(c) + np.abs(s)).astype(np.float64)).astype(F32)
    rcp = rcp * (1 + rng.integers(-1, 2, rcp.shape) * 2.0 ** -23).astype(F32)
    y = (s * rcp).astype(F32)
    return np.where(c >= 0, y, (np.copysign(F32(2), s) - y).astype(F32)).astype(F32)


def key_direction(q):
    a = np.abs(q)
    c = F32(1) - a
    s = np.copysign(np.where(a <= 1, a, F32(2) - a), q).astype(F32)
    inv = F32(1) / np.sqrt(c * c + s * s)
    return c * inv, s * inv


def residual_bin(e):
    t = np.minimum(np.abs(e) + F32(2), F32(511)).astype(F32)
    k = ((t.view(np.uint32) >> 19) & 127).astype(np.int32)
    return (k ^ (e.astype(F32).view(np.int32) >> 31)) + RES // 2


def sigma_of(tau):
    exponent = int(np.float32(tau).view(np.uint32)) >> 23 & 255
    return np.uint32((127 + 127 + 2 - exponent) << 23).view(F32)


def outside(theta, vd, hyps, r, tau, seed, width_factor=F32(0.53)):
    """Number of (hypothesis, float32 inlier) pairs outside the window."""
    rng = np.random.default_rng(seed)
    c, s = np.cos(theta.astype(np.float64)).astype(F32), np.sin(theta.astype(np.float64)).astype(F32)
    q = direction_key(c, s, rng)
    q0, q1 = q.min(), q.max()
    width = np.maximum(q1 - q0, F32(1e-6)) * F32(1 / BINS)
    i = np.arange(BINS, dtype=F32)
    ax, ay = key_direction(q0 + i * width)
    edge = q0 + (i + 1) * width
    edge[-1] = q1
    bx, by = key_direction(edge)
    w = (width_factor * np.sqrt((bx - ax) ** 2 + (by - ay) ** 2) + F32(2.0 ** -15)).astype(F32)
    mx, my = ax + bx, ay + by
    inv = F32(1) / np.sqrt(mx * mx + my * my)
    mx, my = mx * inv, my * inv
    w2 = (F32(0.5) * w * w).max()
    b = np.clip(((q - q0) * (F32(1) / width)).astype(np.int32), 0, BINS - 1)
    sigma = sigma_of(tau)
    rx, ry = F32(r[0]), F32(r[1])
    er = fma(-ry, s, fma(-rx, c, vd))
    kr = residual_bin(er * sigma)
    bad = 0
    inliers = 0
    for hx, hy in hyps.astype(F32):
        e = fma(-hy, s, fma(-hx, c, vd))
        inl = np.abs(e) < F32(tau)
        m = np.abs(hx) + np.abs(hy) + np.abs(rx) + np.abs(ry)
        dx, dy = (hx - rx) * sigma, (hy - ry) * sigma
        band = fma(np.abs(dx) + np.abs(dy), w2, (F32(tau) + F32(2.0 ** -18) * (F32(tau) + m)) * sigma)
        f = fma(dx, mx, dy * my)
        g = fma(dy, mx, -dx * my)
        rad = fma(np.abs(g), w, band)
        lo, hi = residual_bin(f - rad), residual_bin(f + rad)
        inside = (kr >= lo[b]) & (kr <= hi[b])
        bad += int((inl & ~inside).sum())
        inliers += int(inl.sum())
    assert inliers > 0
    return bad


RANGES = [(-1.05, 1.05), (0.3, 0.3 + 1e-5), (-0.02, 0.03), (1.2, 1.9), (-3.14159, 3.14159), (2.9, 3.141)]


def case(seed):
    rng = np.random.default_rng(seed)
    a, z = RANGES[seed % len(RANGES)]
    tau = F32(rng.choice([1e-4, 0.01, 0.15, 0.25, 0.5, 3.0, 1000.0]))
    speed = 10.0 ** rng.uniform(-1, 6)
    n = 3000
    theta = rng.uniform(a, z, n)
    theta[: 64] = np.linspace(a, z, 64)  # edges of every bin among them
    theta = theta.astype(F32)
    r = rng.uniform(-speed, speed, 2)
    step = 10.0 ** rng.uniform(-7, 0.5, (40, 1)) * rng.choice([float(tau), speed], (40, 1))
    hyps = r + rng.normal(size=(40, 2)) * step
    hyps[:5] = rng.uniform(-speed, speed, (5, 2))
    # Points within 1e-7 of tau of a random hypothesis, either sign, and points inside.
    pick = hyps.astype(F32).astype(np.float64)[rng.integers(0, 40, n)]
    edge = np.where(rng.random(n) < 0.7, 1 - np.abs(rng.normal(0, 1e-7, n)), rng.uniform(0, 1, n))
    e = rng.choice([-1.0, 1.0], n) * float(tau) * edge
    t64 = theta.astype(np.float64)
    vd = (pick[:, 0] * np.cos(t64) + pick[:, 1] * np.sin(t64) + e).astype(F32)
    return theta, vd, hyps, r, tau


@pytest.mark.parametrize("seed", range(36))
def test_every_inlier_is_inside_its_window(seed):
    theta, vd, hyps, r, tau = case(seed)
    assert outside(theta, vd, hyps, r, tau, seed) == 0


def test_a_narrower_window_is_caught():
    """The same check finds inliers outside when the direction bins are taken a
    tenth narrower than they are."""
    assert any(outside(*case(seed), seed, width_factor=F32(0.45)) > 0 for seed in range(36))


def test_residual_bin_is_monotone_and_in_range():
    e = np.sort(np.concatenate([-np.logspace(-30, 38, 4000), [0.0], np.logspace(-30, 38, 4000),
                                np.linspace(-600, 600, 20001)])).astype(F32)
    k = residual_bin(e)
    assert (np.diff(k) >= 0).all() and k.min() == 0 and k.max() == RES - 1


def test_scale_takes_tau_into_its_octave():
    for tau in np.logspace(-14.9, 14.9, 200).astype(F32):
        assert 4.0 <= float(tau * sigma_of(tau)) < 8.0
