"""Large clusters counting only possible winners (score_pruned in csrc/rv.hip) on
the GPU: a call without per-hypothesis counts gives, bit for bit, the outputs of
the same call that counts every hypothesis (``hyp_counts`` requested), which the
parity tests compare with the oracle.  Tolerance: none, the kept hypothesis is
the same and everything after it is the same code."""
from __future__ import annotations

import numpy as np
import pytest

from paper_2012_12618_amd import synth

pytestmark = pytest.mark.gpu

KEYS = ("vx", "vy", "heading", "n_inliers", "status", "n_near_tau", "best_hyp", "inlier_bits")


@pytest.fixture(scope="module")
def rv():
    import torch

    if not torch.cuda.is_available():
        pytest.skip("needs a GPU")
    from paper_2012_12618_amd import binding

    binding.load_library()
    return binding


def frame_of(clusters):
    """Clusters (theta, vd) concatenated into one CSR frame."""
    off = np.concatenate([[0], np.cumsum([len(t) for t, _ in clusters])]).astype(np.int32)
    return (np.concatenate([t for t, _ in clusters]).astype(np.float32),
            np.concatenate([v for _, v in clusters]).astype(np.float32), off)


def cluster(n, seed, **kw):
    f = synth.make_frame(synth.FrameSpec(1, "fixed", n, n, **kw), seed)
    return f.theta, f.vd


def compare(rv, theta, vd, off, n_hyp, tau, seed, label, bits=True):
    import torch

    print(f"[gpu] pruned against full count: {label} K={len(off) - 1} N={len(theta)} H={n_hyp} "
          f"tau={tau}", flush=True)
    t, v, o = (torch.from_numpy(np.ascontiguousarray(a)).cuda() for a in (theta, vd, off))
    K, N = len(off) - 1, len(theta)

    def call(counts):
        out = rv.allocate_outputs(K, N, n_hyp, t.device, want_bits=bits, debug=True)
        if not counts:
            del out["hyp_counts"]
        rv.rv_estimate_velocity(t, v, o, n_hyp, tau, seed, out=out)
        torch.cuda.synchronize()
        return {k: out[k].cpu().numpy() for k in KEYS if k in out}

    full, pruned = call(True), call(False)
    for k in full:
        a, b = full[k], pruned[k]
        if a.dtype == np.float32:
            a, b = a.view(np.int32), b.view(np.int32)
        bad = np.nonzero(a != b)[0]
        assert bad.size == 0, f"{label}: {k} differs at {bad[:8]}: {full[k][bad[:8]]} {pruned[k][bad[:8]]}"
    return pruned


SIZES = (255, 256, 257, 319, 320, 321, 383, 384, 385, 512, 513, 1023, 1024, 1025, 2047, 4096, 4097)


@pytest.mark.parametrize("n_hyp", [1, 7, 64, 255, 256, 257, 512, 1000, 1024, 1025, 2500])
def test_sizes_and_hypothesis_counts(rv, n_hyp):
    clusters = [cluster(n, 900 + i, p_uniform=0.15, p_band=0.15) for i, n in enumerate(SIZES)]
    compare(rv, *frame_of(clusters), n_hyp, 0.15, 77 + n_hyp, f"sizes H={n_hyp}")
    # The one-launch path (no mask, at most 256 hypotheses).
    compare(rv, *frame_of(clusters), min(n_hyp, 256), 0.15, 78 + n_hyp, "one launch", bits=False)


def stress_clusters():
    rng = np.random.default_rng(5)
    out = []
    n = 900
    th = rng.uniform(-1, 1, n)
    out.append((th, 3 * np.cos(th) - 4 * np.sin(th)))                     # noiseless: all valid pairs tie
    out.append((np.full(n, 0.3), rng.normal(0, 1, n)))                    # all pairs degenerate
    out.append((np.repeat(rng.uniform(-1, 1, 5), 180), rng.normal(0, 1, n)))  # five directions
    out.append(cluster(1500, 11, p_uniform=0.2, theta_spread_deg=0.5))    # half-degree window
    out.append(cluster(1500, 12, p_uniform=0.2, theta_spread_deg=3.0))
    th = rng.uniform(-np.pi, np.pi, 2000)
    out.append((th, 9 * np.cos(th) + 2 * np.sin(th) + rng.normal(0, 0.05, 2000)))  # whole circle
    th = np.pi + rng.uniform(-0.4, 0.4, 1200)                              # across the cut at pi
    th = np.where(th > np.pi, th - 2 * np.pi, th)
    out.append((th, 9 * np.cos(th) + 2 * np.sin(th) + rng.normal(0, 0.05, 1200)))
    out.append((rng.uniform(-50, 50, 700), rng.normal(0, 5, 700)))         # many turns, no structure
    t, v = cluster(3000, 13, p_uniform=0.3)
    o = np.argsort(t)
    out.append((t[o], v[o]))                                               # sorted by azimuth
    o = np.argsort(v)
    out.append((t[o], v[o]))                                               # sorted by Doppler
    t, v = (a.copy() for a in cluster(1000, 14, p_uniform=0.2))
    t[::7], v[::11], v[::13] = np.nan, np.inf, -np.inf                     # non-finite points
    out.append((t, v))
    t, v = (a.copy() for a in cluster(1000, 15, p_uniform=0.2))
    v[::5] = rng.choice([-1, 1], 200) * 10.0 ** rng.uniform(10, 38, 200)   # enormous outliers
    out.append((t, v.astype(np.float32)))
    t, v = cluster(1000, 16, p_uniform=0.2)
    out.append((t, v * np.float32(1e17)))                                  # no usable reference
    out.append((t, v * np.float32(400.0)))                                 # 12 km/s
    out.append((t, v * np.float32(1e-3)))                                  # everything is an inlier
    out.append((t, np.zeros_like(v)))
    out.append((np.full(600, np.nan), np.zeros(600)))                      # no finite point
    return out


@pytest.mark.parametrize("n_hyp,tau", [(256, 0.15), (1000, 0.15), (1024, 0.01), (512, 3.0),
                                       (512, 1e-31), (512, 1e16), (300, 1e-20), (300, 1e14)])
def test_stress_clusters(rv, n_hyp, tau):
    compare(rv, *frame_of(stress_clusters()), n_hyp, tau, 5, "stress")


@pytest.mark.parametrize("case", range(6))
def test_drawn_frames(rv, case):
    rng = np.random.default_rng(4000 + case)
    spec = synth.FrameSpec(int(rng.integers(3, 60)), "loguniform", 2, int(rng.integers(300, 9000)),
                           p_uniform=float(rng.uniform(0, 0.5)), p_band=float(rng.uniform(0, 0.4)),
                           sigma=float(rng.choice([0.0, 0.02, 0.05, 0.3])),
                           theta_spread_deg=None if case % 2 else float(rng.uniform(0.2, 90)))
    f = synth.make_frame(spec, 4100 + case)
    compare(rv, f.theta, f.vd, f.offsets, int(rng.integers(1, 3000)), float(rng.uniform(0.02, 1.0)),
            case, f"drawn {case}")


def test_long_cluster_and_batch(rv):
    """A 70,000-point cluster beside small ones, and the batched form (with more
    than one workgroup per cluster sharing the best key)."""
    import torch

    clusters = [cluster(70000, 21, p_band=0.4), cluster(40, 22), cluster(5000, 23, p_uniform=0.3)]
    theta, vd, off = frame_of(clusters)
    single = compare(rv, theta, vd, off, 4096, 0.15, 3, "long")
    t, v, o = (torch.from_numpy(a).cuda() for a in (theta, vd, off))
    fo = torch.tensor([0, 3], dtype=torch.int32, device="cuda")
    seeds = torch.tensor([3], dtype=torch.int64, device="cuda")
    for fp16_min in (0, 1024):
        tuning = rv.rv_tuning_default()
        tuning.fp16_min_points = fp16_min
        out = rv.rv_estimate_velocity_batch(t, v, o, fo, seeds, 4096, 0.15, tuning=tuning, want_bits=True)
        torch.cuda.synchronize()
        for k in ("vx", "vy", "heading"):
            assert np.array_equal(out[k].cpu().numpy().view(np.int32), single[k].view(np.int32)), k
        for k in ("n_inliers", "status", "n_near_tau", "inlier_bits"):
            assert np.array_equal(out[k].cpu().numpy(), single[k]), k


@pytest.mark.parametrize("n_hyp,tau", [(1, 0.15), (255, 0.15), (256, 0.15), (512, 0.01), (700, 3.0),
                                       (1024, 0.15), (1100, 0.15), (512, 0.25), (512, 1e-31),
                                       (512, 1e16), (300, 1e-14), (300, 9e14)])
def test_small_clusters(rv, n_hyp, tau):
    """Clusters of 2 to 256 points (score_small: every hypothesis of a workgroup at
    once, the compare as a clamped FMA) against lanes = points (no such form allowed),
    per-hypothesis counts included, with edge clusters and tau at powers of two and
    where the form does not apply."""
    import torch

    sizes = list(range(2, 10)) + [31, 32, 33, 63, 64, 65, 95, 127, 128, 129, 159, 160, 199, 200,
                                  201, 255, 256]
    clusters = [cluster(n, 700 + n, p_uniform=0.2) for n in sizes]
    t, v = (a.copy() for a in cluster(90, 31, p_uniform=0.2))
    t[::7], v[::11], v[::13] = np.nan, np.inf, -np.inf
    clusters.append((t, v))
    # Doppler values at exactly tau, and one unit in the last place either side, from
    # the hypotheses of the others.
    th = np.zeros(60, np.float32)
    th[1::2] = 0.5
    e = np.float32(tau)
    clusters.append((th, np.where(np.arange(60) % 3 == 0, np.nextafter(e, np.float32(0)), e)))
    clusters.append((np.full(40, 0.3), np.linspace(-1, 1, 40)))
    theta, vd, off = frame_of(clusters)
    t, v, o = (torch.from_numpy(a).cuda() for a in (theta, vd, off))
    K = len(off) - 1
    # Enough clusters for several blocks of hypotheses per workgroup.
    copies = 2048 // K + 1
    N = len(theta)
    big_t, big_v = t.repeat(copies), v.repeat(copies)
    base = torch.arange(copies, device="cuda", dtype=torch.int32)[:, None] * N
    big_o = torch.cat([(o[:-1][None] + base).reshape(-1), base[-1:, 0] + N])
    out = {}
    for lanes_max in (0, 64):
        for copy in (False, True):
            tuning = rv.rv_tuning_default()
            tuning.lanes_max_points = lanes_max
            print(f"[gpu] small clusters H={n_hyp} tau={tau} lanes_max={lanes_max} many={copy}", flush=True)
            a, b, c = (big_t, big_v, big_o) if copy else (t, v, o)
            fo = torch.tensor([0, len(c) - 1], dtype=torch.int32, device="cuda")
            seeds = torch.tensor([41], dtype=torch.int64, device="cuda")
            r = rv.rv_estimate_velocity_batch(a, b, c, fo, seeds, n_hyp, tau, tuning=tuning,
                                              want_bits=True, debug=True)
            torch.cuda.synchronize()
            out[lanes_max, copy] = {k: x.cpu().numpy() for k, x in r.items()}
    for copy in (False, True):
        for k, x in out[0, copy].items():
            y = out[64, copy][k]
            assert np.array_equal(x.view(np.uint8), y.view(np.uint8)), (k, copy)
