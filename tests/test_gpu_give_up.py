"""GPU: clusters in which the bound of score_pruned (csrc/rv.hip) excludes too little:
many outliers, a threshold far below the noise, no structure at all.  They are counted
in full after all, in place, by score_small, or deferred to the workgroups behind the
refit (few, long clusters); large clusters of dense frames are split between two scoring
workgroups.  As in test_gpu_pruned, every output equals, bit for bit, that of the call
which counts every hypothesis.  Tolerance: none."""
from __future__ import annotations

import numpy as np
import pytest

from test_gpu_pruned import KEYS, cluster, compare, frame_of, rv  # noqa: F401 (fixture)

pytestmark = pytest.mark.gpu

SIZES = (128, 160, 240, 241, 255, 256, 257, 320, 700, 1023, 1024, 1025, 2047, 2048, 3000)
OUTLIERS = (0.5, 0.65, 0.8, 1.0)


def noisy(sizes, seed):
    return [cluster(n, seed + 7 * i + n, p_uniform=p) for i, p in enumerate(OUTLIERS) for n in sizes]


@pytest.mark.parametrize("n_hyp,tau", [(64, 0.15), (257, 0.15), (1000, 0.15), (1024, 0.005), (2100, 0.15)])
def test_few_clusters(rv, n_hyp, tau):  # noqa: F811
    compare(rv, *frame_of(noisy(SIZES, 10)), n_hyp, tau, 31, f"give up H={n_hyp}")


@pytest.mark.parametrize("n_hyp", [512, 600, 1024, 1025])
def test_many_clusters(rv, n_hyp):  # noqa: F811
    """Two and four blocks of hypotheses per workgroup, split and whole clusters."""
    part = noisy(SIZES, 400)
    few = [cluster(40, 5)] * (2100 - 2 * len(part))
    compare(rv, *frame_of(part + few + part), n_hyp, 0.15, 32, f"give up, many H={n_hyp}")


@pytest.mark.parametrize("n_hyp", [100, 1024, 3000])
@pytest.mark.parametrize("outliers", [0.2, 0.62, 0.7, 0.9])
def test_long_clusters(rv, n_hyp, outliers):  # noqa: F811
    sizes = (1, 2, 300, 1023, 1024, 1500, 8191, 8192, 9000, 30000, 70001)
    long = [cluster(n, 900 + n, p_uniform=outliers) for n in sizes]
    compare(rv, *frame_of(long), n_hyp, 0.15, 33, f"give up, long {outliers} H={n_hyp}")


@pytest.mark.parametrize("fp16_min", [0, 512])
def test_batches(rv, fp16_min):  # noqa: F811
    import torch

    long = [cluster(n, 60 + n, p_uniform=p) for n in (9000, 20000, 1024, 300) for p in (0.3, 0.85)]
    frames = {"long": long, "many": noisy(SIZES, 800) + [cluster(300, 2, p_uniform=0.9)] * 2000}
    for label, clusters in frames.items():
        theta, vd, off = frame_of(clusters)
        t, v, o = (torch.from_numpy(a).cuda() for a in (theta, vd, off))
        K = len(off) - 1
        fo = torch.tensor([0, K // 3, K], dtype=torch.int32, device="cuda")
        seeds = torch.tensor([4, 5], dtype=torch.int64, device="cuda")
        got = []
        for counts in (True, False):
            tuning = rv.rv_tuning_default()
            tuning.fp16_min_points = 0 if counts else fp16_min
            print(f"[gpu] give up, batch {label} fp16_min={fp16_min} counts={counts}", flush=True)
            out = rv.allocate_batch_outputs(2, K, len(theta), 600, t.device, want_bits=True, debug=True)
            if not counts:
                del out["hyp_counts"]
            rv.rv_estimate_velocity_batch(t, v, o, fo, seeds, 600, 0.15, tuning=tuning, out=out)
            torch.cuda.synchronize()
            got.append({k: out[k].cpu().numpy() for k in KEYS if k in out})
        for k, x in got[0].items():
            assert np.array_equal(x.view(np.uint8), got[1][k].view(np.uint8)), (label, k)


def test_graph_of_deferred_clusters(rv):  # noqa: F811
    """A captured batch whose clusters are deferred in one replay and not in the next."""
    import torch

    good = frame_of([cluster(n, n, p_uniform=0.2) for n in (9000, 20000, 1500)])
    bad = frame_of([cluster(n, n, p_uniform=0.9) for n in (9000, 20000, 1500)])
    t, v, o = (torch.from_numpy(a.copy()).cuda() for a in good)
    fo = torch.tensor([0, 3], dtype=torch.int32, device="cuda")
    sd = torch.tensor([5], dtype=torch.int64, device="cuda")
    outs = []
    for _ in range(2):
        out = rv.allocate_batch_outputs(1, 3, t.numel(), 1024, t.device, want_bits=True, debug=True)
        del out["hyp_counts"]
        outs.append(out)
    eager, captured = outs
    graph = rv.rv_graph_capture_batch(t, v, o, fo, sd, 1024, 0.15, captured)
    try:
        for rep, (theta, vd, _) in enumerate((good, bad, bad, good, bad)):
            t.copy_(torch.from_numpy(theta))
            v.copy_(torch.from_numpy(vd))
            rv.rv_estimate_velocity_batch(t, v, o, fo, sd, 1024, 0.15, out=eager)
            torch.cuda.synchronize()
            print(f"[gpu] graph of deferred clusters, replay {rep}", flush=True)
            graph.launch()
            torch.cuda.synchronize()
            for k in KEYS:
                if k in eager:
                    a, b = eager[k].cpu().numpy(), captured[k].cpu().numpy()
                    assert np.array_equal(a.view(np.uint8), b.view(np.uint8)), (rep, k)
    finally:
        graph.destroy()


def test_more_large_clusters_than_points_allow(rv):  # noqa: F811
    """Offsets that go back again and again: more clusters of 2048 points than fit the
    points one after the other (each is a valid range, so each is estimated)."""
    theta, vd = cluster(4096, 77, p_uniform=0.3)
    off = np.resize(np.array([0, 2048, 4096], np.int32), 3001)
    compare(rv, theta, vd, off, 1024, 0.15, 34, "ranges again and again", bits=False)
