"""GPU: a cluster's velocity has the same bits whatever call it is in: the whole frame,
a part of it, a frame of another number of clusters, one of another mean cluster size, a batch of
few or of many clusters, with and without the inlier mask (three launches, or one up to 256
hypotheses), refit by the scoring workgroup or after it.

Nearly all points of a cluster share one azimuth, so that another order of the refit's
float64 sums would change float32 bits of most clusters.
Tolerance: none."""
from __future__ import annotations

import numpy as np
import pytest

from test_gpu_pruned import cluster, frame_of, rv  # noqa: F401 (fixture)

pytestmark = pytest.mark.gpu

OUT = ("vx", "vy", "heading", "n_inliers", "status")


def narrow(sizes, seed):
    """Clusters whose points share one azimuth within a micro-radian, but for one in a
    hundred a little more than the seed separation away."""
    rng = np.random.default_rng(seed)
    out = []
    for n in sizes:
        t = 0.3 + rng.normal(0, 1e-6, n)
        t[rng.permutation(n)[: max(1, n // 100)]] += 1.5e-3
        vx, vy = rng.uniform(-30, 30, 2)
        out.append((t, vx * np.cos(t) + vy * np.sin(t) + rng.normal(0, 0.05, n)))
    return frame_of(out)


def join(*frames):
    off = [np.zeros(1, np.int64)]
    for _, _, o in frames:
        off.append(o[1:].astype(np.int64) + off[-1][-1])
    return (np.concatenate([f[0] for f in frames]), np.concatenate([f[1] for f in frames]),
            np.concatenate(off).astype(np.int32))


def same(label, want, got, k):
    for name in OUT:
        a, b = (np.ascontiguousarray(x[name].cpu().numpy()[:k]) for x in (want, got))
        bad = np.nonzero(a.view(np.uint8).reshape(k, -1) != b.view(np.uint8).reshape(k, -1))[0]
        assert bad.size == 0, f"{label}: {name} differs in {len(set(bad))} of {k} clusters"


@pytest.mark.parametrize("n_hyp", [200, 512])
def test_same_bits_in_every_call(rv, n_hyp):  # noqa: F811
    import torch

    rng = np.random.default_rng(8)
    sizes = np.concatenate([rng.integers(256, 1024, 300), rng.integers(2, 256, 60),
                            rng.integers(1024, 3000, 40), [255, 256, 257, 1023, 1024, 1025]])
    K = len(sizes)
    lead = narrow(sizes, 100)

    def gpu(f):
        return [torch.from_numpy(np.ascontiguousarray(a)).cuda() for a in f]

    def single(label, f, **kw):
        t, v, o = gpu(f)
        print(f"[gpu] refit order: {label} K={len(f[2]) - 1} H={n_hyp}", flush=True)
        r = rv.rv_estimate_velocity(t, v, o, n_hyp, 0.15, 9, **kw)
        torch.cuda.synchronize()
        return r

    want = single("alone", lead, want_bits=True)
    assert (want["status"] == 0).sum() > K // 2
    same("without the mask", want, single("without the mask", lead), K)
    small = frame_of([cluster(5, 1, p_uniform=0.0)] * 3000)
    same("many clusters", want, single("many clusters", join(lead, small), want_bits=True), K)
    same("no order", want, single("no order", join(lead, frame_of([cluster(3, 1)] * 66000)),
                                  want_bits=True), K)
    n_long = 8192 * (K + 1)
    large = frame_of([cluster(n_long, 3, p_uniform=0.1)])
    same("long clusters", want, single("long clusters", join(lead, large), want_bits=True), K)
    # Few enough clusters for the rule of long ones.
    few = narrow(sizes[-60:], 5000)
    large = frame_of([cluster(8192 * 61, 3, p_uniform=0.1)])
    same("few, long", single("few", few, want_bits=True),
         single("few, long", join(few, large), want_bits=True), 60)

    # A small frame (one launch up to 256 hypotheses).
    tiny = narrow(rng.integers(2, 1400, 70), 9000)
    same("one launch", single("three launches", tiny, want_bits=True), single("one launch", tiny), 70)

    # A part of a frame of many clusters.
    whole = join(lead, small)
    t, v, o = gpu(whole)
    first, p0 = 120, int(whole[2][120])
    n1 = int(whole[2][K])
    print(f"[gpu] refit order: part H={n_hyp}", flush=True)
    part = rv.rv_estimate_velocity_part(t[p0:n1], v[p0:n1], o[first:K + 1], first, p0, n_hyp, 0.15, 9)
    torch.cuda.synchronize()
    same("part", {k: want[k][first:] for k in OUT}, part, K - first)

    # Batches: this frame first, then frames that make the batch one of many clusters.
    for label, frames in (("batch of one", [lead]), ("batch of many", [lead, small]),
                          ("long batch", [few, large])):
        t, v, o = gpu(join(*frames))
        ends = np.cumsum([0] + [len(f[2]) - 1 for f in frames]).astype(np.int32)
        print(f"[gpu] refit order: {label} H={n_hyp}", flush=True)
        got = rv.rv_estimate_velocity_batch(t, v, o, torch.from_numpy(ends).cuda(),
                                            torch.full((len(frames),), 9, device="cuda"), n_hyp, 0.15)
        torch.cuda.synchronize()
        k = len(frames[0][2]) - 1
        same(label, single("alone", frames[0], want_bits=True), got, k)
