"""Frames and batches of long clusters on the GPU (mean of 8192 points and more):
scored by workgroups of 1024 threads with a table of 32 directions.  As in
test_gpu_pruned, a call without per-hypothesis counts gives, bit for bit, the
outputs of the same call that counts every hypothesis, which the parity tests
compare with the oracle.  Tolerance: none."""
from __future__ import annotations

import numpy as np
import pytest

from test_gpu_pruned import KEYS, cluster, compare, frame_of, rv, stress_clusters  # noqa: F401

pytestmark = pytest.mark.gpu

SIZES = (0, 1, 2, 5, 63, 64, 65, 127, 128, 129, 200, 319, 320, 1000, 1024, 4097, 30000, 70001, 150000)


def mixed():
    out = []
    for i, n in enumerate(SIZES):
        t, v = cluster(max(n, 1), 300 + i, p_uniform=0.2, p_band=0.2)
        out.append((t[:n], v[:n]))
    return out


@pytest.mark.parametrize("n_hyp", [1, 64, 255, 257, 1023, 1024, 1025, 4100])
def test_mixed_sizes(rv, n_hyp):  # noqa: F811
    theta, vd, off = frame_of(mixed())
    assert len(theta) // (len(off) - 1) >= 8192
    compare(rv, theta, vd, off, n_hyp, 0.15, 19 + n_hyp, "mixed, long")


@pytest.mark.parametrize("tau", [0.15, 0.01, 3.0, 1e-31, 1e16])
def test_stress(rv, tau):  # noqa: F811
    theta, vd, off = frame_of(stress_clusters() + [cluster(250000, 9, p_band=0.4)])
    assert len(theta) // (len(off) - 1) >= 8192
    compare(rv, theta, vd, off, 1500, tau, 23, "stress, long")


@pytest.mark.parametrize("clusters", [256, 257, 520])
def test_cluster_count_rule(rv, clusters):  # noqa: F811
    """Both sides of the rule on the number of clusters (8192-point clusters)."""
    part = [cluster(8192, 40 + i, p_uniform=0.1, p_band=0.1) for i in range(8)]
    theta, vd, off = frame_of([part[i % 8] for i in range(clusters)])
    for n_hyp in (300, 1000):
        compare(rv, theta, vd, off, n_hyp, 0.15, 5, f"rule H={n_hyp}", bits=False)


@pytest.mark.parametrize("fp16_min", [0, 2, 127, 128, 5000])
@pytest.mark.parametrize("lanes_max", [0, 64])
def test_batch(rv, fp16_min, lanes_max):  # noqa: F811
    """The batched form under every tuning that meets the rule, and one that does not."""
    import torch

    frames = [frame_of(mixed()), frame_of([cluster(20000, 3, p_band=0.3), cluster(90, 4)])]
    theta = torch.from_numpy(np.concatenate([f[0] for f in frames])).cuda()
    vd = torch.from_numpy(np.concatenate([f[1] for f in frames])).cuda()
    off, at = [np.zeros(1, np.int32)], 0
    for f in frames:
        off.append(f[2][1:] + at)
        at += f[2][-1]
    off = torch.from_numpy(np.concatenate(off).astype(np.int32)).cuda()
    fo = torch.tensor([0, len(frames[0][2]) - 1, off.numel() - 1], dtype=torch.int32).cuda()
    seeds = torch.tensor([11, 12], dtype=torch.int64, device="cuda")
    tuning = rv.rv_tuning_default()
    tuning.fp16_min_points, tuning.lanes_max_points = fp16_min, lanes_max
    results = []
    for counts in (True, False):
        print(f"[gpu] long batch fp16_min={fp16_min} lanes_max={lanes_max} counts={counts}", flush=True)
        out = rv.allocate_batch_outputs(2, off.numel() - 1, theta.numel(), 1300, theta.device,
                                        want_bits=True, debug=True)
        if not counts:
            del out["hyp_counts"]
        rv.rv_estimate_velocity_batch(theta, vd, off, fo, seeds, 1300, 0.15, tuning=tuning, out=out)
        torch.cuda.synchronize()
        results.append({k: out[k].cpu().numpy() for k in KEYS if k in out})
    for k, x in results[0].items():
        assert np.array_equal(x.view(np.uint8), results[1][k].view(np.uint8)), k
