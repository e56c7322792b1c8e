"""GPU: clusters that score_pruned (csrc/rv.hip) handles without a reference, and the
batched FP16 form with many workgroups per cluster, against the full count, bit for
bit.  tests/test_score_host.py runs the same code on the CPU under many orders of the
waves.  Tolerance: none."""
from __future__ import annotations

import numpy as np
import pytest

from test_gpu_pruned import KEYS, cluster, compare, frame_of, rv  # noqa: F401 (fixture)

pytestmark = pytest.mark.gpu


def sparse(n, seed, finite):
    """A cluster with a share `finite` of finite points."""
    t, v = (a.copy() for a in cluster(n, seed, p_uniform=0.2))
    v[np.random.default_rng(seed).random(n) >= finite] = np.nan
    return t, v


@pytest.mark.parametrize("n_hyp", [256, 700, 1024, 2500])
def test_few_finite_points(rv, n_hyp):  # noqa: F811
    clusters = [sparse(330 + 61 * i, 500 + i, f) for i, f in
                enumerate([0.02, 0.05, 0.08, 0.1, 0.12, 0.2] * 12)]
    # One azimuth but for a few points: nearly every pair degenerate.
    for i in range(8):
        t, v = (a.copy() for a in cluster(600, 600 + i, p_uniform=0.2))
        t[20:] = 0.4
        clusters.append((t, v))
    compare(rv, *frame_of(clusters), n_hyp, 0.15, 21, f"few finite points H={n_hyp}")
    compare(rv, *frame_of(clusters + [sparse(900000, 9, 0.06)]), n_hyp, 0.15, 22,
            f"few finite points, long H={n_hyp}")


@pytest.mark.parametrize("points", [1500, 20000])
def test_fp16_form_with_many_workgroups_per_cluster(rv, points):  # noqa: F811
    """16 (in the large workgroups 4) workgroups of a cluster share its best key."""
    import torch

    theta, vd, off = frame_of([cluster(points + 13 * i, 800 + i, p_uniform=0.3, p_band=0.2)
                               for i in range(24)])
    t, v, o = (torch.from_numpy(a).cuda() for a in (theta, vd, off))
    fo = torch.tensor([0, len(off) - 1], dtype=torch.int32, device="cuda")
    for seed in range(12):
        got = {}
        for fp16_min in (0, 512):
            tuning = rv.rv_tuning_default()
            tuning.fp16_min_points = fp16_min
            print(f"[gpu] fp16 workgroups points={points} seed={seed} fp16_min={fp16_min}", flush=True)
            out = rv.allocate_batch_outputs(1, len(off) - 1, len(theta), 4096, t.device, debug=True)
            del out["hyp_counts"]
            rv.rv_estimate_velocity_batch(t, v, o, fo, torch.tensor([seed], device="cuda"), 4096, 0.15,
                                          tuning=tuning, out=out)
            torch.cuda.synchronize()
            got[fp16_min] = {k: out[k].cpu().numpy() for k in KEYS if k in out}
        for k, x in got[0].items():
            assert np.array_equal(x.view(np.uint8), got[512][k].view(np.uint8)), (seed, k)
