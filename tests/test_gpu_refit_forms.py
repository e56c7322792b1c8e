"""The forms of the refit on the GPU: a cluster is refit by a wave, by a workgroup
of the refit kernel or by its scoring workgroup, by its size and the number of
clusters in the frame.  A cluster's result depends on its id, points and seed
alone, so the same leading clusters are run in frames of different lengths.

Tolerance: whole numbers, status and mask bits equal.  The float64 sums of the two
forms differ in order, which moves a velocity by a few 2^-53 times the solve's
condition number, far below half a float32 step: equal float32 values, or
neighbours where a value lies at a rounding boundary (2^-23 of it, heading too)."""
from __future__ import annotations

import numpy as np
import pytest

from test_gpu_pruned import KEYS, cluster, frame_of, rv  # noqa: F401 (fixture)

pytestmark = pytest.mark.gpu

SIZES = (2, 63, 64, 65, 255, 256, 257, 511, 1023, 1024, 1025, 1100, 3000, 1, 0)


def estimate(rv, theta, vd, off, n_hyp):  # noqa: F811
    import torch

    t, v, o = (torch.from_numpy(np.ascontiguousarray(a)).cuda() for a in (theta, vd, off))
    out = rv.allocate_outputs(len(off) - 1, len(theta), n_hyp, t.device, want_bits=True, debug=True)
    del out["hyp_counts"]
    rv.rv_estimate_velocity(t, v, o, n_hyp, 0.15, 11, out=out)
    torch.cuda.synchronize()
    return {k: out[k].cpu().numpy() for k in KEYS if k in out}


@pytest.mark.parametrize("n_hyp", [64, 512, 1024, 1025])
def test_frames_of_few_and_many_clusters(rv, n_hyp):  # noqa: F811
    lead = [cluster(max(n, 1), 700 + i, p_uniform=0.2, p_band=0.1) for i, n in enumerate(SIZES)]
    lead = [(t[:n], v[:n]) for (t, v), n in zip(lead, SIZES)]
    L, points = len(lead), sum(SIZES)
    want = estimate(rv, *frame_of(lead), n_hyp)
    for total in (2047, 2048, 2300):
        print(f"[gpu] refit forms: K={total} H={n_hyp}", flush=True)
        filler = [cluster(5, 1, p_uniform=0.0)] * (total - L)
        got = estimate(rv, *frame_of(lead + filler), n_hyp)
        for k in want:
            if k == "inlier_bits":
                a, b = (np.unpackbits(x[k].view(np.uint8), bitorder="little")[:points]
                        for x in (want, got))
                assert np.array_equal(a, b), (total, k)
            elif want[k].dtype == np.float32:
                np.testing.assert_allclose(got[k][:L], want[k], rtol=2.0 ** -23, atol=0,
                                           equal_nan=True, err_msg=f"K={total} {k}")
            else:
                np.testing.assert_array_equal(got[k][:L], want[k], err_msg=f"K={total} {k}")
