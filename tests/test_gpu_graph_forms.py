"""HIP graphs of the batched forms that other graph tests do not capture: a batch
ordered beside its staging, long clusters in large workgroups, the FP16 form without
per-hypothesis counts.  Every replay, with new points, new seeds and new cluster
borders in the captured buffers and eager work between, equals the eager call bit
for bit.  Tolerance: none."""
from __future__ import annotations

import numpy as np
import pytest

from test_gpu_pruned import KEYS, cluster, frame_of, rv  # noqa: F401 (fixture)

pytestmark = pytest.mark.gpu

FORMS = {
    "planned": ([3, 40, 130, 500, 1100, 0, 700] * 40, 500, 0),
    "planned fp16": ([3, 40, 130, 500, 1100, 0, 700] * 40, 500, 256),
    "long": ([30000, 9000, 64, 20000, 500], 1500, 0),
    "long fp16": ([30000, 9000, 64, 20000, 500], 1500, 1024),
    "scattered": ([5, 9, 60, 200] * 300, 300, 0),
}


@pytest.mark.parametrize("form", sorted(FORMS))
def test_replays_match_eager(rv, form):  # noqa: F811
    import torch

    sizes, n_hyp, fp16_min = FORMS[form]
    pool = {n: cluster(max(n, 1), 60 + n, p_uniform=0.2) for n in set(sizes)}
    theta, vd, off = frame_of([tuple(a[:n] for a in pool[n]) for n in sizes])
    K, N = len(sizes), len(theta)
    t, v, o = (torch.from_numpy(a).cuda() for a in (theta, vd, off))
    fo = torch.tensor([0, K // 3, K // 3, K], dtype=torch.int32, device="cuda")
    sd = torch.tensor([5, 6, 7], dtype=torch.int64, device="cuda")
    tuning = rv.rv_tuning_default()
    tuning.fp16_min_points = fp16_min
    outs = []
    for _ in range(2):
        out = rv.allocate_batch_outputs(3, K, N, n_hyp, t.device, want_bits=True, debug=True)
        del out["hyp_counts"]
        outs.append(out)
    eager, captured = outs
    graph = rv.rv_graph_capture_batch(t, v, o, fo, sd, n_hyp, 0.15, captured, tuning=tuning)
    try:
        for rep in range(4):
            if rep == 1:
                v.neg_()
            if rep == 2:
                sd.add_(9)
            if rep == 3:  # the last border but one moves: other sizes, another order
                o[K - 1] -= int(off[K - 1] - off[K - 2]) // 2
            rv.rv_estimate_velocity_batch(t, v, o, fo, sd, n_hyp, 0.15, tuning=tuning, out=eager)
            _ = torch.ones(1000, device="cuda").sum().item()
            torch.cuda.synchronize()
            print(f"[gpu] graph of the {form} form, replay {rep}", flush=True)
            graph.launch()
            torch.cuda.synchronize()
            for k in KEYS:
                if k in eager:
                    a, b = eager[k].cpu().numpy(), captured[k].cpu().numpy()
                    assert np.array_equal(a.view(np.uint8), b.view(np.uint8)), (rep, k)
    finally:
        graph.destroy()
