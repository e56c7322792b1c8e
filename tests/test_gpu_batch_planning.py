"""Both ways of ordering a batch's clusters (beside the staging up to 1024 clusters
and frames, by a scatter launch above) on the GPU: every cluster's outputs equal,
bit for bit, those of its frame alone.  Tolerance: none."""
from __future__ import annotations

import numpy as np
import pytest

from test_gpu_pruned import KEYS, cluster, frame_of, rv  # noqa: F401 (fixture)

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("frames,clusters", [(1, 1), (1, 1023), (1, 1024), (1, 1025), (3, 1024),
                                             (300, 255), (1023, 900), (1024, 1024), (1025, 1000),
                                             (1030, 1100)])
def test_batch_equals_its_frames(rv, frames, clusters):  # noqa: F811
    import torch

    rng = np.random.default_rng(clusters * 7 + frames)
    sizes = rng.choice([0, 1, 2, 3, 17, 64, 65, 130, 300, 1100], clusters,
                       p=[.05, .05, .1, .2, .2, .1, .1, .1, .09, .01])
    pool = {n: cluster(max(n, 1), 50 + n, p_uniform=0.2) for n in set(sizes.tolist())}
    theta, vd, off = frame_of([tuple(a[:n] for a in pool[n]) for n in sizes.tolist()])
    if clusters > 500:
        off[100] = off[99] - 1  # clusters 98 and 99: one short span, one that ends before it starts
    # Frames of random lengths, some empty.
    fo = np.concatenate([[0], np.sort(rng.integers(0, clusters + 1, frames - 1)), [clusters]])
    t, v, o = (torch.from_numpy(a).cuda() for a in (theta, vd, off))
    f = torch.from_numpy(fo.astype(np.int32)).cuda()
    seeds = torch.arange(frames, dtype=torch.int64, device="cuda") * 1234567 + 5
    print(f"[gpu] batch planning F={frames} K={clusters}", flush=True)
    got = rv.rv_estimate_velocity_batch(t, v, o, f, seeds, 100, 0.15, want_bits=True, debug=True)
    torch.cuda.synchronize()
    got = {k: x.cpu().numpy() for k, x in got.items() if k in KEYS}
    busy = [i for i in range(frames) if fo[i + 1] > fo[i]]
    for i in busy if len(busy) < 40 else rng.choice(busy, 40, replace=False):
        a, b = int(fo[i]), int(fo[i + 1])
        # The whole point array with this frame's offsets, so that bad ones stay what they are.
        want = rv.rv_estimate_velocity(t, v, o[a:b + 1].contiguous(), 100, 0.15, int(seeds[i]),
                                       debug=True)
        torch.cuda.synchronize()
        for k in KEYS:
            if k in want and k != "inlier_bits":
                x, y = want[k].cpu().numpy(), got[k][a:b]
                assert np.array_equal(x.view(np.uint8), y.view(np.uint8)), (i, k)
