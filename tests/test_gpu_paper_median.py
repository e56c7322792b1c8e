"""GPU: the paper-literal variant's medians (selected from a histogram) and trial
blocks where they can go wrong: thresholds, per-trial counts, kept trials and masks
bit for bit the FP64 oracle's (no tolerance: both sides evaluate the same FP64
expressions in the same order)."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")

pytestmark = pytest.mark.gpu


def _clusters():
    rng = np.random.default_rng(31)
    out = []
    for n in (2, 3, 255, 256, 257, 300, 700, 1025, 4095, 4096):
        th = rng.uniform(-1, 1, n)
        out.append((th, np.round(rng.normal(0, 1, n), 1)))                  # quantised Doppler
        out.append((th, np.where(rng.random(n) < 0.8, 2.5, rng.normal(0, 9, n))))  # one value
        out.append((th, 5.0 + rng.normal(0, 1e-6, n) + 40.0 * (rng.random(n) < 0.01)))
        v = rng.normal(0, 3, n)
        v[rng.random(n) < 0.5] = np.nan                                     # half take no part
        out.append((th, v))
    return out


@pytest.mark.parametrize("n_hyp,bits", [(1, True), (63, True), (64, True), (65, True), (300, True),
                                        (200, False)])
def test_equal_and_crowded_doppler_values(oracle_mod, n_hyp, bits):
    from paper_2012_12618_amd import binding as rv

    if not torch.cuda.is_available():
        pytest.skip("no GPU visible")
    clusters = _clusters()
    off = np.concatenate([[0], np.cumsum([len(t) for t, _ in clusters])]).astype(np.int32)
    theta = np.concatenate([t for t, _ in clusters]).astype(np.float32)
    vd = np.concatenate([v for _, v in clusters]).astype(np.float32)
    print(f"[gpu] paper variant, crowded Doppler values, H={n_hyp} bits={bits}", flush=True)
    r = rv.rv_estimate_velocity_paper(torch.from_numpy(theta).cuda(), torch.from_numpy(vd).cuda(),
                                      torch.from_numpy(off).cuda(), n_hyp, 9, want_bits=bits,
                                      debug=True)
    torch.cuda.synchronize()
    g = {k: x.cpu().numpy() for k, x in r.items()}
    o = oracle_mod.estimate_velocity_paper(theta, vd, off, n_hyp, 9, debug=True)
    assert np.array_equal(g["status"], o.status)
    assert np.array_equal(g["thresh"], o.thresh, equal_nan=True)
    assert np.array_equal(g["best_hyp"], o.best_hyp)
    assert np.array_equal(g["n_inliers"], o.n_inliers)
    assert np.array_equal(g["hyp_counts"].reshape(len(clusters), n_hyp), o.hyp_count)
    if bits:
        mask = np.unpackbits(g["inlier_bits"].view(np.uint8), bitorder="little")[:len(theta)]
        assert np.array_equal(mask.astype(bool), o.inlier_mask.astype(bool))
