"""GPU: the paper-literal variant's launches at the ends of their sizes: more trials than
a grid of 64 each has room for (a grid's threads stay below 2^32), and a frame-wide mask
far larger than its clusters' points.  Tolerance: none."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def rv():
    if not torch.cuda.is_available():
        pytest.skip("no GPU visible")
    from paper_2012_12618_amd import binding

    binding.load_library()
    return binding


def test_most_trials_of_many_clusters(rv):
    """1024 clusters with 2^20 trials each: 2^22 blocks of 256 trials, 2^24 of 64.  Two
    valid points make one line whatever the trial, so the first valid trial is kept."""
    K, H = 1024, 1 << 20
    theta = torch.tensor([0.1, 0.5] * K, dtype=torch.float32, device="cuda")
    vd = torch.linspace(-5, 5, 2 * K, device="cuda")
    off = torch.arange(0, 2 * K + 1, 2, dtype=torch.int32, device="cuda")
    print("[gpu] paper variant, 1024 clusters of 2 points, 2^20 trials", flush=True)
    got = rv.rv_estimate_velocity_paper(theta, vd, off, H, 3, want_bits=True)
    few = rv.rv_estimate_velocity_paper(theta, vd, off, 300, 3, want_bits=True)
    torch.cuda.synchronize()
    for k in ("vx", "vy", "heading", "n_inliers", "status", "inlier_bits"):
        assert torch.equal(got[k], few[k]), k
    assert int(got["status"].max()) == 0


@pytest.mark.parametrize("points", [31, 4096, 40_000_000])
def test_mask_beyond_the_clusters_points(rv, points):
    """Every word of the mask is cleared, also those of points in no cluster."""
    theta = torch.zeros(points, device="cuda")
    vd = torch.zeros(points, device="cuda")
    theta[:20] = torch.linspace(-1, 1, 20)
    vd[:20] = 3 * torch.cos(theta[:20])
    off = torch.tensor([0, 20], dtype=torch.int32, device="cuda")
    print(f"[gpu] paper variant, mask of {points} points", flush=True)
    out = rv.allocate_paper_outputs(1, points, 100, theta.device, want_bits=True)
    out["inlier_bits"].fill_(-1)
    rv.rv_estimate_velocity_paper(theta, vd, off, 100, 3, out=out)
    torch.cuda.synchronize()
    bits = out["inlier_bits"]
    assert bin(int(bits[0]) & 0xFFFFFFFF).count("1") == int(out["n_inliers"][0])
    assert int(bits[0]) >> 20 == 0 and int(bits[1:].ne(0).sum()) == 0
