"""GPU: the paper-literal variant with more trials than a grid of 64 each has room for (a
grid's threads stay below 2^32).  Tolerance: none."""
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
