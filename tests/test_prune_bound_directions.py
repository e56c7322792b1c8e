"""CPU: the bound of test_prune_bound with the 32 direction bins that the large
workgroups of long clusters use (narrower bins: less slack beside the rounding of
the direction key).  No tolerance: one point outside its window fails."""
import pytest

import test_prune_bound as bound


@pytest.mark.parametrize("seed", range(36))
def test_every_inlier_is_inside_its_window(seed, monkeypatch):
    monkeypatch.setattr(bound, "BINS", 32)
    theta, vd, hyps, r, tau = bound.case(seed)
    assert bound.outside(theta, vd, hyps, r, tau, seed) == 0
