"""The tuner times each set of kernels once: a plan with the matrix-core flag is dropped
where the plan without it launches the same kernels (digits of 4 primes or more)."""
import pytest

import paper_2603_16692_amd as ks
from paper_2603_16692_amd import autotune

from test_autotune_cpu import FakeParams


@pytest.mark.parametrize("dnum,log_n,ell,top_ell,same", [
    (4, 16, 32, None, True), (8, 16, 32, None, True), (8, 16, 24, None, False), (2, 13, 6, None, False),
    (4, 16, 4, 32, True), (4, 16, 3, 32, False)])  # at level 3 ModUp has 3 sources, though P has 8
def test_flag_twins_are_dropped_from_four_sources_on(dnum, log_n, ell, top_ell, same):
    P = FakeParams(dnum, log_n, ell, top_ell)
    plans = autotune.candidate_plans(P, 8)
    kept = autotune.distinct_plans(P, plans)
    flagged = [p for p in plans if p.flags & ks.PLAN_MFMA_BCONV]
    assert flagged
    if same:
        assert [p.key() for p in kept] == [p.key() for p in plans if not p.flags & ks.PLAN_MFMA_BCONV]
        assert autotune.distinct_plans(P, flagged) == flagged  # nothing without the plan that stands for it
    else:
        assert kept == plans


def test_tune_enumerates_distinct_plans(monkeypatch):
    P, seen = FakeParams(4, 16, 32), []

    class Stop(Exception):
        pass

    def order(params, batch, plans, *a):
        seen.extend(plans)
        raise Stop

    monkeypatch.setattr(autotune, "prior_order", order)
    with pytest.raises(Stop):
        autotune.tune(P, None, None, 8)
    assert seen and not any(p.flags & ks.PLAN_MFMA_BCONV for p in seen)
