"""The growth class of rpm_stats: one timed interval per growth event, from the
differences of the iterates to the grown basis, results unchanged by the timing; a
solve that stops at a growth point leaves none behind."""
import numpy as np
import pytest
import torch

from paper_2003_07720_amd import binding as B
from paper_2003_07720_amd import microstructure as M

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("prec", ["fp64", "fp32"])
@pytest.mark.parametrize("max_iter", [40, 23])
def test_one_interval_per_event(prec, max_iter):
    """n_max = 6: growth at step 7 and every 7 after; 23 steps stop between events,
    at 40 the cap of 4 columns has ended growth."""
    shape = (12, 16, 18)
    ph = torch.from_numpy(M.random_phases(shape, 2, 4)).to("cuda")
    lt = np.array([B.lame_from_young(1.0, 0.3), B.lame_from_young(20.0, 0.3)])
    l0 = B.lame_from_young(20.0, 0.3)
    E = np.array([0.0, 0.0, 0.01, 0.0, 0.0, 0.0])
    kw = dict(precision=prec, tol=1e-30, n_max=6, p_max=4, refine=0, max_iter=max_iter)
    plain = B.fft_solve(ph, lt, l0, E, B.make_options(**kw))
    timed = B.fft_solve(ph, lt, l0, E, B.make_options(profile=1, **kw))
    only = B.fft_solve(ph, lt, l0, E, B.make_options(profile=1, profile_classes=1 << B.KERNEL_NAMES.index("growth"), **kw))
    for r in (timed, only):
        assert torch.equal(r["eps"], plain["eps"]) and r["growth_events"] == plain["growth_events"] > 0
        assert r["kernel_launches"]["growth"] == r["growth_events"] and r["kernel_ms"]["growth"] > 0
    assert all(only["kernel_launches"][c] == 0 for c in B.KERNEL_NAMES if c != "growth")
