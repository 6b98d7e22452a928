"""The form of the fused step that a System is made with is the one its runs take."""
import pytest

import workloads as W
from paper_1912_08569_amd import System

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("form", ["walk", "sums"])
def test_system_is_made_in_its_form(form):
    s = W.small_reactive(N=5000, density=0.25, seed=3, min_dist=0.95)
    S = System.from_workload(s, step_form=form)
    assert S.ctx.step_form == form
    r = S.run(20, S.integrator(dt=0.001, kT=0.1, gamma=1.0, seed=1), time_kernels=True)
    assert (r.stats.sums_ms > 0.0) is (form == "sums")    # two launches a step, or one
    S.build()
    assert S.ctx.step_form == form
