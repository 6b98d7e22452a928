"""Calls on a stream other than the current one: what they allocate belongs to that stream, and the results are the
same as on the current one."""
import numpy as np
import pytest
import torch

import workloads as W
from paper_1912_08569_amd import System, _lib as rcl, api

pytestmark = pytest.mark.gpu


@pytest.fixture()
def system():
    S = System.from_workload(W.small_reactive(N=1000, density=0.2, seed=9))
    S.build()
    return S


CALLS = {
    # 6000 rows and 700 lags: the form of the autocorrelation that takes scratch
    "stress": lambda S, x, stream: api.rc_stress_autocorrelation(S.ctx, x["rows"], 900.0, 1.0, 700, x["G"],
                                                                 stream=stream) or x["G"],
    "to_tags": lambda S, x, stream: api.rc_to_tags(S.ctx, S.pos, S.rtag, stream=stream),
    "from_tags": lambda S, x, stream: api.rc_from_tags(S.ctx, x["v"], S.pos, stream=stream),
    "normals": lambda S, x, stream: api.rc_thermostat_normals(3, 0, 2, 1000, stream=stream),
}


@pytest.mark.parametrize("name", sorted(CALLS))
def test_side_stream(system, name, monkeypatch):
    S = system
    rng = np.random.default_rng(2)
    x = dict(rows=torch.from_numpy(rng.standard_normal((6000, 13))).cuda(),
             G=torch.zeros(701, dtype=torch.float64, device="cuda"),
             v=torch.from_numpy(rng.standard_normal((S.N, 3)).astype(np.float32)).cuda())
    want = CALLS[name](S, x, None).clone()
    side = torch.cuda.Stream()
    made = []
    for fn in ("empty", "empty_like"):
        real = getattr(torch, fn)
        monkeypatch.setattr(torch, fn, lambda *a, _real=real, **k: (made.append(torch.cuda.current_stream()),
                                                                    _real(*a, **k))[1])
    side.wait_stream(torch.cuda.current_stream())
    got = CALLS[name](S, x, side)
    monkeypatch.undo()
    torch.cuda.current_stream().wait_stream(side)
    assert made and all(s == side for s in made)
    assert torch.equal(got, want)
    torch.cuda.synchronize()


def test_moved_flag_is_the_last_loads(system):
    """rc_load_moved answers for the context's last load, whatever other calls did to the words and events that they
    share, and refuses a context that made none."""
    S = system
    cfg = S.integrator(dt=0.001, kT=0.1, gamma=1.0, seed=4)
    S.run(4, cfg)
    with pytest.raises(api.RcError) as e:
        api.rc_load_moved(S.ctx)
    assert e.value.code == rcl.RC_ERR_ARG
    # a load that has not begun, and a status read on another stream meanwhile
    pos = S.pos.clone()
    ref = api.rc_to_tags(S.ctx, pos, S.rtag)
    far = ref + 0.5
    side = torch.cuda.Stream()
    side.wait_stream(torch.cuda.current_stream())
    with torch.cuda.stream(side):
        torch.cuda._sleep(100_000_000)       # some tens of milliseconds
        api.rc_load_by_tag(S.ctx, pos, far, ref, S.box, 0.1)
    S.run(4, cfg, step0=4)
    assert not side.query()                  # the load is still to come
    assert api.rc_load_moved(S.ctx) is True
    assert api.rc_load_moved(S.ctx) is True
    torch.cuda.synchronize()


def test_moved_flag_after_a_run_of_rigid_bodies():
    from paper_1912_08569_amd import RigidBodies
    s = W.patchy_mixture(seed=1014)
    S = System.from_workload(s)
    R = RigidBodies(S, s.meta["bodies"], s.meta["theta"], s.meta["omega"])
    S.build()
    x = api.rc_to_tags(S.ctx, S.pos, S.rtag)
    api.rc_load_by_tag(S.ctx, S.pos, x, x, S.box, 0.1)
    R.run(1, S.integrator(dt=0.001, kT=1.0, gamma=1.0, seed=21, dim=2))
    assert api.rc_load_moved(S.ctx) is False
