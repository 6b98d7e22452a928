"""Steps without a thermostat through every form of the driver, bit for bit."""
import numpy as np
import pytest
import torch

import workloads as W
from paper_1912_08569_amd import RigidBodies, System
from paper_1912_08569_amd import _lib as rcl, api

pytestmark = pytest.mark.gpu


def _same(a, b):
    assert all(torch.equal(x.view(torch.int32), y.view(torch.int32)) for x, y in zip(a, b))


@pytest.mark.parametrize("form", ["walk", "sums"])
@pytest.mark.parametrize("N,kind", [(40, "pair"), (513, "pair"), (1024, "pair"), (600, "drop")])
def test_one_workgroup_steps(N, kind, form):
    # rows in registers, entries in LDS and (a drop) read from the list, against launches
    s = W.dumbbell_mixture(N=N, seed=N) if kind == "pair" else W.small_reactive(N=N, density=0.3, seed=N, min_dist=0.95)
    L = s.L if kind == "pair" else float(np.float32(2.2 * s.L))
    out = []
    for one in (False, True):
        S = System(s.pos, s.types, L, s.table, vel=s.vel, mass=s.mass, step_form=form)
        cfg = S.integrator(kind="nve", dt=0.001)
        ev = [S.run(n, cfg, step0=k, log_period=17, one_block=one, max_chunk=29, adapt=False).ev.copy()
              for k, n in ((0, 37), (37, 1), (38, 90))]
        out.append((S.pos, S.vel, S.image, torch.from_numpy(np.concatenate(ev)).view(torch.int32)))
    _same(*out)


@pytest.mark.parametrize("name", ["drop-1100", "reactive-20481", "assembly-5003"])
def test_driver_forms(name):
    # a step per launch with its log row, queued and replayed stretches; 64 to 8 particles per wavefront and the
    # two-pass form in one launch, which the log steps do not take
    kind, N = name.split("-")
    N = int(N)
    s = W.assembly_mixture(N=N, seed=N) if kind == "assembly" else W.small_reactive(N=N, density=0.3, seed=N, min_dist=0.95)
    L = float(np.float32(s.L * (1.45 if kind == "drop" else 1.0)))
    for form in ("walk", "sums"):
        out = []
        for period, graph in ((1, False), (0, False), (0, True)):
            S = System(s.pos, s.types, L, s.table, vel=s.vel, mass=s.mass, step_form=form)
            S.run(40, S.integrator(kind="nve", dt=0.001), log_period=period, use_graph=graph, max_chunk=18, adapt=False)
            out.append((S.pos, S.vel, S.image))
        for other in out[1:]:
            _same(out[0], other)


@pytest.mark.parametrize("B", [1, 17, 130])
def test_rigid_run(B):
    # the queued run against single half steps, over rebuilds
    from test_gpu_rigid import _wheels
    bodies, theta, omega, pos, types, vel, L = _wheels(B, 1017)
    table, steps, frac = W.patchy_table(), 60, 0.8

    def fresh():
        S = System(pos, types, L, table, vel=vel)
        S.build()
        return S, RigidBodies(S, bodies, theta, omega), S.integrator(kind="nve", dt=0.002, dim=2)

    S, R, cfg = fresh()
    got = R.run(steps, cfg, step0=5, soft_frac=frac)
    T, Q, cfg = fresh()
    T.compute_forces(gather=True, ev=False)
    builds = 0
    for k in range(steps):
        for half in (rcl.RC_HALF_FIRST, rcl.RC_HALF_SECOND):
            api.rc_rigid_step(T.ctx, T.pos, T.vel, T.force, T.image, T.rtag, Q.b, Q.theta, Q.omega, T.box, cfg, 5 + k,
                              half, T.status)
            if half == rcl.RC_HALF_FIRST:
                if float(T.vel[:, 3].max()) > 0.5 * T.r_buff * frac:
                    T.build()
                    builds += 1
                T.compute_forces(gather=True, ev=False)
    assert got["rebuilds"] == builds >= 1
    for a, b in ((S.pos, T.pos), (S.vel, T.vel), (S.image, T.image), (R.theta, Q.theta), (R.omega, Q.omega),
                 (S.force, T.force)):
        assert bool((a == b).all())
