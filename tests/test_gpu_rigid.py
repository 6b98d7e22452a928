"""Rigid planar bodies (the patchy colloids of Sec. 3.2) on the GPU: one body step
against the oracle, and a Langevin run that keeps the bodies rigid, the plane
and equipartition.  All calls go through the C ABI (rc_compute_forces,
rc_rigid_step)."""
import numpy as np
import pytest

import workloads as W
from oracle import rigid_ref, swap_ref

pytestmark = pytest.mark.gpu


_FRESH = r"""
import sys
sys.path.insert(0, {root!r})
import numpy as np
import workloads as W
s = W.patchy_mixture()                        # host-side set-up first, torch not imported yet
from paper_1912_08569_amd import System       # then the engine (it brings torch's HIP runtime first)
S = System.from_workload(s)
F, ev = S.compute_forces()
print("ok", s.N, bool(np.isfinite(F.cpu().numpy()).all()))
"""


def test_fresh_process_sets_up_the_workload_before_the_device():
    # a process that generates the patchy mixture before its first device use, with torch imported only by
    # the engine package (the order that once mapped two HIP runtimes and failed to bring up the device)
    import os
    import subprocess
    root = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
    print("fresh process: patchy_mixture, then System and compute_forces", flush=True)
    out = subprocess.run(["python", "-c", _FRESH.format(root=root)], capture_output=True, text=True, timeout=240)
    assert out.returncode == 0, out.stderr[-3000:]
    assert out.stdout.split()[0] == "ok" and out.stdout.split()[-1] == "True", out.stdout


def _bodies(s):
    from paper_1912_08569_amd import RigidBodies, System
    S = System.from_workload(s)
    return S, RigidBodies(S, s.meta["bodies"], s.meta["theta"], s.meta["omega"])


def _owner(b):
    return np.repeat(np.arange(len(b["centre"])), np.diff(b["first"]))


@pytest.mark.parametrize("kind", ["langevin", "nve"])
def test_rigid_step_matches_oracle(kind):
    s = W.patchy_mixture(seed=1014)
    S, R = _bodies(s)
    gamma = 1.0 if kind == "langevin" else 0.0
    cfg = S.integrator(kind=kind, dt=0.001, kT=1.0, gamma=gamma, seed=21, dim=2)
    S.build()
    x0, v0, _, ty = S.state_by_tag()
    th0, w0 = R.theta.cpu().numpy().copy(), R.omega.cpu().numpy().copy()
    R.run(1, cfg, step0=7)
    x1, v1, _, _ = S.state_by_tag()
    th1, w1 = R.theta.cpu().numpy(), R.omega.cpu().numpy()
    ref = rigid_ref.step(x0, v0, th0, w0, ty, s.meta["bodies"], s.box, s.table, s.mass, 0.001, 1.0, gamma, 21, 7)
    dx = np.abs(swap_ref.min_image(ref["pos"], x1.astype(np.float64), s.box))
    kx = int(np.argmax(np.max(dx, axis=1)))
    b = s.meta["bodies"]
    ob = int(np.searchsorted(b["first"], kx - len(b["centre"]), side="right") - 1) if kx >= len(b["centre"]) else kx
    assert dx.max() < 1e-5, (f"tag {kx} body {ob}: gpu {x1[kx]} oracle {ref['pos'][kx]} start {x0[kx]}; "
                             f"centre gpu {x1[ob]} oracle {ref['pos'][ob]} start {x0[ob]}; "
                             f"theta gpu {th1[ob]} oracle {ref['theta'][ob]} start {th0[ob]}; "
                             f"{int(np.sum(np.max(dx, axis=1) > 1e-5))} particles off")
    dv = np.abs(v1 - ref["vel"])
    k = int(np.argmax(np.max(dv / (1.0 + np.abs(ref["vel"])), axis=1)))
    nb = len(s.meta["bodies"]["centre"])
    assert np.all(dv <= 1e-4 * (1.0 + np.abs(ref["vel"]))), (
        f"tag {k} ({'centre' if k < nb else 'member'}): gpu {v1[k]} oracle {ref['vel'][k]} start {v0[k]}; "
        f"{int(np.sum(np.any(dv > 1e-4 * (1.0 + np.abs(ref['vel'])), axis=1)))} particles off")
    dth = np.abs(np.mod(th1 - ref["theta"] + np.pi, 2 * np.pi) - np.pi)
    assert dth.max() < 1e-5, dth.max()
    assert np.all(np.abs(w1 - ref["omega"]) <= 1e-4 * (1.0 + np.abs(ref["omega"])))
    assert np.all(x1[:, 2] == 0.0) and np.all(v1[:, 2] == 0.0)


def test_rigid_run_keeps_bodies_plane_and_temperature():
    # weak patches (eps 1) so that bonding heats little: equipartition of translation and rotation
    s = W.patchy_mixture(seed=1015, table=W.patchy_table(eps_patch=1.0))
    S, R = _bodies(s)
    cfg = S.integrator(dt=0.001, kT=1.0, gamma=1.0, seed=5, dim=2)
    out = R.run(3000, cfg)
    print(f"rigid patchy mixture: {3000 / out['seconds']:.0f} steps/s, {out['rebuilds']} rebuilds")
    assert out["rebuilds"] >= 1
    x, v, img, ty = S.state_by_tag()
    b = s.meta["bodies"]
    d = swap_ref.min_image(x[b["centre"][_owner(b)]].astype(np.float64), x[b["member"]].astype(np.float64),
                           s.box)
    assert np.allclose(np.linalg.norm(d[:, :2], axis=1), 0.5, atol=2e-5)
    assert np.all(x[:, 2] == 0.0) and np.all(v[:, 2] == 0.0)
    vc = v[b["centre"]].astype(np.float64)
    w = R.omega.cpu().numpy().astype(np.float64)
    kt_trans = float(np.mean(np.sum(vc[:, :2] ** 2, axis=1)) / 2.0)   # unit masses, two degrees of freedom
    kt_rot = float(np.mean(b["inertia"] * w ** 2))
    assert abs(kt_trans - 1.0) < 0.15 and abs(kt_rot - 1.0) < 0.2, (kt_trans, kt_rot)


def test_rigid_argument_errors():
    from paper_1912_08569_amd import RcError
    s = W.patchy_mixture(n_tri=40, n_di=60, L=12.5, seed=1016)
    S, R = _bodies(s)
    with pytest.raises(RcError):   # rigid planar bodies need dim 2
        R.run(1, S.integrator(dt=0.001, kT=1.0, gamma=1.0, seed=5, dim=3))


def _wheels(B, seed):
    """B bodies on a jittered lattice with 0 to 6 rim members each (more and fewer than four lanes hold)."""
    rng = np.random.default_rng(seed)
    arms = (np.arange(B) * 5 + 3) % 7
    first = np.concatenate([[0], np.cumsum(arms)]).astype(np.int32)
    own = np.repeat(np.arange(B), arms)
    side = max(4, int(np.ceil(np.sqrt(B))))
    L = (float(np.float32(1.6 * side)), float(np.float32(1.6 * side)), 8.0)
    cen = np.zeros((B, 3))
    at = np.arange(B)
    cen[:, 0] = (at % side + 0.5) * 1.6 - 0.5 * L[0] + rng.uniform(-0.1, 0.1, B)
    cen[:, 1] = (at // side + 0.5) * 1.6 - 0.5 * L[1] + rng.uniform(-0.1, 0.1, B)
    ang = 2.0 * np.pi * (np.arange(len(own)) - first[own]) / np.maximum(arms[own], 1)
    offset = (0.5 * np.stack([np.cos(ang), np.sin(ang)], axis=1)).astype(np.float32)
    bodies = dict(centre=np.arange(B, dtype=np.int32), first=first, offset=offset,
                  member=np.arange(B, B + len(own), dtype=np.int32), inertia=rng.uniform(0.1, 0.2, B).astype(np.float32))
    theta = rng.uniform(-3.0, 3.0, B).astype(np.float32)
    omega = (2.0 * rng.standard_normal(B)).astype(np.float32)
    pos = rigid_ref.place(np.concatenate([cen, np.zeros((len(own), 3))]), bodies, theta, np.array(L))
    types = np.concatenate([np.zeros(B, np.int32), np.full(len(own), 2, np.int32)])
    vel = np.zeros(pos.shape, np.float32)
    vel[:B, :2] = 2.0 * rng.standard_normal((B, 2))
    return bodies, theta, omega, pos.astype(np.float32), types, vel, L


@pytest.mark.parametrize("B", [1, 15, 17, 130])
def test_rigid_run_equals_single_half_steps(B):
    # the queued run (fused halves, device-side stop at a list build) against rc_rigid_step and
    # rc_compute_forces called one by one, bit for bit, over several rebuilds; the first step to the oracle
    from paper_1912_08569_amd import RigidBodies, System
    from paper_1912_08569_amd import _lib as rcl
    from paper_1912_08569_amd import api
    bodies, theta, omega, pos, types, vel, L = _wheels(B, 1017)
    print(f"case: B={B} N={len(pos)}", flush=True)
    table, steps, frac = W.patchy_table(), 60, 0.8

    def fresh():
        S = System(pos, types, L, table, vel=vel)
        S.build()
        return S, RigidBodies(S, bodies, theta, omega), S.integrator(dt=0.002, kT=1.0, gamma=1.0, seed=3, dim=2)

    S, R, cfg = fresh()
    x0, v0, _, ty = S.state_by_tag()
    R.run(1, cfg, step0=5)
    x1 = S.state_by_tag()[0]
    ref = rigid_ref.step(x0, v0, theta, omega, ty, bodies, S.edges, table, S.mass, 0.002, 1.0, 1.0, 3, 5)
    dx = np.abs(swap_ref.min_image(ref["pos"], x1.astype(np.float64), np.array(S.edges)))
    assert dx.max() < 1e-5, dx.max()

    S, R, cfg = fresh()
    got = R.run(steps, cfg, step0=5, soft_frac=frac)
    T, Q, cfg = fresh()
    T.compute_forces(gather=True, ev=False)
    builds = 0
    for k in range(steps):
        for half in (rcl.RC_HALF_FIRST, rcl.RC_HALF_SECOND):
            api.rc_rigid_step(T.ctx, T.pos, T.vel, T.force, T.image, T.rtag, Q.b, Q.theta, Q.omega, T.box, cfg,
                              5 + k, half, T.status)
            if half == rcl.RC_HALF_FIRST:
                if float(T.vel[:, 3].max()) > 0.5 * T.r_buff * frac:
                    T.build()
                    builds += 1
                T.compute_forces(gather=True, ev=False)
    assert got["rebuilds"] == builds >= 1
    for a, b in ((S.pos, T.pos), (S.vel, T.vel), (S.image, T.image), (R.theta, Q.theta), (R.omega, Q.omega),
                 (S.force, T.force)):
        assert bool((a == b).all())


def test_rigid_run_step_counts(monkeypatch):
    # a count that is no whole number is refused, a count past the library's is split, and a run split into
    # short calls equals one call, bit for bit
    from paper_1912_08569_amd import RigidBodies, System, api, rigid
    bodies, theta, omega, pos, types, vel, L = _wheels(17, 1018)

    def fresh():
        S = System(pos, types, L, W.patchy_table(), vel=vel)
        S.build()
        return S, RigidBodies(S, bodies, theta, omega), S.integrator(dt=0.002, kT=1.0, gamma=1.0, seed=3, dim=2)

    S, R, cfg = fresh()
    for bad in (2.0, 2.5, "3"):
        with pytest.raises(TypeError):
            R.run(bad, cfg)
    whole = R.run(np.int64(60), cfg)
    T, Q, cfg = fresh()
    monkeypatch.setattr(rigid, "_CALL_STEPS", 7)
    parts = Q.run(60, cfg)
    assert parts["rebuilds"] == whole["rebuilds"] >= 1
    for a, b in ((S.pos, T.pos), (S.vel, T.vel), (S.image, T.image), (R.theta, Q.theta), (R.omega, Q.omega),
                 (S.force, T.force)):
        assert bool((a == b).all())
    monkeypatch.undo()
    asked = []
    monkeypatch.setattr(api, "rc_rigid_run", lambda *a: (asked.append((a[13], a[14])), (0, a[14]))[1])
    R.run(2 ** 31 + 5, cfg, step0=3)
    assert max(n for _, n in asked) < 2 ** 31 and sum(n for _, n in asked) == 2 ** 31 + 5
    assert [s for s, _ in asked] == list(range(3, 3 + 2 ** 31 + 5, asked[0][1]))
