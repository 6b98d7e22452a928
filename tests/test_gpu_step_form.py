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


@pytest.mark.parametrize("name", ["reactive-1000", "reactive-20481", "reactive-81921", "assembly-5003", "network-300"])
def test_kernels_chosen_by_list_length_give_the_same_step(name):
    # one step by every kernel that a list length can choose (64, 32, 16 and 8 particles per wavefront, the two-pass
    # form in one launch), Langevin and NVE, bit for bit; the length is a hint, so wrong ones have to do as well
    import torch
    from test_gpu_kernel_edges import _step_system
    from paper_1912_08569_amd import _lib as rcl, api
    s = _step_system(name)
    for form in ("walk", "sums"):
        S = System.from_workload(s, step_form=form)
        for kind in ("langevin", "nve"):
            cfg = S.integrator(kind=kind, dt=2e-4, kT=0.1, gamma=1.0, seed=6)
            S.build()
            x0, v0, im0 = S.pos.clone(), S.vel.clone(), S.image.clone()
            out = []
            for entries in (0.0, 1.0, 1.2, 2.0, 2.4, 3.0, 5.0, 50.0, -1.0):
                S.ctx.set_list_length(-1.0)
                S.ctx.set_list_length(entries)
                S.vel.copy_(v0)
                S.image.copy_(im0)
                S.pos_alt.fill_(float("nan"))
                for k, (a, b) in enumerate(((x0, S.pos_alt), (S.pos_alt, S.pos))):
                    api.rc_step_fused(S.ctx, a, b, S.vel, S.image, S.nlist, S.nn, S.box, cfg, 7 + k,
                                      rcl.RC_STEP_CONT if k else rcl.RC_STEP_START, status=S.status)
                out.append((S.pos.clone(), S.vel.clone(), S.image.clone()))
                S.pos.copy_(x0)
            S.vel.copy_(v0)
            S.image.copy_(im0)
            for other in out[1:]:
                assert all(torch.equal(a.view(torch.int32), b.view(torch.int32)) for a, b in zip(out[0], other))


def test_list_length_word():
    # the status word of all list entries, by the few-particle and the one-thread list kernels and batches, and
    # what it is refused for
    import numpy as np
    from paper_1912_08569_amd import Batch, RcError, _lib as rcl, api
    for N in (1, 900, 5000, 80001):
        s = W.small_reactive(N=N, density=0.25, seed=N, min_dist=0.9) if N > 1 else W.cluster([[0.0, 0.0, 0.0]])
        S = System.from_workload(s)
        S.build()
        _, st = api.rc_read_status(S.status)
        nn = S.nn.cpu().numpy()
        assert st[rcl.RC_ST_NLIST] == int(((nn & 0xFFFF) + (nn >> 16)).sum())
        assert st[rcl.RC_ST_NSWAP] == int((nn & 0xFFFF).sum())
    B = Batch([W.small_reactive(N=n, density=0.3, seed=n) for n in (300, 64, 5000)])
    B.build()
    _, st = api.rc_read_status(B.status)
    nn = B.nn.cpu().numpy()
    assert st[rcl.RC_ST_NLIST] == int(((nn & 0xFFFF) + (nn >> 16)).sum())
    with pytest.raises(RcError):
        S.ctx.set_list_length(float("nan"))
    S.ctx.set_list_length(float("inf"))
    S.ctx.set_list_length(np.float64(3.0))


@pytest.mark.parametrize("N", [1, 100, 6145, 12289, 24577, 32769, 65601])
def test_forces_by_list_length(N):
    # the gather kernel with 8, 16, 32 and 64 particles per wavefront, in blocks of one, two and four wavefronts
    # (energies from 768 on) and ragged last blocks: forces and per-particle energies bit for bit, sums in FP64 of
    # the same terms in another order (|difference| <= 2 N u sum |terms|), adding up or not, with a status word
    import torch
    from paper_1912_08569_amd import _lib as rcl, api
    s = W.small_reactive(N=N, density=0.25, seed=N, min_dist=0.9) if N > 1 else W.cluster([[0.0, 0.0, 0.0]])
    S = System.from_workload(s)
    S.build()
    for flag in (rcl.RC_FORCE_GATHER, rcl.RC_FORCE_SUMS):
        out = []
        for entries in (0.0, 1.0, 2.0, 5.0):
            S.ctx.set_list_length(-1.0)
            S.ctx.set_list_length(entries)
            F, ev = torch.full_like(S.force, float("nan")), torch.full((7,), float("nan"), dtype=torch.float64,
                                                                       device="cuda")
            api.rc_compute_forces(S.ctx, S.pos, S.nlist, S.nn, S.box, F, ev, flag, S.status)
            G = F.clone()
            api.rc_compute_forces(S.ctx, S.pos, S.nlist, S.nn, S.box, G, None, flag | rcl.RC_FORCE_ACCUMULATE,
                                  S.status)
            H, ew = torch.empty_like(F), torch.empty_like(ev)
            api.rc_compute_forces_noalloc(S.ctx, S.pos, S.nlist, S.nn, S.box, H, ew, flag, S.status)
            assert torch.equal(F[:, :3], H[:, :3]) and torch.equal(ev, ew)
            out.append((F[:, :3].clone(), G[:, :3].clone(), F[:, 3].double().clone(), ev.clone()))
        bound = 2.0 * N * 2.0 ** -53 * (float(out[0][2].abs().sum()) + 1.0) * 50.0    # virials: terms up to 50 times E's
        for o in out[1:]:
            assert torch.equal(o[0], out[0][0]) and torch.equal(o[1], out[0][1])
            assert bool(((o[3] - out[0][3]).abs() <= bound).all())


@pytest.mark.parametrize("name", ["reactive-2003", "reactive-65601", "dense-1000", "network-21", "network-300"])
def test_triplet_kernel_by_list_length(name):
    # entries of both kinds in flat passes and the kinds apart (lists named short and long), a lane's ordinary entries in
    # several rounds of four (the network's), ragged last wavefronts, pools that hold the swap ranges and do not
    from paper_1912_08569_amd import api
    from oracle import swap_ref
    from parity_util import assert_energy, assert_forces, assert_pe, assert_virial
    from test_gpu_kernel_edges import _step_system
    kind, n = name.split("-")
    s = W.small_reactive(N=int(n), density=0.6, seed=9, min_dist=0.85) if kind == "dense" else _step_system(name)
    S = System.from_workload(s)
    S.build()
    ns, no = S.nn.cpu() & 0xffff, S.nn.cpu() >> 16
    if kind == "network":
        assert int(no.max()) > 4
    elif kind == "dense":
        assert int(ns[:64].sum()) > 512
    x, _, _, ty = S.state_by_tag()
    ref = swap_ref.evaluate(x, ty, s.L, s.table)
    for entries in (0.5, 50.0):
        S.ctx.set_list_length(-1.0)
        S.ctx.set_list_length(entries)
        api.rc_compute_forces(S.ctx, S.pos, S.nlist, S.nn, S.box, S.force, S.ev, 0, S.status)   # without springs
        F = S.by_tag(S.force)
        assert_forces(F, ref)
        assert_pe(F[:, 3], ref)
        assert_energy(float(S.ev[0]), ref)
        assert_virial(S.ev[1:7].cpu().numpy(), ref)


@pytest.mark.parametrize("N,density", [(1, 0.01), (63, 0.05), (4099, 0.2), (30001, 0.05), (72003, 0.2), (140003, 0.3)])
def test_both_list_kernels_build_the_same_list(N, density):
    # lists named short and long choose the kernel where the density does not: one thread per particle and few
    # particles per wavefront, with and without a crowded corner, ragged last blocks; every word of the list alike
    import numpy as np
    import torch
    rng = np.random.default_rng(N)
    t = W.PairTable.empty(2)
    t.set(0, 0, W.KIND_SWAP, 1.0, 1.0, 10, 1.5, 1.0)
    t.set(0, 1, W.KIND_WCA, 1.0, 0.9, 6)
    L = max(6.0, float(np.float32((N / density) ** (1.0 / 3.0))))
    pos = (rng.uniform(-0.5, 0.5, (N, 3)) * L).astype(np.float32)
    pos[: N // 20] *= np.float32(0.5)
    types = (rng.random(N) < 0.3).astype(np.int32)
    out = []
    for entries in (0.0, 500.0):
        S = System(pos, types, L, t, vel=rng.standard_normal((N, 3)).astype(np.float32) * 0, k_max=200)
        S.ctx.set_list_length(entries)
        S.build()
        slots = torch.arange(S.nlist.numel() // N, device=S.nn.device)[:, None]
        live = (slots < (S.nn & 0xffff)) | (slots >= slots.numel() - (S.nn >> 16))
        out.append((S.pos.clone(), S.nn.clone(), torch.where(live, S.nlist.view(-1, N), -1), S.mean_list_length()))
    for a, b in zip(out[0][:3], out[1][:3]):
        assert torch.equal(a.view(torch.int32), b.view(torch.int32))
    assert out[0][3] == out[1][3]
