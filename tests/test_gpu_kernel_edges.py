"""Kernels at the sizes where their tiling can go wrong (edges of tiles, remainders, the smallest and
the largest of a range), against the FP64 oracle or the general path of the same quantity."""
import numpy as np
import pytest
import torch

import workloads as W
from oracle import observables_ref

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("T,max_lag", [(1, 0), (2, 1), (300, 255), (2047, 256), (2049, 2048), (4111, 287),
                                       (6200, 4096), (6145, 6144)])
def test_stress_autocorrelation_tiles(T, max_lag):
    # tiles of 2048 origins and 16 or 32 lags; a row whose stress is not a number reaches exactly the
    # lags that read it.  Both sides add n = 3 (T - t) products in FP64: |difference| <= 2 n u sum |products|
    from paper_1912_08569_amd import System
    S = System.from_workload(W.small_reactive(N=300, density=0.2, seed=1))
    V = float(S.edges[0]) ** 3
    rng = np.random.default_rng(T)
    rows = rng.standard_normal((T, 13)) * 50.0
    bad = T - 1 if T > 100 else None
    if bad is not None:
        rows[bad, 5] = np.nan
    G = S.stress_autocorrelation(rows, 0.7, max_lag)
    s = observables_ref.shear_stress(rows, V)
    for t in sorted({0, 1, 15, 16, 31, 32, max_lag // 2, max_lag - 1, max_lag} & set(range(max_lag + 1))):
        p = s[:T - t] * s[t:]
        ref = V / 0.7 * p.sum() / (3 * (T - t))
        if np.isnan(ref):
            assert np.isnan(G[t])
        else:
            n = 3 * (T - t)
            assert abs(G[t] - ref) <= 2 * (n + 8) * 2.0 ** -53 * V / 0.7 * np.abs(p).sum() / n, (t, G[t], ref)


@pytest.mark.parametrize("T,max_lag", [(300, 256), (2049, 2048), (4111, 287), (9000, 1000)])
def test_stress_autocorrelation_without_scratch(T, max_lag):
    # the form that reads the rows (no scratch given) against the one with scratch: the same products in another
    # order, |difference| <= 2 n u sum |products|; a scratch of the wrong size is refused
    from paper_1912_08569_amd import System, api
    from paper_1912_08569_amd import _lib as rcl
    S = System.from_workload(W.small_reactive(N=300, density=0.2, seed=1))
    V = float(S.edges[0]) ** 3
    r = torch.from_numpy(np.random.default_rng(T).standard_normal((T, 13)) * 50.0).cuda()
    G, H = (torch.empty(max_lag + 1, dtype=torch.float64, device="cuda") for _ in range(2))
    api.rc_stress_autocorrelation(S.ctx, r, V, 0.7, max_lag, G)
    args = (S.ctx.handle, api._ptr(r), T, V, 0.7, max_lag, api._ptr(H))
    assert rcl.load().rc_stress_autocorrelation(*args, api._stream()) == rcl.RC_OK
    s = torch.from_numpy(np.abs(observables_ref.shear_stress(r.cpu().numpy(), V)))
    t = torch.arange(max_lag + 1)
    size = torch.stack([(s[:T - k] * s[k:]).sum() for k in t.tolist()]) * V / 0.7 / (3 * (T - t))
    bound = 2 * (3 * (T - t) + 8) * 2.0 ** -53 * size
    assert bool(((G - H).abs().cpu() <= bound).all())
    assert rcl.load().rc_stress_autocorrelation_ws(*args, api._ptr(r), 8, api._stream()) == rcl.RC_ERR_WORKSPACE


@pytest.mark.parametrize("T,max_lag,plain", [
    (1000, 256, True), (2000, 400, True), (5000, 511, True), (5001, 511, False), (5000, 512, False),
    (3333, 767, True), (3334, 767, False), (10001, 255, True), (40, 30, True)])
def test_stress_autocorrelation_of_short_series(T, max_lag, plain, monkeypatch):
    # a block per lag (no scratch is made) or tiles of lags, at the limits of rows times groups of 256 lags; FP64
    # sums of n = 3 (T - t) products in another order: |difference| <= 2 n u sum |products|
    from paper_1912_08569_amd import System
    S = System.from_workload(W.small_reactive(N=300, density=0.2, seed=1))
    V = float(S.edges[0]) ** 3
    rows = np.random.default_rng(T).standard_normal((T, 13)) * 50.0
    made, real = [], torch.empty
    monkeypatch.setattr(torch, "empty", lambda *a, **k: (made.append(k.get("dtype")), real(*a, **k))[1])
    G = S.stress_autocorrelation(rows, 0.7, max_lag)
    assert (torch.uint8 in made) is not plain
    s = observables_ref.shear_stress(rows, V)
    for t in range(max_lag + 1):
        p, n = s[:T - t] * s[t:], 3 * (T - t)
        assert abs(G[t] - V / 0.7 * p.sum() / n) <= 2 * (n + 8) * 2.0 ** -53 * V / 0.7 * np.abs(p).sum() / n, t


@pytest.mark.parametrize("nvec", [33, 65])
def test_hvp_vectors_per_thread(nvec):
    # two and four vectors per thread with one vector left over, a ragged last block, several types: each
    # product equals the single product (one vector per thread) bit for bit
    from paper_1912_08569_amd import System
    S = System.from_workload(W.unequal_lambda_mixture(N=8195))
    S.build()
    gen = torch.Generator().manual_seed(nvec)
    V = torch.randn((nvec, S.N, 4), generator=gen).to(S.device)
    H = S.hvp_batch(V)
    for k in (0, 1, nvec // 2, nvec - 2, nvec - 1):
        assert torch.equal(H[k], S.hvp(V[k])), k


@pytest.mark.parametrize("N,density,gather", [
    (90, 0.05, False), (90, 0.05, True), (90, 0.05, "sums"), (2003, 0.6, False), (4097, 0.25, False),
    (32768, 0.25, True), (32769, 0.25, True), (65537, 0.25, True), (65537, 0.25, "sums")])
def test_forces_per_wavefront(N, density, gather):
    # gather: 8, 16 and 32 particles per wavefront and their limits; triplet kernel: partner pools that
    # hold the wavefront's swap ranges and (density 0.6) that do not; ragged last wavefronts
    from oracle import swap_ref
    from paper_1912_08569_amd import System
    from parity_util import assert_energy, assert_forces, assert_pe, assert_virial
    s = W.small_reactive(N=N, density=density, seed=N, min_dist=0.85)
    S = System.from_workload(s)
    F, ev = S.compute_forces(gather=gather)
    x, _, _, ty = S.state_by_tag()
    ref = swap_ref.evaluate(x, ty, s.L, s.table)
    F = S.by_tag(F)
    assert_forces(F, ref)
    assert_pe(F[:, 3], ref)
    assert_energy(float(ev[0]), ref)
    assert_virial(ev[1:7].cpu().numpy(), ref)


@pytest.mark.parametrize("N,density", [(65535, 0.25), (65536, 0.25), (65601, 0.25), (65537, 0.6)])
def test_triplet_kernel_sends_partner_forces(N, density):
    # partners' forces sent one by one (below 65536 particles) and a row at a time: ragged last wavefronts,
    # swap ranges that fit the pools and (density 0.6) do not, adding to what is there
    from oracle import swap_ref
    from paper_1912_08569_amd import System, api
    from paper_1912_08569_amd import _lib as rcl
    from parity_util import assert_energy, assert_forces, assert_pe, assert_virial
    s = W.small_reactive(N=N, density=density, seed=N, min_dist=0.85)
    S = System.from_workload(s)
    F, ev = S.compute_forces(gather=False)
    x, _, _, ty = S.state_by_tag()
    ref = swap_ref.evaluate(x, ty, s.L, s.table)
    f = S.by_tag(F)
    assert_forces(f, ref)
    assert_pe(f[:, 3], ref)
    assert_energy(float(ev[0]), ref)
    assert_virial(ev[1:7].cpu().numpy(), ref)
    A = F.clone()
    api.rc_compute_forces(S.ctx, S.pos, S.nlist, S.nn, S.box, A, None, rcl.RC_FORCE_ACCUMULATE, S.status)
    assert_forces(S.by_tag(A * 0.5), ref)


def _step_system(name):
    kind, n = name.split("-")
    n = int(n)
    if kind == "dumbbells":
        return W.dumbbell_mixture(N=n, seed=n)
    if kind == "assembly":
        return W.assembly_mixture(N=n, seed=n)
    if kind == "reactive":
        return W.small_reactive(N=n, density=0.25, seed=n, min_dist=0.95)
    return W.vitrimer_network(n_chains=n, n_dimers=3, seed=n)


@pytest.mark.parametrize("form", ["walk", "sums"])
@pytest.mark.parametrize("name", ["dumbbells-70", "dumbbells-511", "dumbbells-512", "dumbbells-513", "dumbbells-1024",
                                  "dumbbells-1025", "assembly-333", "assembly-20001", "reactive-100", "reactive-700",
                                  "reactive-20481", "reactive-41000", "network-9", "network-300"])
def test_few_particles_per_wavefront_equal_64(name, form):
    # plain steps of small systems (8, 16 or 32 particles per wavefront, the one-workgroup replays, springs)
    # against the same steps taken as log steps, which always run 64 particles per wavefront: bit for bit,
    # in the plain and the graph replayed form
    from paper_1912_08569_amd import System
    s = _step_system(name)
    dt = 2e-4 if name.startswith("network") else 0.001
    out = []
    for period, graph in ((1, False), (0, False), (0, True)):
        S = System.from_workload(s, step_form=form)
        cfg = S.integrator(dt=dt, kT=0.05, gamma=1.0, seed=11)
        S.run(50, cfg, log_period=period, use_graph=graph, max_chunk=18, adapt=False)
        out.append((S.pos.clone(), S.vel.clone(), S.image.clone()))
    for other in out[1:]:
        assert all(torch.equal(a.view(torch.int32), b.view(torch.int32)) for a, b in zip(out[0], other))


@pytest.mark.parametrize("N,cells", [(1, 3), (63, 3), (64, 4), (65, 3), (700, 5), (72000, 17), (72001, 16), (72003, 17)])
def test_list_holds_every_pair_once(N, cells):
    # the list of both kernels (few particles per wavefront up to 72000) against a k-d tree: odd and even
    # numbers of cells (an even last cell's right neighbour wraps), three cells an edge, partly filled blocks,
    # empty and crowded cells; the state and rtag it leaves, and a second build of the same state
    from scipy.spatial import cKDTree
    from paper_1912_08569_amd import System
    rng = np.random.default_rng(N)
    t = W.PairTable.empty(2)
    t.set(0, 0, W.KIND_SWAP, 1.0, 1.0, 10, 1.5, 1.0)
    t.set(0, 1, W.KIND_WCA, 1.0, 0.9, 6)
    L = [float(np.float32(1.8 * 1.01 * c)) for c in (cells, cells + 1, cells)]
    pos = (rng.uniform(-0.5, 0.5, (N, 3)) * L).astype(np.float32)
    pos[: N // 10] = (0.3 * pos[: N // 10]).astype(np.float32)
    types = (rng.random(N) < 0.3).astype(np.int32)
    print(f"case: N={N} cells={cells}", flush=True)
    S = System(pos, types, L, t, vel=rng.standard_normal((N, 3)).astype(np.float32), k_max=500)
    v0 = S.vel[:, :3].cpu().numpy().copy()
    S.build()
    x, _, tags = S.pos[:, :3].cpu().numpy(), None, (S.pos[:, 3].view(torch.int32) >> 4).cpu().numpy()
    assert np.array_equal(x, pos[tags]) and np.array_equal(S.vel[:, :3].cpu().numpy(), v0[tags])
    assert np.array_equal(S.rtag.cpu().numpy()[tags], np.arange(N)) and bool((S.vel[:, 3] == 0).all())
    nn = S.nn.cpu().numpy()
    ns, no = nn & 0xFFFF, nn >> 16
    nl = S.nlist.cpu().numpy().reshape(-1, N)
    ty = types[tags]
    edge = np.array(L)
    tree = cKDTree(np.mod(x.astype(np.float64) + 0.5 * edge, edge), boxsize=edge)
    r_wca = 0.9 * 2.0 ** (1.0 / 6.0) + 0.3
    P = tree.query_pairs(1.8, output_type="ndarray")
    d = x[P[:, 1]].astype(np.float64) - x[P[:, 0]]
    d -= edge * np.round(d / edge)
    r = np.sqrt((d * d).sum(axis=1))
    kind = ty[P[:, 0]] + ty[P[:, 1]]               # 0 swap, 1 WCA, 2 none
    lim = np.where(kind == 0, 1.8, np.where(kind == 1, r_wca, 0.0))
    sure = P[(r < lim) & (kind < 2)]
    key = lambda a, b: a.astype(np.int64) * N + b  # noqa: E731
    want = np.concatenate([key(sure[:, 0], sure[:, 1]), key(sure[:, 1], sure[:, 0])])
    k = np.arange(nl.shape[0])[:, None]
    swap, other = k < ns[None], k >= nl.shape[0] - no[None]
    got = []
    for mask, is_swap in ((swap, True), (other, False)):
        s, i = np.nonzero(mask)
        j = nl[s, i]
        assert np.array_equal((ty[i] == 0) & (ty[j] == 0), np.full(len(i), is_swap))
        got.append(key(i, j))
    got = np.concatenate(got)
    assert len(np.unique(got)) == len(got)
    assert np.isin(want, got).all()
    extra = got[~np.isin(got, want)]               # the radius carries a 1e-5 margin
    i, j = extra // N, extra % N
    d = x[j].astype(np.float64) - x[i]
    d -= edge * np.round(d / edge)
    lim = np.where(ty[i] + ty[j] == 0, 1.8, r_wca) * (1.0 + 2e-5)
    assert np.all((ty[i] + ty[j] < 2) & (np.sqrt((d * d).sum(axis=1)) <= lim))
    first = (S.pos.clone(), S.nn.clone(), S.nlist.clone())
    S.build()
    assert all(torch.equal(a, b) for a, b in zip(first, (S.pos, S.nn, S.nlist)))


@pytest.mark.parametrize("N,grow", [(1100, 1.45), (3001, 1.6), (40953, 1.7), (81921, 1.7)])
def test_one_launch_of_the_two_pass_form_equals_two(N, grow):
    # a dense drop in a large box: short lists by the mean density, so the one-launch form runs, but rows of
    # entries past those it keeps in registers and swap ranges longer than a walk's first four slots; against
    # log steps, which take two launches, bit for bit
    from paper_1912_08569_amd import System
    s = W.small_reactive(N=N, density=0.3, seed=N, min_dist=0.95)
    L = float(np.float32(s.L * grow))
    print(f"case: N={N} grow={grow}", flush=True)
    out = []
    for period, graph in ((1, False), (0, False), (0, True)):
        S = System(s.pos, s.types, L, s.table, vel=s.vel, mass=s.mass, step_form="sums")
        cfg = S.integrator(dt=0.001, kT=0.1, gamma=1.0, seed=12)
        S.run(40, cfg, log_period=period, use_graph=graph, max_chunk=18, adapt=False)
        out.append((S.pos.clone(), S.vel.clone(), S.image.clone()))
    assert S.mean_swap_length() > 4.0
    for other in out[1:]:
        assert all(torch.equal(a.view(torch.int32), b.view(torch.int32)) for a, b in zip(out[0], other))


@pytest.mark.parametrize("N,kind", [(40, "pair"), (512, "drop"), (600, "drop"), (1024, "mix"), (512, "types")])
def test_one_workgroup_steps_equal_launched_ones(N, kind):
    # the one-workgroup form (rows of entries in registers, noise drawn a step ahead, any number of steps per
    # launch) against launches, bit for bit: one short row, wavefronts past the rows kept (a dense drop), two
    # rows and a half, a table that leaves no room for the staging; odd stretches between log rows
    from paper_1912_08569_amd import System
    if kind == "drop":
        s = W.small_reactive(N=N, density=0.3, seed=N, min_dist=0.95)
        L, types, table, mass = float(np.float32(s.L * 2.2)), s.types, s.table, s.mass
    else:
        s = W.dumbbell_mixture(N=N, seed=N)
        L, types, table, mass = s.L, s.types, s.table, s.mass
        if kind == "types":     # the same two species spread over 16 types
            types = (s.types + 2 * (np.arange(N) % 8)).astype(np.int32)
            table = W.PairTable.empty(16)
            for a in range(16):
                for b in range(a, 16):
                    p, q = a % 2, b % 2
                    table.set(a, b, int(s.table.kind[p, q]), s.table.epsilon[p, q], s.table.sigma[p, q],
                              int(s.table.n[p, q]), s.table.rcut[p, q], s.table.lam[p, q])
            mass = np.ones(16)
    print(f"case: N={N} {kind}", flush=True)
    out = []
    for one in (False, True):
        S = System(s.pos, types, L, table, vel=s.vel, mass=mass, step_form="sums")
        cfg = S.integrator(dt=0.001, kT=0.05, gamma=1.0, seed=13)
        for k, n in enumerate((37, 1, 90)):
            r = S.run(n, cfg, step0=(0, 37, 38)[k], log_period=17, one_block=one, max_chunk=29, adapt=False)
            out.append((S.pos.clone(), S.vel.clone(), S.image.clone(), torch.from_numpy(r.ev.copy())))
    for a, b in zip(out[:3], out[3:]):
        assert all(torch.equal(x, y) for x, y in zip(a, b))
