// Forces, energy and virial of the swap potential; the fused MD step; bond
// counting.  gfx950, wave64.
//
// Notation: for a centre c and a swap partner a inside r_cut, w_ca =
// sqrt(Lambda_ca) vhat(r_ca) and w'_ca/r = sqrt(Lambda_ca) vhat'(r_ca)/r_ca,
// so that a triplet term is w_ca w_cb (eq. 3bp with
// Lambda_cab = sqrt(Lambda_ca Lambda_cb)).  d = x_a - x_c (minimum image).
//   force on partner a from (c; a, b):  -w'_ca/r_ca w_cb d_ca
//   force on the centre:                minus the sum of the two
#include <hip/hip_ext.h>

#include "rc_internal.h"
#include "rc_gather.h"
#include "rc_step.h"

namespace rc {

static inline int nblk(long n, int b) { return (int)((n + b - 1) / b); }

// ---------------------------------------------------------------------------
// atomic-free gather force kernel (RC_FORCE_GATHER)
// ---------------------------------------------------------------------------
// A wavefront owns OW particles: 64, or fewer where 64 would leave most of
// the chip without a wavefront (gather_owners).  A block is one wavefront, or
// NW of them where that leaves the row reduction fewer partial sums of energy
// and virial to read (gather_waves).
template <bool EV, bool BATCH, bool SF, int OW, int NW>
__global__ __launch_bounds__(kWave * NW) void k_forces_gather(ForceArgs a) {
    static_assert(!BATCH || (OW == kWave && NW == 1), "a batch chunk has 64 slots");
    extern __shared__ DevEntry s_tab[];
    const int blk = xcd_block(gridDim.x);
    Box box_r;
    int lim = a.N;
    if constexpr (BATCH) {
        const RepDesc& d = a.rep[a.chunk_rep[blk]];
        box_r = d.box;
        lim = d.off + d.n;
        load_table(s_tab, Table{a.tab.e + d.tab, a.tab.nt});
    } else {
        box_r = a.box;
        load_table(s_tab, a.tab);
    }
    const int lane = threadIdx.x & (kWave - 1), wv = NW > 1 ? (int)threadIdx.x / kWave : 0;
    const int m = (blk * NW + wv) * OW + lane;
    const bool live = lane < OW && m < lim;
    const float4 pm = live ? a.pos[m] : make_float4(0.f, 0.f, 0.f, 0.f);
    const int packed = live ? a.nn[m] : 0;
    Acc acc = {};
    const OneSystem sys{s_tab, a.tab.nt, box_r};
    wave_gather<EV, kDefaultWidth, SF, OneSystem, NW, false, 4, OW>(m - lane, live, pm, packed, a.pos, a.nlist, a.nn,
                                                                    a.k_max, a.N, sys, acc, a.ssum);
    if (live) {
        float4 f = make_float4(acc.fx, acc.fy, acc.fz, acc.e);
        if (a.accumulate) {
            const float4 o = a.force[m];
            f.x += o.x;
            f.y += o.y;
            f.z += o.z;
            f.w += o.w;
        }
        a.force[m] = f;
        if (a.status && !(isfinite(f.x) && isfinite(f.y) && isfinite(f.z)))
            atomicOr(&a.status[RC_ST_FLAGS], RC_FLAG_NONFINITE);
    }
    if constexpr (EV) {
        double v[7] = {acc.e, acc.w[0], acc.w[1], acc.w[2], acc.w[3], acc.w[4], acc.w[5]};
        double* row = a.ev_part + (size_t)blk * kEvWords;
        if constexpr (NW == 1) {
            wave_sum_store<7>(v, row);
        } else {   // the wavefronts' sums one after the other
            __shared__ double s_ev[NW][7];
            wave_sum_store<7>(v, s_ev[wv]);
            __syncthreads();
            if (threadIdx.x < 7) {
                double t = s_ev[0][threadIdx.x];
#pragma unroll
                for (int w = 1; w < NW; ++w) t += s_ev[w][threadIdx.x];
                row[threadIdx.x] = t;
            }
        }
    }
}

// ---------------------------------------------------------------------------
// triplet kernel (default of rc_compute_forces): one wavefront per block.
// The swap entries of its 64 centres are evaluated flat, two or eight per lane
// and pass as in wave_gather (a lane per centre evaluated its own before: the
// wavefront took its longest list's time), and every lane sums its centre's
// terms from LDS in slot order.  The ordinary entries, which need no sum over
// them, follow the same way in short lists (FLAT); else they stay with their
// centre's lane, four requested at a time and the first four on their way beside
// the swap partners: flat they took passes that short swap ranges leave no others
// for, 23.4 us against 14.5 at 4032 beads of the network (9.6 entries each, few
// of them swap) and 26.9 against 16.9 at 67200.  The active partners of centres
// with two or more of them are kept in an LDS pool; the wave then enumerates every (j<k)
// triplet of its 64 centres across its lanes for the energy and the virial,
// and adds up each partner's w of the others, which gives the force on it in
// one product.  It leaves with global atomics, or stays in LDS for a partner
// among the wavefront's own 64.  Those atomics bound the kernel: with the six
// of every triplet it took 142 us at 200003 particles of three types, 90 of
// them in the atomics (20 without any).  An instruction's atomics go out as one
// request per line they touch, so the centres' rows leave as 64 consecutive
// floats per instruction, and (SPREAD) the partners' rows by four lanes each: 71
// -> 60 us, and 1000003 of the assembly mixture, which has few partners, 88 -> 69
// per call.  The XCD-aware block order gained nothing on top.  The pool is filled
// while the entries are summed when the wavefront's swap ranges fit it, else in
// rounds by walks of the lists.
// ---------------------------------------------------------------------------
constexpr int kPool = 512;   // staged partners per wave and round

template <bool SPREAD, int PL, bool FLAT>
__global__ __launch_bounds__(kWave) void k_forces_triplet(ForceArgs a, int want_ev) {
    constexpr int W = PL * kWave, AH = 4;   // flat entries per pass, a lane's own entries requested at a time
    extern __shared__ DevEntry s_tab[];
    __shared__ int p_j[kPool];
    __shared__ float p_w[kPool], p_g[kPool], p_dx[kPool], p_dy[kPool], p_dz[kPool], p_s[kPool];
    __shared__ int l_pool[kWave], l_k[kWave], l_tri[kWave + 1], l_out;
    __shared__ float l_f[kWave][4];
    __shared__ int s_off[kWave], s_ns[FLAT ? kWave : 1], s_j[W];
    __shared__ unsigned char s_own[W];
    __shared__ float4 s_pos[kWave];
    __shared__ float s_c[8][W];   // phi'/r, phi, d, w, w'/r, 1 for an active swap partner
    load_table(s_tab, a.tab);
    const int nt = a.tab.nt;
    const int lane = threadIdx.x;
    const int i = blockIdx.x * kWave + lane;
    const bool live = i < a.N;
    float4 pi = live ? a.pos[i] : make_float4(0.f, 0.f, 0.f, 0.f);
    const int ti = ptype(pi.w);
    const int packed = live ? a.nn[i] : 0;
    const int ns = nn_swap(packed), cnt = FLAT ? ns + nn_other(packed) : ns, no = FLAT ? 0 : nn_other(packed);
    auto other = [&](int b, int (&j)[AH]) {   // the other range's entries from b on
#pragma unroll
        for (int u = 0; u < AH; ++u) j[u] = b + u < no ? a.nlist[(size_t)(a.k_max - 1 - (b + u)) * a.N + i] : i;
    };
    auto other_pos = [&](int b, const int (&j)[AH], float4 (&p)[AH]) {
#pragma unroll
        for (int u = 0; u < AH; ++u) p[u] = b + u < no ? a.pos[j[u]] : pi;
    };
    int oj[AH];
    float4 op[AH];
    if (!FLAT) other(0, oj);
    const int inc = wave_inclusive_scan(cnt), my_off = inc - cnt;
    const int T = __builtin_amdgcn_readlane(inc, kWave - 1);
    const int pinc = FLAT ? wave_inclusive_scan(ns) : inc, poff = pinc - ns;   // in the pool
    const bool fits = __builtin_amdgcn_readlane(pinc, kWave - 1) <= kPool;
    s_off[lane] = my_off;
    if (FLAT) s_ns[lane] = ns;
    s_pos[lane] = pi;
    float fx = 0.f, fy = 0.f, fz = 0.f, en = 0.f;
    float w6[6] = {0.f, 0.f, 0.f, 0.f, 0.f, 0.f};
    int nact = 0;
    auto add_pair = [&](float g, float phi, float dx, float dy, float dz) {
        fx += g * dx;
        fy += g * dy;
        fz += g * dz;
        en += 0.5f * phi;
        const float c = -0.5f * g;
        w6[0] += c * dx * dx; w6[1] += c * dy * dy; w6[2] += c * dz * dz;
        w6[3] += c * dx * dy; w6[4] += c * dx * dz; w6[5] += c * dy * dz;
    };
    __syncthreads();
    for (int base = 0; base < T; base += W) {
        const int lo = max(my_off, base) - base, hi = min(my_off + cnt, base + W) - base;
        for (int q = lo; q < hi; ++q) s_own[q] = (unsigned char)lane;
        __syncthreads();
        int own[PL], jj[PL];
        float4 pj[PL];
#pragma unroll
        for (int u = 0; u < PL; ++u) {
            const int e = base + u * kWave + lane;
            own[u] = -1;
            jj[u] = 0;
            if (e < T) {
                own[u] = s_own[e - base];
                int slot = e - s_off[own[u]];
                if (FLAT && slot >= s_ns[own[u]]) slot = a.k_max - 1 - (slot - s_ns[own[u]]);
                jj[u] = a.nlist[(size_t)slot * a.N + (i - lane) + own[u]];
            }
        }
        if (!FLAT && base == 0) other_pos(0, oj, op);   // on their way beside the swap partners
#pragma unroll
        for (int u = 0; u < PL; ++u) {
            pj[u] = pi;
            if (own[u] >= 0) {
                const unsigned lj = (unsigned)(jj[u] - (i - lane));
                if (lj < (unsigned)kWave) pj[u] = s_pos[lj];
                else pj[u] = a.pos[jj[u]];
            }
        }
#pragma unroll
        for (int u = 0; u < PL; ++u) {
            float c[8] = {0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f};
            if (own[u] >= 0) {
                const float4 po = s_pos[own[u]];
                const DevEntry& e = s_tab[ptype(po.w) * nt + ptype(pj[u].w)];
                if (e.kind != RC_KIND_NONE) {
                    const PairGeom pg = pair_geom<true>(po, pj[u], a.box, e);
                    if (pg.cut) {
                        pair_eval(e, pg.r2, c[1], c[0]);
                        c[2] = pg.dx;
                        c[3] = pg.dy;
                        c[4] = pg.dz;
                        if (e.kind == RC_KIND_SWAP) {
                            float v, v1r;
                            vhat_eval(e, pg.inside, pg.r2, v, v1r);
                            c[5] = e.sqrt_lam * v;
                            c[6] = e.sqrt_lam * v1r;
                            c[7] = 1.0f;
                        }
                    }
                }
            }
            s_j[u * kWave + lane] = jj[u];
#pragma unroll
            for (int q = 0; q < 8; ++q) s_c[q][u * kWave + lane] = c[q];
        }
        __syncthreads();
        for (int q = lo; q < hi; ++q) {
            const float dx = s_c[2][q], dy = s_c[3][q], dz = s_c[4][q];
            add_pair(s_c[0][q], s_c[1][q], dx, dy, dz);
            if (s_c[7][q] != 0.0f) {
                if (fits) {
                    const int at = poff + nact;   // at most ns active partners
                    p_j[at] = s_j[q];
                    p_w[at] = s_c[5][q];
                    p_g[at] = s_c[6][q];
                    p_dx[at] = dx;
                    p_dy[at] = dy;
                    p_dz[at] = dz;
                }
                ++nact;
            }
        }
        __syncthreads();
    }
    if (!FLAT && T == 0) other_pos(0, oj, op);
    for (int b = 0; b < no; b += AH) {
        if (b > 0) {
            other(b, oj);
            other_pos(b, oj, op);
        }
#pragma unroll
        for (int u = 0; u < AH; ++u) {
            const DevEntry& e = s_tab[ti * nt + ptype(op[u].w)];
            if (b + u >= no || e.kind == RC_KIND_NONE) continue;
            const PairGeom pg = pair_geom<true>(pi, op[u], a.box, e);
            if (!pg.cut) continue;
            float phi, g;
            pair_eval(e, pg.r2, phi, g);
            add_pair(g, phi, pg.dx, pg.dy, pg.dz);
        }
    }
    // ---- wave-wide triplet stage -------------------------------------------
    const int k = (nact >= 2) ? nact : 0;
    const int incl = wave_inclusive_scan(k);
    const int off = incl - k;
    const int total = __builtin_amdgcn_readlane(incl, kWave - 1);
    l_f[lane][0] = l_f[lane][1] = l_f[lane][2] = l_f[lane][3] = 0.f;
    int round_start = 0;
    bool done = (k == 0);
    while (round_start < total) {
        bool mine = !done;
        int next = total, pool = poff;
        if (!fits) {
            // the admitted lanes form a run; the next round starts at the first lane left out
            mine = !done && off >= round_start && off + k <= round_start + kPool;
            int cand = (!done && !mine) ? off : total;
#pragma unroll
            for (int o = 32; o > 0; o >>= 1) cand = min(cand, __shfl_xor(cand, o, kWave));
            next = cand;
            pool = off - round_start;
            if (mine) {
                int q = pool;
                walk_list<true, 4>(i, pi, ti, a.nlist, packed, a.k_max, a.N, a.pos, s_tab, nt, a.box, -1,
                                   [&](int j, const float4&, const DevEntry& e, const PairGeom& pg) {
                                       float u, u1r;
                                       vhat_eval(e, pg.inside, pg.r2, u, u1r);
                                       p_j[q] = j;
                                       p_w[q] = e.sqrt_lam * u;
                                       p_g[q] = e.sqrt_lam * u1r;
                                       p_dx[q] = pg.dx;
                                       p_dy[q] = pg.dy;
                                       p_dz[q] = pg.dz;
                                       ++q;
                                   });
            }
        }
        const int tcount = mine ? k * (k - 1) / 2 : 0;
        int tinc = tcount;
#pragma unroll
        for (int o = 1; o < kWave; o <<= 1) {
            int t = __shfl_up(tinc, o, kWave);
            if (lane >= o) tinc += t;
        }
        l_tri[lane] = tinc - tcount;
        if (lane == kWave - 1) l_tri[kWave] = tinc;
        l_pool[lane] = pool;
        if (mine)
            for (int q = pool; q < pool + k; ++q) p_s[q] = 0.0f;
        l_k[lane] = mine ? k : 0;
        if (SPREAD && lane == 0) l_out = 0;
        __syncthreads();
        const int T = l_tri[kWave];
        for (int t = lane; t < T; t += kWave) {
            int lo = 0, hi = kWave - 1;  // owner: last lane with l_tri <= t
            while (lo < hi) {
                int mid = (lo + hi + 1) >> 1;
                if (l_tri[mid] <= t) lo = mid;
                else hi = mid - 1;
            }
            const int c = lo, kc = l_k[c];
            int loc = t - l_tri[c], aa = 0;
            while (loc >= kc - 1 - aa) {
                loc -= kc - 1 - aa;
                ++aa;
            }
            const int qa = l_pool[c] + aa, qb = l_pool[c] + aa + 1 + loc;
            const float wa = p_w[qa], wb = p_w[qb];
            const float ca = -p_g[qa] * wb, cb = -p_g[qb] * wa;  // force on a = ca d_a
            atomicAdd(&p_s[qa], wb);
            atomicAdd(&p_s[qb], wa);
            atomicAdd(&l_f[c][3], wa * wb);
            w6[0] += ca * p_dx[qa] * p_dx[qa] + cb * p_dx[qb] * p_dx[qb];
            w6[1] += ca * p_dy[qa] * p_dy[qa] + cb * p_dy[qb] * p_dy[qb];
            w6[2] += ca * p_dz[qa] * p_dz[qa] + cb * p_dz[qb] * p_dz[qb];
            w6[3] += ca * p_dx[qa] * p_dy[qa] + cb * p_dx[qb] * p_dy[qb];
            w6[4] += ca * p_dx[qa] * p_dz[qa] + cb * p_dx[qb] * p_dz[qb];
            w6[5] += ca * p_dy[qa] * p_dz[qa] + cb * p_dy[qb] * p_dz[qb];
        }
        __syncthreads();
        int* out = reinterpret_cast<int*>(p_w);   // read for the last time above
        if (mine) {   // the forces on the centre's partners, and minus their sum on the centre
            for (int q = pool; q < pool + k; ++q) {
                const float c = -p_g[q] * p_s[q];
                if (c == 0.0f) continue;   // a bonded partner (w' = 0): most of them
                const float gx = c * p_dx[q], gy = c * p_dy[q], gz = c * p_dz[q];
                const unsigned lj = (unsigned)(p_j[q] - (i - lane));
                if (!SPREAD || lj < (unsigned)kWave) {
                    float* F = lj < (unsigned)kWave ? l_f[lj] : reinterpret_cast<float*>(a.force + p_j[q]);
                    atomicAdd(F + 0, gx);
                    atomicAdd(F + 1, gy);
                    atomicAdd(F + 2, gz);
                } else {   // noted for the wavefront to send
                    p_dx[q] = gx;
                    p_dy[q] = gy;
                    p_dz[q] = gz;
                    out[atomicAdd(&l_out, 1)] = q;
                }
                fx -= gx;
                fy -= gy;
                fz -= gz;
            }
            done = true;
        }
        if constexpr (SPREAD) {
            __syncthreads();
            for (int t = lane; t < 4 * l_out; t += kWave) {
                const int q = out[t >> 2], x = t & 3;
                const float g = x == 0 ? p_dx[q] : x == 1 ? p_dy[q] : p_dz[q];
                if (x < 3) atomicAdd(reinterpret_cast<float*>(a.force + p_j[q]) + x, g);
            }
        }
        __syncthreads();
        round_start = next;
    }
    __syncthreads();
    fx += l_f[lane][0];
    fy += l_f[lane][1];
    fz += l_f[lane][2];
    en += l_f[lane][3];
    if (live && a.status && !(isfinite(fx) && isfinite(fy) && isfinite(fz)))
        atomicOr(&a.status[RC_ST_FLAGS], RC_FLAG_NONFINITE);
    // the wavefront's 64 rows as they lie in memory, 64 consecutive floats per instruction
    l_f[lane][0] = fx;
    l_f[lane][1] = fy;
    l_f[lane][2] = fz;
    l_f[lane][3] = en;
    __syncthreads();
    float* F0 = reinterpret_cast<float*>(a.force + (i - lane));
    const int words = 4 * min(kWave, a.N - (i - lane));
#pragma unroll
    for (int q = 0; q < 4; ++q) {
        const int at = q * kWave + lane;
        if (at < words) atomicAdd(F0 + at, (&l_f[0][0])[at]);
    }
    if (want_ev) {
        double v[7] = {en, w6[0], w6[1], w6[2], w6[3], w6[4], w6[5]};
#pragma unroll
        for (int q = 0; q < 7; ++q) v[q] = wave_sum(v[q]);
        if (lane == 0) {
#pragma unroll
            for (int q = 0; q < 7; ++q) a.ev_part[(size_t)blockIdx.x * kEvWords + q] = v[q];
        }
    }
}

__global__ __launch_bounds__(kBlock) void k_zero_f4(float4* __restrict__ p, int n) {
    for (int i = blockIdx.x * blockDim.x + threadIdx.x; i < n; i += gridDim.x * blockDim.x)
        p[i] = make_float4(0.f, 0.f, 0.f, 0.f);
}

hipError_t launch_forces_triplet(const ForceArgs& a, hipStream_t s) {
    if (!a.accumulate)
        hipLaunchKernelGGL(k_zero_f4, dim3(std::min(nblk(a.N, kBlock), 4096)), dim3(kBlock), 0, s,
                           a.force, a.N);
    const size_t shm = sizeof(DevEntry) * a.tab.nt * a.tab.nt;
    // sending the partners' forces together costs a barrier and pays where the atomics are the bound: us per call
    // apart and together, 32768 unequal 24.2, 24.8, 8000 22.7, 23.4; 200003 unequal 73.3, 68.0, reactive 53.8, 50.4.
    // Lists whose entries fill a pass or two stay flat: taking the kinds apart adds the reads of the ordinary ones to
    // the chain.  us per call, flat and apart: 0.6 entries (assembly) 16000 7.7, 8.6, 1000003 46.7, 54.9; 0.9
    // (dumbbells) 16000 8.6, 9.1; 1.7 (reactive) 16000 10.1, 10.2; 4.9 (unequal) 100003 39.0, 27.2; 5.9 (network) 16000
    // 14.4, 9.4, 200003 33.0, 17.7.  The long ones take eight swap entries per lane and pass below 65536: two passes
    // more of a wavefront's entries cost 2 us, a lane's unused places 0.4 (two and eight: lists of 2.4 entries 11.6,
    // 10.8, of 4.9 17.9, 15.2, of 7.3 28.7, 23.1).  Above, the wavefronts hide the passes and eight entries' LDS takes
    // their places: 100003 of 4.9 23.3, 32.2.
    const bool flat = a.list_len < 2.2f;
    auto kernel = flat ? k_forces_triplet<true, 2, true> : k_forces_triplet<true, 2, false>;
    if (a.N < 65536) kernel = flat ? k_forces_triplet<false, 2, true> : k_forces_triplet<false, 8, false>;
    hipLaunchKernelGGL(kernel, dim3(nblk(a.N, kWave)), dim3(kWave), shm, s, a, a.ev_part ? 1 : 0);
    return hipGetLastError();
}

// First pass of the sums form: S_m of every particle into a.ssum (one thread
// per particle, one wavefront per block so that a batch chunk names the table).
template <bool BATCH>
__global__ __launch_bounds__(kWave) void k_swap_sums(ForceArgs a) {
    extern __shared__ DevEntry s_tab[];
    // as in k_step: xcd_block's order from N (the grid is N / 64 blocks rounded up) with selects, and the
    // particle's own data requested before the table is staged (13.27 -> 13.12 us per dumbbell step at 8192)
    const int nbl = (a.N + kWave - 1) / kWave;
    const int per = nbl / 8;
    const int bx = blockIdx.x;
    const int blk = bx < per * 8 ? (bx & 7) * per + (bx >> 3) : bx;
    const int m = blk * kWave + threadIdx.x;
    const int mc = min(m, a.N - 1);   // in bounds; lanes past the end return below
    const float4 pm = a.pos[mc];
    const int packed = a.nn[mc];
    Box box_r;
    int lim = a.N;
    if constexpr (BATCH) {
        const RepDesc& d = a.rep[a.chunk_rep[blk]];
        box_r = d.box;
        lim = d.off + d.n;
        load_table(s_tab, Table{a.tab.e + d.tab, a.tab.nt});
    } else {
        box_r = a.box;
        load_table(s_tab, a.tab);
    }
    if (m >= lim) return;
    a.ssum[m] = swap_sum(m, pm, packed, a.pos, a.nlist, a.N, s_tab, a.tab.nt, box_r);
}

// The same sums from the packed list (the steps' first pass), OW particles per
// wavefront as in k_step_few.  A lane per particle took the wavefront's longest
// swap range in fours (8.6 us per launch at 5000 particles of density 0.25; now
// 4.8, about a launch's own time).
template <bool BATCH, int OW, int PL = 2>   // PL: entries per lane and pass
__global__ __launch_bounds__(kWave) void k_swap_sums_packed(ForceArgs a) {
    static_assert(!BATCH || OW == kWave, "a batch chunk has 64 slots");
    constexpr int G = kWave / OW;
    extern __shared__ DevEntry s_tab[];
    __shared__ float4 s_pos[OW];
    __shared__ float s_w[2][PL * kWave];
    const int lane = threadIdx.x, nt = a.tab.nt;
    const int ngr = (a.N + OW - 1) / OW;   // the grid
    const int per = ngr / 8, bx = blockIdx.x;
    const int gr = bx < per * 8 ? (bx & 7) * per + (bx >> 3) : bx;
    const int blk = gr / G, h = gr % G, base_m = gr * OW;
    const int m = base_m + lane;
    const int mc = min(base_m + min(lane, OW - 1), a.N - 1), m64 = blk * kWave + lane;
    const float4 pm0 = a.pos[mc];
    const int nn64 = a.nn[min(m64, a.N - 1)];
    Box box_r;
    int lim = a.N;
    if constexpr (BATCH) {
        const RepDesc& d = a.rep[a.chunk_rep[blk]];
        box_r = d.box;
        lim = d.off + d.n;
        load_table(s_tab, Table{a.tab.e + d.tab, nt});
    } else {
        box_r = a.box;
        load_table(s_tab, a.tab);
    }
    const int cnt64 = m64 < lim ? nn_swap(nn64) + nn_other(nn64) : 0;
    const int inc64 = wave_inclusive_scan(cnt64);
    const int before = h > 0 ? __builtin_amdgcn_readlane(inc64, h * OW - 1) : 0;
    const int T = __builtin_amdgcn_readlane(inc64, h * OW + OW - 1) - before;
    const int from = h * OW + min(lane, OW - 1);
    const bool live = lane < OW && m < lim;
    const int my_off = __shfl(inc64 - cnt64, from, kWave) - before;
    const int ns_any = nn_swap(__shfl(nn64, from, kWave));
    const int ns = live ? ns_any : 0;
    if (lane < OW) s_pos[lane] = pm0;
    __syncthreads();
    const float S = packed_sums<PL, OW, false>(base_m, s_pos, my_off, ns, T, h * OW,
                                               (size_t)blk * kWave * a.k_max + before, a.pos, a.pl_j, a.pl_o, s_tab, nt,
                                               box_r, s_w);
    if (live) a.ssum[m] = S;
}

static hipError_t launch_sums(const ForceArgs& a, bool batch, hipStream_t s) {
    const size_t shm = sizeof(DevEntry) * a.tab.nt * a.tab.nt;
    if (batch)
        hipLaunchKernelGGL((k_swap_sums<true>), dim3(nblk(a.N, kWave)), dim3(kWave), shm, s, a);
    else
        hipLaunchKernelGGL((k_swap_sums<false>), dim3(nblk(a.N, kWave)), dim3(kWave), shm, s, a);
    return hipGetLastError();
}

// Particles per wavefront, by the lists' mean length: those that hold about half a row of 64 entries (8 to 32) while
// that makes at most 4096 wavefronts (four per SIMD); lists shorter than a particle or so leave too little to share
// once a few thousand particles fill the chip's compute units.
// A wavefront's time is its rows of 64 entries one after the other, each as long as its longest partner walk, so a
// chip with idle SIMDs wants more wavefronts with fewer rows.  us without ev at 8, 16, 32, 64 particles per wavefront
// (entries per particle): 0.6 (assembly) 4000 particles 5.8, 5.7, 5.8, 6.0; 32000 6.9, 6.5, 6.4, 6.3; 128000 13.5, 9.9,
// 7.5, 6.8; 0.9 (dumbbells) 4000 6.7, 6.6, 7.0, 8.0; 64000 10.8, 8.3, 7.8, 8.5; 4.8 (reactive, density 0.25) 4000 14.2,
// 18.8, 26.0, 38.8; 32000 16.8, 20.8, 25.6, 38.7; 64000 28.3, 23.7, 27.7, 39.8; 256000 79.5, 65.0, 53.7, 48.8.
static int gather_owners(int N, float list_len) {
    if (list_len < 0.8f) return N <= 5120 ? 16 : kWave;
    int ow = 32;
    while (ow > 8 && (float)ow * list_len > 44.0f) ow /= 2;
    while (ow < kWave && (long)N > 4096L * ow) ow *= 2;
    return ow;
}

// Wavefronts per block with ev: several from 768 wavefronts on, where the rows cost the reduction more than blocks of
// one gain by spreading over the compute units.  us at blocks of one and of four: reactive particles of density 0.25
// (8 per wavefront) 1000 16.4, 19.3; 4000 17.9, 18.9; 8000 19.3, 18.5; 32000 24.7, 21.1; 64000 (16) 32.1, 28.3;
// 128000 (32, blocks of two) 40.0, 37.6.  (Without ev 1000 13.0, 15.6; 32000 16.8, 16.8.)
constexpr int gather_waves(int ow) { return ow == kWave ? 1 : (ow == 32 ? 2 : 4); }
static bool gather_wide(int N, int ow) { return (long)N > 768L * ow; }

int gather_particles(int N, float list_len) {
    const int ow = gather_owners(N, list_len);
    return gather_wide(N, ow) ? ow * gather_waves(ow) : ow;
}

template <bool BATCH, int OW>
static void launch_gather_ow(const ForceArgs& a, hipStream_t s) {
    const size_t shm = sizeof(DevEntry) * a.tab.nt * a.tab.nt;
    constexpr int NW = BATCH ? 1 : gather_waves(OW);
    if (a.ev_part) {
        const int w = !BATCH && gather_wide(a.N, OW) ? NW : 1;
        const dim3 g(nblk(a.N, OW * w)), b(kWave * w);
        if (w > 1 && a.ssum)
            hipLaunchKernelGGL((k_forces_gather<true, BATCH, true, OW, NW>), g, b, shm, s, a);
        else if (w > 1)
            hipLaunchKernelGGL((k_forces_gather<true, BATCH, false, OW, NW>), g, b, shm, s, a);
        else if (a.ssum)
            hipLaunchKernelGGL((k_forces_gather<true, BATCH, true, OW, 1>), g, b, shm, s, a);
        else
            hipLaunchKernelGGL((k_forces_gather<true, BATCH, false, OW, 1>), g, b, shm, s, a);
    } else {
        const dim3 g(nblk(a.N, OW)), b(kWave);
        if (a.ssum)
            hipLaunchKernelGGL((k_forces_gather<false, BATCH, true, OW, 1>), g, b, shm, s, a);
        else
            hipLaunchKernelGGL((k_forces_gather<false, BATCH, false, OW, 1>), g, b, shm, s, a);
    }
}

hipError_t launch_forces_gather(const ForceArgs& a, hipStream_t s) {
    if (a.ssum) {
        hipError_t e = launch_sums(a, false, s);
        if (e != hipSuccess) return e;
    }
    switch (gather_owners(a.N, a.list_len)) {
        case 8: launch_gather_ow<false, 8>(a, s); break;
        case 16: launch_gather_ow<false, 16>(a, s); break;
        case 32: launch_gather_ow<false, 32>(a, s); break;
        default: launch_gather_ow<false, kWave>(a, s);
    }
    return hipGetLastError();
}

hipError_t launch_forces_gather_batch(const ForceArgs& a, hipStream_t s) {
    if (a.ssum) {
        hipError_t e = launch_sums(a, true, s);
        if (e != hipSuccess) return e;
    }
    launch_gather_ow<true, kWave>(a, s);
    return hipGetLastError();
}

// ---------------------------------------------------------------------------
// fused MD step: gather forces at x_in, finish the previous step's final half
// kick, then B A O A into pos_out.  One kernel per step, no atomics on data.
// ---------------------------------------------------------------------------
// With BATCH the wave's 64-slot chunk names its replica, which supplies the
// box, the coefficient table, the slot bound and the noise key; the noise
// counter uses the tag relative to the replica's first slot, so a replica
// draws the same numbers as the same system run on its own.
// Seven wavefronts per SIMD: the walk-form kernel at width 2 then fits 72
// VGPRs without spilling (74 otherwise, six wavefronts) and runs ~2 % faster
// at 1M particles; the other instantiations are unchanged by the hint.
// The particle's own data is requested before the table is staged in LDS,
// so that the table's load and barrier overlap it instead of preceding it
// (24.9 -> 24.3 us per step at 1M particles).
template <bool EV, bool BATCH, int PL, bool SF>
__global__ __launch_bounds__(kWave) __attribute__((amdgpu_waves_per_eu(7))) void k_step(StepArgs a) {
    extern __shared__ DevEntry s_tab[];
    const int nt = a.tab.nt;
    // Wavefronts in their load and gather part run at raised issue priority and drop it for the
    // integrator, so a SIMD's newer wavefronts get their loads out ahead of older ones' arithmetic
    // (24.52-24.70 -> 24.29-24.36 us per step at 1M particles, any raised level alike).
    __builtin_amdgcn_s_setprio(2);
    // xcd_block's order, from N (every launch's grid is N / 64 blocks rounded up) and without branches,
    // so that the arguments the own data needs come in one round of scalar loads (24.84 -> 24.68 us)
    const int nbl = (a.N + kWave - 1) / kWave;
    const int per = nbl / 8;
    const int bx = blockIdx.x;
    const int blk = bx < per * 8 ? (bx & 7) * per + (bx >> 3) : bx;
    const int m = blk * kWave + threadIdx.x;
    const int mc = min(m, a.N - 1);   // in bounds; lanes past a replica's end or N are dropped below
    const float4 pm0 = a.pos_in[mc];
    const float4 vm0 = a.vel[mc];
    const int packed0 = a.nn[mc];
    Box box_r;
    int lim = a.N, tag0 = 0;
    uint64_t seed = a.seed;
    if constexpr (BATCH) {
        const int r = a.chunk_rep[blk];
        const RepDesc& d = a.rep[r];
        box_r = d.box;
        lim = d.off + d.n;
        tag0 = d.off;
        seed = a.seeds[r];
        load_table(s_tab, Table{a.tab.e + d.tab, nt});
    } else {
        box_r = a.box;
        load_table(s_tab, a.tab);
    }
    const Box& box = box_r;
    const bool live = m < lim;
    const uint64_t step = a.step + (a.step_base ? *a.step_base : 0ull);
    Acc acc = {};
    const float4 pm = live ? pm0 : make_float4(0.f, 0.f, 0.f, 0.f);
    const float4 vm = live ? vm0 : make_float4(0.f, 0.f, 0.f, 0.f);
    const int packed = live ? packed0 : 0;
    const OneSystem sys{s_tab, nt, box};
    // the entries come from the packed copy of the list
    wave_gather<EV, PL, SF, OneSystem, 1, true>(m - (int)threadIdx.x, live, pm, packed, a.pos_in, a.nlist, a.nn,
                                                     a.k_max, a.N, sys, acc, a.ssum, a.pl_j, a.pl_o);
    if (!BATCH && a.bonds && live)
        fene_add<EV>(ptag(pm.w), pm, a.bonds, a.rtag, a.pos_in, box, a.fene_k, a.fene_r02, acc);
    __builtin_amdgcn_s_setprio(0);
    step_finish<EV>(a, a.pos_out, m, blk, live, pm, vm, acc, box, tag0, seed, step);
    // the chunk's reset, when this launch carries it (no kernel of the launch reads those words); at the
    // end, so that its argument's load does not hold up the start of every wavefront (25.15 -> 24.79 us)
    if (a.reset_status && blockIdx.x == 0 && threadIdx.x == 0) chunk_reset(a.reset_status, a.reset_base, a.reset_to);
}

// The plain step with few particles per wavefront, for systems whose 64-particle
// wavefronts would hold many entries and not fill the chip: a wavefront's time
// is its rows of 64 entries one after the other.  Same arithmetic and order as
// k_step (bit for bit); the thermostat normals are drawn and the spring
// partners read while the list reads are under way.
// us per step as a run sees it (one launch for every 64 particles -> this):
// network of 67200 beads 33.7 -> 24.2, of 5000 beads 27.9 -> 15.4; 30000
// reactive particles (density 0.25) 21.4 -> 17.2; 20011 dumbbells 11.0 -> 10.6.
template <bool SF, int OW>
__global__ __launch_bounds__(kWave) void k_step_few(StepArgs a) {
    extern __shared__ DevEntry s_tab[];
    const int nt = a.tab.nt, lane = threadIdx.x;
    const int ngr = (a.N + OW - 1) / OW;   // the grid
    const int per = ngr / 8, bx = blockIdx.x;
    const int gr = bx < per * 8 ? (bx & 7) * per + (bx >> 3) : bx;
    constexpr int G = kWave / OW;
    const int blk = gr / G, h = gr % G;    // the 64-particle block of the packed list and the group in it
    const int m = gr * OW + lane;
    const bool live = lane < OW && m < a.N;
    const int mc = min(gr * OW + min(lane, OW - 1), a.N - 1);
    const int m64 = blk * kWave + lane;
    const float4 pm0 = a.pos_in[mc];
    const float4 vm0 = a.vel[mc];
    const int nn64 = a.nn[min(m64, a.N - 1)];
    const uint64_t step = a.step + (a.step_base ? *a.step_base : 0ull);
    load_table(s_tab, a.tab);
    const float4 pm = live ? pm0 : make_float4(0.f, 0.f, 0.f, 0.f);
    const float4 vm = live ? vm0 : make_float4(0.f, 0.f, 0.f, 0.f);
    // this group's entries within the block's
    const int cnt64 = m64 < a.N ? nn_swap(nn64) + nn_other(nn64) : 0;
    const int inc64 = wave_inclusive_scan(cnt64);
    const int before = h > 0 ? __builtin_amdgcn_readlane(inc64, h * OW - 1) : 0;
    const int packed_any = __shfl(nn64, h * OW + min(lane, OW - 1), kWave);
    const int packed = live ? packed_any : 0;
    Acc acc = {};
    const OneSystem sys{s_tab, nt, a.box};
    int2 bond = make_int2(-1, -1);
    if (a.bonds && live) bond = a.bonds[ptag(pm.w)];
    float nz[3] = {0.f, 0.f, 0.f};
    int bi[2] = {-1, -1};
    float4 bp[2] = {pm, pm};
    wave_gather<false, 1, SF, OneSystem, 1, true, 4, OW>(
        m - lane, live, pm, packed, a.pos_in, a.nlist, a.nn, a.k_max, a.N, sys, acc, a.ssum, a.pl_j, a.pl_o,
        (size_t)blk * kWave * a.k_max + before, h * OW, [&](int at) {
            if (at == 0) {
                if (a.bonds) {
                    if (bond.x >= 0) bi[0] = a.rtag[bond.x];
                    if (bond.y >= 0) bi[1] = a.rtag[bond.y];
                }
                if (a.langevin) {
                    thermostat_normals(a.seed, (uint32_t)ptag(pm.w), step, nz[0], nz[1], nz[2]);
                    asm volatile("" : "+v"(nz[0]), "+v"(nz[1]), "+v"(nz[2]));   // drawn here, not where they are used
                }
            } else if (a.bonds) {
#pragma unroll
                for (int q = 0; q < 2; ++q)
                    if (bi[q] >= 0) bp[q] = a.pos_in[bi[q]];
            }
        });
    if (a.bonds && live) fene_pair(bi, bp, pm, a.box, a.fene_k, a.fene_r02, acc);
    step_finish<false, true, true>(a, a.pos_out, m, blk, live, pm, vm, acc, a.box, 0, a.seed, step, nz);
    if (a.reset_status && blockIdx.x == 0 && threadIdx.x == 0) chunk_reset(a.reset_status, a.reset_base, a.reset_to);
}

// k_step_few of the two-pass form in one launch: a wavefront adds up the sums S
// of its own particles from its entries, keeps a row of entries in registers,
// and takes the sum of a partner outside the wavefront from a walk of the
// partner's swap range (the same terms in the same order, so the same bits as
// the launch that computed every S).  Only entries between r_min and r_cut need
// their partner's sum, half of the bonded ones of stiff dumbbells: the walk costs
// less than the first launch's own time while lists are short (fused_sums).
// Bound by one wavefront's instructions and reads.  Records of the entries with
// fixed places and the partners' own partners, which take three dependent reads
// out, gained 0.3 us; 32 particles per wavefront lost once the mixture had
// aggregated, as some then hold two rows (20011 dumbbells: 13.1 us per step; 10.0
// with 16, 11.9 in two launches).
constexpr int kFusedOwn = 16;
__global__ __launch_bounds__(kWave) void k_step_fused(StepArgs a) {
    constexpr int OW = kFusedOwn;
    extern __shared__ DevEntry s_tab[];
    __shared__ float4 s_pos[OW];
    __shared__ float s_S[OW];
    __shared__ float s_w[2][kWave], s_c[3][kWave];
    const int nt = a.tab.nt, lane = threadIdx.x;
    const int ngr = (a.N + OW - 1) / OW;   // the grid
    const int per = ngr / 8, bx = blockIdx.x;
    const int gr = bx < per * 8 ? (bx & 7) * per + (bx >> 3) : bx;
    constexpr int G = kWave / OW;
    const int blk = gr / G, h = gr % G;    // the 64-particle block of the packed list and the group in it
    const int base_m = gr * OW, m = base_m + lane;
    const bool live = lane < OW && m < a.N;
    const int mc = min(base_m + min(lane, OW - 1), a.N - 1);
    const int m64 = blk * kWave + lane;
    const float4 pm0 = a.pos_in[mc];
    const float4 vm0 = a.vel[mc];
    const int nn64 = a.nn[min(m64, a.N - 1)];
    const uint64_t step = a.step + (a.step_base ? *a.step_base : 0ull);
    load_table(s_tab, a.tab);
    const float4 pm = live ? pm0 : make_float4(0.f, 0.f, 0.f, 0.f);
    const float4 vm = live ? vm0 : make_float4(0.f, 0.f, 0.f, 0.f);
    // this group's entries within the block's
    const int cnt64 = m64 < a.N ? nn_swap(nn64) + nn_other(nn64) : 0;
    const int inc64 = wave_inclusive_scan(cnt64);
    const int before = h > 0 ? __builtin_amdgcn_readlane(inc64, h * OW - 1) : 0;
    const int T = __builtin_amdgcn_readlane(inc64, h * OW + OW - 1) - before;
    const int from = h * OW + min(lane, OW - 1);
    const int my_off = __shfl(inc64 - cnt64, from, kWave) - before;
    const int packed_any = __shfl(nn64, from, kWave);
    const int ns = live ? nn_swap(packed_any) : 0, cnt = live ? ns + nn_other(packed_any) : 0;
    const size_t first = (size_t)blk * kWave * a.k_max + before;
    if (lane < OW) s_pos[lane] = pm;
    int2 bond = make_int2(-1, -1);
    if (a.bonds && live) bond = a.bonds[ptag(pm.w)];
    __syncthreads();

    struct Entry {
        int own, j, nnj;             // owner lane (-1: none), neighbour, its list lengths
        float4 pj;
        SwapEntry t;
    };
    auto index = [&](int row, Entry& x) {
        const int e = row * kWave + lane;
        x.own = -1;
        x.j = base_m;
        if (e < T) {
            x.own = a.pl_o[first + e] - h * OW;
            x.j = a.pl_j[first + e];
        }
    };
    auto request = [&](Entry& x) {
        x.pj = pm;
        x.nnj = 0;
        if (x.own >= 0) {
            const unsigned lj = (unsigned)(x.j - base_m);
            if (lj < (unsigned)OW) {
                x.pj = s_pos[lj];
            } else {
                x.pj = a.pos_in[x.j];
                x.nnj = a.nn[x.j];
            }
        }
    };
    // the entry's terms (zero outside its cutoff) and its share of S
    auto terms = [&](Entry& x) {
        x.t = SwapEntry{0.0f, 0.0f, 0.0f, 0.0f, 0.0f, 0.0f, 0.0f};
        if (x.own >= 0) x.t = swap_entry(s_pos[x.own], x.pj, s_tab, nt, a.box);
        s_w[0][lane] = x.t.sl;
        s_w[1][lane] = x.t.u;
    };
    float S = 0.0f;
    auto add_sums = [&](int row) {
        __syncthreads();
        const int b = row * kWave, lo = max(my_off, b) - b, hi = min(my_off + ns, b + kWave) - b;
        for (int q = lo; q < hi; ++q) S = __fmaf_rn(s_w[0][q], s_w[1][q], S);
        __syncthreads();
    };

    Entry x;   // the first row's; further ones are read again
    index(0, x);
    // while the indices are on their way: the spring partners' and the noise
    int bi[2] = {-1, -1};
    float4 bp[2] = {pm, pm};
    float nz[3] = {0.f, 0.f, 0.f};
    if (a.bonds) {
        if (bond.x >= 0) bi[0] = a.rtag[bond.x];
        if (bond.y >= 0) bi[1] = a.rtag[bond.y];
    }
    if (a.langevin) {
        thermostat_normals(a.seed, (uint32_t)ptag(pm.w), step, nz[0], nz[1], nz[2]);
        asm volatile("" : "+v"(nz[0]), "+v"(nz[1]), "+v"(nz[2]));   // drawn here, not where they are used
    }
    request(x);
    if (a.bonds) {
#pragma unroll
        for (int q = 0; q < 2; ++q)
            if (bi[q] >= 0) bp[q] = a.pos_in[bi[q]];
    }
    terms(x);
    add_sums(0);
    for (int r = 1; r * kWave < T; ++r) {
        Entry y;
        index(r, y);
        request(y);
        terms(y);
        add_sums(r);
    }
    if (lane < OW) s_S[lane] = S;
    __syncthreads();

    Acc acc = {};
    auto force = [&](int row, const Entry& x) {
        float f = x.t.g;
        if (needs_sums(x.t)) {
            const unsigned lj = (unsigned)(x.j - base_m);
            const float Sj = lj < (unsigned)OW
                                 ? s_S[lj]
                                 : swap_sum(x.j, x.pj, x.nnj, a.pos_in, a.nlist, a.N, s_tab, nt, a.box);
            f = swap_factor(x.t, s_S[x.own], Sj);
        }
        s_c[0][lane] = f * x.t.dx;
        s_c[1][lane] = f * x.t.dy;
        s_c[2][lane] = f * x.t.dz;
        __syncthreads();
        const int b = row * kWave, lo = max(my_off, b) - b, hi = min(my_off + cnt, b + kWave) - b;
        for (int q = lo; q < hi; ++q) {
            acc.fx += s_c[0][q];
            acc.fy += s_c[1][q];
            acc.fz += s_c[2][q];
        }
        __syncthreads();
    };
    force(0, x);
    for (int r = 1; r * kWave < T; ++r) {
        Entry y;
        index(r, y);
        request(y);
        terms(y);
        force(r, y);
    }
    if (a.bonds && live) fene_pair(bi, bp, pm, a.box, a.fene_k, a.fene_r02, acc);
    step_finish<false, true, true>(a, a.pos_out, m, blk, live, pm, vm, acc, a.box, 0, a.seed, step, nz);
    if (a.reset_status && blockIdx.x == 0 && threadIdx.x == 0) chunk_reset(a.reset_status, a.reset_base, a.reset_to);
}

// Step kernels by (ev, batch, width, form); log steps use the default width.
template <bool BATCH, bool SF>
static const void* step_fn_form(bool ev, int width) {
    if (ev) return reinterpret_cast<const void*>(&k_step<true, BATCH, kDefaultWidth, SF>);
    switch (width) {
        case 1: return reinterpret_cast<const void*>(&k_step<false, BATCH, 1, SF>);
        case 4: return reinterpret_cast<const void*>(&k_step<false, BATCH, 4, SF>);
        default: return reinterpret_cast<const void*>(&k_step<false, BATCH, 2, SF>);
    }
}

template <bool BATCH>
static const void* step_fn(bool ev, int width, int form) {
    return form == RC_FORM_SUMS ? step_fn_form<BATCH, true>(ev, width) : step_fn_form<BATCH, false>(ev, width);
}

// arguments of the first pass of the sums form for a step reading pos_in
static ForceArgs sums_args(const StepArgs& a) {
    ForceArgs f{};
    f.pos = a.pos_in;
    f.nlist = a.nlist;
    f.nn = a.nn;
    f.N = a.N;
    f.k_max = a.k_max;
    f.tab = a.tab;
    f.box = a.box;
    f.rep = a.rep;
    f.chunk_rep = a.chunk_rep;
    f.ssum = a.ssum;
    f.pl_j = a.pl_j;
    f.pl_o = a.pl_o;
    return f;
}

template <bool SF>
static const void* few_fn(int ow) {
    switch (ow) {
        case 8: return reinterpret_cast<const void*>(&k_step_few<SF, 8>);
        case 16: return reinterpret_cast<const void*>(&k_step_few<SF, 16>);
        default: return reinterpret_cast<const void*>(&k_step_few<SF, 32>);
    }
}

// Particles per wavefront of a plain step; list_len: mean list entries per particle.  k_step_few at the particles
// that hold about half a row of 64 entries (8 to 32), as long as that makes at most 5120 wavefronts (five per SIMD; 3584
// for lists of about one entry, which have less to gain); lists of fewer entries than particles leave too little to
// share.  By the length, not by the density: the walk kernel of the assembly mixture, whose colloids make the largest
// list radius a poor guide, was slower by 5-9 %.
// us per step of a run with 64, 32, 16, 8 particles per wavefront:
//   walk   0.8 entries (assembly mixture) 8000 particles 8.0, 8.1, 8.1, 8.1; 30000 8.4, 8.7, 9.0, 9.8; 80000 9.0,
//          9.6, 10.7, 14.7
//          0.84 (dumbbells, thin skin) 8000 7.9, 8.4; 100000 9.8, 9.7; 160000 9.4, 11.0; 0.89 (dumbbells) 40000 10.3, 9.4;
//          110000 10.1, 9.9; 0.93 (assembly, thick skin) 8000 7.8, 7.5, 7.5; 100000 9.3, 8.8; 131072 9.2, 9.4
//          1.2 (assembly, aggregated) 8000 8.7, 7.8, 7.7; 80000 10.3, 8.9, 9.5; 160000 10.8, 10.4
//          1.2 (reactive, density 0.1) 4000 13.4, 10.3, 10.2, 9.8; 80000 14.7, 12.5, 13.4, 18.4; 160000 17.2, 15.3, ..
//          2.3 (0.15) 4000 21.5, 16.2, 12.4, 12.2; 80000 23.8, 19.0, 17.2, 24.8; 110000 24.1, 20.3, 23.1, 30.5
//          4.8 (0.25) 4000 47.8, 29.7, 22.5, 17.3; 45000 48.4, 33.2, 26.5, 29.0; 110000 52.5, 35.7, 42.5, 46.2
//          10 (network) 4000 29.0, 23.3, 17.6, 15.1; 60000 31.1, 25.7, 21.1, 23.6; 160000 36.3, 31.7, 34.5, 43.3
//   sums   0.9 (dumbbells) 110000 12.1, 12.4, 15.2, 21.7; 4.8 16000 20.4, 15.4, 12.8, 11.1; 80000 22.1, 18.3, 17.1, 19.6
//          1.3 (dumbbells, aggregated) 90000 13.0, 13.1; 131072 13.8, 14.4; 150000 14.1, 15.1; 1.7 (reactive, 0.13)
//          110000 12.1, 12.7; 2.1 (0.15) 96000 13.8, 13.1 (such lists up to 81920 particles take one launch, fused_sums,
//          but for log steps: the sums of 512 dumbbells 5.1, 4.9)
static int step_particles(int N, int form, float list_len) {
    if (list_len < (form == RC_FORM_SUMS && N > 5120 * kFusedOwn ? 1.9f : 0.87f)) return kStepBlock;
    int ow = 32;
    while (ow > 8 && (float)ow * list_len > 44.0f) ow /= 2;
    const long wavefronts = list_len < 1.1f ? 3584 : 5120;
    while (ow < kStepBlock && (long)N > wavefronts * ow) ow *= 2;
    return ow;
}

// Batches of lists longer than a pass of two entries per lane holds take four (16.8 -> 15.6 us per launch at 96
// replicas, five entries per particle; 131072 dumbbells, 1.7 entries: 12.5 -> 12.7 per step).  (A batch's length is
// that of uniform replicas at their largest list radii.)
static const void* sums_fn(bool batch, int ow, float list_len) {
    if (batch)
        return list_len > 3.0f ? reinterpret_cast<const void*>(&k_swap_sums_packed<true, kWave, 4>)
                               : reinterpret_cast<const void*>(&k_swap_sums_packed<true, kWave>);
    switch (ow) {
        case 8: return reinterpret_cast<const void*>(&k_swap_sums_packed<false, 8>);
        case 16: return reinterpret_cast<const void*>(&k_swap_sums_packed<false, 16>);
        case 32: return reinterpret_cast<const void*>(&k_swap_sums_packed<false, 32>);
        default: return reinterpret_cast<const void*>(&k_swap_sums_packed<false, kWave>);
    }
}

// Whether the two-pass form takes one launch: while a row holds 16 particles' entries with some room for a denser spot,
// and the wavefronts are at most five per SIMD.  us per step, two launches (best particles per wavefront) and one:
// 0.8 entries per particle (assembly) 1500 8.6, 6.8; 80000 10.3, 9.5; 110000 10.6, 11.5; 0.9 (dumbbells) 20000 9.5, 8.1;
// 80000 11.4, 10.7; 1.2 (reactive, density 0.1) 4000 9.4, 8.3; 80000 11.8, 11.4; 2.3 (0.15) 1500 9.4, 9.6; 30000 10.9,
// 10.8; 80000 13.7, 13.1; 4.1 (a drop of density 0.25 in a box eight times as large) 1340 9.4, 16.5; 78000 16.1, 23.2.
static bool fused_sums(int N, float list_len) { return list_len <= 2.5f && N <= 5120 * kFusedOwn; }

StepKernel step_kernel(bool batch, bool ev, int width, int form, int N, float list_len) {
    StepKernel k;
    const int few = batch ? kStepBlock : step_particles(N, form, list_len);
    if (!batch && !ev && form == RC_FORM_SUMS && fused_sums(N, list_len)) {
        k.particles = kFusedOwn;
        k.fn = reinterpret_cast<const void*>(&k_step_fused);
        return k;
    }
    if (!ev) k.particles = few;
    if (k.particles < kStepBlock)
        k.fn = form == RC_FORM_SUMS ? few_fn<true>(few) : few_fn<false>(few);
    else
        k.fn = batch ? step_fn<true>(ev, width, form) : step_fn<false>(ev, width, form);
    if (form == RC_FORM_SUMS) {
        k.sums_fn = sums_fn(batch, few, list_len);
        k.sums_particles = few;
    }
    return k;
}

static hipError_t launch_step_any(const StepArgs& a, bool batch, bool ev, hipStream_t s) {
    const StepKernel k = step_kernel(batch, ev, a.width, a.form, a.N, a.list_len);
    const size_t shm = sizeof(DevEntry) * a.tab.nt * a.tab.nt;
    if (k.sums_fn) {
        ForceArgs f = sums_args(a);
        void* fargs[] = {&f};
        hipError_t e = hipLaunchKernel(k.sums_fn, dim3(nblk(a.N, k.sums_particles)), dim3(kWave), fargs, shm, s);
        if (e != hipSuccess) return e;
    }
    StepArgs arg = a;
    void* args[] = {&arg};
    return hipLaunchKernel(k.fn, dim3(nblk(a.N, k.particles)), dim3(kStepBlock), args, shm, s);
}

hipError_t launch_step(const StepArgs& a, bool ev, hipStream_t s) { return launch_step_any(a, false, ev, s); }
hipError_t launch_step_batch(const StepArgs& a, bool ev, hipStream_t s) { return launch_step_any(a, true, ev, s); }

// A plain (no ev) step launch whose kernels each run between an event pair
// (hipExtLaunchKernel records them around the kernel alone).
hipError_t launch_step_timed(const StepArgs& a, bool batch, hipStream_t s, hipEvent_t* sums, hipEvent_t* step) {
    const size_t shm = sizeof(DevEntry) * a.tab.nt * a.tab.nt;
    const StepKernel k = step_kernel(batch, false, a.width, a.form, a.N, a.list_len);
    if (k.sums_fn) {
        ForceArgs f = sums_args(a);
        void* fargs[] = {&f};
        hipError_t e = sums ? hipExtLaunchKernel(k.sums_fn, dim3(nblk(a.N, k.sums_particles)), dim3(kWave), fargs, shm,
                                                 s, sums[0], sums[1], 0)
                            : hipLaunchKernel(k.sums_fn, dim3(nblk(a.N, k.sums_particles)), dim3(kWave), fargs, shm, s);
        if (e != hipSuccess) return e;
    }
    StepArgs arg = a;
    void* args[] = {&arg};
    return hipExtLaunchKernel(k.fn, dim3(nblk(a.N, k.particles)), dim3(kStepBlock), args, shm, s, step[0], step[1], 0);
}

ForceArgs step_sums_args(const StepArgs& a) { return sums_args(a); }

// ---------------------------------------------------------------------------
// bond count: swap pairs i<j with canonical r^2 < r_min^2
// ---------------------------------------------------------------------------
__global__ __launch_bounds__(kBlock) void k_bonds(const float4* __restrict__ pos,
                                                 const int* __restrict__ nlist,
                                                 const int* __restrict__ nn, int k_max, int N, Table tab, Box box,
                                                 unsigned long long* __restrict__ part) {
    extern __shared__ DevEntry s_tab[];
    __shared__ unsigned s_w[kBlock / kWave];
    load_table(s_tab, tab);
    const int i = blockIdx.x * blockDim.x + threadIdx.x;
    unsigned c = 0;
    if (i < N) {
        const float4 pi = pos[i];
        walk_list<true, 4>(i, pi, ptype(pi.w), nlist, nn[i], k_max, N, pos, s_tab, tab.nt, box, -1,
                        [&](int j, const float4&, const DevEntry&, const PairGeom& pg) {
                            if (j > i && pg.bond) ++c;
                        });
    }
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) c += __shfl_xor(c, o, kWave);
    if ((threadIdx.x & (kWave - 1)) == 0) s_w[threadIdx.x / kWave] = c;
    __syncthreads();
    if (threadIdx.x == 0) {
        unsigned long long t = 0;
        for (int w = 0; w < kBlock / kWave; ++w) t += s_w[w];
        part[blockIdx.x] = t;
    }
}

// bond partner of every particle, by tag: the tag of its one bonded swap partner
// (canonical r^2 < r_min^2), -1 when it has none, -2 when it has several
__global__ __launch_bounds__(kBlock) void k_bond_partners(const float4* __restrict__ pos,
                                                         const int* __restrict__ nlist,
                                                         const int* __restrict__ nn, int k_max, int N, Table tab,
                                                         Box box, int* __restrict__ partner) {
    extern __shared__ DevEntry s_tab[];
    load_table(s_tab, tab);
    const int i = blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= N) return;
    const float4 pi = pos[i];
    int p = -1;
    walk_list<true, 4>(i, pi, ptype(pi.w), nlist, nn[i], k_max, N, pos, s_tab, tab.nt, box, -1,
                    [&](int, const float4& pj, const DevEntry&, const PairGeom& pg) {
                        if (pg.bond) p = (p == -1) ? ptag(pj.w) : -2;
                    });
    const int t = ptag(pi.w);
    if (t >= 0 && t < N) partner[t] = p;   // tags >= N have no slot (documented requirement: tags < N)
}

hipError_t launch_bond_partners(const float4* pos, const int* nlist, const int* nn, int k_max, int N, Table tab,
                                Box box, int* partner, hipStream_t s) {
    const size_t shm = sizeof(DevEntry) * tab.nt * tab.nt;
    hipLaunchKernelGGL(k_bond_partners, dim3(nblk(N, kBlock)), dim3(kBlock), shm, s, pos, nlist, nn, k_max, N, tab,
                       box, partner);
    return hipGetLastError();
}

// one block: sum nb partial counts into *out (fixed order: exact either way)
__global__ __launch_bounds__(1024) void k_sum_u64(const unsigned long long* __restrict__ part, int nb,
                                                 unsigned long long* __restrict__ out) {
    __shared__ unsigned long long red[1024];
    unsigned long long s = 0;
    for (int b = threadIdx.x; b < nb; b += blockDim.x) s += part[b];
    red[threadIdx.x] = s;
    __syncthreads();
    for (int w = 512; w > 0; w >>= 1) {
        if (threadIdx.x < w) red[threadIdx.x] += red[threadIdx.x + w];
        __syncthreads();
    }
    if (threadIdx.x == 0) *out = red[0];
}

hipError_t launch_bonds(const float4* pos, const int* nlist, const int* nn, int k_max, int N, Table tab, Box box,
                        unsigned long long* count, unsigned long long* part, hipStream_t s) {
    const size_t shm = sizeof(DevEntry) * tab.nt * tab.nt;
    const int nb = nblk(N, kBlock);
    hipLaunchKernelGGL(k_bonds, dim3(nb), dim3(kBlock), shm, s, pos, nlist, nn, k_max, N, tab, box, part);
    hipLaunchKernelGGL(k_sum_u64, dim3(1), dim3(1024), 0, s, part, nb, count);
    return hipGetLastError();
}

// FENE springs alone (one thread per particle; accumulates into force)
template <bool EV>
__global__ __launch_bounds__(kWave) void k_fene(const float4* __restrict__ pos, const int2* __restrict__ bonds,
                                               const int* __restrict__ rtag, int N, Box box, float K, float R02,
                                               float4* __restrict__ force, double* __restrict__ ev_part) {
    const int m = blockIdx.x * kWave + threadIdx.x;
    Acc acc = {};
    if (m < N) {
        const float4 pm = pos[m];
        fene_add<EV>(ptag(pm.w), pm, bonds, rtag, pos, box, K, R02, acc);
        float4 f = force[m];
        f.x += acc.fx;
        f.y += acc.fy;
        f.z += acc.fz;
        f.w += acc.e;
        force[m] = f;
    }
    if (EV) {
        double v[7] = {acc.e, acc.w[0], acc.w[1], acc.w[2], acc.w[3], acc.w[4], acc.w[5]};
        wave_sum_store<7>(v, ev_part + (size_t)blockIdx.x * kEvWords);
    }
}

hipError_t launch_fene(const float4* pos, const int2* bonds, const int* rtag, int N, Box box, float K, float R02,
                       float4* force, double* ev_part, hipStream_t s) {
    if (ev_part)
        hipLaunchKernelGGL(k_fene<true>, dim3(nblk(N, kWave)), dim3(kWave), 0, s, pos, bonds, rtag, N, box, K, R02,
                           force, ev_part);
    else
        hipLaunchKernelGGL(k_fene<false>, dim3(nblk(N, kWave)), dim3(kWave), 0, s, pos, bonds, rtag, N, box, K, R02,
                           force, ev_part);
    return hipGetLastError();
}

// Bond counts of a batch: one 64-slot chunk per block (a chunk lies in one
// replica), a count per chunk, then one exact integer sum per replica.
__global__ __launch_bounds__(kWave) void k_bonds_batch(const float4* __restrict__ pos,
                                                      const int* __restrict__ nlist, const int* __restrict__ nn,
                                                      int k_max, int N, Table tab, const RepDesc* __restrict__ rep,
                                                      const int* __restrict__ chunk_rep,
                                                      unsigned long long* __restrict__ part) {
    extern __shared__ DevEntry s_tab[];
    const RepDesc& d = rep[chunk_rep[blockIdx.x]];
    load_table(s_tab, Table{tab.e + d.tab, tab.nt});
    const int i = blockIdx.x * kWave + threadIdx.x;
    unsigned c = 0;
    if (i < d.off + d.n) {
        const float4 pi = pos[i];
        walk_list<true, 4>(i, pi, ptype(pi.w), nlist, nn[i], k_max, N, pos, s_tab, tab.nt, d.box, -1,
                        [&](int j, const float4&, const DevEntry&, const PairGeom& pg) {
                            if (j > i && pg.bond) ++c;
                        });
    }
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) c += __shfl_xor(c, o, kWave);
    if (threadIdx.x == 0) part[blockIdx.x] = c;
}

__global__ __launch_bounds__(kBlock) void k_sum_u64_batch(const unsigned long long* __restrict__ part,
                                                         const RepDesc* __restrict__ rep,
                                                         unsigned long long* __restrict__ out) {
    __shared__ unsigned long long red[kBlock];
    const RepDesc& d = rep[blockIdx.x];
    const int c0 = d.off / kWave, nc = (d.n + kWave - 1) / kWave;
    unsigned long long s = 0;
    for (int b = threadIdx.x; b < nc; b += blockDim.x) s += part[c0 + b];
    red[threadIdx.x] = s;
    __syncthreads();
    for (int w = kBlock / 2; w > 0; w >>= 1) {
        if (threadIdx.x < w) red[threadIdx.x] += red[threadIdx.x + w];
        __syncthreads();
    }
    if (threadIdx.x == 0) out[blockIdx.x] = red[0];
}

hipError_t launch_bonds_batch(const float4* pos, const int* nlist, const int* nn, int k_max, int N, Table tab,
                              const RepDesc* rep, const int* chunk_rep, int R, unsigned long long* count,
                              unsigned long long* part, hipStream_t s) {
    const size_t shm = sizeof(DevEntry) * tab.nt * tab.nt;
    hipLaunchKernelGGL(k_bonds_batch, dim3(nblk(N, kWave)), dim3(kWave), shm, s, pos, nlist, nn, k_max, N, tab,
                       rep, chunk_rep, part);
    hipLaunchKernelGGL(k_sum_u64_batch, dim3(R), dim3(kBlock), 0, s, part, rep, count);
    return hipGetLastError();
}

// Fold the per-block slots of the step kernel into the status word (OR of
// flags, min of first steps), reset the slots, and raise status[MAXPATH] to
// the largest vel.w (path lengths only grow between list builds, and a build
// zeroes the status word).  One launch per chunk; one atomic per block and word.
__global__ __launch_bounds__(kBlock) void k_fold_status(int* __restrict__ blk, int nb,
                                                       const float4* __restrict__ vel, int N,
                                                       int* __restrict__ status) {
    __shared__ int r_fl[kBlock / kWave], r_s[kBlock / kWave], r_h[kBlock / kWave];
    __shared__ float r_p[kBlock / kWave];
    const int tid = blockIdx.x * blockDim.x + threadIdx.x, stride = gridDim.x * blockDim.x;
    int fl = 0, fs = 0x7fffffff, fh = 0x7fffffff;
    for (int b = tid; b < nb; b += stride) {
        fl |= blk[3 * b];
        fs = min(fs, blk[3 * b + 1]);
        fh = min(fh, blk[3 * b + 2]);
        blk[3 * b] = 0;
        blk[3 * b + 1] = 0x7fffffff;
        blk[3 * b + 2] = 0x7fffffff;
    }
    float pm = 0.0f;
    if (vel) {   // sixteen path lengths in flight per thread (a maximum: exact in any order)
        constexpr int U = 16;
        int i = tid;
        for (; i + (U - 1) * stride < N; i += U * stride) {
            float v[U];
#pragma unroll
            for (int u = 0; u < U; ++u) v[u] = vel[i + u * stride].w;
#pragma unroll
            for (int u = 0; u < U; ++u) pm = fmaxf(pm, v[u]);
        }
        for (; i < N; i += stride) pm = fmaxf(pm, vel[i].w);
    }
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) {
        fl |= __shfl_xor(fl, o, kWave);
        fs = min(fs, __shfl_xor(fs, o, kWave));
        fh = min(fh, __shfl_xor(fh, o, kWave));
        pm = fmaxf(pm, __shfl_xor(pm, o, kWave));
    }
    const int w = threadIdx.x / kWave;
    if ((threadIdx.x & (kWave - 1)) == 0) {
        r_fl[w] = fl;
        r_s[w] = fs;
        r_h[w] = fh;
        r_p[w] = pm;
    }
    __syncthreads();
    if (threadIdx.x == 0) {
        for (int q = 1; q < kBlock / kWave; ++q) {
            fl |= r_fl[q];
            fs = min(fs, r_s[q]);
            fh = min(fh, r_h[q]);
            pm = fmaxf(pm, r_p[q]);
        }
        fl |= r_fl[0];
        fs = min(fs, r_s[0]);
        fh = min(fh, r_h[0]);
        pm = fmaxf(pm, r_p[0]);
        if (fl) atomicOr(&status[RC_ST_FLAGS], fl);
        if (fs != 0x7fffffff) atomicMin(&status[RC_ST_FIRST_SOFT], fs);
        if (fh != 0x7fffffff) atomicMin(&status[RC_ST_FIRST_HARD], fh);
        if (vel) atomicMax(&status[RC_ST_MAXPATH], __float_as_int(pm));
    }
}

hipError_t launch_fold_status(int* blk, int nb, const float4* vel, int N, int* status, hipStream_t s) {
    // at most 256 blocks: each ends with atomics on the same status words (2048 blocks took 26 us at 1M
    // particles against 8.5 us)
    const int work = vel ? std::max(N, nb) : nb;
    hipLaunchKernelGGL(k_fold_status, dim3(std::max(1, std::min(nblk(work, kBlock), 256))), dim3(kBlock), 0, s,
                       blk, nb, vel, N, status);
    return hipGetLastError();
}

// Per-replica fold of a batch chunk, before k_fold_status resets the block
// slots, in two launches: the largest path length of every 64-slot chunk
// (one wavefront per chunk, all chunks in parallel), then one workgroup per
// replica over its chunks' maxima and block flags, which stores the flag of
// any block that crossed the rebuild threshold and the largest path length;
// status[MAXPATH] is raised to the largest of all.  Path lengths are
// non-negative, so their float bits order like ints.
__global__ __launch_bounds__(kBlock) void k_chunk_paths(const float4* __restrict__ vel, int nb,
                                                       float* __restrict__ chunk_path) {
    const int ch = (blockIdx.x * blockDim.x + threadIdx.x) / kWave;
    if (ch >= nb) return;   // uniform per wavefront
    const float p = wave_maxf(vel[(size_t)ch * kWave + (threadIdx.x & (kWave - 1))].w);
    if ((threadIdx.x & (kWave - 1)) == 0) chunk_path[ch] = p;
}

__global__ __launch_bounds__(kBlock) void k_fold_reps(const int* __restrict__ blk,
                                                     const float* __restrict__ chunk_path,
                                                     const RepDesc* __restrict__ rep, int* __restrict__ rep_flag,
                                                     int* __restrict__ rep_path, int* __restrict__ status) {
    __shared__ float r_p[kBlock / kWave];
    __shared__ int r_f[kBlock / kWave];
    const int r = blockIdx.x;
    const int c0 = rep[r].off / kWave, c1 = (rep[r].off + rep[r].n + kWave - 1) / kWave;
    float pm = 0.0f;
    int fl = 0;
    for (int c = c0 + (int)threadIdx.x; c < c1; c += blockDim.x) {
        pm = fmaxf(pm, chunk_path[c]);
        fl |= blk[3 * c] & RC_FLAG_REBUILD;
    }
    pm = wave_maxf(pm);
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) fl |= __shfl_xor(fl, o, kWave);
    if ((threadIdx.x & (kWave - 1)) == 0) {
        r_p[threadIdx.x / kWave] = pm;
        r_f[threadIdx.x / kWave] = fl;
    }
    __syncthreads();
    if (threadIdx.x == 0) {
        for (int q = 1; q < kBlock / kWave; ++q) {
            pm = fmaxf(pm, r_p[q]);
            fl |= r_f[q];
        }
        rep_flag[r] = fl != 0;
        rep_path[r] = __float_as_int(pm);
        atomicMax(&status[RC_ST_MAXPATH], __float_as_int(pm));
    }
}

hipError_t launch_fold_reps(const int* blk, const float4* vel, int nb, const RepDesc* rep, int R, int* out,
                            float* chunk_path, int* status, hipStream_t s) {
    hipLaunchKernelGGL(k_chunk_paths, dim3(nblk((long)nb * kWave, kBlock)), dim3(kBlock), 0, s, vel, nb, chunk_path);
    hipLaunchKernelGGL(k_fold_reps, dim3(R), dim3(kBlock), 0, s, blk, chunk_path, rep, out, out + R, status);
    return hipGetLastError();
}

// the driver's snapshot of (pos, vel, image) and its restore, in one launch
__global__ __launch_bounds__(kBlock) void k_copy_state(const float4* __restrict__ pos, const float4* __restrict__ vel,
                                                      const int4* __restrict__ image, float4* __restrict__ pos_to,
                                                      float4* __restrict__ vel_to, int4* __restrict__ image_to,
                                                      int N, int zero_path) {
    const int i = blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= N) return;
    pos_to[i] = pos[i];
    float4 v = vel[i];
    if (zero_path) v.w = 0.0f;
    vel_to[i] = v;
    if (image && image_to) image_to[i] = image[i];
}

hipError_t launch_copy_state(const float4* pos, const float4* vel, const int4* image, float4* pos_to, float4* vel_to,
                             int4* image_to, int N, hipStream_t s, bool zero_path) {
    hipLaunchKernelGGL(k_copy_state, dim3(nblk(N, kBlock)), dim3(kBlock), 0, s, pos, vel, image, pos_to, vel_to,
                       image_to, N, zero_path ? 1 : 0);
    return hipGetLastError();
}

__global__ __launch_bounds__(kBlock) void k_blk_reset(int* __restrict__ blk, int nb) {
    for (int b = blockIdx.x * blockDim.x + threadIdx.x; b < nb; b += gridDim.x * blockDim.x) {
        blk[3 * b] = 0;
        blk[3 * b + 1] = 0x7fffffff;
        blk[3 * b + 2] = 0x7fffffff;
    }
}

hipError_t launch_blk_reset(int* blk, int nb, hipStream_t s) {
    hipLaunchKernelGGL(k_blk_reset, dim3(std::min(nblk(nb, kBlock), 1024)), dim3(kBlock), 0, s, blk, nb);
    return hipGetLastError();
}

// ---------------------------------------------------------------------------
// fixed-order FP64 reduction of block partial rows
// ---------------------------------------------------------------------------
// Thread t's slice of one word: rows t, t + 256, t + 512, ... added in that
// order; the loads of 32 rows are issued before their adds (the same sum,
// without a load round trip per row).
__device__ __forceinline__ double strided_row_sum(const double* __restrict__ p, int nblocks, int q) {
    constexpr int U = 32;
    double s = 0.0;
    int b = threadIdx.x;
    for (; b + (U - 1) * kBlock < nblocks; b += U * kBlock) {
        double v[U];
#pragma unroll
        for (int u = 0; u < U; ++u) v[u] = p[(size_t)(b + u * kBlock) * kEvWords + q];
#pragma unroll
        for (int u = 0; u < U; ++u) s += v[u];
    }
    for (; b < nblocks; b += kBlock) s += p[(size_t)b * kEvWords + q];
    return s;
}

__global__ __launch_bounds__(kBlock) void k_reduce_rows(const double* __restrict__ part, int nblocks,
                                                       int first, int count, double* __restrict__ out) {
    // one block per output word; each thread sums a strided slice, then a tree
    __shared__ double red[kBlock];
    const int q = first + blockIdx.x;
    const double s = strided_row_sum(part, nblocks, q);
    red[threadIdx.x] = s;
    __syncthreads();
    for (int w = kBlock / 2; w > 0; w >>= 1) {
        if (threadIdx.x < w) red[threadIdx.x] += red[threadIdx.x + w];
        __syncthreads();
    }
    if (threadIdx.x == 0) out[blockIdx.x] = red[0];
}

// The same sums in two launches, for the driver's log rows: first every
// (thread slice t, word q) sum of k_reduce_rows, one thread each, with the
// threads of a wavefront on consecutive words of consecutive rows (coalesced
// reads spread over many CUs instead of 13 CUs each reading every row), then
// per word the same tree over the 256 slices.  Bit for bit k_reduce_rows.
// With bonds, one more column sums the per-block bond counts (64-bit integers,
// exact in any order) into *bonds_out.
__global__ __launch_bounds__(kWave) void k_row_slices(const double* __restrict__ part, int nblocks, int first,
                                                     int count, double* __restrict__ slice,
                                                     const unsigned* __restrict__ bonds) {
    const int cols = count + (bonds ? 1 : 0);
    const int i = blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= kBlock * cols) return;
    const int t = i / cols, qc = i % cols;
    constexpr int U = 16;
    if (qc == count) {
        unsigned long long n = 0;
        int b = t;
        for (; b + (U - 1) * kBlock < nblocks; b += U * kBlock) {
            unsigned v[U];
#pragma unroll
            for (int u = 0; u < U; ++u) v[u] = bonds[b + u * kBlock];
#pragma unroll
            for (int u = 0; u < U; ++u) n += v[u];
        }
        for (; b < nblocks; b += kBlock) n += bonds[b];
        reinterpret_cast<unsigned long long*>(slice)[i] = n;
        return;
    }
    const int q = first + qc;
    double s = 0.0;
    int b = t;
    for (; b + (U - 1) * kBlock < nblocks; b += U * kBlock) {
        double v[U];
#pragma unroll
        for (int u = 0; u < U; ++u) v[u] = part[(size_t)(b + u * kBlock) * kEvWords + q];
#pragma unroll
        for (int u = 0; u < U; ++u) s += v[u];
    }
    for (; b < nblocks; b += kBlock) s += part[(size_t)b * kEvWords + q];
    slice[i] = s;
}

__global__ __launch_bounds__(kBlock) void k_row_tree(const double* __restrict__ slice, int count,
                                                    double* __restrict__ out,
                                                    unsigned long long* __restrict__ bonds_out) {
    const int cols = count + (bonds_out ? 1 : 0);
    if ((int)blockIdx.x == count) {   // the bond column (launched with bonds_out only)
        __shared__ unsigned long long redn[kBlock];
        redn[threadIdx.x] = reinterpret_cast<const unsigned long long*>(slice)[threadIdx.x * cols + count];
        __syncthreads();
        for (int w = kBlock / 2; w > 0; w >>= 1) {
            if (threadIdx.x < w) redn[threadIdx.x] += redn[threadIdx.x + w];
            __syncthreads();
        }
        if (threadIdx.x == 0) *bonds_out = redn[0];
        return;
    }
    __shared__ double red[kBlock];
    red[threadIdx.x] = slice[threadIdx.x * cols + blockIdx.x];
    __syncthreads();
    for (int w = kBlock / 2; w > 0; w >>= 1) {
        if (threadIdx.x < w) red[threadIdx.x] += red[threadIdx.x + w];
        __syncthreads();
    }
    if (threadIdx.x == 0) out[blockIdx.x] = red[0];
}

hipError_t launch_reduce_rows(const double* part, int nblocks, int first, int count, double* out,
                              hipStream_t s, double* slice, const unsigned* bonds, unsigned long long* bonds_out) {
    if ((bonds != nullptr) != (bonds_out != nullptr) || (bonds && !slice)) return hipErrorInvalidValue;
    if (slice && count <= kEvWords) {
        const int cols = count + (bonds ? 1 : 0);   // kBlock * cols <= kRowSlices
        hipLaunchKernelGGL(k_row_slices, dim3(nblk((long)kBlock * cols, kWave)), dim3(kWave), 0, s, part, nblocks,
                           first, count, slice, bonds);
        hipLaunchKernelGGL(k_row_tree, dim3(cols), dim3(kBlock), 0, s, slice, count, out, bonds_out);
    } else {
        hipLaunchKernelGGL(k_reduce_rows, dim3(count), dim3(kBlock), 0, s, part, nblocks, first, count, out);
    }
    return hipGetLastError();
}

// The same fixed-order sum per replica over its own chunk rows (grid: words x
// replicas), so a replica's sums equal those of the system run on its own.
// bonds: per-chunk bond counts, summed by one more column of blocks (NULL: none).
__global__ __launch_bounds__(kBlock) void k_reduce_rows_batch(const double* __restrict__ part,
                                                             const RepDesc* __restrict__ rep, int first,
                                                             double* __restrict__ out, int out_stride,
                                                             const unsigned* __restrict__ bonds,
                                                             unsigned long long* __restrict__ bonds_out) {
    __shared__ double red[kBlock];
    const RepDesc& d = rep[blockIdx.y];
    const double* p = part + (size_t)(d.off / kWave) * kEvWords;
    const int nblocks = (d.n + kWave - 1) / kWave;
    if (bonds && blockIdx.x == gridDim.x - 1) {   // whole numbers below 2^53: exact in FP64
        double t = 0.0;
        for (int b = threadIdx.x; b < nblocks; b += blockDim.x) t += (double)bonds[d.off / kWave + b];
        t = wave_sum(t);
        if ((threadIdx.x & (kWave - 1)) == 0) red[threadIdx.x / kWave] = t;
        __syncthreads();
        if (threadIdx.x == 0) {
            for (int w = 1; w < kBlock / kWave; ++w) t += red[w];
            bonds_out[blockIdx.y] = (unsigned long long)t;
        }
        return;
    }
    const int q = first + blockIdx.x;
    const double s = strided_row_sum(p, nblocks, q);
    red[threadIdx.x] = s;
    __syncthreads();
    for (int w = kBlock / 2; w > 0; w >>= 1) {
        if (threadIdx.x < w) red[threadIdx.x] += red[threadIdx.x + w];
        __syncthreads();
    }
    if (threadIdx.x == 0) out[(size_t)blockIdx.y * out_stride + blockIdx.x] = red[0];
}

hipError_t launch_reduce_rows_batch(const double* part, const RepDesc* rep, int R, int first, int count,
                                    double* out, int out_stride, hipStream_t s, const unsigned* bonds,
                                    unsigned long long* bonds_out) {
    hipLaunchKernelGGL(k_reduce_rows_batch, dim3(count + (bonds ? 1 : 0), R), dim3(kBlock), 0, s, part, rep, first, out,
                       out_stride, bonds, bonds_out);
    return hipGetLastError();
}

__global__ void k_status_reset_chunk(int* st, unsigned long long* base, unsigned long long step) {
    chunk_reset(st, base, step);
}
hipError_t launch_status_reset_chunk(int* status, hipStream_t s, unsigned long long* step_base,
                                     unsigned long long step) {
    hipLaunchKernelGGL(k_status_reset_chunk, dim3(1), dim3(1), 0, s, status, step_base, step);
    return hipGetLastError();
}

__global__ void k_zero_words(int* p, int n) {
    for (int i = threadIdx.x; i < n; i += blockDim.x) p[i] = 0;
}
hipError_t launch_zero_words(int* p, int n, hipStream_t s) {
    hipLaunchKernelGGL(k_zero_words, dim3(1), dim3(64), 0, s, p, n);
    return hipGetLastError();
}

__global__ void k_add_step(unsigned long long* p, unsigned long long v) { *p += v; }
hipError_t launch_add_step(unsigned long long* p, unsigned long long v, hipStream_t s) {
    hipLaunchKernelGGL(k_add_step, dim3(1), dim3(1), 0, s, p, v);
    return hipGetLastError();
}
// The module is loaded with the first use of one of its functions: 2.7 ms once per process, and a run that follows
// within half a millisecond was seen to stall for 0.14 ms (20 steps of 1048576 particles after 5: 31.2-32.0 us per
// step with the module loaded before, else 38.1-39.3 in most processes).  A context's creation asks for it, so that
// no run pays.
hipError_t load_step_kernels() {
    hipFuncAttributes at{};
    return hipFuncGetAttributes(&at, reinterpret_cast<const void*>(&k_add_step));
}
void add_step_kernel_info(const void** fn) { *fn = reinterpret_cast<const void*>(&k_add_step); }

__global__ void k_set_step(unsigned long long* p, unsigned long long v) { *p = v; }
hipError_t launch_set_step(unsigned long long* p, unsigned long long v, hipStream_t s) {
    hipLaunchKernelGGL(k_set_step, dim3(1), dim3(1), 0, s, p, v);
    return hipGetLastError();
}

}  // namespace rc
