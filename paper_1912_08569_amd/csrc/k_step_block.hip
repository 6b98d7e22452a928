// Small systems in one workgroup.  A system of at most kBlockMaxN particles
// (key order) is advanced by G plain steps of the fused step in a single
// launch: the positions live in LDS for the whole replay (two buffers), the
// switching sums of the two-pass form too, the velocities in registers, and the
// steps are separated by workgroup barriers.  Every wavefront runs the same
// gather and integrator code as k_step on its particles, with its own LDS
// slices and wavefront-level barriers inside the gather, and writes the status
// slot of its 64-particle block, so the result is the same, bit for bit, as G
// launches of k_step (and of the switching sums first, in the two-pass form).
// At these sizes a step is bound by the latency of its dependent reads and of
// its arithmetic; LDS reads and workgroup barriers replace the global reads of
// data written by the previous launch on another XCD and the launches
// themselves.  512 dumbbells, us per step: launched 7.4, here 3.4.
#include <algorithm>

#include "rc_step.h"

namespace rc {

static inline int nblk(long n, int b) { return (int)((n + b - 1) / b); }

__host__ __device__ static inline size_t block_tab_bytes(int nt) {
    return (sizeof(DevEntry) * (size_t)nt * nt + 15) & ~size_t(15);
}

// particles per wavefront: the fewest of 32 and 64 that fit one workgroup
static int block_particles(int N) { return N <= 32 * kGatherMaxWaves ? 32 : kWave; }

// entries per wavefront kept in LDS (block_steps), and rows of entries kept in registers (block_steps_row)
constexpr int kBlockEntries = 256;
__host__ __device__ constexpr int block_rows(int ow) { return ow == kWave ? 3 : 2; }

// Dynamic LDS: the coefficient table, two position buffers, the sums, and per
// wavefront its entries or (rows) the staging of block_steps_row.
static size_t step_block_dyn_lds(int N, int nt, bool rows) {
    const size_t nthr = (size_t)((N + kWave - 1) / kWave) * kWave;
    const int ow = block_particles(N);
    const size_t ent = (sizeof(int) + 1) * kBlockEntries, stage = 3 * sizeof(float) * block_rows(ow) * kWave;
    return block_tab_bytes(nt) + 2 * sizeof(float4) * nthr + sizeof(float) * nthr +
           (size_t)nblk(N, ow) * (rows ? std::max(ent, stage) : ent);
}

// OW particles per wavefront: 64, or 32 where that still fits one workgroup (a
// wavefront's time is its rows of 64 entries one after the other).  The
// velocities stay in registers; the wavefront's entries of the packed list are
// kept in LDS when every wavefront's fit kBlockEntries, else read from
// the list every step.
template <bool SF, int OW>
__device__ __forceinline__ void block_steps(const StepArgs& a, const DevEntry* s_tab, float4* s_p0, float4* s_p1,
                                            float* s_S, const int* ent_j, const unsigned char* ent_o, size_t first,
                                            int lane0, int T, int my_off, int packed, int m, int w, bool live,
                                            uint64_t base, int G) {
    const int nt = a.tab.nt;
    const int lane = (int)threadIdx.x & (kWave - 1);
    const float4 zero = make_float4(0.f, 0.f, 0.f, 0.f);
    const OneSystem sys{s_tab, nt, a.box};
    __shared__ float s_w_w[SF ? kGatherMaxWaves : 1][2][kDefaultWidth * kWave];
    float4 vm = zero;
    if (live) vm = a.vel[m];
    for (int k = 0; k < G; ++k) {
        const float4* pin = (k & 1) ? s_p1 : s_p0;
        float4* pout = (k & 1) ? s_p0 : s_p1;
        float4 pm = zero;
        if (live) pm = pin[m];
        if constexpr (SF) {
            const float S = packed_sums<kDefaultWidth, OW, true>(m - lane, pin + (m - lane), my_off, nn_swap(packed), T,
                                                                 lane0, first, pin, ent_j, ent_o, s_tab, nt, a.box,
                                                                 s_w_w[w]);
            if (live) s_S[m] = S;
            __syncthreads();
        }
        Acc acc = {};
        wave_gather<false, kDefaultWidth, SF, OneSystem, kGatherMaxWaves, true, 1, OW>(m - lane, live, pm, packed, pin, a.nlist, a.nn,
                                                                            a.k_max, a.N, sys, acc, s_S, ent_j, ent_o,
                                                                            first, lane0);
        if (a.bonds && live)
            fene_add<false>(ptag(pm.w), pm, a.bonds, a.rtag, pin, a.box, a.fene_k, a.fene_r02, acc);
        step_finish<false, false, (OW < kWave)>(a, pout, m, m / kWave, live, pm, vm, acc, a.box, 0, a.seed,
                                                base + (uint64_t)k, nullptr, &vm);
        __syncthreads();
    }
}

// The two-pass form with a wavefront's entries in registers for the whole replay
// (at most NR rows of 64): an entry's terms are evaluated once per step, for the
// sums and for the forces, and with 32 particles per wavefront the idle half of
// the lanes draws the next step's noise.  s_w: 3 NR 64 floats of the wavefront's.
// us per step, block_steps and this: 512 dumbbells 5.6, 3.4 (aggregated 6.0, 3.9),
// 1000 of them 6.5, 4.6 (8.3, 5.6).
template <int OW, int NR>
__device__ __forceinline__ void block_steps_row(const StepArgs& a, const DevEntry* s_tab, float4* s_p0, float4* s_p1,
                                                float* s_S, const int* pl_j, const unsigned char* pl_o, size_t first,
                                                int lane0, int T, int my_off, int packed, int m, bool live,
                                                uint64_t base, int G, float (*s_w)[NR * kWave]) {
    const int nt = a.tab.nt;
    const int lane = (int)threadIdx.x & (kWave - 1);
    const int base_m = m - lane, ns = nn_swap(packed), cnt = ns + nn_other(packed);
    const float4 zero = make_float4(0.f, 0.f, 0.f, 0.f);
    int own[NR], j[NR];
#pragma unroll
    for (int r = 0; r < NR; ++r) {
        const int e = r * kWave + lane;
        own[r] = -1;
        j[r] = base_m;
        if (e < T) {
            own[r] = pl_o[first + e] - lane0;
            j[r] = pl_j[first + e];
        }
    }
    float4 vm = zero;
    if (live) vm = a.vel[m];
    float nz[3] = {0.f, 0.f, 0.f};
    for (int k = 0; k < G; ++k) {
        const float4* pin = (k & 1) ? s_p1 : s_p0;
        float4* pout = (k & 1) ? s_p0 : s_p1;
        float4 pm = zero;
        if (live) pm = pin[m];
        SwapEntry x[NR];
#pragma unroll
        for (int r = 0; r < NR; ++r) {
            if (r > 0 && T <= r * kWave) break;
            x[r] = SwapEntry{0.0f, 0.0f, 0.0f, 0.0f, 0.0f, 0.0f, 0.0f};
            if (own[r] >= 0) x[r] = swap_entry(pin[base_m + own[r]], pin[j[r]], s_tab, nt, a.box);
            s_w[0][r * kWave + lane] = x[r].sl;
            s_w[1][r * kWave + lane] = x[r].u;
        }
        gather_sync<true>();
        float S = 0.0f;
        for (int q = my_off; q < my_off + ns; ++q) S = __fmaf_rn(s_w[0][q], s_w[1][q], S);
        if (live) s_S[m] = S;
        // the noise while other wavefronts finish their sums
        float z[3] = {0.f, 0.f, 0.f};
        if (a.langevin) {
            if (OW == kWave || (k & 1) == 0) {
                const int ahead = lane / OW, mz = min(base_m + lane % OW, a.N - 1);
                thermostat_normals(a.seed, (uint32_t)ptag(pin[mz].w), base + (uint64_t)(k + ahead), nz[0], nz[1], nz[2]);
            }
            for (int q = 0; q < 3; ++q) z[q] = OW < kWave && (k & 1) ? __shfl(nz[q], lane % OW + OW % kWave, kWave) : nz[q];
        }
        __syncthreads();
#pragma unroll
        for (int r = 0; r < NR; ++r) {
            if (r > 0 && T <= r * kWave) break;
            float f = x[r].g;
            if (needs_sums(x[r])) f = swap_factor(x[r], s_S[base_m + own[r]], s_S[j[r]]);
            s_w[0][r * kWave + lane] = f * x[r].dx;
            s_w[1][r * kWave + lane] = f * x[r].dy;
            s_w[2][r * kWave + lane] = f * x[r].dz;
        }
        gather_sync<true>();
        Acc acc = {};
        for (int q = my_off; q < my_off + cnt; ++q) {
            acc.fx += s_w[0][q];
            acc.fy += s_w[1][q];
            acc.fz += s_w[2][q];
        }
        if (a.bonds && live)
            fene_add<false>(ptag(pm.w), pm, a.bonds, a.rtag, pin, a.box, a.fene_k, a.fene_r02, acc);
        step_finish<false, true, (OW < kWave)>(a, pout, m, m / kWave, live, pm, vm, acc, a.box, 0, a.seed,
                                               base + (uint64_t)k, z, &vm);
        __syncthreads();
    }
}

template <bool SF, int OW>
__global__ __launch_bounds__(kBlockMaxN) void k_step_block(StepArgs a, float4* __restrict__ pos_final,
                                                           unsigned long long* __restrict__ step_base, int G,
                                                           int stage) {
    extern __shared__ __align__(16) unsigned char s_dyn[];
    const int nt = a.tab.nt;
    const int np = ((a.N + kWave - 1) / kWave) * kWave;   // particles, rounded up
    DevEntry* s_tab = reinterpret_cast<DevEntry*>(s_dyn);
    float4* s_p0 = reinterpret_cast<float4*>(s_dyn + block_tab_bytes(nt));
    float4* s_p1 = s_p0 + np;
    float* s_S = reinterpret_cast<float*>(s_p1 + np);
    int* s_ej = reinterpret_cast<int*>(s_S + np);   // or block_steps_row's staging
    unsigned char* s_eo = reinterpret_cast<unsigned char*>(s_ej + (blockDim.x / kWave) * kBlockEntries);
    load_table(s_tab, a.tab);  // ends with a workgroup barrier
    const int lane = (int)threadIdx.x & (kWave - 1);
    const int w = (int)threadIdx.x / kWave;
    const int m = w * OW + lane, blk = w * OW / kWave, lane0 = w * OW % kWave;
    const bool live = lane < OW && m < a.N;
    const float4 zero = make_float4(0.f, 0.f, 0.f, 0.f);
    // (branches, not selects of the loaded value: a select becomes a select of addresses)
    float4 p_first = zero;
    if (live) p_first = a.pos_in[m];
    if (lane < OW && m < np) {
        s_p0[m] = p_first;
        s_p1[m] = zero;
    }
    // this wavefront's entries within those of its 64-particle block
    int nn64 = 0;
    if (blk * kWave + lane < a.N) nn64 = a.nn[blk * kWave + lane];
    const int cnt64 = nn_swap(nn64) + nn_other(nn64), inc64 = wave_inclusive_scan(cnt64);
    const int before = lane0 > 0 ? __builtin_amdgcn_readlane(inc64, lane0 - 1) : 0;
    const int T = __builtin_amdgcn_readlane(inc64, lane0 + OW - 1) - before;
    const int from = lane0 + min(lane, OW - 1);
    const int my_off = __shfl(inc64 - cnt64, from, kWave) - before;
    const int packed_any = __shfl(nn64, from, kWave);
    const int packed = live ? packed_any : 0;
    const size_t first = (size_t)blk * kWave * a.k_max + before;
    const uint64_t base = *step_base;
    constexpr int NR = block_rows(OW);
    const bool rows = SF && __syncthreads_and(stage && T <= NR * kWave) != 0;
    const bool fits = !rows && __syncthreads_and(T <= kBlockEntries) != 0;
    if (rows) {
        if constexpr (SF)
            block_steps_row<OW, NR>(a, s_tab, s_p0, s_p1, s_S, a.pl_j, a.pl_o, first, lane0, T, my_off, packed, m,
                                    live, base, G, reinterpret_cast<float(*)[NR * kWave]>(s_ej) + 3 * w);
    } else if (fits) {
        for (int e = lane; e < T; e += kWave) {
            s_ej[w * kBlockEntries + e] = a.pl_j[first + e];
            s_eo[w * kBlockEntries + e] = a.pl_o[first + e];
        }
        __syncthreads();
        block_steps<SF, OW>(a, s_tab, s_p0, s_p1, s_S, s_ej, s_eo, (size_t)w * kBlockEntries, lane0, T, my_off, packed,
                            m, w, live, base, G);
    } else {
        block_steps<SF, OW>(a, s_tab, s_p0, s_p1, s_S, a.pl_j, a.pl_o, first, lane0, T, my_off, packed, m, w,
                            live, base, G);
    }
    if (live) pos_final[m] = (G & 1) ? s_p1[m] : s_p0[m];   // the buffer the last step wrote
    if (threadIdx.x == 0) *step_base = base + (uint64_t)G;
}

static const void* block_fn(int N, int form) {
    if (block_particles(N) == 32)
        return form == RC_FORM_SUMS ? reinterpret_cast<const void*>(&k_step_block<true, 32>)
                                    : reinterpret_cast<const void*>(&k_step_block<false, 32>);
    return form == RC_FORM_SUMS ? reinterpret_cast<const void*>(&k_step_block<true, kWave>)
                                : reinterpret_cast<const void*>(&k_step_block<false, kWave>);
}

// Whether a system fits: particle count, form and the LDS the kernel needs
// (its static gather slices plus the dynamic part) within one workgroup.
bool step_block_fits(int N, int nt, int form, float list_len) {
    if (N < 1 || N > kBlockMaxN) return false;
    // A wavefront here holds 32 or 64 particles, launches of k_step_few as few as 8.  The two-pass form is faster here
    // while the entries of an average wavefront fit the registers (block_steps_row) but for an eighth, the walk form,
    // which evaluates every row by itself, up to about one row.  us per step here and launched (entries per wavefront):
    // sums 1000 of the assembly mixture (51) 4.1, 8.6; 1000 reactive of density 0.15 (148) 6.7, 9.6 and of density 0.25 (310) 16.1,
    // 9.9; 433 in a drop (126) 7.9, 9.3; 500 of density 0.25 (158) 10.5, 9.7; walk 1000 dumbbells (62) 7.9, 8.8; 300
    // reactive of density 0.1 (41) 7.9, 9.4; 1000 of them (79) 10.0, 9.4; 300 of density 0.15 (77) 13.1, 11.0
    const int ow = block_particles(N);
    if ((float)ow * list_len > (form == RC_FORM_SUMS ? 1.125f * (float)(block_rows(ow) * kWave) : 72.0f)) return false;
    const void* fn = block_fn(N, form);
    hipFuncAttributes at{};
    if (hipFuncGetAttributes(&at, fn) != hipSuccess) return false;
    int dev = 0, max_lds = 0;
    if (hipGetDevice(&dev) != hipSuccess ||
        hipDeviceGetAttribute(&max_lds, hipDeviceAttributeMaxSharedMemoryPerBlock, dev) != hipSuccess)
        return false;
    return at.sharedSizeBytes + step_block_dyn_lds(N, nt, false) <= (size_t)max_lds;
}

hipError_t launch_step_block(const StepArgs& a, float4* pos_final, unsigned long long* step_base, int G,
                             hipStream_t s) {
    if (a.N < 1 || a.N > kBlockMaxN || G < 1) return hipErrorInvalidValue;
    const void* fn = block_fn(a.N, a.form);
    const int ow = block_particles(a.N), waves = nblk(a.N, ow);
    size_t shm = step_block_dyn_lds(a.N, a.tab.nt, false);
    // with the staging of block_steps_row where it fits the LDS (a large table may leave no room)
    hipFuncAttributes at{};
    int dev = 0, max_lds = 0;
    hipError_t e = hipFuncGetAttributes(&at, fn);
    if (e == hipSuccess) e = hipGetDevice(&dev);
    if (e == hipSuccess) e = hipDeviceGetAttribute(&max_lds, hipDeviceAttributeMaxSharedMemoryPerBlock, dev);
    if (e != hipSuccess) return e;
    const size_t with_rows = step_block_dyn_lds(a.N, a.tab.nt, true);
    int stage = a.form == RC_FORM_SUMS && at.sharedSizeBytes + with_rows <= (size_t)max_lds;
    if (stage) shm = with_rows;
    e = hipFuncSetAttribute(fn, hipFuncAttributeMaxDynamicSharedMemorySize, (int)shm);
    if (e != hipSuccess) return e;
    const int nthr = waves * kWave;
    StepArgs arg = a;
    void* args[] = {&arg, &pos_final, &step_base, &G, &stage};
    return hipLaunchKernel(fn, dim3(1), dim3(nthr), args, shm, s);
}

}  // namespace rc
