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
// themselves.  512 dumbbells 7.1 -> 5.7 us per step, 1000 8.2 -> 7.3 (32
// particles per wavefront, flat switching sums, entries in LDS).
#include "rc_step.h"

namespace rc {

static inline int nblk(long n, int b) { return (int)((n + b - 1) / b); }

__host__ __device__ static inline size_t block_tab_bytes(int nt) {
    return (sizeof(DevEntry) * (size_t)nt * nt + 15) & ~size_t(15);
}

// Dynamic LDS: the coefficient table, two position buffers and the sums.
size_t step_block_dyn_lds(int N, int nt) {
    const size_t nthr = (size_t)((N + kWave - 1) / kWave) * kWave;
    return block_tab_bytes(nt) + 2 * sizeof(float4) * nthr + sizeof(float) * nthr;
}

// OW particles per wavefront: 64, or 32 where that still fits one workgroup (a
// wavefront's time is its rows of 64 entries one after the other).  The
// velocities stay in registers; the wavefront's entries of the packed list are
// kept in LDS when every wavefront's fit kBlockEntries (ENT), else read from
// the list every step.
template <bool SF, int OW, bool ENT>
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
        wave_gather<false, kDefaultWidth, SF, OneSystem, true, true, 1, OW>(m - lane, live, pm, packed, pin, a.nlist, a.nn,
                                                                            a.k_max, a.N, sys, acc, s_S, ent_j, ent_o,
                                                                            first, lane0);
        if (a.bonds && live)
            fene_add<false>(ptag(pm.w), pm, a.bonds, a.rtag, pin, a.box, a.fene_k, a.fene_r02, acc);
        step_finish<false, false, (OW < kWave)>(a, pout, m, m / kWave, live, pm, vm, acc, a.box, 0, a.seed,
                                                base + (uint64_t)k, nullptr, &vm);
        __syncthreads();
    }
}

constexpr int kBlockEntries = 256;

template <bool SF, int OW>
__global__ __launch_bounds__(kBlockMaxN) void k_step_block(StepArgs a, float4* __restrict__ pos_final,
                                                           unsigned long long* __restrict__ step_base, int G) {
    extern __shared__ __align__(16) unsigned char s_dyn[];
    __shared__ int s_ej[kGatherMaxWaves * kBlockEntries];
    __shared__ unsigned char s_eo[kGatherMaxWaves * kBlockEntries];
    const int nt = a.tab.nt;
    const int np = ((a.N + kWave - 1) / kWave) * kWave;   // particles, rounded up
    DevEntry* s_tab = reinterpret_cast<DevEntry*>(s_dyn);
    float4* s_p0 = reinterpret_cast<float4*>(s_dyn + block_tab_bytes(nt));
    float4* s_p1 = s_p0 + np;
    float* s_S = reinterpret_cast<float*>(s_p1 + np);
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
    const bool fits = __syncthreads_and(T <= kBlockEntries) != 0;
    if (fits) {
        for (int e = lane; e < T; e += kWave) {
            s_ej[w * kBlockEntries + e] = a.pl_j[first + e];
            s_eo[w * kBlockEntries + e] = a.pl_o[first + e];
        }
        __syncthreads();
        block_steps<SF, OW, true>(a, s_tab, s_p0, s_p1, s_S, s_ej, s_eo, (size_t)w * kBlockEntries, lane0, T, my_off,
                                  packed, m, w, live, base, G);
    } else {
        block_steps<SF, OW, false>(a, s_tab, s_p0, s_p1, s_S, a.pl_j, a.pl_o, first, lane0, T, my_off, packed, m, w,
                                   live, base, G);
    }
    if (live) pos_final[m] = s_p0[m];  // G is even: the last step wrote buffer 0
    if (threadIdx.x == 0) *step_base = base + (uint64_t)G;
}

// particles per wavefront: the fewest of 32 and 64 that fit one workgroup
static int block_particles(int N) { return N <= 32 * kGatherMaxWaves ? 32 : kWave; }

static const void* block_fn(int N, int form) {
    if (block_particles(N) == 32)
        return form == RC_FORM_SUMS ? reinterpret_cast<const void*>(&k_step_block<true, 32>)
                                    : reinterpret_cast<const void*>(&k_step_block<false, 32>);
    return form == RC_FORM_SUMS ? reinterpret_cast<const void*>(&k_step_block<true, kWave>)
                                : reinterpret_cast<const void*>(&k_step_block<false, kWave>);
}

// Whether a system fits: particle count, form and the LDS the kernel needs
// (its static gather slices plus the dynamic part) within one workgroup.
bool step_block_fits(int N, int nt, int form, float list_est) {
    if (N < 1 || N > kBlockMaxN) return false;
    // A wavefront here holds 32 or 64 particles, launches of k_step_few as few as 8: lists that make more than
    // about two rows of entries (three in the walk form, one launch per step there) are faster launched (us per
    // step here, launched: 1000 dumbbells 7.3, 9.3; 1000 of the assembly mixture 5.6, 8.2; reactive particles of
    // density 0.25, 300 of them 9.9, 10.0 and 1000 16.1, 10.0)
    if ((float)block_particles(N) * list_est > (form == RC_FORM_SUMS ? 160.0f : 240.0f)) return false;
    const void* fn = block_fn(N, form);
    hipFuncAttributes at{};
    if (hipFuncGetAttributes(&at, fn) != hipSuccess) return false;
    int dev = 0, max_lds = 0;
    if (hipGetDevice(&dev) != hipSuccess ||
        hipDeviceGetAttribute(&max_lds, hipDeviceAttributeMaxSharedMemoryPerBlock, dev) != hipSuccess)
        return false;
    return at.sharedSizeBytes + step_block_dyn_lds(N, nt) <= (size_t)max_lds;
}

hipError_t launch_step_block(const StepArgs& a, float4* pos_final, unsigned long long* step_base, int G,
                             hipStream_t s) {
    if (a.N < 1 || a.N > kBlockMaxN || (G & 1) || G < 2) return hipErrorInvalidValue;
    const void* fn = block_fn(a.N, a.form);
    const size_t shm = step_block_dyn_lds(a.N, a.tab.nt);
    hipError_t e = hipFuncSetAttribute(fn, hipFuncAttributeMaxDynamicSharedMemorySize, (int)shm);
    if (e != hipSuccess) return e;
    const int nthr = nblk(a.N, block_particles(a.N)) * kWave;
    StepArgs arg = a;
    void* args[] = {&arg, &pos_final, &step_base, &G};
    return hipLaunchKernel(fn, dim3(1), dim3(nthr), args, shm, s);
}

}  // namespace rc
