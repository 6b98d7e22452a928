// Observables built on the step.
//
// Bond-partner statistics between two tag-indexed partner snapshots (as
// rc_bond_partners writes them): over the selected tags, the particles bonded
// at 0, those whose partner is unchanged (the numerator of the bond
// autocorrelation, Sec. 3.1 / Fig. 3) and those whose single partner is now
// another particle (a swap event).  Wavefront ballots give per-block counts;
// a second kernel adds the block counts (integers: the order does not
// matter).
//
// The stress autocorrelation G(t) (the relaxation modulus by the
// autocorrelation method, Sec. 2.2 after eq. p3) of a series of logged rows
// (E, W(6), K(6)): V/kT times the average over the off-diagonal components
// xy, xz, yz and over every time origin of sigma(t0) sigma(t0 + t), with
// sigma_ab = -(K_ab + W_ab)/V.  FP64, a lag or a tile of lags per block, a fixed order
// of additions.
#include "rc_gather.h"

namespace rc {

static inline int nblk(long n, int b) { return (int)((n + b - 1) / b); }

__global__ __launch_bounds__(kBlock) void k_partner_counts(const int* __restrict__ p0, const int* __restrict__ pt,
                                                           const unsigned char* __restrict__ sel, int N,
                                                           unsigned long long* __restrict__ part) {
    const int i = blockIdx.x * blockDim.x + threadIdx.x;
    bool b = false, u = false, w = false;
    if (i < N && (!sel || sel[i])) {
        const int a = p0[i];
        if (a >= 0) {
            const int c = pt[i];
            b = true;
            u = c == a;
            w = c >= 0 && c != a;
        }
    }
    const unsigned long long bb = __ballot(b), bu = __ballot(u), bw = __ballot(w);
    __shared__ unsigned long long s_cnt[kBlock / kWave][3];
    const int lane = threadIdx.x & (kWave - 1), wv = threadIdx.x / kWave;
    if (lane == 0) {
        s_cnt[wv][0] = (unsigned long long)__popcll(bb);
        s_cnt[wv][1] = (unsigned long long)__popcll(bu);
        s_cnt[wv][2] = (unsigned long long)__popcll(bw);
    }
    __syncthreads();
    if (threadIdx.x < 3) {
        unsigned long long t = 0;
        for (int q = 0; q < kBlock / kWave; ++q) t += s_cnt[q][threadIdx.x];
        part[(size_t)blockIdx.x * 3 + threadIdx.x] = t;
    }
}

__global__ __launch_bounds__(kBlock) void k_sum_counts3(const unsigned long long* __restrict__ part, int nb,
                                                        unsigned long long* __restrict__ out) {
    __shared__ unsigned long long red[3][kBlock];
    unsigned long long s[3] = {0, 0, 0};
    for (int b = threadIdx.x; b < nb; b += blockDim.x)
        for (int q = 0; q < 3; ++q) s[q] += part[(size_t)b * 3 + q];
    for (int q = 0; q < 3; ++q) red[q][threadIdx.x] = s[q];
    __syncthreads();
    for (int w = kBlock / 2; w > 0; w >>= 1) {
        if (threadIdx.x < w)
            for (int q = 0; q < 3; ++q) red[q][threadIdx.x] += red[q][threadIdx.x + w];
        __syncthreads();
    }
    if (threadIdx.x < 3) out[threadIdx.x] = red[threadIdx.x][0];
}

hipError_t launch_partner_counts(const int* p0, const int* pt, const unsigned char* sel, int N,
                                 unsigned long long* part, unsigned long long* out, hipStream_t s) {
    const int nb = nblk(N, kBlock);
    hipLaunchKernelGGL(k_partner_counts, dim3(nb), dim3(kBlock), 0, s, p0, pt, sel, N, part);
    hipLaunchKernelGGL(k_sum_counts3, dim3(1), dim3(kBlock), 0, s, part, nb, out);
    return hipGetLastError();
}

// The off-diagonal stresses of the rows, s[c][t] for c = xy, xz, yz (W at 4 + c, K at 10 + c of a row)
__device__ __forceinline__ double row_stress(const double* r, int c, double inv_v) {
    return -(r[10 + c] + r[4 + c]) * inv_v;
}

__global__ __launch_bounds__(kBlock) void k_stress_rows(const double* __restrict__ rows, int T, double inv_v,
                                                        double* __restrict__ s) {
    const int t = blockIdx.x * blockDim.x + threadIdx.x;
    if (t >= T) return;
#pragma unroll
    for (int c = 0; c < 3; ++c) s[(size_t)c * T + t] = row_stress(rows + (size_t)t * kEvWords, c, inv_v);
}

// One block per lag, from the rows: the better form for at most one lag per CU (100000 rows, 101 lags 148 us,
// 2000 rows 7.7; from the stresses of a launch before 156 and 11), and for short series (plain_stress).
__global__ __launch_bounds__(kBlock) void k_stress_acf_few(const double* __restrict__ rows, int T, double inv_v,
                                                           double v_over_kt, double* __restrict__ G) {
    const int t = blockIdx.x;  // lag
    double acc = 0.0;
    for (int t0 = threadIdx.x; t0 < T - t; t0 += blockDim.x) {
        const double* a = rows + (size_t)t0 * kEvWords;
        const double* b = rows + (size_t)(t0 + t) * kEvWords;
        for (int c = 0; c < 3; ++c) acc += row_stress(a, c, inv_v) * row_stress(b, c, inv_v);
    }
    __shared__ double red[kBlock];
    red[threadIdx.x] = acc;
    __syncthreads();
    for (int w = kBlock / 2; w > 0; w >>= 1) {
        if (threadIdx.x < w) red[threadIdx.x] += red[threadIdx.x + w];
        __syncthreads();
    }
    if (threadIdx.x == 0) G[t] = v_over_kt * red[0] / (3.0 * (double)(T - t));
}

// A block of 512 threads computes 32 consecutive lags of one component (two
// groups of threads, 16 lags each).  It walks the time origins in chunks: the
// stresses of the chunk's origins and of the rows its lags reach are staged in
// LDS, and each thread multiplies 8 consecutive origins with 16 lags out of a
// register window: 31 LDS reads for 128 products, about what the LDS and the
// FP64 units of a CU take the same time for.  Read from the 104-byte rows, a
// block per 32 lags for the three components, the reads took four times the
// products (an address unit takes a cycle for each lane of such a stride) and
// 5001 lags made 157 blocks.  The next chunk is requested before this one is
// multiplied.  The LDS index skips one double in every 8, so that lanes 8 apart
// fall on different banks.
// us, a block per lag, from the rows, and this with its two small launches (rows, lags): (8000, 2001) 96, 21, 15;
// (20000, 1001) 126, 43, 21; (20000, 5001) 549, 56, 37.
constexpr int kAcfThreads = 512;
constexpr int kAcfLags = 16;
constexpr int kAcfRows = 2048;   // rows of each series in LDS

// ROWS: without scratch, a block per 32 lags takes the three components from the rows, one after the other.
template <bool ROWS>
__global__ __launch_bounds__(kAcfThreads) void k_stress_acf(const double* __restrict__ src, int T, int max_lag,
                                                            double inv_v, double v_over_kt, double* __restrict__ out) {
    constexpr int LG = 2;
    constexpr int kGroup = kAcfThreads / LG;           // threads per group of lags
    constexpr int kOwn = kAcfRows / kGroup;            // origins per thread
    constexpr int kChunk = kAcfRows - LG * kAcfLags;   // origins per chunk
    constexpr int kFlight = kAcfRows / kAcfThreads;    // rows per thread and series
    auto at = [](int i) { return i + i / kOwn; };
    constexpr int kS = kAcfRows + kAcfRows / kOwn;
    __shared__ double s_a[kS];
    __shared__ double s_b[kS];
    __shared__ double s_sum[kAcfThreads / kWave][kAcfLags];
    const int l0 = blockIdx.x * (LG * kAcfLags);   // the block's first lag (<= max_lag < T)
    const int grp = threadIdx.x / kGroup, own = (threadIdx.x % kGroup) * kOwn;
    const int off = own + grp * kAcfLags;
    // kAcfRows stresses from r0 on (the last one in place of those past the end)
    auto request = [&](int c, int r0, double (&v)[kFlight]) {
#pragma unroll
        for (int u = 0; u < kFlight; ++u) {
            const size_t t = min(r0 + (int)threadIdx.x + u * kAcfThreads, T - 1);
            v[u] = ROWS ? row_stress(src + t * kEvWords, c, inv_v) : src[(size_t)c * T + t];
        }
    };
    auto store = [&](const double (&v)[kFlight], double* d) {
#pragma unroll
        for (int u = 0; u < kFlight; ++u) d[at(threadIdx.x + u * kAcfThreads)] = v[u];
    };
    double acc[kAcfLags] = {};
    for (int c = ROWS ? 0 : blockIdx.y, end = ROWS ? 3 : c + 1; c < end; ++c) {
        double ra[kFlight], rb[kFlight];
        request(c, 0, ra);
        request(c, l0, rb);
        for (int t0 = 0; t0 < T - l0; t0 += kChunk) {
            __syncthreads();
            store(ra, s_a);
            store(rb, s_b);
            __syncthreads();
            if (t0 + kChunk < T - l0) {
                request(c, t0 + kChunk, ra);
                request(c, t0 + kChunk + l0, rb);
            }
            const int i0 = t0 + own, lag = l0 + grp * kAcfLags;   // the thread's first origin and lag
            if (own >= kChunk || i0 + lag >= T) continue;
            if (i0 + kOwn - 1 + lag + kAcfLags - 1 < T) {   // every product of the thread exists
                double a[kOwn], b[kOwn + kAcfLags - 1];
#pragma unroll
                for (int u = 0; u < kOwn; ++u) a[u] = s_a[at(own) + u];
#pragma unroll
                for (int u = 0; u < kOwn + kAcfLags - 1; ++u) b[u] = s_b[at(off) + at(u)];
#pragma unroll
                for (int u = 0; u < kOwn; ++u)
#pragma unroll
                    for (int l = 0; l < kAcfLags; ++l) acc[l] += a[u] * b[u + l];
            } else {   // products past the series' end are cleared bitwise (whatever they are; no branches)
                const int live = T - i0 - lag;   // row u + l of the thread's lags exists when below this
#pragma unroll
                for (int u = 0; u < kOwn; ++u) {
                    const double a = s_a[at(own) + u];
#pragma unroll
                    for (int l = 0; l < kAcfLags; ++l) {
                        const long long p = __double_as_longlong(a * s_b[at(off) + at(u + l)]);
                        acc[l] += __longlong_as_double(p & (long long)((u + l - live) >> 31));
                    }
                }
            }
        }
    }
    // fixed order: the wavefront's sums, then the group's wavefronts one after the other
    wave_sum_store<kAcfLags>(acc, s_sum[threadIdx.x / kWave]);
    __syncthreads();
    const int t = l0 + (int)threadIdx.x;
    if (threadIdx.x < LG * kAcfLags && t <= max_lag) {
        constexpr int nw = kGroup / kWave;
        const int g = threadIdx.x / kAcfLags, l = threadIdx.x % kAcfLags;
        double sum = 0.0;
        for (int w = 0; w < nw; ++w) sum += s_sum[g * nw + w][l];
        if (ROWS) out[t] = v_over_kt * sum / (3.0 * (double)(T - t));
        else out[(size_t)blockIdx.y * (max_lag + 1) + t] = sum;
    }
}

__global__ __launch_bounds__(kBlock) void k_stress_sum(const double* __restrict__ part, int T, int n, double v_over_kt,
                                                       double* __restrict__ G) {
    const int t = blockIdx.x * blockDim.x + threadIdx.x;
    if (t < n) G[t] = v_over_kt * (part[t] + part[n + t] + part[2 * (size_t)n + t]) / (3.0 * (double)(T - t));
}

size_t stress_scratch_doubles(int T, int max_lag) {
    return max_lag < RC_STRESS_PLAIN_LAGS ? 0 : 3 * ((size_t)T + (size_t)max_lag + 1);
}

// Whether a block per lag takes the series.  Its time goes with the rows times the rounds of 256 lags; the tiles take
// three launches and a scratch whatever the length, and a few dozen blocks when it is short.  us, kernels and whole
// call from host rows, a block per lag and tiles: (rows, lags) (1000, 256) 4.3 and 52, 9.4 and 62; (2000, 500) 7.5 and
// 58, 9.6 and 63; (3000, 750) 14.7 and 68, 10.9 and 68; (5000, 416) 15.3 and 75, 12.0 and 76; (5000, 625) 22 and 83,
// 12.2 and 76; (7000, 256) 19 and 85, 13.2 and 83; (20000, 1000) 122 and 245, 21 and 137.
static bool plain_stress(int T, int n) {
    constexpr int g = RC_STRESS_PLAIN_LAGS;
    return n <= g || (long long)T * nblk(n, g) <= RC_STRESS_PLAIN_WORK;
}

hipError_t launch_stress_acf(const double* rows, int T, double volume, double kT, int max_lag, double* G,
                             double* scratch, hipStream_t s) {
    const int n = max_lag + 1;
    const double inv_v = 1.0 / volume, v_over_kt = volume / kT;
    const dim3 tiles(nblk(n, 2 * kAcfLags), 3), threads(kAcfThreads);
    if (plain_stress(T, n)) {
        hipLaunchKernelGGL(k_stress_acf_few, dim3(n), dim3(kBlock), 0, s, rows, T, inv_v, v_over_kt, G);
    } else if (!scratch) {
        hipLaunchKernelGGL(k_stress_acf<true>, dim3(tiles.x), threads, 0, s, rows, T, max_lag, inv_v, v_over_kt, G);
    } else {
        double* part = scratch + 3 * (size_t)T;
        hipLaunchKernelGGL(k_stress_rows, dim3(nblk(T, kBlock)), dim3(kBlock), 0, s, rows, T, inv_v, scratch);
        hipLaunchKernelGGL(k_stress_acf<false>, tiles, threads, 0, s, scratch, T, max_lag, inv_v, v_over_kt, part);
        hipLaunchKernelGGL(k_stress_sum, dim3(nblk(n, kBlock)), dim3(kBlock), 0, s, part, T, n, v_over_kt, G);
    }
    return hipGetLastError();
}

}  // namespace rc
