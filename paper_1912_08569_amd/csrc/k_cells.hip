// Cell binning (counting sort along a Morton curve of the cell grid) and the
// full neighbour list.  gfx950, wave64.
#include "rc_internal.h"

namespace rc {

// ---------------------------------------------------------------------------
// binning
// ---------------------------------------------------------------------------
// The status words before a list build (kStatusFold: the words of earlier work stay, the list's own are cleared).
__device__ __forceinline__ void status_begin(int* st, int mode) {
    if (mode != kStatusFold) {
        for (int w = 0; w < RC_STATUS_WORDS; ++w) st[w] = 0;
        if (mode == kStatusFresh) {
            st[RC_ST_FIRST_SOFT] = 0x7fffffff;
            st[RC_ST_FIRST_HARD] = 0x7fffffff;
        }
    }
    st[RC_ST_NSWAP] = 0;
    st[RC_ST_NLIST] = 0;
}

// counts cleared (n a multiple of 4); with status, its words for the list build that follows
__global__ __launch_bounds__(kBlock) void k_clear_counts(int* __restrict__ p, int n, int* status, int mode) {
    int4* p4 = reinterpret_cast<int4*>(p);
    for (int i = blockIdx.x * blockDim.x + threadIdx.x; i < n / 4; i += gridDim.x * blockDim.x)
        p4[i] = make_int4(0, 0, 0, 0);
    if (status && blockIdx.x == 0 && threadIdx.x == 0) status_begin(status, mode);
}

__global__ void k_status_begin(int* status, int mode) { status_begin(status, mode); }

// cell key of every particle and its arrival rank inside the cell
__device__ __forceinline__ int cell_key(const float4& p, const Box& b, const Grid& g) {
    const int cx = cell_coord(p.x, b.hf[0], g.inv_w[0], g.nc[0]);
    const int cy = cell_coord(p.y, b.hf[1], g.inv_w[1], g.nc[1]);
    const int cz = cell_coord(p.z, b.hf[2], g.inv_w[2], g.nc[2]);
    return (int)morton3(cx, cy, cz);
}

__global__ __launch_bounds__(kBlock) void k_bin(const float4* __restrict__ pos, int N, Box b, Grid g,
                                               int* __restrict__ counts, int* __restrict__ keys,
                                               int* __restrict__ rank) {
    int i = blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= N) return;
    const int key = cell_key(pos[i], b, g);
    keys[i] = key;
    rank[i] = atomicAdd(&counts[key], 1);
}

// ---- three-phase exclusive scan of counts[0..n) -----------------------------
__device__ __forceinline__ int wave_incl_scan(int v) {
    const int lane = threadIdx.x & (kWave - 1);
#pragma unroll
    for (int o = 1; o < kWave; o <<= 1) {
        int t = __shfl_up(v, o, kWave);
        if (lane >= o) v += t;
    }
    return v;
}

// exclusive block scan of one value per thread; returns the block total too
__device__ __forceinline__ int block_excl_scan(int v, int& total) {
    __shared__ int wsum[kBlock / kWave];
    const int lane = threadIdx.x & (kWave - 1), wid = threadIdx.x / kWave;
    int inc = wave_incl_scan(v);
    if (lane == kWave - 1) wsum[wid] = inc;
    __syncthreads();
    int off = 0, tot = 0;
#pragma unroll
    for (int w = 0; w < kBlock / kWave; ++w) {
        int s = wsum[w];
        off += (w < wid) ? s : 0;
        tot += s;
    }
    __syncthreads();
    total = tot;
    return off + inc - v;
}

// The tiles hold kScanItems = 8 counts per thread, read and written as two int4 (n is a multiple of 8: every
// grid has 8^k keys); one by one, 32 bytes apart, they took 12.0 us instead of 5.3 for 2.1 million keys.
struct Items {
    int v[kScanItems];
};
__device__ __forceinline__ Items load_items(const int* p) {
    static_assert(kScanItems == 8, "two int4");
    const int4 a = reinterpret_cast<const int4*>(p)[0], b = reinterpret_cast<const int4*>(p)[1];
    return Items{{a.x, a.y, a.z, a.w, b.x, b.y, b.z, b.w}};
}

__global__ __launch_bounds__(kBlock) void k_scan_reduce(const int* __restrict__ counts, int n,
                                                       int* __restrict__ block_sums) {
    const int base = blockIdx.x * kScanTile + threadIdx.x * kScanItems;
    int s = 0;
    if (base < n) {
        const Items t = load_items(counts + base);
#pragma unroll
        for (int q = 0; q < kScanItems; ++q) s += t.v[q];
    }
    int total;
    block_excl_scan(s, total);
    if (threadIdx.x == 0) block_sums[blockIdx.x] = total;
}

// one block of 1024 threads scans up to 8192 block sums; also writes start[n]
__global__ __launch_bounds__(1024) void k_scan_top(int* __restrict__ block_sums, int nb,
                                                  int* __restrict__ start, int n) {
    __shared__ int wsum[1024 / kWave];
    const int lane = threadIdx.x & (kWave - 1), wid = threadIdx.x / kWave;
    int v[8];
    int s = 0;
#pragma unroll
    for (int q = 0; q < 8; ++q) {
        int idx = threadIdx.x * 8 + q;
        v[q] = idx < nb ? block_sums[idx] : 0;
        s += v[q];
    }
    int inc = wave_incl_scan(s);
    if (lane == kWave - 1) wsum[wid] = inc;
    __syncthreads();
    int off = 0, tot = 0;
    for (int w = 0; w < 1024 / kWave; ++w) {
        off += (w < wid) ? wsum[w] : 0;
        tot += wsum[w];
    }
    int run = off + inc - s;
#pragma unroll
    for (int q = 0; q < 8; ++q) {
        int idx = threadIdx.x * 8 + q;
        if (idx < nb) block_sums[idx] = run;
        run += v[q];
    }
    if (threadIdx.x == 0) start[n] = tot;
}

// Exclusive prefixes of the counts; nb: tiles whose sums are summed here (0: block_sums holds their prefixes
// already).  Up to kScanFlat tiles every block adds up the sums before its own, which costs less than a launch.
constexpr int kScanFlat = 4 * kBlock;
__global__ __launch_bounds__(kBlock) void k_scan_down(const int* __restrict__ counts, int n,
                                                     const int* __restrict__ block_sums, int nb,
                                                     int* __restrict__ start) {
    const int base = blockIdx.x * kScanTile + threadIdx.x * kScanItems;
    Items t{};
    if (base < n) t = load_items(counts + base);
    int before = 0;
    if (nb > 0) {
        int p = 0;
#pragma unroll
        for (int q = 0; q < kScanFlat / kBlock; ++q) {
            const int b = q * kBlock + threadIdx.x;
            if (b < (int)blockIdx.x) p += block_sums[b];
        }
        block_excl_scan(p, before);
    } else {
        before = block_sums[blockIdx.x];
    }
    int s = 0;
#pragma unroll
    for (int q = 0; q < kScanItems; ++q) s += t.v[q];
    int total;
    int run = block_excl_scan(s, total) + before;
    if (nb > 0 && (int)blockIdx.x == nb - 1 && threadIdx.x == 0) start[n] = before + total;
    if (base < n) {
        int o[kScanItems];
#pragma unroll
        for (int q = 0; q < kScanItems; ++q) {
            o[q] = run;
            run += t.v[q];
        }
        int4* d = reinterpret_cast<int4*>(start + base);
        d[0] = make_int4(o[0], o[1], o[2], o[3]);
        d[1] = make_int4(o[4], o[5], o[6], o[7]);
    }
}

static void launch_scan(const int* counts, int nk, int* block_sums, int* start, hipStream_t s) {
    const int nsb = (nk + kScanTile - 1) / kScanTile;
    hipLaunchKernelGGL(k_scan_reduce, dim3(nsb), dim3(kBlock), 0, s, counts, nk, block_sums);
    const bool flat = nsb <= kScanFlat;
    if (!flat) hipLaunchKernelGGL(k_scan_top, dim3(1), dim3(1024), 0, s, block_sums, nsb, start, nk);
    hipLaunchKernelGGL(k_scan_down, dim3(nsb), dim3(kBlock), 0, s, counts, nk, block_sums, flat ? nsb : 0, start);
}

__global__ __launch_bounds__(kBlock) void k_scatter(const int* __restrict__ keys,
                                                   const int* __restrict__ rank,
                                                   const int* __restrict__ start, int N,
                                                   int* __restrict__ order) {
    int i = blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= N) return;
    order[start[keys[i]] + rank[i]] = i;
}

// One thread per entry q of the scattered order: gather the particle's data
// to its place in key order.  Inside a cell the places go by previous index
// (the arrival order of the binning atomics is not deterministic): an entry's
// is the number of smaller ones among the cell's few, counted here instead of in
// a sorting launch of its own.  Writes are coalesced but for the order inside a
// cell; the reads follow the previous order, which is close to the new one after
// the first build.  The particle's key is formed again from the position it has
// read: another read in the previous order would fetch a line per particle when
// that order is a new state's (1M of the assembly mixture in random order: 106 us
// with the stored keys, 73.5 so; sorted, 28.5 and 27).  The path lengths since the last list build (vel.w) restart at
// zero for the particles whose list is rebuilt; a batch replica that keeps its
// list (build[r] == 0) keeps its order (order[q] == q) and its path lengths.
// The temporaries are the state the rebuild leaves, which the driver restores
// on a rollback.
struct PermuteArgs {
    const int* order;
    const int* cell_start;
    int N;
    Box box;                // single systems; a batch's are its replicas'
    Grid grid;
    const float4* pos;
    const float4* vel;
    const int4* image;
    float4* tpos;
    float4* tvel;
    int4* timage;
    int* rtag;
    const int* build;       // batches only
    const RepDesc* rep;
    const int* chunk_rep;
};

template <bool BATCH>
__global__ __launch_bounds__(kBlock) void k_permute(PermuteArgs a) {
    const int q = blockIdx.x * blockDim.x + threadIdx.x;
    if (q >= a.N) return;
    const int o = a.order[q];
    if (o < 0) {   // an unused slot of a batch: zeroed
        a.tpos[q] = make_float4(0.f, 0.f, 0.f, 0.f);
        if (a.vel) a.tvel[q] = make_float4(0.f, 0.f, 0.f, 0.f);
        if (a.image) a.timage[q] = make_int4(0, 0, 0, 0);
        return;
    }
    bool rebuilt = true;
    int shift = 0;
    if constexpr (BATCH) {
        const int r = a.chunk_rep[q / kWave];
        rebuilt = !a.build || a.build[r] != 0;
        if (rebuilt) shift = a.rep[r].off - a.cell_start[a.rep[r].key_base];
    }
    const float4 p = a.pos[o];
    float4 v = make_float4(0.f, 0.f, 0.f, 0.f);
    int4 im = make_int4(0, 0, 0, 0);
    if (a.vel) v = a.vel[o];
    if (a.image) im = a.image[o];
    int d = q;
    if (rebuilt) {
        v.w = 0.0f;
        int k;
        if constexpr (BATCH) {
            const RepDesc& d = a.rep[a.chunk_rep[q / kWave]];
            k = (int)d.key_base + cell_key(p, d.box, d.grid);
        } else {
            k = cell_key(p, a.box, a.grid);
        }
        const int s = a.cell_start[k] + shift, e = a.cell_start[k + 1] + shift;
        if (e - s > 1) {
            d = s;
            for (int t = s; t < e; ++t) d += a.order[t] < o ? 1 : 0;
        }
    }
    a.tpos[d] = p;
    if (a.vel) a.tvel[d] = v;
    if (a.image) a.timage[d] = im;
    if (a.rtag) {
        const int tg = ptag(p.w);
        if (tg >= 0 && tg < a.N) a.rtag[tg] = d;
    }
}

// ---- batches: the same counting sort over the concatenated key ranges ------
// Only the replicas with build[r] != 0 (every replica when build is NULL) are
// binned and re-ordered; the others keep their order and their lists.  A
// replica's particles go to its own slots: slot = off + (the cell start of
// its key) - (the cell start of its first key) + rank, so the order does not
// depend on which other replicas take part.
__device__ __forceinline__ bool rep_builds(const int* build, int r) { return !build || build[r] != 0; }

// order[q]: -1 for unused slots, q for the slots of replicas that keep their
// order; the scatter fills the rest
__global__ __launch_bounds__(kBlock) void k_order_init_batch(CellsArgsB a) {
    const int q = blockIdx.x * blockDim.x + threadIdx.x;
    if (q >= a.N) return;
    const int r = a.chunk_rep[q / kWave];
    const RepDesc& d = a.rep[r];
    a.order[q] = (q < d.off + d.n && !rep_builds(a.build, r)) ? q : -1;
}

__global__ __launch_bounds__(kBlock) void k_bin_batch(CellsArgsB a) {
    const int i = blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= a.N) return;
    const int r = a.chunk_rep[i / kWave];
    if (!rep_builds(a.build, r)) return;
    const RepDesc& d = a.rep[r];
    if (i >= d.off + d.n) return;
    const int key = (int)d.key_base + cell_key(a.pos[i], d.box, d.grid);
    a.keys[i] = key;
    a.rank[i] = atomicAdd(&a.counts[key], 1);
}

// scatter into the replica's own slots
__global__ __launch_bounds__(kBlock) void k_scatter_batch(CellsArgsB a) {
    const int i = blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= a.N) return;
    const int r = a.chunk_rep[i / kWave];
    if (!rep_builds(a.build, r)) return;
    const RepDesc& d = a.rep[r];
    if (i >= d.off + d.n) return;
    a.order[a.cell_start[a.keys[i]] - a.cell_start[d.key_base] + a.rank[i] + d.off] = i;
}

static inline int nblk(long n, int b) { return (int)((n + b - 1) / b); }

// The permuted state back from the temporaries, in one launch (vel and image may be NULL)
__global__ __launch_bounds__(kBlock) void k_copy_back(const float4* __restrict__ tpos, const float4* __restrict__ tvel,
                                                     const int4* __restrict__ timage, float4* __restrict__ pos,
                                                     float4* __restrict__ vel, int4* __restrict__ image, int N) {
    const int i = blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= N) return;
    pos[i] = tpos[i];
    if (vel) vel[i] = tvel[i];
    if (image) image[i] = timage[i];
}

template <class Args>
static PermuteArgs permute_args(const Args& a) {
    PermuteArgs p{};
    p.order = a.order;
    p.cell_start = a.cell_start;
    p.N = a.N;
    p.pos = a.pos;
    p.vel = a.vel;
    p.image = a.image;
    p.tpos = a.tpos;
    p.tvel = a.tvel;
    p.timage = a.timage;
    p.rtag = a.rtag;
    return p;
}

hipError_t launch_cells_batch(const CellsArgsB& a, hipStream_t s) {
    const int nk = (int)a.nkeys;
    if (nblk(nk, kScanTile) > 8192) return hipErrorInvalidValue;
    hipLaunchKernelGGL(k_clear_counts, dim3(std::min(nblk(nk / 4, kBlock), 2048)), dim3(kBlock), 0, s, a.counts, nk,
                       a.status, a.status_mode);
    hipLaunchKernelGGL(k_order_init_batch, dim3(nblk(a.N, kBlock)), dim3(kBlock), 0, s, a);
    hipLaunchKernelGGL(k_bin_batch, dim3(nblk(a.N, kBlock)), dim3(kBlock), 0, s, a);
    launch_scan(a.counts, nk, a.block_sums, a.cell_start, s);
    hipLaunchKernelGGL(k_scatter_batch, dim3(nblk(a.N, kBlock)), dim3(kBlock), 0, s, a);
    PermuteArgs p = permute_args(a);
    p.build = a.build;
    p.rep = a.rep;
    p.chunk_rep = a.chunk_rep;
    hipLaunchKernelGGL(k_permute<true>, dim3(nblk(a.N, kBlock)), dim3(kBlock), 0, s, p);
    if (!a.list_follows)
        hipLaunchKernelGGL(k_copy_back, dim3(nblk(a.N, kBlock)), dim3(kBlock), 0, s, a.tpos, a.tvel, a.timage, a.pos,
                           a.vel, a.image, a.N);
    return hipGetLastError();
}

hipError_t launch_cells(const CellsArgs& a, hipStream_t s) {
    const int nk = (int)a.g.nkeys;
    if (nblk(nk, kScanTile) > 8192) return hipErrorInvalidValue;
    hipLaunchKernelGGL(k_clear_counts, dim3(std::min(nblk(nk / 4, kBlock), 2048)), dim3(kBlock), 0, s, a.counts, nk,
                       a.status, a.status_mode);
    hipLaunchKernelGGL(k_bin, dim3(nblk(a.N, kBlock)), dim3(kBlock), 0, s, a.pos, a.N, a.box, a.g,
                       a.counts, a.keys, a.rank);
    launch_scan(a.counts, nk, a.block_sums, a.cell_start, s);
    hipLaunchKernelGGL(k_scatter, dim3(nblk(a.N, kBlock)), dim3(kBlock), 0, s, a.keys, a.rank,
                       a.cell_start, a.N, a.order);
    PermuteArgs p = permute_args(a);
    p.box = a.box;
    p.grid = a.g;
    hipLaunchKernelGGL(k_permute<false>, dim3(nblk(a.N, kBlock)), dim3(kBlock), 0, s, p);
    if (!a.list_follows)
        hipLaunchKernelGGL(k_copy_back, dim3(nblk(a.N, kBlock)), dim3(kBlock), 0, s, a.tpos, a.tvel, a.timage, a.pos,
                           a.vel, a.image, a.N);
    return hipGetLastError();
}

// p[i] by a 32-bit byte offset from the uniform base (i < 2^28 for 16-byte elements: N < 2^27)
template <class T>
__device__ __forceinline__ T at(const T* p, uint32_t i) {
    return *reinterpret_cast<const T*>(reinterpret_cast<const char*>(p) + (size_t)(i * (uint32_t)sizeof(T)));
}

// ---------------------------------------------------------------------------
// neighbour list
// ---------------------------------------------------------------------------
// List of one particle i (key order): scan the 27 cells around i's cell and
// keep every j != i inside r_list(t_i, t_j).  Cells are visited in (z, y, x)
// offset order and each cell's particles in memory order, so the list order
// is fixed.  For a cell that does not wrap around the box the difference
// x_j - x_i is one FP32 subtraction (a single rounding of the exact value);
// across a periodic face it is the FP64 difference folded by the box (exact
// image choice).  The square is FP32; the list radius carries a 1e-5 relative
// margin for that rounding.  Cell k's particles sit at cell_start[key_base +
// k] + shift onwards.  rl(q, rl2, swap) gives entry q's squared list radius
// and whether it is a swap pair.  Returns the full neighbour count and stores
// nn[i] (clipped to k_max).
//
// A cell whose nearest point is farther from i than i's largest list radius
// (over all partner types) is skipped: its count is taken as zero.  The gaps
// to the cell faces are shrunk by 1e-3 cell widths, far above the FP32
// rounding of the cell coordinates, so no cell that holds a listable
// neighbour is skipped.
//
// Per z slab the cells form NR ranges of memory in visiting order: the nine
// cells themselves, or (PAIR) two per row, since along x the cells 2k and 2k + 1
// follow each other on the curve: the row's middle cell and its even-odd partner
// are one range, trimmed where the partner is too far, and the third cell the
// other.  That fails only for an even last cell, whose right neighbour wraps.
// The ranges' candidates are numbered t = 0 .. tot-1 (exclusive prefix pre[q] of
// the lengths), and candidate t is located without branches: the last range q
// with pre[q] <= t gives j = t + (start_q - pre_q).  The offset and the range's
// wrap flag are packed in one word, so a candidate costs NR - 1 compare/select
// pairs and a wavefront runs one uniform loop per slab instead of a
// data-dependent cursor.  Bound by its instructions and the reads of the bounds:
// with two ranges per row, both bounds read without branches and 32-bit offsets
// 2161 -> 1967 VALU instructions per wavefront at 1M particles and 80 -> 74 us,
// the copy of the sorted state (14 us by itself) included.  Keeping the entries
// found as bits and storing them after the test was slower (93 us).
template <bool PAIR, class Radii>
__device__ __forceinline__ int list_scan(int i, const float4& pi, const Box& b, const Grid& g, uint32_t key_base,
                                        int shift, const int* __restrict__ cell_start, const float4* __restrict__ pos,
                                        int nt, int k_max, int N, int* __restrict__ nlist, int* __restrict__ nn,
                                        Radii rl) {
    int ns = 0, no = 0;
    const int ti = ptype(pi.w);
    const int cx = cell_coord(pi.x, b.hf[0], g.inv_w[0], g.nc[0]);
    const int cy = cell_coord(pi.y, b.hf[1], g.inv_w[1], g.nc[1]);
    const int cz = cell_coord(pi.z, b.hf[2], g.inv_w[2], g.nc[2]);
    float rmax2 = 0.0f;  // i's largest squared list radius
    for (int t = 0; t < nt; ++t) {
        float r2t;
        bool sw;
        rl(ti * nt + t, r2t, sw);
        rmax2 = fmaxf(rmax2, r2t);
    }
    // squared gaps from i to the cells at offsets -1, 0, +1 along an axis
    auto gaps = [&](float x, float h, float inv_w, int c, float& g0, float& g2) {
        const float f = (x + h) * inv_w - (float)c;  // place in the cell, in widths
        const float w = __builtin_amdgcn_rcpf(inv_w);   // its last bit is far below the margin
        const float lo = fmaxf(f - 1e-3f, 0.0f) * w, hi = fmaxf(1.0f - f - 1e-3f, 0.0f) * w;
        g0 = lo * lo;
        g2 = hi * hi;
    };
    float gx0, gx2, gy0, gy2, gz0, gz2;
    gaps(pi.x, b.hf[0], g.inv_w[0], cx, gx0, gx2);
    gaps(pi.y, b.hf[1], g.inv_w[1], cy, gy0, gy2);
    gaps(pi.z, b.hf[2], g.inv_w[2], cz, gz0, gz2);
    // Morton parts of the three cell coordinates per axis, and whether the offset wraps
    int wxy = 0;  // bit o: x offset o wraps; bit 3 + o: y offset o wraps
    auto axis = [&](int c, int o, int nc, int bit) {
        int x = c + o - 1;
        wxy |= (x < 0 || x >= nc) ? bit : 0;
        x += (x < 0) ? nc : 0;
        x -= (x >= nc) ? nc : 0;
        return spread3((uint32_t)x);
    };
    const uint32_t kx0 = axis(cx, 0, g.nc[0], 1), kx1 = axis(cx, 1, g.nc[0], 2), kx2 = axis(cx, 2, g.nc[0], 4);
    const uint32_t ky0 = axis(cy, 0, g.nc[1], 8) << 1, ky1 = axis(cy, 1, g.nc[1], 16) << 1,
                   ky2 = axis(cy, 2, g.nc[1], 32) << 1;
    constexpr int NR = PAIR ? 6 : 9;
    const bool odd = cx & 1;
    auto consider = [&](int j, const float4& pj, bool wrapped) {
        float dx, dy, dz;
        if (wrapped) {
            dx = (float)fold((double)pj.x - (double)pi.x, b.L[0], b.h[0]);
            dy = (float)fold((double)pj.y - (double)pi.y, b.L[1], b.h[1]);
            dz = (float)fold((double)pj.z - (double)pi.z, b.L[2], b.h[2]);
        } else {
            dx = pj.x - pi.x;
            dy = pj.y - pi.y;
            dz = pj.z - pi.z;
        }
        const float r2 = dx * dx + dy * dy + dz * dz;
        float rl2;
        bool swap;
        rl(ti * nt + ptype(pj.w), rl2, swap);
        if (r2 < rl2 && j != i) {
            // swap kind from the front, the rest from the back (counters stay in registers)
            const int slot = swap ? ns : k_max - 1 - no;
            if (ns + no < k_max) nlist[(size_t)slot * N + i] = j;
            ns += swap ? 1 : 0;
            no += swap ? 0 : 1;
        }
    };
    for (int oz = -1; oz <= 1; ++oz) {
        const float dz2 = oz < 0 ? gz0 : (oz > 0 ? gz2 : 0.0f);
        if (dz2 >= rmax2) continue;
        int z = cz + oz;
        const bool wz = z < 0 || z >= g.nc[2];
        z += (z < 0) ? g.nc[2] : 0;
        z -= (z >= g.nc[2]) ? g.nc[2] : 0;
        const uint32_t kz = spread3((uint32_t)z) << 2;
        // range 0's packed word, then ranges 1 .. NR - 1: exclusive prefix of the lengths and
        // (start - prefix) * 2 + wraps (vector values, so they stay in registers)
        typedef int intv __attribute__((ext_vector_type(8)));
        int ow0 = 0, tot = 0;
        intv pre, ow;
        auto range = [&](int q, uint32_t kb, uint32_t ke, bool near, bool wraps) {
            const int st = at(cell_start, kb) + shift, end = at(cell_start, ke) + shift;
            const int en = near ? end : st;
            const int o = (st - tot) * 2 + (wraps ? 1 : 0);  // st - tot may be negative: >> 1 is arithmetic
            if (q == 0) {
                ow0 = o;
            } else {
                pre[q - 1] = tot;
                ow[q - 1] = o;
            }
            tot += en - st;
        };
#pragma unroll
        for (int y = 0; y < 3; ++y) {
            const uint32_t kyz = key_base + ((y == 0 ? ky0 : (y == 1 ? ky1 : ky2)) | kz);
            const bool wyz = wz || (wxy & (8 << y)) != 0;
            const float d2 = dz2 + (y == 0 ? gy0 : (y == 2 ? gy2 : 0.0f));
            const bool row = d2 < rmax2, left = d2 + gx0 < rmax2, right = d2 + gx2 < rmax2;
            const uint32_t ka = kyz + kx0, km = kyz + kx1, kc = kyz + kx2;
            const bool wl = wyz || (wxy & 1) != 0, wr = wyz || (wxy & 4) != 0;
            if constexpr (PAIR) {
                range(2 * y, odd && !left ? km : ka, (odd ? km : ka) + 1, odd ? row : left, wl);
                range(2 * y + 1, odd ? kc : km, odd ? kc + 1 : km + (right ? 2 : 1), odd ? right : row, wr);
            } else {
                range(3 * y, ka, ka + 1, left, wl);
                range(3 * y + 1, km, km + 1, row, wyz);
                range(3 * y + 2, kc, kc + 1, right, wr);
            }
        }
        auto locate = [&](int t) {
            int o = ow0;
#pragma unroll
            for (int q = 0; q < NR - 1; ++q) o = t >= pre[q] ? ow[q] : o;
            return o;
        };
        // candidates in groups of four, all four positions requested before any is tested (in candidate
        // order, so the list is the same): 102 -> 95 us per build at 1M particles; one ahead, two, three,
        // six or eight at a time, or the next group requested during the current one, were slower
        constexpr int kAhead = 4;
        for (int t0 = 0; t0 < tot; t0 += kAhead) {
            int oq[kAhead];
            float4 pq[kAhead];
#pragma unroll
            for (int u = 0; u < kAhead; ++u) {
                oq[u] = 0;
                pq[u] = pi;
                if (t0 + u < tot) {
                    oq[u] = locate(t0 + u);
                    pq[u] = at(pos, (uint32_t)(t0 + u + (oq[u] >> 1)));
                }
            }
#pragma unroll
            for (int u = 0; u < kAhead; ++u)
                if (t0 + u < tot) consider(t0 + u + (oq[u] >> 1), pq[u], (oq[u] & 1) != 0);
        }
    }
    const int total = ns + no;
    // on overflow the stored prefix is what fitted (the status reports it)
    if (ns + no > k_max) {
        const int keep_s = min(ns, k_max);
        ns = keep_s;
        no = k_max - keep_s;
    }
    nn[i] = ns | (no << 16);
    return total;
}

template <class Radii>
__device__ __forceinline__ int list_one(int i, const float4& pi, const Box& b, const Grid& g, uint32_t key_base,
                                        int shift, const int* __restrict__ cell_start, const float4* __restrict__ pos,
                                        int nt, int k_max, int N, int* __restrict__ nlist, int* __restrict__ nn,
                                        Radii rl) {
    const int cx = cell_coord(pi.x, b.hf[0], g.inv_w[0], g.nc[0]);
    if (__any((cx & 1) == 0 && cx + 1 == g.nc[0]))
        return list_scan<false>(i, pi, b, g, key_base, shift, cell_start, pos, nt, k_max, N, nlist, nn, rl);
    return list_scan<true>(i, pi, b, g, key_base, shift, cell_start, pos, nt, k_max, N, nlist, nn, rl);
}

// The list's status words: KMAX and the overflow flag from the largest list, NSWAP the swap ranges' entries and
// NLIST all entries (saturating).  A launch of at most kStatusBlocks blocks sets them by atomics as its blocks end; the blocks of
// a larger one leave their values to k_list_status, since atomics on one address follow each other about 45 ns
// apart (the list kernel at 1M particles, 3907 blocks: 80 us with them left to a launch of 4 us, 262 with atomics).
constexpr int kStatusBlocks = 64;

template <int THREADS = kBlock>   // of the block, which take part
__device__ __forceinline__ void block_list_status(int cnt, int packed, int* status, int k_max, int4* per_block) {
    constexpr int W = THREADS / kWave;
    __shared__ int s_m[W], s_n[W], s_a[W];
    int m = cnt;
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) m = max(m, __shfl_xor(m, o, kWave));
    const int t_ns = __builtin_amdgcn_readlane(wave_inclusive_scan(nn_swap(packed)), kWave - 1);
    const int t_all = t_ns + __builtin_amdgcn_readlane(wave_inclusive_scan(nn_other(packed)), kWave - 1);
    if (W > 1) {
        if ((threadIdx.x & (kWave - 1)) == 0) {
            s_m[threadIdx.x / kWave] = m;
            s_n[threadIdx.x / kWave] = t_ns;
            s_a[threadIdx.x / kWave] = t_all;
        }
        __syncthreads();
    }
    if (threadIdx.x == 0) {
        int t = m, u = t_ns, a = t_all;
#pragma unroll
        for (int w = 1; w < W; ++w) {
            t = max(t, s_m[w]);
            u += s_n[w];
            a += s_a[w];
        }
        if (gridDim.x > kStatusBlocks) {
            per_block[blockIdx.x] = make_int4(t, u, a, 0);
        } else {   // at most 64 blocks of 256 lists of 512 entries: the sums fit
            atomicMax(&status[RC_ST_KMAX], t);
            if (t > k_max) atomicOr(&status[RC_ST_FLAGS], RC_FLAG_NLIST_OVERFLOW);
            atomicAdd(&status[RC_ST_NSWAP], u);
            atomicAdd(&status[RC_ST_NLIST], a);
        }
    }
}

__global__ __launch_bounds__(1024) void k_list_status(const int4* __restrict__ per_block, int nb, int k_max,
                                                     int* __restrict__ status) {
    __shared__ int red[1024 / kWave];
    __shared__ double red_ns[1024 / kWave], red_all[1024 / kWave];
    int m = 0;
    double t = 0, all = 0;   // whole numbers below 2^53
    for (int b = threadIdx.x; b < nb; b += 4 * 1024) {   // four reads under way
        int4 v[4];
#pragma unroll
        for (int u = 0; u < 4; ++u) v[u] = b + u * 1024 < nb ? per_block[b + u * 1024] : make_int4(0, 0, 0, 0);
#pragma unroll
        for (int u = 0; u < 4; ++u) {
            m = max(m, v[u].x);
            t += v[u].y;
            all += v[u].z;
        }
    }
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) m = max(m, __shfl_xor(m, o, kWave));
    t = wave_sum(t);
    all = wave_sum(all);
    if ((threadIdx.x & (kWave - 1)) == 0) {
        red[threadIdx.x / kWave] = m;
        red_ns[threadIdx.x / kWave] = t;
        red_all[threadIdx.x / kWave] = all;
    }
    __syncthreads();
    if (threadIdx.x >= kWave) return;
    const bool in = threadIdx.x < 1024 / kWave;
    m = in ? red[threadIdx.x] : 0;
    t = wave_sum(in ? red_ns[threadIdx.x] : 0.0);
    all = wave_sum(in ? red_all[threadIdx.x] : 0.0);
#pragma unroll
    for (int o = 1024 / kWave / 2; o > 0; o >>= 1) m = max(m, __shfl_xor(m, o, kWave));
    if (threadIdx.x == 0) {
        status[RC_ST_KMAX] = max(status[RC_ST_KMAX], m);
        if (m > k_max) status[RC_ST_FLAGS] |= RC_FLAG_NLIST_OVERFLOW;
        status[RC_ST_NSWAP] = (int)fmin(t, 2147483647.0);
        status[RC_ST_NLIST] = (int)fmin(all, 2147483647.0);
    }
}

// A state the cell sort left in its temporaries, of which pos is one, written back by the list build (its
// arithmetic hides the copy: 14 us of its own at 1M particles)
__device__ __forceinline__ void write_back(const StateBack& b, int i, const float4& p) {
    b.pos[i] = p;
    if (b.vel) b.vel[i] = b.tvel[i];
    if (b.image) b.image[i] = b.timage[i];
}

// One thread per particle (key order).
__global__ __launch_bounds__(kBlock) void k_nlist(NlistArgs a) {
    extern __shared__ float s_rl2[];  // [nt*nt] list radii^2, then [nt*nt] swap flags
    const int nt = a.tab.nt;
    int* s_swap = reinterpret_cast<int*>(s_rl2 + nt * nt);
    for (int q = threadIdx.x; q < nt * nt; q += blockDim.x) {
        s_rl2[q] = a.tab.e[q].rlist2;
        s_swap[q] = a.tab.e[q].kind == RC_KIND_SWAP;
    }
    __syncthreads();
    const int nb = gridDim.x;
    const int i = xcd_block(nb) * blockDim.x + threadIdx.x;
    int total = 0, packed = 0;
    if (i < a.N) {
        const float4 pi = a.pos[i];
        if (a.back.pos) write_back(a.back, i, pi);
        total = list_one(i, pi, a.box, a.g, 0u, 0, a.cell_start, a.pos, nt, a.k_max, a.N, a.nlist, a.nn,
                         [&](int q, float& rl2, bool& swap) {
                             rl2 = s_rl2[q];
                             swap = s_swap[q] != 0;
                         });
        packed = a.nn[i];
        if (!a.back.pos && a.vel) a.vel[i].w = 0.0f;
    }
    if (a.pl_j) pack_wave_lists(i, i < a.N, packed, a.nlist, a.k_max, a.N, a.pl_j, a.pl_o);
    if (a.status) block_list_status(total, packed, a.status, a.k_max, a.per_block);
}

// LDS writes of a wavefront before its own reads, without the block's barrier
__device__ __forceinline__ void wave_sync() {
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "workgroup");
}

// The same list for systems whose one-thread-per-particle wavefronts would not
// fill the chip: there a build lasts as long as one wavefront's three slabs of
// dependent reads (17 to 58 us whatever the size).  A block holds 64 particles
// and 64 / OW wavefronts of OW particles.  SL lanes per particle read its 27
// cells' bounds at once, the wavefront lays its candidates out flat in LDS
// (particle by particle, cells in visiting order), and tests 64 PL of them at a
// time with their positions requested together; an entry's slot is the
// particle's count so far plus the entries before it in the same row of 64.
// us per launch, one thread per particle and now: 512 dumbbells 20.6, 8.5; 3000
// and 32768 reactive particles of density 0.25 31.7, 10.8 and 28.4, 13.5; 67200
// beads of a network 44.8, 29.0.
constexpr int kFewOwn = 8;   // OW; with 16 and 32 the 32768 took 16.0 and 26.0
__global__ __launch_bounds__(kWave * (kWave / kFewOwn)) void k_nlist_few(NlistArgs a) {
    constexpr int OW = kFewOwn, NW = kWave / OW, SL = kWave / OW, R = (27 + SL - 1) / SL, PL = 4, CAP = 64 * OW;
    extern __shared__ float s_rl2[];  // [nt*nt] list radii^2, then [nt*nt] swap flags
    __shared__ float4 s_pos[kWave];
    __shared__ int s_ns[kWave], s_no[kWave];        // entries found so far, not clipped
    __shared__ int s_off[NW][OW + 1];               // a particle's first candidate of its wavefront's
    __shared__ uint32_t s_cand[NW][CAP];            // index << 6 | wraps << 5 | particle
    const int nt = a.tab.nt;
    int* s_swap = reinterpret_cast<int*>(s_rl2 + nt * nt);
    const int lane = threadIdx.x % kWave, wv = threadIdx.x / kWave, sub = lane % SL;
    const int first = xcd_block(gridDim.x) * kWave;
    const int p = wv * OW + lane / SL;              // this lane's particle in the block
    const int i = first + p;
    const bool live = i < a.N;
    const float4 pi = a.pos[min(i, a.N - 1)];
    if (a.back.pos) {                               // the block's 64 particles, an array per wavefront
        const int q = first + lane;
        if (q < a.N) {
            if (wv == 0) a.back.pos[q] = a.pos[q];
            if (a.back.vel && wv == 1 % NW) a.back.vel[q] = a.back.tvel[q];
            if (a.back.image && wv == 2 % NW) a.back.image[q] = a.back.timage[q];
        }
    } else if (a.vel && wv == 0 && first + lane < a.N) {
        a.vel[first + lane].w = 0.0f;
    }
    for (int q = threadIdx.x; q < nt * nt; q += blockDim.x) {
        s_rl2[q] = a.tab.e[q].rlist2;
        s_swap[q] = a.tab.e[q].kind == RC_KIND_SWAP;
    }
    if (sub == 0) {
        s_pos[p] = pi;
        s_ns[p] = 0;
        s_no[p] = 0;
    }
    __syncthreads();
    const Box& b = a.box;
    const Grid& g = a.g;
    // the lane's cells sub R .. sub R + R - 1: their candidates
    int st[R], len[R];
    uint32_t wraps = 0;
    int mine = 0;
    {
        const int ti = ptype(pi.w);
        float rmax2 = 0.0f;
        for (int t = 0; t < nt; ++t) rmax2 = fmaxf(rmax2, s_rl2[ti * nt + t]);
        const int cx = cell_coord(pi.x, b.hf[0], g.inv_w[0], g.nc[0]);
        const int cy = cell_coord(pi.y, b.hf[1], g.inv_w[1], g.nc[1]);
        const int cz = cell_coord(pi.z, b.hf[2], g.inv_w[2], g.nc[2]);
        // squared gap from the particle to the cells at offset o along an axis, as in list_scan
        auto gap = [&](float x, float h, float inv_w, int c, int o) {
            const float f = (x + h) * inv_w - (float)c;
            const float d = fmaxf((o < 0 ? f : 1.0f - f) - 1e-3f, 0.0f) * __builtin_amdgcn_rcpf(inv_w);
            return o == 0 ? 0.0f : d * d;
        };
        auto part = [&](int c, int o, int nc, bool& wrap) {
            int x = c + o;
            wrap = wrap || x < 0 || x >= nc;
            x += x < 0 ? nc : 0;
            x -= x >= nc ? nc : 0;
            return spread3((uint32_t)x);
        };
#pragma unroll
        for (int q = 0; q < R; ++q) {
            const int c = sub * R + q;
            const int oz = c / 9 - 1, oy = c / 3 % 3 - 1, ox = c % 3 - 1;
            bool wrap = false;
            const uint32_t key = part(cx, ox, g.nc[0], wrap) | part(cy, oy, g.nc[1], wrap) << 1 |
                                 part(cz, oz, g.nc[2], wrap) << 2;
            const float d2 = gap(pi.z, b.hf[2], g.inv_w[2], cz, oz) + gap(pi.y, b.hf[1], g.inv_w[1], cy, oy) +
                             gap(pi.x, b.hf[0], g.inv_w[0], cx, ox);
            const bool near = live && c < 27 && d2 < rmax2;
            st[q] = near ? at(a.cell_start, key) : 0;
            len[q] = near ? at(a.cell_start, key + 1) : 0;
            wraps |= wrap ? 1u << q : 0u;
        }
#pragma unroll
        for (int q = 0; q < R; ++q) {
            len[q] -= st[q];
            mine += len[q];
        }
    }
    const int inc = wave_inclusive_scan(mine);
    const int off = inc - mine, T = __builtin_amdgcn_readlane(inc, kWave - 1);
    if (sub == 0) s_off[wv][lane / SL] = off;
    if (lane == 0) s_off[wv][OW] = T;
    wave_sync();
    uint32_t* cand = s_cand[wv];
    for (int w0 = 0; w0 < T; w0 += CAP) {
        const int tw = min(T - w0, CAP);
        // candidates w0 .. w0 + tw - 1
        int o = off - w0;
#pragma unroll
        for (int q = 0; q < R; ++q) {
            const uint32_t tail = ((wraps >> q) & 1u) << 5 | (uint32_t)(lane / SL);
            const int k0 = max(0, -o), k1 = min(len[q], tw - o);
            for (int k = k0; k < k1; ++k) cand[o + k] = (uint32_t)(st[q] + k) << 6 | tail;
            o += len[q];
        }
        wave_sync();
        for (int e0 = 0; e0 < tw; e0 += PL * kWave) {
            uint32_t c[PL];
            float4 pj[PL];
#pragma unroll
            for (int u = 0; u < PL; ++u) {
                const int e = e0 + u * kWave + lane;
                c[u] = e < tw ? cand[e] : 0u;
            }
#pragma unroll
            for (int u = 0; u < PL; ++u) {
                pj[u] = make_float4(0.f, 0.f, 0.f, 0.f);
                if (e0 + u * kWave + lane < tw) pj[u] = at(a.pos, c[u] >> 6);
            }
#pragma unroll
            for (int u = 0; u < PL; ++u) {
                const int row = e0 + u * kWave;
                if (row >= tw) break;   // uniform
                const bool on = row + lane < tw;
                const int own = c[u] & (OW - 1), j = (int)(c[u] >> 6), m = wv * OW + own;
                bool hit = false, swap = false;
                if (on) {
                    const float4 po = s_pos[m];
                    float dx, dy, dz;
                    if (c[u] & 32u) {
                        dx = (float)fold((double)pj[u].x - (double)po.x, b.L[0], b.h[0]);
                        dy = (float)fold((double)pj[u].y - (double)po.y, b.L[1], b.h[1]);
                        dz = (float)fold((double)pj[u].z - (double)po.z, b.L[2], b.h[2]);
                    } else {
                        dx = pj[u].x - po.x;
                        dy = pj[u].y - po.y;
                        dz = pj[u].z - po.z;
                    }
                    const float r2 = dx * dx + dy * dy + dz * dz;
                    const int q = ptype(po.w) * nt + ptype(pj[u].w);
                    hit = r2 < s_rl2[q] && j != first + m;
                    swap = hit && s_swap[q] != 0;
                }
                const unsigned long long ms = __ballot(swap), mo = __ballot(hit && !swap);
                if (on) {
                    // the row's entries of the same particle before this one
                    const int lo = max(0, s_off[wv][own] - w0 - row);
                    const unsigned long long mask = ((1ull << lane) - 1ull) & ~((1ull << lo) - 1ull);
                    const int ns = s_ns[m] + __popcll(ms & mask), no = s_no[m] + __popcll(mo & mask);
                    if (hit && ns + no < a.k_max)
                        a.nlist[(size_t)(swap ? ns : a.k_max - 1 - no) * a.N + first + m] = j;
                    const int next = row + lane + 1;   // the particle's last entry of the row keeps its counts
                    if (lane == kWave - 1 || next == tw || w0 + next == s_off[wv][own + 1]) {
                        s_ns[m] = ns + (swap ? 1 : 0);
                        s_no[m] = no + (hit && !swap ? 1 : 0);
                    }
                }
                wave_sync();
            }
        }
    }
    __syncthreads();
    // the block's 64 lists: lane l of every wavefront looks at particle l
    int ns = s_ns[lane], no = s_no[lane];
    const int total = ns + no;
    if (total > a.k_max) {   // on overflow the stored prefix is what fitted
        ns = min(ns, a.k_max);
        no = a.k_max - ns;
    }
    if (wv == 0) {
        if (first + lane < a.N) a.nn[first + lane] = ns | (no << 16);
        if (a.status) block_list_status<kWave>(total, ns | (no << 16), a.status, a.k_max, a.per_block);
    }
    if (a.pl_j) {            // the packed copy (pack_wave_lists), SL lanes per particle
        const int before = wave_inclusive_scan(ns + no) - (ns + no);
        const int p_ns = __shfl(ns, p, kWave), p_cnt = p_ns + __shfl(no, p, kWave);
        const size_t base = (size_t)first * a.k_max + __shfl(before, p, kWave);
        for (int s = sub; s < p_cnt; s += SL) {
            const int slot = s < p_ns ? s : a.k_max - 1 - (s - p_ns);
            a.pl_j[base + s] = a.nlist[(size_t)slot * a.N + i];
            a.pl_o[base + s] = (unsigned char)p;
        }
    }
}

__global__ __launch_bounds__(kBlock) void k_pack_list(const int* __restrict__ nlist, const int* __restrict__ nn,
                                                      int k_max, int N, int* __restrict__ pl_j,
                                                      unsigned char* __restrict__ pl_o) {
    const int i = blockIdx.x * blockDim.x + threadIdx.x;
    const bool live = i < N;
    pack_wave_lists(i, live, live ? nn[i] : 0, nlist, k_max, N, pl_j, pl_o);
}

hipError_t launch_pack_list(const int* nlist, const int* nn, int k_max, int N, int* pl_j, unsigned char* pl_o,
                            hipStream_t s) {
    hipLaunchKernelGGL(k_pack_list, dim3(nblk(N, kBlock)), dim3(kBlock), 0, s, nlist, nn, k_max, N, pl_j, pl_o);
    return hipGetLastError();
}

// Batches: each wave lies in one replica, which gives the box, grid, key
// range and table (its list radii staged in the wavefront's LDS slice); empty
// slots get an empty list.  A replica that keeps its list (build[r] == 0)
// keeps its lists, packed copy and path lengths; its list lengths still count
// towards the status words.
__global__ __launch_bounds__(kBlock) void k_nlist_batch(NlistArgsB a) {
    extern __shared__ float s_rl2b[];  // per wavefront: [nt*nt] list radii^2, then [nt*nt] swap flags
    const int nt = a.tab.nt, nt2 = nt * nt;
    const int i = blockIdx.x * blockDim.x + threadIdx.x;
    const int lane = threadIdx.x & (kWave - 1), wv = threadIdx.x / kWave;
    const int r = i < a.N ? a.chunk_rep[i / kWave] : 0;
    float* rl2s = s_rl2b + 2 * nt2 * wv;
    int* sws = reinterpret_cast<int*>(rl2s + nt2);
    if (i < a.N) {
        const DevEntry* t = a.tab.e + a.rep[r].tab;
        for (int q = lane; q < nt2; q += kWave) {
            rl2s[q] = t[q].rlist2;
            sws[q] = t[q].kind == RC_KIND_SWAP;
        }
    }
    __syncthreads();
    int total = 0, packed = 0;
    const bool builds = i < a.N && rep_builds(a.build, r);   // uniform over the wavefront
    if (i < a.N) {
        const RepDesc& d = a.rep[r];
        if (a.back.pos) write_back(a.back, i, a.pos[i]);
        if (!builds) {
            packed = a.nn[i];
            total = nn_swap(packed) + nn_other(packed);
        } else if (i < d.off + d.n) {
            const int shift = d.off - a.cell_start[d.key_base];
            total = list_one(i, a.pos[i], d.box, d.grid, d.key_base, shift, a.cell_start, a.pos, nt, a.k_max,
                             a.N, a.nlist, a.nn, [&](int q, float& rl2, bool& swap) {
                                 rl2 = rl2s[q];
                                 swap = sws[q] != 0;
                             });
            packed = a.nn[i];
        } else {
            a.nn[i] = 0;
        }
        if (!a.back.pos && builds && a.vel) a.vel[i].w = 0.0f;
    }
    if (a.pl_j && (builds || i >= a.N)) pack_wave_lists(i, i < a.N, packed, a.nlist, a.k_max, a.N, a.pl_j, a.pl_o);
    if (a.status) block_list_status(total, packed, a.status, a.k_max, a.per_block);
}

// A list laid out for k_old slots per particle copied into the layout of
// k_new >= k_old slots (swap range at the front, the rest at the back), and
// its packed copy for k_new.  One thread per slot; every lane of a
// wavefront takes part (the packing scans the wavefront's lengths).
__global__ __launch_bounds__(kBlock) void k_relayout_list(const int* __restrict__ old_list, int k_old,
                                                         int* __restrict__ new_list, int k_new,
                                                         const int* __restrict__ nn, int N, int* __restrict__ pl_j,
                                                         unsigned char* __restrict__ pl_o) {
    const int i = blockIdx.x * blockDim.x + threadIdx.x;
    const bool live = i < N;
    int packed = 0;
    if (live) {
        packed = nn[i];
        const int ns = min(nn_swap(packed), k_old);
        const int no = min(nn_other(packed), k_old - ns);
        for (int q = 0; q < ns; ++q) new_list[(size_t)q * N + i] = old_list[(size_t)q * N + i];
        for (int q = 0; q < no; ++q) new_list[(size_t)(k_new - 1 - q) * N + i] = old_list[(size_t)(k_old - 1 - q) * N + i];
    }
    if (pl_j) pack_wave_lists(i, live, packed, new_list, k_new, N, pl_j, pl_o);
}

hipError_t launch_relayout_list(const int* old_list, int k_old, int* new_list, int k_new, const int* nn, int N,
                                int* pl_j, unsigned char* pl_o, hipStream_t s) {
    hipLaunchKernelGGL(k_relayout_list, dim3(nblk(N, kBlock)), dim3(kBlock), 0, s, old_list, k_old, new_list, k_new,
                       nn, N, pl_j, pl_o);
    return hipGetLastError();
}

// status words first, unless the cell sort of the same build wrote them
static void begin_status(int* status, int mode, bool begun, hipStream_t s) {
    if (status && !begun) hipLaunchKernelGGL(k_status_begin, dim3(1), dim3(1), 0, s, status, mode);
}

static void end_status(int* status, int k_max, const int4* per_block, int nb, hipStream_t s) {
    if (status && nb > kStatusBlocks)
        hipLaunchKernelGGL(k_list_status, dim3(1), dim3(1024), 0, s, per_block, nb, k_max, status);
}

// Systems the list kernel of few particles per wavefront takes; cand: mean particles within the largest list radius.
// One thread per particle takes the time of its serial reads, the longer the more candidates there are, until its
// wavefronts fill the chip; the flat layout's time goes by the particles.  They meet at (us, few and one per thread)
// cand 2.1 (dumbbells) 60000 18.4, 19.4 and 72000 20.6, 19.2; 3.6 (assembly mixture) 72000 21.7, 22.1 and 90000 24.1,
// 23.2; 6.1 (reactive, density 0.25) 110000 31.5, 31.5; 8.6 (three reactive types) 130000 39.3, 41.1 and 160000 45.8,
// 44.1; 9.8 (reactive, 0.4) 160000 49.8, 50.9 and 200000 59.3, 55.2; 10.3 (network) 160000 49.6, 52.9 and 200000 62.0,
// 59.5.  The line goes through those.
static bool few_list(int N, float cand) { return (float)N <= 33000.0f + 12800.0f * cand; }

hipError_t launch_nlist(const NlistArgs& a, hipStream_t s) {
    begin_status(a.status, a.status_mode, a.back.pos != nullptr, s);
    const size_t shm = 2 * sizeof(float) * a.tab.nt * a.tab.nt;
    const bool few = few_list(a.N, a.cand);
    const int nb = nblk(a.N, few ? kWave : kBlock);
    if (few)
        hipLaunchKernelGGL(k_nlist_few, dim3(nb), dim3(kWave * (kWave / kFewOwn)), shm, s, a);
    else
        hipLaunchKernelGGL(k_nlist, dim3(nb), dim3(kBlock), shm, s, a);
    end_status(a.status, a.k_max, a.per_block, nb, s);
    return hipGetLastError();
}

hipError_t launch_nlist_batch(const NlistArgsB& a, hipStream_t s) {
    begin_status(a.status, a.status_mode, a.back.pos != nullptr, s);
    const int nb = nblk(a.N, kBlock);
    const size_t shm = (size_t)(kBlock / kWave) * 2 * sizeof(float) * a.tab.nt * a.tab.nt;
    hipLaunchKernelGGL(k_nlist_batch, dim3(nb), dim3(kBlock), shm, s, a);
    end_status(a.status, a.k_max, a.per_block, nb, s);
    return hipGetLastError();
}

}  // namespace rc
