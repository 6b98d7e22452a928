// Differentiation of the swap-potential energy: Hessian-vector products and
// parameter gradients, both as atomic-free per-particle gathers.
//
// With w_ma = sqrt(Lambda_ma) vhat(r_ma) for swap partners inside r_cut and
// S_m = sum_a w_ma, the gradient of E with respect to x_m is
//     grad_m E = - sum_a rhat_ma G_ma,
//     G_ma = phi'(r_ma) + w'_ma (S_m + S_a - 2 w_ma)
// (the triplet sum of eq. 3bp over j<k regrouped per centre), so
//     (H v)_m = - sum_a [ dG_ma rhat_ma + G_ma (D_ma - dr_ma rhat_ma) / r_ma ],
//     D_ma = v_a - v_m,  dr_ma = rhat_ma . D_ma,
//     dG_ma = phi'' dr + w'' dr (S_m + S_a - 2 w) + w' (dS_m + dS_a - 2 w' dr),
//     dS_m = sum_b w'_mb dr_mb.
// A first pass stores (S, dS) of every particle; the second reads S_a and dS_a
// of a partner from there instead of walking a's list (the two-hop walk of
// the one-pass form; the values are those of the same walk, so the result is
// the same).
#include "rc_internal.h"

namespace rc {

static inline int nblk(long n, int b) { return (int)((n + b - 1) / b); }

__device__ __forceinline__ void load_table_adj(DevEntry* s_tab, const Table& t) {
    const int n = t.nt * t.nt;
    for (int q = threadIdx.x; q < n; q += blockDim.x) s_tab[q] = t.e[q];
    __syncthreads();
}

struct Deriv {  // value and first two r-derivatives of one term, plus geometry
    float r, rx, ry, rz;  // r and rhat
};

// The Hessian-vector kernels' term arithmetic is written with explicit fused multiply-adds and contraction
// off, so that every number of vectors per thread gives the same bits.
// 2n(2n+1) q^2 - n(n+1) q
__device__ __forceinline__ float curvature(float n, float q, float q2) {
#pragma clang fp contract(off)
    const float a = 2.0f * n * __fmaf_rn(2.0f, n, 1.0f), b = n * (n + 1.0f);
    return __fmaf_rn(a, q2, -(b * q));
}

// pair: phi'(r), phi''(r)
__device__ __forceinline__ void pair_d12(const DevEntry& e, float r2, float r, float& d1, float& d2) {
#pragma clang fp contract(off)
    const float q = qpow(e.sig2 / r2, e.n);
    const float q2 = q * q, n = (float)e.n;
    d1 = 4.0f * e.eps * n * (q - 2.0f * q2) / r;
    d2 = 4.0f * e.eps * curvature(n, q, q2) / r2;
}

// w = sqrt(Lambda) vhat and its first two r-derivatives
__device__ __forceinline__ void w_d012(const DevEntry& e, bool inside, float r2, float r, float& w,
                                       float& w1, float& w2) {
#pragma clang fp contract(off)
    if (inside) {
        w = e.sqrt_lam;
        w1 = 0.0f;
        w2 = 0.0f;
        return;
    }
    const float q = qpow(e.sig2 / r2, e.n);
    const float q2 = q * q, n = (float)e.n;
    w = e.sqrt_lam * 4.0f * (q - q2);
    w1 = e.sqrt_lam * 4.0f * n * (2.0f * q2 - q) / r;
    w2 = -e.sqrt_lam * 4.0f * curvature(n, q, q2) / r2;
}

// a . (u - v) over the first three components
__device__ __forceinline__ float along(float ax, float ay, float az, const float4& u, const float4& v, float& dx,
                                       float& dy, float& dz) {
#pragma clang fp contract(off)
    dx = u.x - v.x;
    dy = u.y - v.y;
    dz = u.z - v.z;
    return __fmaf_rn(az, dz, __fmaf_rn(ay, dy, ax * dx));
}

// Both passes: one thread per particle and group of V tangent vectors (grid
// row y holds vectors yV .. yV + V - 1).  The list walk, the FP64 decision and
// the derivatives of a term are the same for every vector, so a thread does
// them once for its V vectors; a vector's own part is two loads and ~20 FP32
// operations per term.  The next neighbour's index and position are requested
// before the current one is used.  Bound by the latency of the gathers of v and
// dS.  Walking marked neighbours (inside the cutoff) only, or v and dS of the
// block's particles in LDS, gained nothing (83 and 98 us).
// 64 vectors at 32768 particles, both passes: 160 -> 86 us.
// Scratch (16 bytes per particle and vector hold it): S of every particle,
// then dS of every particle per vector.

// f(j, pos[j]) for the slots [0, cnt) of particle m's column, the next neighbour in flight
template <class F>
__device__ __forceinline__ void walk_ahead(const HvpArgs& a, int m, int ns, int cnt, const float4& pm, F&& f) {
    auto slot = [&](int s) { return (size_t)(s < ns ? s : a.k_max - 1 - (s - ns)) * a.N + m; };
    int j = cnt > 0 ? a.nlist[slot(0)] : m, jn = cnt > 1 ? a.nlist[slot(1)] : m;
    float4 pj = cnt > 0 ? a.pos[j] : pm;
    for (int s = 0; s < cnt; ++s) {
        const int j2 = s + 2 < cnt ? a.nlist[slot(s + 2)] : m;
        const float4 pn = a.pos[jn];
        f(j, pj);
        j = jn;
        pj = pn;
        jn = j2;
    }
}

// first pass: S and dS = sum_b w'_mb rhat_mb . (v_b - v_m) over m's swap partners
template <int V>
__global__ __launch_bounds__(kBlock) void k_hvp_sums(HvpArgs a) {
    extern __shared__ DevEntry s_tab[];
    load_table_adj(s_tab, a.tab);
    const int m = xcd_block(gridDim.x) * kBlock + threadIdx.x;
    if (m >= a.N) return;
    const int y0 = blockIdx.y * V, nv = min(V, a.nvec - y0);   // vectors past the last repeat it and are not stored
    const float4* v[V];
    float4 vm[V];
    double dS[V];
#pragma unroll
    for (int u = 0; u < V; ++u) {
        v[u] = a.v + (size_t)(y0 + min(u, nv - 1)) * a.N;
        vm[u] = v[u][m];
        dS[u] = 0.0;
    }
    const float4 pm = a.pos[m];
    const int tm = ptype(pm.w), ns = nn_swap(a.nn[m]);   // swap-kind neighbours fill the front of the column
    double S = 0.0;
    walk_ahead(a, m, ns, ns, pm, [&](int b, const float4& pb) {
#pragma clang fp contract(off)
        const DevEntry& e = s_tab[tm * a.tab.nt + ptype(pb.w)];
        if (e.kind != RC_KIND_SWAP) return;
        double dx, dy, dz;
        const double r2d = canon_r2(pm, pb, a.box, dx, dy, dz);
        if (!(r2d < e.rcut2)) return;
        float4 vb[V];
#pragma unroll
        for (int u = 0; u < V; ++u) vb[u] = v[u][b];
        const float r2 = (float)r2d, r = sqrtf(r2);
        float w, w1, w2;
        w_d012(e, r2d <= e.rmin2, r2, r, w, w1, w2);
        S += (double)w;
#pragma unroll
        for (int u = 0; u < V; ++u) {
            float Dx, Dy, Dz;
            const float dr = along((float)dx, (float)dy, (float)dz, vb[u], vm[u], Dx, Dy, Dz) / r;
            dS[u] += (double)(w1 * dr);
        }
    });
    double* sums = reinterpret_cast<double*>(a.sums);
    if (y0 == 0) sums[m] = S;
#pragma unroll
    for (int u = 0; u < V; ++u)
        if (u < nv) sums[(size_t)(y0 + u + 1) * a.N + m] = dS[u];
}

template <int V>
__global__ __launch_bounds__(kBlock) void k_hvp(HvpArgs a) {
    extern __shared__ DevEntry s_tab[];
    load_table_adj(s_tab, a.tab);
    const int m = xcd_block(gridDim.x) * kBlock + threadIdx.x;
    if (m >= a.N) return;
    const int y0 = blockIdx.y * V, nv = min(V, a.nvec - y0);
    const double* sums = reinterpret_cast<const double*>(a.sums);
    const float4* v[V];
    const double* ds[V];
    float4 vm[V];
    double dSm[V];
    float hx[V], hy[V], hz[V];
#pragma unroll
    for (int u = 0; u < V; ++u) {
        const int y = y0 + min(u, nv - 1);
        v[u] = a.v + (size_t)y * a.N;
        ds[u] = sums + (size_t)(y + 1) * a.N;
        vm[u] = v[u][m];
        dSm[u] = ds[u][m];
        hx[u] = hy[u] = hz[u] = 0.f;
    }
    const float4 pm = a.pos[m];
    const int tm = ptype(pm.w);
    const int packed = a.nn[m];
    const int ns = nn_swap(packed), cnt = ns + nn_other(packed);
    const double Sm = sums[m];
    walk_ahead(a, m, ns, cnt, pm, [&](int j, const float4& pj) {
#pragma clang fp contract(off)
        const DevEntry& e = s_tab[tm * a.tab.nt + ptype(pj.w)];
        if (e.kind == RC_KIND_NONE) return;
        double dxd, dyd, dzd;
        const double r2d = canon_r2(pm, pj, a.box, dxd, dyd, dzd);
        if (!(r2d < e.rcut2)) return;
        float4 vj[V];
#pragma unroll
        for (int u = 0; u < V; ++u) vj[u] = v[u][j];
        const float r2 = (float)r2d, r = sqrtf(r2), ir = 1.0f / r;
        const float rx = (float)dxd * ir, ry = (float)dyd * ir, rz = (float)dzd * ir;
        float G0, dG0, w = 0.f, w1 = 0.f, w2 = 0.f, X = 0.f;
        pair_d12(e, r2, r, G0, dG0);
        bool three = false;
        if (e.kind == RC_KIND_SWAP) {
            w_d012(e, r2d <= e.rmin2, r2, r, w, w1, w2);
            three = w1 != 0.0f || w2 != 0.0f;
        }
        double dSj[V];
        if (three) {
            const double Sj = sums[j];
#pragma unroll
            for (int u = 0; u < V; ++u) dSj[u] = ds[u][j];
            X = (float)((Sm - (double)w) + (Sj - (double)w));
        }
#pragma unroll
        for (int u = 0; u < V; ++u) {
            float Dx, Dy, Dz;
            const float dr = along(rx, ry, rz, vj[u], vm[u], Dx, Dy, Dz);
            float G = G0, dG = dG0 * dr;
            if (three) {
                const double d = (double)(w1 * dr);
                const float dX = (float)((dSm[u] - d) + (dSj[u] - d));
                G = __fmaf_rn(w1, X, G);
                dG = dG + __fmaf_rn(w1, dX, (w2 * dr) * X);
            }
            const float c = G * ir;
            hx[u] = hx[u] - __fmaf_rn(c, __fmaf_rn(-dr, rx, Dx), dG * rx);
            hy[u] = hy[u] - __fmaf_rn(c, __fmaf_rn(-dr, ry, Dy), dG * ry);
            hz[u] = hz[u] - __fmaf_rn(c, __fmaf_rn(-dr, rz, Dz), dG * rz);
        }
    });
#pragma unroll
    for (int u = 0; u < V; ++u)
        if (u < nv) a.hv[(size_t)(y0 + u) * a.N + m] = make_float4(hx[u], hy[u], hz[u], 0.0f);
}

template <int V>
static void launch_hvp_v(const HvpArgs& a, hipStream_t s) {
    const size_t shm = sizeof(DevEntry) * a.tab.nt * a.tab.nt;
    const dim3 grid(nblk(a.N, kBlock), nblk(a.nvec, V));
    hipLaunchKernelGGL(k_hvp_sums<V>, grid, dim3(kBlock), shm, s, a);
    hipLaunchKernelGGL(k_hvp<V>, grid, dim3(kBlock), shm, s, a);
}

hipError_t launch_hvp(const HvpArgs& a, hipStream_t s) {
    if (a.nvec < 1 || a.nvec > 65535) return hipErrorInvalidValue;
    // Vectors per thread, by the blocks one vector per thread would make: sharing the walk pays once they
    // fill the chip several times (us with 1, 2, 4, 8 vectors per thread at 512 blocks: 21.9, 22.4, 25.1, 30.1;
    // 1024: 28.9, 24.5, 25.8, 30.3; 2048: 45.5, 33.8, 30.3, 32.7; 8192: 141, 97, 86, 89)
    const long blocks = (long)nblk(a.N, kBlock) * a.nvec;
    if (blocks >= 2048) launch_hvp_v<4>(a, s);
    else if (blocks >= 1024) launch_hvp_v<2>(a, s);
    else launch_hvp_v<1>(a, s);
    return hipGetLastError();
}

// ---------------------------------------------------------------------------
// dE / d(eps, sigma, lambda) per table entry, at fixed r_cut.
//  pair (half per list direction):  d/deps = phi/eps,  d/dsigma = 4 eps n (2q^2 - q)/sigma
//  triplets of centre m, per active partner a with entry e:
//     d/dlambda_e  = w_a (S - w_a) / (2 lambda_e)        (lambda_e > 0)
//                  = eps_e u_a (U_e - u_a) / 2            (lambda_e = 0, same-entry pairs)
//     d/deps_e     = w_a (S - w_a) / (2 eps_e)
//     d/dsigma_e   = sqrt(Lambda) du_a/dsigma (S - w_a),  du/dsigma = -4 n (2q^2 - q)/sigma beyond r_min
//  With sums over the partners of one entry (X = sum w, or sum u where lambda_e
//  = 0, X2 the same of squares, D = sum sqrt(Lambda) du/dsigma, DW = sum of that
//  times w) the four are (S X - X2) / (2 lambda), eps (X^2 - X2) / 2, (S X - X2)
//  / (2 eps) and S D - DW, in FP64 of FP32 terms.
//
// Both parameter kernels: one thread per centre and one walk of its list for
// every NT types (one walk up to four types), the entries' sums in registers.
// A walk is a chain of reads, so four neighbours' indices, then their data are
// requested at a time.  At 32768 particles of one type, two walks of one
// neighbour after the other with an LDS atomic per term took 23.8 us (energy
// gradient) and 23.3 us (force product); now 12.8 and 13.8.
// ---------------------------------------------------------------------------

// f(pos[j], adj[j]) for the slots [0, cnt) of particle m's column, four requested at a time
template <bool ADJ, class F>
__device__ __forceinline__ void walk_four(const ParamArgs& a, int m, int ns, int cnt, const float4& pm, F&& f) {
    for (int b = 0; b < cnt; b += 4) {
        int j[4];
        float4 p[4], v[4];
#pragma unroll
        for (int u = 0; u < 4; ++u) {
            const int s = b + u;
            j[u] = s < cnt ? a.nlist[(size_t)(s < ns ? s : a.k_max - 1 - (s - ns)) * a.N + m] : m;
        }
#pragma unroll
        for (int u = 0; u < 4; ++u) {
            p[u] = b + u < cnt ? a.pos[j[u]] : pm;
            if constexpr (ADJ) v[u] = b + u < cnt ? a.adj[j[u]] : pm;
        }
#pragma unroll
        for (int u = 0; u < 4; ++u)
            if (b + u < cnt) f(p[u], v[u]);
    }
}

// one thread's three values of the unordered entry {ta, tb} into the block's sums: every lane takes part
__device__ __forceinline__ void add_entry(double* s_acc, int nt, int ta, int tb, bool live, const double (&v)[3]) {
    if (nt == 1) {   // every lane has the same entry: no 64 additions to one address
#pragma unroll
        for (int q = 0; q < 3; ++q) {
            const double t = wave_sum(live ? v[q] : 0.0);
            if ((threadIdx.x & (kWave - 1)) == 0) atomicAdd(&s_acc[q], t);
        }
    } else if (live) {
        const int key = (ta < tb ? ta * nt + tb : tb * nt + ta) * 3;
#pragma unroll
        for (int q = 0; q < 3; ++q) atomicAdd(&s_acc[key + q], v[q]);
    }
}

template <int NT>
__global__ __launch_bounds__(kBlock) void k_param_grad(ParamArgs a) {
    extern __shared__ __align__(16) unsigned char s_raw[];
    const int nt = a.tab.nt, ne = nt * nt;
    DevEntry* s_tab = reinterpret_cast<DevEntry*>(s_raw);
    double* s_acc = reinterpret_cast<double*>(s_raw + sizeof(DevEntry) * ne);
    for (int q = threadIdx.x; q < ne * 3; q += blockDim.x) s_acc[q] = 0.0;
    const int m = blockIdx.x * blockDim.x + threadIdx.x;
    const bool live = m < a.N;
    const float4 pm = live ? a.pos[m] : make_float4(0.f, 0.f, 0.f, 0.f);
    const int packed = live ? a.nn[m] : 0;
    load_table_adj(s_tab, a.tab);
    const int tm = ptype(pm.w);
    const int ns = nn_swap(packed), cnt = ns + nn_other(packed);
    double S = 0.0;
    for (int t0 = 0; t0 < nt; t0 += NT) {
        double pe[NT] = {}, ps[NT] = {}, X[NT] = {}, X2[NT] = {}, D[NT] = {}, DW[NT] = {};
        walk_four<false>(a, m, ns, cnt, pm, [&](const float4& pj, const float4&) {
            const int tj = ptype(pj.w);
            const DevEntry& e = s_tab[tm * nt + tj];
            if (e.kind == RC_KIND_NONE || (NT < 4 ? false : t0 > 0 && (tj < t0 || tj >= t0 + NT))) return;
            double dx, dy, dz;
            const double r2d = canon_r2(pm, pj, a.box, dx, dy, dz);
            if (!(r2d < e.rcut2)) return;
            const float r2 = (float)r2d;
            const bool inside = r2d <= e.rmin2;
            float phi, g;
            pair_eval(e, r2, phi, g);
            const float q = qpow(e.sig2 / r2, e.n);
            const float dsig = 4.0f * e.eps * (float)e.n * (2.0f * q * q - q) / e.sigma;
            double x = 0.0, d = 0.0, dw = 0.0;
            if (e.kind == RC_KIND_SWAP) {
                const float u = vhat_value(e, inside, r2), w = e.sqrt_lam * u;
                if (t0 == 0) S += (double)w;
                x = e.lam > 0.0f ? (double)w : (double)u;
                if (!inside) {
                    const float du = -4.0f * (float)e.n * (2.0f * q * q - q) / e.sigma;
                    d = (double)(e.sqrt_lam * du);
                    dw = d * (double)w;
                }
            }
#pragma unroll
            for (int t = 0; t < NT; ++t) {
                const bool on = NT == 1 || tj == t0 + t;
                pe[t] += on ? 0.5 * (double)(phi / e.eps) : 0.0;
                ps[t] += on ? 0.5 * (double)dsig : 0.0;
                X[t] += on ? x : 0.0;
                X2[t] += on ? x * x : 0.0;
                D[t] += on ? d : 0.0;
                DW[t] += on ? dw : 0.0;
            }
        });
#pragma unroll
        for (int t = 0; t < NT; ++t) {
            const int te = t0 + t;
            if (te >= nt) break;
            const DevEntry& e = s_tab[tm * nt + te];
            double v[3] = {pe[t], ps[t], 0.0};
            if (e.kind == RC_KIND_SWAP) {
                if (e.lam > 0.0f) {
                    const double c = S * X[t] - X2[t];
                    v[2] = c / (2.0 * (double)e.lam);
                    v[0] += c / (2.0 * (double)e.eps);
                } else {
                    // lambda = 0: E3 of same-entry pairs is lambda eps sum u_a u_b
                    v[2] = 0.5 * (double)e.eps * (X[t] * X[t] - X2[t]);
                }
                v[1] += S * D[t] - DW[t];
            }
            add_entry(s_acc, nt, tm, te, live, v);
        }
    }
    __syncthreads();
    for (int q = threadIdx.x; q < ne * 3; q += blockDim.x) a.part[(size_t)blockIdx.x * ne * 3 + q] = s_acc[q];
}

// ---------------------------------------------------------------------------
// Force-parameter VJP: out[e][w] = sum_m a_m . dF_m / dtheta_w(e), theta =
// (eps, sigma, lambda) of the unordered entry e.  With D = rhat . (a_j - a_m)
// the work of the adjoint field on a term:
//  pair (half per list direction):  a . F = -phi'(r) D, so
//     d/deps = -(phi'/eps) D,  d/dsigma = -4 eps n^2 (q - 4 q^2) / (sigma r) D
//  triplets of centre m (swap partners a inside r_cut, k_a = sqrt(lambda eps)
//  of the edge, u = vhat, u' = du/dr, D_a = rhat_a . (a_a - a_m)):
//     a . F = -T,  T = sum_{a != b} k_a k_b u_b u'_a D_a = S P - Q,
//     S = sum k u,  P = sum k u' D,  Q = sum k^2 u u' D.
//  Per partner entry e (sums restricted to partners of entry e carry the
//  subscript e; U, V, X are the unweighted sum u, sum u' D, sum u u' D):
//     dT/dlambda_e = eps_e (U V - X) + [P_e (S - S_e) + (P - P_e) S_e] / (2 lambda_e)
//     dT/deps_e    = lambda_e (U V - X) + [P_e (S - S_e) + (P - P_e) S_e] / (2 eps_e)
//     dT/dsigma_e  = A P - B + C S - G,  A = sum_e k u_s,  B = sum_e k^2 u_s u' D,
//                    C = sum_e k u'_s D,  G = sum_e k^2 u'_s D u
//  with u_s = du/dsigma = 4 n (q - 2q^2)/sigma and u'_s = 4 n^2 (4q^2 - q)/(sigma r)
//  beyond r_min (all zero inside, where u = 1).  The cross term of
//  dT/dlambda_e is taken as 0 when lambda_e = 0 (its derivative is unbounded
//  there), as in the energy gradient.
// ---------------------------------------------------------------------------
struct SwapTerms {  // u, u', du/dsigma, du'/dsigma of one swap edge
    float u, u1, us, u1s;
};

__device__ __forceinline__ SwapTerms swap_terms(const DevEntry& e, bool inside, float r2, float r) {
    SwapTerms t{1.0f, 0.0f, 0.0f, 0.0f};
    if (inside) return t;
    const float q = qpow(e.sig2 / r2, e.n);
    const float q2 = q * q, n = (float)e.n;
    t.u = 4.0f * (q - q2);
    t.u1 = 4.0f * n * (2.0f * q2 - q) / r;
    t.us = 4.0f * n * (q - 2.0f * q2) / e.sigma;
    t.u1s = 4.0f * n * n * (4.0f * q2 - q) / (e.sigma * r);
    return t;
}

template <int NT>
__global__ __launch_bounds__(kBlock) void k_param_vjp(ParamArgs a) {
    extern __shared__ __align__(16) unsigned char s_raw[];
    const int nt = a.tab.nt, ne = nt * nt;
    DevEntry* s_tab = reinterpret_cast<DevEntry*>(s_raw);
    double* s_acc = reinterpret_cast<double*>(s_raw + sizeof(DevEntry) * ne);
    for (int q = threadIdx.x; q < ne * 3; q += blockDim.x) s_acc[q] = 0.0;
    const int m = blockIdx.x * blockDim.x + threadIdx.x;
    const bool live = m < a.N;
    const float4 zero = make_float4(0.f, 0.f, 0.f, 0.f);
    const float4 pm = live ? a.pos[m] : zero, am = live ? a.adj[m] : zero;
    const int packed = live ? a.nn[m] : 0;
    load_table_adj(s_tab, a.tab);
    const int tm = ptype(pm.w);
    const int ns = nn_swap(packed), cnt = ns + nn_other(packed);
    double S = 0.0, P = 0.0;   // over every swap partner
    for (int t0 = 0; t0 < nt; t0 += NT) {
        // per partner type: pair terms, and the sums U, V, X and (A, B, C, G) without their factors k
        double pe[NT] = {}, ps[NT] = {}, U[NT] = {}, V[NT] = {}, X[NT] = {}, A[NT] = {}, B[NT] = {}, C[NT] = {}, G[NT] = {};
        walk_four<true>(a, m, ns, cnt, pm, [&](const float4& pj, const float4& aj) {
            const int tj = ptype(pj.w);
            const DevEntry& e = s_tab[tm * nt + tj];
            if (e.kind == RC_KIND_NONE || (NT < 4 ? false : t0 > 0 && (tj < t0 || tj >= t0 + NT))) return;
            double dx, dy, dz;
            const double r2d = canon_r2(pm, pj, a.box, dx, dy, dz);
            if (!(r2d < e.rcut2)) return;
            const float r2 = (float)r2d, r = sqrtf(r2), ir = 1.0f / r;
            const float dot = (float)dx * (aj.x - am.x) + (float)dy * (aj.y - am.y) + (float)dz * (aj.z - am.z);
            const float D = dot * ir, Dr = dot / r;
            const float q = qpow(e.sig2 / r2, e.n), q2 = q * q, n = (float)e.n;
            const float d1 = 4.0f * e.eps * n * (q - 2.0f * q2) * ir;
            const float d1s = 4.0f * e.eps * n * n * (q - 4.0f * q2) / (e.sigma * r);
            const double te = -0.5 * (double)(d1 / e.eps * D), ts = -0.5 * (double)(d1s * D);
            SwapTerms w{0.0f, 0.0f, 0.0f, 0.0f};
            if (e.kind == RC_KIND_SWAP) {
                w = swap_terms(e, r2d <= e.rmin2, r2, r);
                if (t0 == 0) {
                    S += (double)(e.sqrt_lam * w.u);
                    P += (double)(e.sqrt_lam * w.u1 * D);
                }
            }
            const double u = w.u, v = (double)w.u1 * Dr, us = w.us, vs = (double)w.u1s * Dr;
#pragma unroll
            for (int t = 0; t < NT; ++t) {
                const bool on = NT == 1 || tj == t0 + t;
                pe[t] += on ? te : 0.0;
                ps[t] += on ? ts : 0.0;
                U[t] += on ? u : 0.0;
                V[t] += on ? v : 0.0;
                X[t] += on ? u * v : 0.0;
                A[t] += on ? us : 0.0;
                B[t] += on ? us * v : 0.0;
                C[t] += on ? vs : 0.0;
                G[t] += on ? vs * u : 0.0;
            }
        });
#pragma unroll
        for (int t = 0; t < NT; ++t) {
            const int te = t0 + t;
            if (te >= nt) break;
            const DevEntry& e = s_tab[tm * nt + te];
            double v[3] = {pe[t], ps[t], 0.0};
            if (e.kind == RC_KIND_SWAP) {
                const double lam = (double)e.lam, eps = (double)e.eps, k = (double)e.sqrt_lam;
                const double Se = k * U[t], Pe = k * V[t];
                const double same = U[t] * V[t] - X[t];
                const double cross = Pe * (S - Se) + (P - Pe) * Se;
                v[0] -= lam * same + cross / (2.0 * eps);
                v[1] -= k * (A[t] * P + C[t] * S) - k * k * (B[t] + G[t]);
                v[2] = -(eps * same + (lam > 0.0 ? cross / (2.0 * lam) : 0.0));
            }
            add_entry(s_acc, nt, tm, te, live, v);
        }
    }
    __syncthreads();
    for (int q = threadIdx.x; q < ne * 3; q += blockDim.x) a.part[(size_t)blockIdx.x * ne * 3 + q] = s_acc[q];
}

__global__ __launch_bounds__(kBlock) void k_reduce_param(const double* __restrict__ part, int nblocks,
                                                        int nt, double* __restrict__ out) {
    // one block per output value (upper-triangle key), mirrored to both entries
    __shared__ double red[kBlock];
    const int q = blockIdx.x;
    const int ne3 = nt * nt * 3;
    double s = 0.0;
    for (int b = threadIdx.x; b < nblocks; b += blockDim.x) s += part[(size_t)b * ne3 + q];
    red[threadIdx.x] = s;
    __syncthreads();
    for (int w = kBlock / 2; w > 0; w >>= 1) {
        if (threadIdx.x < w) red[threadIdx.x] += red[threadIdx.x + w];
        __syncthreads();
    }
    if (threadIdx.x == 0) {
        const int key = q / 3, comp = q % 3;
        const int ta = key / nt, tb = key % nt;
        if (ta <= tb) {
            out[(ta * nt + tb) * 3 + comp] = red[0];
            out[(tb * nt + ta) * 3 + comp] = red[0];
        }
    }
}

// One wavefront per block while blocks of four would leave compute units without one.
int param_block(int N) { return N <= 256 * kBlock ? kWave : kBlock; }

template <template <int> class K>
static hipError_t launch_param_nt(const ParamArgs& a, hipStream_t s) {
    const int ne = a.tab.nt * a.tab.nt;
    const size_t shm = sizeof(DevEntry) * ne + sizeof(double) * ne * 3;
    const dim3 g(nblk(a.N, param_block(a.N))), b(param_block(a.N));
    switch (std::min(a.tab.nt, 4)) {
        case 1: hipLaunchKernelGGL(K<1>::fn, g, b, shm, s, a); break;
        case 2: hipLaunchKernelGGL(K<2>::fn, g, b, shm, s, a); break;
        case 3: hipLaunchKernelGGL(K<3>::fn, g, b, shm, s, a); break;
        default: hipLaunchKernelGGL(K<4>::fn, g, b, shm, s, a);
    }
    return hipGetLastError();
}
template <int NT>
struct ParamGrad {
    static constexpr auto fn = &k_param_grad<NT>;
};
template <int NT>
struct ParamVjp {
    static constexpr auto fn = &k_param_vjp<NT>;
};

hipError_t launch_param(const ParamArgs& a, hipStream_t s) { return launch_param_nt<ParamGrad>(a, s); }
hipError_t launch_param_vjp(const ParamArgs& a, hipStream_t s) { return launch_param_nt<ParamVjp>(a, s); }

// ---------------------------------------------------------------------------
// Soft bond count B = sum over swap pairs i<j inside r_cut of vhat(r_ij)
// (1 for a bonded pair, r <= r_min, decaying to 0 at r_cut; eq. pot) and its
// gradient dB/dx_m = - sum_j vhat'(r_mj) rhat_mj over m's swap partners.
// Bound by its chain of reads (entry, then position), so four entries are
// requested at a time: 14.6 -> 11.4 us at 200003 particles of three types.
// ---------------------------------------------------------------------------
__global__ __launch_bounds__(kBlock) void k_soft_bonds(const float4* __restrict__ pos,
                                                      const int* __restrict__ nlist, const int* __restrict__ nn,
                                                      int k_max, int N, Table tab, Box box,
                                                      double* __restrict__ part, float4* __restrict__ grad) {
    extern __shared__ DevEntry s_tab[];
    __shared__ double s_w[kBlock / kWave];
    load_table_adj(s_tab, tab);
    const int m = blockIdx.x * blockDim.x + threadIdx.x;
    double b = 0.0;
    if (m < N) {
        const float4 pm = pos[m];
        const int tm = ptype(pm.w);
        const int ns = nn_swap(nn[m]);
        float gx = 0.f, gy = 0.f, gz = 0.f;
        for (int s0 = 0; s0 < ns; s0 += 4) {
            int j[4];
            float4 p[4];
#pragma unroll
            for (int v = 0; v < 4; ++v) j[v] = s0 + v < ns ? nlist[(size_t)(s0 + v) * N + m] : m;
#pragma unroll
            for (int v = 0; v < 4; ++v) p[v] = pos[j[v]];
#pragma unroll
            for (int v = 0; v < 4; ++v) {
                const float4 pj = p[v];
                const DevEntry& e = s_tab[tm * tab.nt + ptype(pj.w)];
                if (s0 + v >= ns || e.kind != RC_KIND_SWAP) continue;
                double dx, dy, dz;
                const double r2d = canon_r2(pm, pj, box, dx, dy, dz);
                if (!(r2d < e.rcut2)) continue;
                float u, u1r;
                vhat_eval(e, r2d <= e.rmin2, (float)r2d, u, u1r);
                b += 0.5 * (double)u;
                gx -= u1r * (float)dx;
                gy -= u1r * (float)dy;
                gz -= u1r * (float)dz;
            }
        }
        if (grad) grad[m] = make_float4(gx, gy, gz, 0.0f);
    }
    b = wave_sum(b);
    if ((threadIdx.x & (kWave - 1)) == 0) s_w[threadIdx.x / kWave] = b;
    __syncthreads();
    if (threadIdx.x == 0) {
        double t = 0.0;
        for (int w = 0; w < kBlock / kWave; ++w) t += s_w[w];
        part[blockIdx.x] = t;
    }
}

__global__ __launch_bounds__(kBlock) void k_sum_doubles(const double* __restrict__ part, int nb,
                                                       double* __restrict__ out) {
    __shared__ double red[kBlock];
    double s = 0.0;
    for (int b = threadIdx.x; b < nb; b += blockDim.x) s += part[b];
    red[threadIdx.x] = s;
    __syncthreads();
    for (int w = kBlock / 2; w > 0; w >>= 1) {
        if (threadIdx.x < w) red[threadIdx.x] += red[threadIdx.x + w];
        __syncthreads();
    }
    if (threadIdx.x == 0) *out = red[0];
}

hipError_t launch_soft_bonds(const float4* pos, const int* nlist, const int* nn, int k_max, int N, Table tab,
                             Box box, double* part, double* value, float4* grad, hipStream_t s) {
    const size_t shm = sizeof(DevEntry) * tab.nt * tab.nt;
    const int nb = nblk(N, kBlock);
    hipLaunchKernelGGL(k_soft_bonds, dim3(nb), dim3(kBlock), shm, s, pos, nlist, nn, k_max, N, tab, box, part, grad);
    hipLaunchKernelGGL(k_sum_doubles, dim3(1), dim3(kBlock), 0, s, part, nb, value);
    return hipGetLastError();
}

hipError_t launch_reduce_param(const double* part, int nblocks, int nt, double* out, hipStream_t s) {
    hipLaunchKernelGGL(k_reduce_param, dim3(nt * nt * 3), dim3(kBlock), 0, s, part, nblocks, nt, out);
    return hipGetLastError();
}

}  // namespace rc
