// Tag-ordered views of a system's state, for callers that keep positions and
// per-particle vectors by tag (the differentiable bindings): positions loaded
// into the engine's order and checked against those of the last list build, and
// float4 arrays read or written in tag order.  One pass each over the particles,
// bound by its launch below ~10^5 particles; written with tensor operations, a
// load took a dozen launches and a reordering three (a differentiated evaluation
// of energy and forces at 32768 particles: 127 launches and 1.2-1.3 ms; now 34 and
// 0.60 ms).
#include "rc_host.h"

#include <climits>

namespace rc {

// Position of tag t folded into the box, rounded as x - L floor((x + L/2) / L)
// is, operation by operation, with the upper edge excluded.
__device__ __forceinline__ float fold_edge(float x, float L) {
#pragma clang fp contract(off)
    const float h = 0.5f * L;
    const float w = x - L * floorf((x + h) / L);
    return w >= h ? w - L : w;
}

// d - L rint(d / L)
__device__ __forceinline__ float nearest(float d, float L) {
#pragma clang fp contract(off)
    return d - L * rintf(d / L);
}

// host (pinned): [0] some particle farther than sqrt(far2) from its ref, [1] some distance not a number.  Stores
// to host memory go over the bus one by one: from every wavefront that has such a particle they took 440 us at
// 262144 particles which all moved, so only the first that sets mark[q] to this load's number stores.
__device__ __forceinline__ void report_once(int* mark, int number, int* host) {
    if (__hip_atomic_load(mark, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) == number) return;
    if (atomicExch(mark, number) != number) __hip_atomic_store(host, 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_SYSTEM);
}

__global__ __launch_bounds__(kBlock) void k_load_by_tag(float4* __restrict__ pos, const float* __restrict__ xyz,
                                                        const float* __restrict__ ref, int N, Box box, float far2,
                                                        int* mark, int number, int* host) {
    const int i = blockIdx.x * blockDim.x + threadIdx.x;
    bool far = false, nan = false;
    if (i < N) {
        const float w = pos[i].w;
        const int t = ptag(w);
        if (t >= 0 && t < N) {
            float x[3], r2 = 0.0f;
#pragma unroll
            for (int q = 0; q < 3; ++q) {
                x[q] = fold_edge(xyz[3 * (size_t)t + q], box.Lf[q]);
                const float d = nearest(x[q] - ref[3 * (size_t)t + q], box.Lf[q]);
                r2 += d * d;
            }
            pos[i] = make_float4(x[0], x[1], x[2], w);
            far = r2 > far2;
            nan = !(r2 == r2);
        }
    }
    const unsigned long long bf = __ballot(far), bn = __ballot(nan);
    if ((threadIdx.x & (kWave - 1)) == 0) {
        if (bf) report_once(mark, number, host);
        if (bn) report_once(mark + 1, number, host + 1);
    }
}

// out[t] = sign arr[rtag[t]], three components
__global__ __launch_bounds__(kBlock) void k_to_tags(const float4* __restrict__ arr, const int* __restrict__ rtag,
                                                    int N, int negate, float* __restrict__ out) {
    const int t = blockIdx.x * blockDim.x + threadIdx.x;
    if (t >= N) return;
    const float4 v = arr[rtag[t]];
    out[3 * (size_t)t] = negate ? -v.x : v.x;
    out[3 * (size_t)t + 1] = negate ? -v.y : v.y;
    out[3 * (size_t)t + 2] = negate ? -v.z : v.z;
}

// out[i] = (v[tag of i], 0)
__global__ __launch_bounds__(kBlock) void k_from_tags(const float* __restrict__ v, const float4* __restrict__ pos,
                                                      int N, float4* __restrict__ out) {
    const int i = blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= N) return;
    const int t = ptag(pos[i].w);
    const bool ok = t >= 0 && t < N;
    const float* p = v + 3 * (size_t)(ok ? t : 0);
    out[i] = ok ? make_float4(p[0], p[1], p[2], 0.0f) : make_float4(0.f, 0.f, 0.f, 0.f);
}

}  // namespace rc

using namespace rc;
using namespace rc::host;

extern "C" int rc_load_by_tag(rc_ctx* c, float* pos, const float* xyz, const float* ref, int N, rc_box box,
                              double reach, void* stream) {
    if (!c) return RC_ERR_ARG;
    c->md.valid = false;   // the state changes outside the driver
    if (N < 1 || N >= RC_MAX_TAG) return fail(c, RC_ERR_ARG, "need 1 <= N < 2^27 (N = %d)", N);
    if (!pos || !xyz || !ref) return fail(c, RC_ERR_ARG, "rc_load_by_tag: a required array is NULL");
    if (reinterpret_cast<uintptr_t>(pos) & 15) return fail(c, RC_ERR_ARG, "positions not 16-byte aligned");
    Box b;
    int r = make_box(c, box, b);
    if (r || (r = ensure_host_words(c))) return r;
    hipStream_t s = S(stream);
    if (c->ev_load) {   // an earlier load's words may not have been asked for
        if ((r = wait_event(c, c->ev_load))) return r;
    } else {
        HIP_TRY(c, hipEventCreateWithFlags(&c->ev_load, hipEventDisableTiming));
    }
    volatile int* host = c->h_status + kLoadWords;
    host[0] = host[1] = 0;
    c->load_mark = c->load_mark == INT_MAX ? 1 : c->load_mark + 1;
    hipLaunchKernelGGL(k_load_by_tag, dim3(nblocks(N, kBlock)), dim3(kBlock), 0, s, reinterpret_cast<float4*>(pos), xyz,
                       ref, N, b, (float)(reach * reach), reinterpret_cast<int*>(c->d_step_base + 2), c->load_mark,
                       c->h_status + kLoadWords);
    HIP_TRY(c, hipGetLastError());
    HIP_TRY(c, hipEventRecord(c->ev_load, s));
    return RC_OK;
}

extern "C" int rc_load_moved(rc_ctx* c, int* moved) {
    if (!c || !moved) return RC_ERR_ARG;
    if (!c->ev_load) return fail(c, RC_ERR_ARG, "rc_load_moved follows rc_load_by_tag");
    int r = wait_event(c, c->ev_load);
    if (r) return r;
    const volatile int* host = c->h_status + kLoadWords;
    *moved = host[0] && !host[1];
    return RC_OK;
}

extern "C" int rc_to_tags(rc_ctx* c, const float* arr, const int* rtag, int N, int negate, float* out, void* stream) {
    if (!c) return RC_ERR_ARG;
    if (N < 1 || !arr || !rtag || !out || (reinterpret_cast<uintptr_t>(arr) & 15))
        return fail(c, RC_ERR_ARG, "rc_to_tags: N >= 1, arrays not NULL, arr 16-byte aligned");
    hipLaunchKernelGGL(k_to_tags, dim3(nblocks(N, kBlock)), dim3(kBlock), 0, S(stream),
                       reinterpret_cast<const float4*>(arr), rtag, N, negate, out);
    HIP_TRY(c, hipGetLastError());
    return RC_OK;
}

extern "C" int rc_from_tags(rc_ctx* c, const float* v, const float* pos, int N, float* out, void* stream) {
    if (!c) return RC_ERR_ARG;
    if (N < 1 || !v || !pos || !out || ((reinterpret_cast<uintptr_t>(pos) | reinterpret_cast<uintptr_t>(out)) & 15))
        return fail(c, RC_ERR_ARG, "rc_from_tags: N >= 1, arrays not NULL, pos and out 16-byte aligned");
    hipLaunchKernelGGL(k_from_tags, dim3(nblocks(N, kBlock)), dim3(kBlock), 0, S(stream), v,
                       reinterpret_cast<const float4*>(pos), N, reinterpret_cast<float4*>(out));
    HIP_TRY(c, hipGetLastError());
    return RC_OK;
}
