// Rigid planar bodies for the patchy colloids of Sec. 3.2: a disk (the body's
// centre particle) carrying massless patch particles at fixed body-frame
// offsets.  The forces on every particle come from the stand-alone force
// kernel; this file sums them per body into a force and a torque, advances
// the body's (x, y, angle) by the BAOAB half steps of the particle integrator
// (with the angle driven by the torque, the body's moment of inertia and a
// rotational friction equal to the translational one), and places the patches
// at the new pose.  Members are found by tag (rtag).
#include <cmath>

#include "rc_host.h"

namespace rc {

struct RigidArgs {
    float4* pos;
    float4* vel;
    const float4* force;
    int4* image;            // NULL ok
    const int* rtag;
    const int* centre;      // [B] tag of each body's centre particle
    const int* first;       // [B + 1] member range of each body
    const int* member;      // [M] member tags
    const float* offset;    // [M][2] body-frame offsets
    const float* inertia;   // [B]
    float* theta;           // [B] angle in [-pi, pi)
    float* omega;           // [B] angular velocity
    int* status;            // NULL ok
    int B;
    Box box;
    float minv[RC_MAX_TYPES];
    float c2[RC_MAX_TYPES];
    float dt, c1, kT;
    int langevin;
    uint64_t seed, step;    // step: the one whose first half this launch does
    int second, firsth;     // halves done, in this order: the second one of a step, the first one of the next
    // runs only (NULL otherwise): the step a path length passed soft at, on the device and for the host
    int* stop;
    int* host;              // pinned: [0] as stop, [1] the last launch that began, [2] a non-finite path length
    int at;                 // the step (within the run) whose second half this launch does
    float soft;
};

// minimum image of a separation in the plane (FP32; members lie well within half a box of their centre)
__device__ __forceinline__ float mi(float d, float L, float h) {
    if (d >= h) d -= L;
    else if (d < -h) d += L;
    return d;
}

__device__ __forceinline__ float wrap_coord(float x, float L, float h, int& im) {
    if (x >= h) {
        x -= L;
        ++im;
    } else if (x < -h) {
        x += L;
        --im;
    }
    return x;
}

__device__ __forceinline__ void tell_host(int* p, int v) {
    __hip_atomic_store(p, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_SYSTEM);
}

// Path lengths past the rebuild threshold (NaN included) end the run before step `at`'s forces.
__device__ __forceinline__ void check_paths(bool past, bool bad, int* stop, int* host, int at) {
    const unsigned long long p = __ballot(past), q = __ballot(bad);
    if (p && (int)(threadIdx.x & (kWave - 1)) == __ffsll(p) - 1) {
        __hip_atomic_store(stop, at, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        if (q) tell_host(host + 2, 1);
        tell_host(host, at);
    }
}

// Four lanes per body: the launch is a chain of dependent reads (body, members,
// their indices, their data), so the members of a body are read side by side and
// the normals are drawn meanwhile; a thread per body read them one after the
// other and twice (7.4 us per launch for 1000 bodies; now
// 5.3, for both halves).  The second
// half of a step and the first one of the next need the same forces and share a
// launch.  The members' forces are added in member order.
constexpr int kBodyLanes = 4;

__global__ __launch_bounds__(kWave) void k_rigid(RigidArgs a) {
    if (a.stop) {
        if (blockIdx.x == 0 && threadIdx.x == 0) tell_host(a.host + 1, a.at);
        if (__hip_atomic_load(a.stop, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) <= a.at) return;
    }
    const int q = threadIdx.x % kBodyLanes;
    const int b = (blockIdx.x * kWave + threadIdx.x) / kBodyLanes;
    if (b >= a.B) return;   // a body's lanes leave together
    const Box& bx = a.box;
    const int ctag = a.centre[b];
    const int m0 = a.first[b], m1 = a.first[b + 1];
    const int c = a.rtag[ctag];
    // the lane's member of the first four
    const bool has0 = m0 + q < m1;
    int j0 = 0;
    float2 o0 = make_float2(0.f, 0.f);
    if (has0) {
        j0 = a.rtag[a.member[m0 + q]];
        o0 = make_float2(a.offset[2 * (m0 + q)], a.offset[2 * (m0 + q) + 1]);
    }
    const float4 pc = a.pos[c];
    const float4 vc = a.vel[c];
    float4 p0 = pc, f0 = make_float4(0.f, 0.f, 0.f, 0.f);
    float path0 = 0.0f;
    float fx = a.force[c].x, fy = a.force[c].y, tau = 0.0f;
    if (has0) {
        p0 = a.pos[j0];
        f0 = a.force[j0];
        path0 = a.vel[j0].w;
    }
    const float inv_i = 1.0f / a.inertia[b];
    float w = a.omega[b], th = a.theta[b];
    float z0 = 0.f, z1 = 0.f, z2 = 0.f;   // the centre's z normal drives the angle
    if (a.firsth && a.langevin) {
        thermostat_normals(a.seed, (uint32_t)ctag, a.step, z0, z1, z2);
        asm volatile("" : "+v"(z0), "+v"(z1), "+v"(z2));   // drawn here, while the reads are under way
    }
    const float minv = a.minv[ptype(pc.w)];
    // force and torque (about the centre) of the body
    for (int base = m0; base < m1; base += kBodyLanes) {
        float4 pm = p0, fm = f0;
        if (base > m0 && base + q < m1) {
            const int j = a.rtag[a.member[base + q]];
            pm = a.pos[j];
            fm = a.force[j];
        }
        const float dx = mi(pm.x - pc.x, bx.Lf[0], bx.hf[0]), dy = mi(pm.y - pc.y, bx.Lf[1], bx.hf[1]);
        const float t = __fmaf_rn(fm.y, dx, -__fmul_rn(fm.x, dy));
        for (int u = 0; u < kBodyLanes; ++u) {
            const float ux = __shfl(fm.x, u, kBodyLanes), uy = __shfl(fm.y, u, kBodyLanes);
            const float ut = __shfl(t, u, kBodyLanes);
            if (base + u < m1) {
                fx += ux;
                fy += uy;
                tau += ut;
            }
        }
    }
    const float hdt = 0.5f * a.dt;
    float vx = vc.x, vy = vc.y;
    // roundings written out from here on, so that the bits do not depend on which halves a launch holds
    if (a.second) {   // B of the step that ends
        vx = __fmaf_rn(hdt * fx, minv, vx);
        vy = __fmaf_rn(hdt * fy, minv, vy);
        w = __fmaf_rn(hdt * tau, inv_i, w);
    }
    float x = pc.x, y = pc.y, path = vc.w;
    if (a.firsth) {
        vx = __fmaf_rn(hdt * fx, minv, vx);  // B
        vy = __fmaf_rn(hdt * fy, minv, vy);
        w = __fmaf_rn(hdt * tau, inv_i, w);
        float sx = __fmul_rn(hdt, vx), sy = __fmul_rn(hdt, vy), st = __fmul_rn(hdt, w);  // A
        if (a.langevin) {                                   // O
            const float c2 = a.c2[ptype(pc.w)];
            vx = __fmaf_rn(a.c1, vx, __fmul_rn(c2, z0));
            vy = __fmaf_rn(a.c1, vy, __fmul_rn(c2, z1));
            const float cw = sqrtf(__fmul_rn(__fmul_rn(__fmaf_rn(-a.c1, a.c1, 1.0f), a.kT), inv_i));
            w = __fmaf_rn(a.c1, w, __fmul_rn(cw, z2));
        }
        sx = __fadd_rn(sx, __fmul_rn(hdt, vx));  // A
        sy = __fadd_rn(sy, __fmul_rn(hdt, vy));
        st = __fadd_rn(st, __fmul_rn(hdt, w));
        int ix = 0, iy = 0;
        x = wrap_coord(pc.x + sx, bx.Lf[0], bx.hf[0], ix);
        y = wrap_coord(pc.y + sy, bx.Lf[1], bx.hf[1], iy);
        path += sqrtf(__fmaf_rn(sy, sy, __fmul_rn(sx, sx)));
        th += st;
        const float pi = 3.14159265358979f;
        if (th >= pi) th -= 2.0f * pi;
        else if (th < -pi) th += 2.0f * pi;
        if (q == 0) {
            a.pos[c] = make_float4(x, y, pc.z, pc.w);
            if (a.image && (ix | iy)) {
                int4 im = a.image[c];
                im.x += ix;
                im.y += iy;
                a.image[c] = im;
            }
            a.theta[b] = th;
            const bool bad = !(isfinite(x) && isfinite(y) && isfinite(vx) && isfinite(vy) && isfinite(w));
            if (bad && a.status) atomicOr(&a.status[RC_ST_FLAGS], RC_FLAG_NONFINITE);
        }
    }
    if (q == 0) {
        a.vel[c] = make_float4(vx, vy, 0.0f, path);
        a.omega[b] = w;
    }
    bool past = !(path <= a.soft), nonf = !isfinite(path);
    // members: placed at the pose (first half), velocities v + w x d (both halves)
    float sn, cs;
    sincosf(th, &sn, &cs);
    for (int m = m0 + q; m < m1; m += kBodyLanes) {
        int j = j0;
        float ox = o0.x, oy = o0.y, pmw = path0;
        float4 pm = p0;
        if (m >= m0 + kBodyLanes) {
            j = a.rtag[a.member[m]];
            ox = a.offset[2 * m];
            oy = a.offset[2 * m + 1];
            pm = a.pos[j];
            pmw = a.vel[j].w;
        }
        const float dx = __fmaf_rn(cs, ox, -__fmul_rn(sn, oy)), dy = __fmaf_rn(sn, ox, __fmul_rn(cs, oy));
        if (a.firsth) {
            int ix = 0, iy = 0;
            const float xm = wrap_coord(x + dx, bx.Lf[0], bx.hf[0], ix);
            const float ym = wrap_coord(y + dy, bx.Lf[1], bx.hf[1], iy);
            const float ex = mi(xm - pm.x, bx.Lf[0], bx.hf[0]), ey = mi(ym - pm.y, bx.Lf[1], bx.hf[1]);
            pmw += sqrtf(__fmaf_rn(ex, ex, __fmul_rn(ey, ey)));
            a.pos[j] = make_float4(xm, ym, pm.z, pm.w);
            if (a.image) {  // a member's image follows its own crossings
                const int mx = (xm - pm.x > bx.hf[0]) ? -1 : ((xm - pm.x < -bx.hf[0]) ? 1 : 0);
                const int my = (ym - pm.y > bx.hf[1]) ? -1 : ((ym - pm.y < -bx.hf[1]) ? 1 : 0);
                if (mx | my) {
                    int4 im = a.image[j];
                    im.x += mx;
                    im.y += my;
                    a.image[j] = im;
                }
            }
        }
        a.vel[j] = make_float4(__fmaf_rn(-w, dy, vx), __fmaf_rn(w, dx, vy), 0.0f, pmw);
        past = past || !(pmw <= a.soft);
        nonf = nonf || !isfinite(pmw);
    }
    if (a.stop && a.firsth) check_paths(past, nonf, a.stop, a.host, a.at + 1);
}

// A run's start: no step stopped at, or step 0 where a path length is past the
// threshold already (want: the first step's first half came before this).
__global__ __launch_bounds__(kBlock) void k_rigid_paths(const float4* __restrict__ vel, int N, float soft, int* stop,
                                                        int* host) {
    const int i = blockIdx.x * blockDim.x + threadIdx.x;
    const float p = i < N ? vel[i].w : 0.0f;
    check_paths(!(p <= soft), !isfinite(p), stop, host, 0);
}

}  // namespace rc

using namespace rc;
using namespace rc::host;

namespace {

// the launch arguments of body steps, checked (halves, step and the run's words are the caller's)
int body_args(rc_ctx* c, float* pos, float* vel, const float* force, int* image, const int* rtag, int B,
              const int* centre, const int* first, const int* member, const float* offset, const float* inertia,
              float* theta, float* omega, int N, rc_box box, const rc_integrator* cfg, int* status, RigidArgs& a) {
    if (N < 1 || B < 1 || B > N) return fail(c, RC_ERR_ARG, "need 1 <= B <= N (B = %d, N = %d)", B, N);
    if (!pos || !vel || !force || !rtag || !centre || !first || !member || !offset || !inertia || !theta ||
        !omega)
        return fail(c, RC_ERR_ARG, "rigid bodies: a required array is NULL");
    if (!cfg || cfg->dim != 2) return fail(c, RC_ERR_ARG, "rigid planar bodies need an integrator of dim 2");
    int lang = 0;
    float nz = 0.0f;
    int r = check_integrator(c, cfg, a.minv, a.c2, a.c1, lang, nz);
    if (r) return r;
    if ((r = make_box(c, box, a.box))) return r;
    a.pos = reinterpret_cast<float4*>(pos);
    a.vel = reinterpret_cast<float4*>(vel);
    a.force = reinterpret_cast<const float4*>(force);
    a.image = reinterpret_cast<int4*>(image);
    a.rtag = rtag;
    a.centre = centre;
    a.first = first;
    a.member = member;
    a.offset = offset;
    a.inertia = inertia;
    a.theta = theta;
    a.omega = omega;
    a.status = status;
    a.B = B;
    a.dt = (float)cfg->dt;
    a.kT = (float)cfg->kT;
    a.langevin = lang;
    a.seed = cfg->seed;
    return RC_OK;
}

hipError_t launch_bodies(const RigidArgs& a, hipStream_t s) {
    hipLaunchKernelGGL(k_rigid, dim3(nblocks((long)a.B * kBodyLanes, kWave)), dim3(kWave), 0, s, a);
    return hipGetLastError();
}

}  // namespace

extern "C" int rc_rigid_step(rc_ctx* c, float* pos, float* vel, const float* force, int* image, const int* rtag,
                             int B, const int* centre, const int* first, const int* member, const float* offset,
                             const float* inertia, float* theta, float* omega, int N, rc_box box,
                             const rc_integrator* cfg, uint64_t step, int half, int* status, void* stream) {
    if (c) c->md.valid = false;   // the state changes outside the driver
    if (!c) return RC_ERR_ARG;
    if (half != RC_HALF_FIRST && half != RC_HALF_SECOND) return fail(c, RC_ERR_ARG, "half must be 0 or 1");
    RigidArgs a{};
    int r = body_args(c, pos, vel, force, image, rtag, B, centre, first, member, offset, inertia, theta, omega, N,
                      box, cfg, status, a);
    if (r) return r;
    a.step = step;
    a.firsth = half == RC_HALF_FIRST;
    a.second = half == RC_HALF_SECOND;
    HIP_TRY(c, launch_bodies(a, S(stream)));
    return RC_OK;
}

extern "C" int rc_rigid_run(rc_ctx* c, float* pos, float* vel, float* force, int* image, const int* rtag,
                            const int* nlist, const int* nn, int k_max, int B, const int* centre, const int* first,
                            const int* member, const float* offset, const float* inertia, float* theta, float* omega,
                            int N, rc_box box, const rc_integrator* cfg, uint64_t step0, int n_steps, int pending,
                            double soft, int* status, int* done, void* stream) {
    if (c) c->md.valid = false;   // the state changes outside the driver
    if (!c) return RC_ERR_ARG;
    if (n_steps < 1 || !done) return fail(c, RC_ERR_ARG, "rc_rigid_run: n_steps >= 1 and done not NULL");
    *done = 0;
    hipStream_t s = S(stream);
    RigidArgs a{};
    int r = body_args(c, pos, vel, force, image, rtag, B, centre, first, member, offset, inertia, theta, omega, N,
                      box, cfg, status, a);
    if (r) return r;
    if ((r = check_list(c, nlist, nn, k_max))) return r;
    if (reinterpret_cast<uintptr_t>(pos) & 15) return fail(c, RC_ERR_ARG, "positions not 16-byte aligned");
    // (every launch that writes the words has ended: a run waits for its own)
    if ((r = ensure_host_words(c)) || (r = wait_event(c, c->ev_sync))) return r;
    volatile int* host = c->h_status + kRigidWords;
    host[0] = n_steps;
    host[1] = -1;
    host[2] = 0;
    a.stop = reinterpret_cast<int*>(c->d_step_base + 1);
    a.host = c->h_status + kRigidWords;
    // p > soft in FP64 for an FP32 p: the largest FP32 value that is not above soft (never for NaN)
    a.soft = std::isnan(soft) ? INFINITY : (float)soft;
    if ((double)a.soft > soft) a.soft = std::nextafterf(a.soft, -INFINITY);
    HIP_TRY(c, launch_set_step(c->d_step_base + 1, (unsigned long long)n_steps, s));
    if (!pending) {
        RigidArgs f = a;
        f.firsth = 1;
        f.step = step0;
        f.stop = nullptr;   // the paths of every particle are looked at below
        HIP_TRY(c, launch_bodies(f, s));
        hipLaunchKernelGGL(k_rigid_paths, dim3(nblocks(N, kBlock)), dim3(kBlock), 0, s, a.vel, N, a.soft, a.stop, a.host);
        HIP_TRY(c, hipGetLastError());
    }
    // Steps are queued ahead of the device: once a path length passes soft, the body launches that
    // follow return at once (their forces, of the step that waits for its list, are evaluated anew
    // after the build).  At most kLead steps ahead, so that few are queued in vain; the queue stays full.
    constexpr int kLead = 4;
    for (int k = 0; k < n_steps && host[0] >= n_steps; ++k) {
        while (host[1] < k - kLead && host[0] >= n_steps) {
            const hipError_t e = hipStreamQuery(s);
            if (e == hipSuccess) break;
            if (e != hipErrorNotReady) return hip_fail(c, e, "waiting for the body steps");
        }
        r = rc_compute_forces(c, pos, nlist, nn, k_max, N, box, force, nullptr, RC_FORCE_GATHER, status, stream);
        if (!r && c->bonds) r = rc_fene_forces(c, pos, N, box, force, nullptr, stream);
        if (r) {
            (void)wait_spin(c, s);   // the words stay in use until the queued launches end
            return r;
        }
        RigidArgs f = a;
        f.second = 1;
        f.firsth = k + 1 < n_steps;
        f.step = step0 + (uint64_t)k + 1;
        f.at = k;
        HIP_TRY(c, launch_bodies(f, s));
    }
    if ((r = wait_spin(c, s))) return r;
    *done = host[0];
    if (host[2]) return fail(c, RC_ERR_NONFINITE, "non-finite path length");
    return RC_OK;
}
