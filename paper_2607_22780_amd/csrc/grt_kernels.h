// grt_kernels.h -- per-hit work shared by the trace and render kernels:
// front-to-back compositing (forward) and its gradient (backward).
#pragma once

#include "grt_internal.h"

namespace grt {

// A visitor takes a ray's hits in order, each in parts (Walker::composite):
//   item   what does not depend on the ray's other hits, by any lane: kIn
//          values for the ray's own lane, and an Item that the lane keeps;
//   step   the ray's own lane, in order: true when compositing stops after
//          the hit, and kOut values for the lane that has the Item;
//   emit   by that lane again, with those and the ray's kRay terms: what
//          remains (a gradient's chain rule), and kBack values that
//   collect, by the ray's lane, sums.
struct NoTables {};
struct VisitBase {
    static constexpr int kOut = 0, kRay = 0, kBack = 0;
    struct Item {};
    static __device__ __forceinline__ NoTables tables(int) { return {}; }
};

// Forward compositing (Sec. 3.2, Eq. trace; Eq. alpha_blending along the ray).
// Where to stop is decided on the transmittance of the canonical
// single-precision alphas (Td); the composited values use alphas from the
// double-precision crossing.  kHitList: the visitor also records the record
// positions of the composited hits in the ray's stored hit list (hl); the
// plain forward carries no list pointer at all.
template <bool kHitList>
struct CompositeVisit : VisitBase {
    static constexpr int kIn = 5;  // alpha, canonical alpha, colour
    float tcut;
    float3 C;
    float T, Td;
    int cnt;
    int32_t *did = nullptr;
    float *dtau = nullptr;
    int cap = 0;
    uint32_t *hl = nullptr;  // stored hit list of the ray (record positions)
    int hcap = 0;

    __device__ CompositeVisit() {}
    __device__ explicit CompositeVisit(float t_cut) : tcut(t_cut) {}

    __device__ __forceinline__ void reset()
    {
        C = make_float3(0.f, 0.f, 0.f);
        T = 1.0f;
        Td = 1.0f;
        cnt = 0;
    }

    static __device__ __forceinline__ void item(const SceneDev &S, NoTables, uint32_t p, const float4 r0,
                                                const float4 r1, const float4 r2, const float4 r3, float crho2,
                                                const float3 o, const float3 d, Item &, float (&in)[kIn])
    {
        const float4 c = S.col[p];
        HitGeo g;
        value_geo(r0, r1, r2, r3, o, d, g);
        in[0] = r1.w * expf(-0.5f * g.rho2);
        in[1] = hit_alpha(r1.w, crho2);
        in[2] = c.x; in[3] = c.y; in[4] = c.z;
    }

    __device__ __forceinline__ bool step(const float (&in)[kIn], uint32_t p, uint32_t id, float tau, float *)
    {
        const float a = in[0], w = T * a;
        C.x += w * in[2]; C.y += w * in[3]; C.z += w * in[4];
        if (did && cnt < cap) { did[cnt] = (int32_t)id; dtau[cnt] = tau; }
        if (kHitList && hl && cnt < hcap) hl[cnt] = p;
        ++cnt;
        T = T * (1.0f - a);
        Td = trans_step(Td, in[1]);
        return Td < tcut;
    }
};

__device__ __forceinline__ float dot3(float3 a, float3 b) { return a.x * b.x + a.y * b.y + a.z * b.z; }

// Attribute query of a ray (Eq. trace_attr, Gaussian backend): along the same
// ordered hits and cut-off as the radiance trace, the material attributes of
// the composited surfels summed with blending weights w = T alpha (Eq.
// deferred_maps), each normal turned to face the ray origin; the caller
// normalizes by the summed weight.  T ends as the visibility V of the
// environment.
//
// kPerRayArgs: the attribute tables belong to the lane's ray, so a helper
// takes them from the lane that it helps.
struct AttrTables {
    const float *albedo, *rough, *metal;  // per surfel id
};

template <class P>
__device__ __forceinline__ P *lane_pull_ptr(int address, P *x)
{
    const uint64_t v = (uint64_t)(uintptr_t)x;
    const uint32_t lo = (uint32_t)__builtin_amdgcn_ds_bpermute(address, (int)(uint32_t)v);
    const uint32_t hi = (uint32_t)__builtin_amdgcn_ds_bpermute(address, (int)(uint32_t)(v >> 32));
    return (P *)(uintptr_t)((uint64_t)hi << 32 | lo);
}

template <bool kPerRayArgs = false>
struct AttrVisitT : VisitBase {
    static constexpr int kIn = 10;  // alpha, canonical alpha, albedo, roughness, metallic, normal
    AttrTables t;
    float tcut;
    float T, Td, W, R, M;
    float3 A, N;

    __device__ AttrVisitT() {}
    __device__ AttrVisitT(float t_cut, const float *al, const float *ro, const float *me) : t{al, ro, me}, tcut(t_cut)
    {
    }

    __device__ __forceinline__ AttrTables tables(int from) const
    {
        if (!kPerRayArgs) return t;
        return {lane_pull_ptr(from, t.albedo), lane_pull_ptr(from, t.rough), lane_pull_ptr(from, t.metal)};
    }

    __device__ __forceinline__ void reset()
    {
        T = 1.0f;
        Td = 1.0f;
        W = 0.0f; R = 0.0f; M = 0.0f;
        A = make_float3(0.f, 0.f, 0.f);
        N = make_float3(0.f, 0.f, 0.f);
    }

    static __device__ __forceinline__ void item(const SceneDev &, const AttrTables &t, uint32_t, const float4 r0,
                                                const float4 r1, const float4 r2, const float4 r3, float crho2,
                                                const float3 o, const float3 d, Item &, float *in)
    {
        HitGeo g;
        value_geo(r0, r1, r2, r3, o, d, g);
        in[0] = r1.w * expf(-0.5f * g.rho2);
        in[1] = hit_alpha(r1.w, crho2);
        const bool away = g.den > 0.0f;  // normal toward the ray origin
        in[7] = away ? -r1.x : r1.x; in[8] = away ? -r1.y : r1.y; in[9] = away ? -r1.z : r1.z;
        // the record is done with before the attributes need registers
        __builtin_amdgcn_sched_barrier(0);
        const size_t i = __float_as_uint(r2.w);
        in[2] = t.albedo[3 * i]; in[3] = t.albedo[3 * i + 1]; in[4] = t.albedo[3 * i + 2];
        in[5] = t.rough[i];
        in[6] = t.metal[i];
    }

    __device__ __forceinline__ bool step(const float *in, uint32_t, uint32_t, float, float *)
    {
        const float a = in[0], w = T * a;
        W += w;
        A.x += w * in[2]; A.y += w * in[3]; A.z += w * in[4];
        R += w * in[5];
        M += w * in[6];
        N.x += w * in[7]; N.y += w * in[8]; N.z += w * in[9];
        T = T * (1.0f - a);
        Td = trans_step(Td, in[1]);
        return Td < tcut;
    }
};

using AttrVisit = AttrVisitT<>;

// Primary-ray G-buffer (Eq. deferred_maps on traced camera rays): the
// attribute sums plus the depth tau and the colour of each composited hit,
// with the same weights.
struct GBufVisit : AttrVisit {
    static constexpr int kIn = AttrVisit::kIn + 3;  // and the colour
    float Dsum;
    float3 Csum;

    __device__ GBufVisit() {}
    __device__ GBufVisit(float t_cut, const float *al, const float *ro, const float *me) : AttrVisit(t_cut, al, ro, me)
    {
    }

    __device__ __forceinline__ void reset()
    {
        AttrVisit::reset();
        Dsum = 0.0f;
        Csum = make_float3(0.f, 0.f, 0.f);
    }

    static __device__ __forceinline__ void item(const SceneDev &S, const AttrTables &t, uint32_t p, const float4 r0,
                                                const float4 r1, const float4 r2, const float4 r3, float crho2,
                                                const float3 o, const float3 d, Item &it, float *in)
    {
        const float4 c = S.col[p];
        AttrVisit::item(S, t, p, r0, r1, r2, r3, crho2, o, d, it, in);
        in[10] = c.x; in[11] = c.y; in[12] = c.z;
    }

    __device__ __forceinline__ bool step(const float *in, uint32_t p, uint32_t id, float tau, float *out)
    {
        const float w = T * in[0];
        Dsum += w * tau;
        Csum.x += w * in[10]; Csum.y += w * in[11]; Csum.z += w * in[12];
        return AttrVisit::step(in, p, id, tau, out);
    }
};

// Gradient terms reach global memory through per-wavefront LDS staging.
// Device FP32 atomics are limited by the cache lines they touch (one line per
// lane-atomic when lanes update unrelated surfels), not by the dwords: 16
// lanes adding to the 16 floats of one line cost what one lane does.  So each
// surfel owns a 16-float line of a scratch buffer (13 terms used), a hit's
// terms are staged in LDS where it is composited (any subset of lanes), and a
// flush has 16 lanes add one staged hit to its line in one instruction, four
// hits per instruction.  Flushes run at wavefront-uniform points; a step
// stages at most one hit per lane, so flushing whenever the list could not
// take another full step keeps it from overflowing.
constexpr int kStageStride = 16;  // 13 terms, then the surfel id (16-byte aligned entries)
template <int Cap>
struct WaveStageN {
    static constexpr int kCap = Cap;
    alignas(16) float v[Cap * kStageStride];
    int count;
};
// 80 entries of 64 bytes: with the backward's 16-deep stacks, 52 KB of LDS
// per workgroup, three workgroups per CU
using WaveStage = WaveStageN<80>;

// Active lanes: stage one hit each (13 terms of surfel id).
template <class Stage>
__device__ __forceinline__ void stage_add(Stage *s, uint32_t id, const float (&t)[13])
{
    const uint64_t m = __ballot(1);
    const int rank = (int)__builtin_amdgcn_mbcnt_hi((uint32_t)(m >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)m, 0u));
    volatile int *cnt = &s->count;
    const int base = __builtin_amdgcn_readfirstlane(*cnt);
    // four 16-byte stores per entry; stage_sync's fences order them
    float4 *e = reinterpret_cast<float4 *>(&s->v[(base + rank) * kStageStride]);
    e[0] = make_float4(t[0], t[1], t[2], t[3]);
    e[1] = make_float4(t[4], t[5], t[6], t[7]);
    e[2] = make_float4(t[8], t[9], t[10], t[11]);
    e[3] = make_float4(t[12], __uint_as_float(id), 0.0f, 0.0f);
    if (rank == 0) *cnt = base + __popcll(m);
}

// All 64 lanes of the wavefront: start with an empty list.
template <class Stage>
__device__ __forceinline__ void stage_init(Stage *s)
{
    if ((threadIdx.x & 63) == 0) *(volatile int *)&s->count = 0;
    __builtin_amdgcn_fence(__ATOMIC_SEQ_CST, "wavefront");
}

// All 64 lanes of the wavefront, at a wavefront-uniform point: add the staged
// hits to their surfels' lines once the list is past half full (all of it
// when `all`), then empty it.
template <class Stage>
__device__ __forceinline__ void stage_sync(float *acc, Stage *s, bool all)
{
    __builtin_amdgcn_fence(__ATOMIC_SEQ_CST, "wavefront");
    const int n = __builtin_amdgcn_readfirstlane(*(volatile int *)&s->count);
    if (n == 0 || (!all && n <= Stage::kCap - 64)) return;
    const int lane = threadIdx.x & 63, c = lane & 15;
    const volatile float *v = s->v;
    if (c < 13)
        for (int e = lane >> 4; e < n; e += 4) {
            const uint32_t id = reinterpret_cast<const volatile uint32_t *>(v)[e * kStageStride + 13];
            unsafeAtomicAdd(&acc[16 * (size_t)id + c], v[e * kStageStride + c]);
        }
    __builtin_amdgcn_fence(__ATOMIC_SEQ_CST, "wavefront");
    if (lane == 0) *(volatile int *)&s->count = 0;
    __builtin_amdgcn_fence(__ATOMIC_SEQ_CST, "wavefront");
}

// Backward of g_C . C + g_T . T_fin through every composited hit, with the
// hit set, order and stop index of the forward.
// Chain rule of one composited hit: from dL/dalpha (dA) -- and, for callers
// that also read the hit's depth tau and normal n, a direct dL/dtau (dtau)
// and dL/dn (dnx) -- to the surfel's stored parameters, out[0..9] = (mu xyz,
// s_u, s_v, q wxyz, opacity).  alpha = o G(u, v) at the tangent-plane
// crossing x = o + tau d, tau = n.(mu - o) / n.d, so tau moves with mu and n.
template <bool kDirect>
__device__ __forceinline__ void hit_param_grads(const HitGeo &hg, const float4 r1, const float4 r2, const float4 r3,
                                                float3 d, float a, float G, float dA, float dtau, float3 dnx,
                                                float4 q, float su, float sv, float out[10])
{
    const float3 n = make_float3(r1.x, r1.y, r1.z);
    const float den = hg.den;
    const float3 D = hg.D;
    const float3 au = make_float3(r2.x, r2.y, r2.z), av = make_float3(r3.x, r3.y, r3.z);
    const float u = hg.u, v = hg.v;
    const float gamma = -0.5f * a * dA;  // dL/d(rho^2)
    const float du = 2.0f * u * gamma, dv = 2.0f * v * gamma;
    // parameters of the surfel in its stored form (q, su, sv from the record order)
    const float ql = sqrtf(q.x * q.x + q.y * q.y + q.z * q.z + q.w * q.w);
    const float iq = 1.0f / ql;
    const float qw = q.x * iq, qx = q.y * iq, qy = q.z * iq, qz = q.w * iq;
    const float dsu = -(u / su) * du, dsv = -(v / sv) * dv;
    const float3 gD = make_float3(du * au.x + dv * av.x, du * au.y + dv * av.y, du * au.z + dv * av.z);
    const float gDd = kDirect ? (dot3(gD, d) + dtau) / den : dot3(gD, d) / den;
    const float3 dmu = make_float3(gDd * n.x - gD.x, gDd * n.y - gD.y, gDd * n.z - gD.z);
    const float ku = du / su, kv = dv / sv;
    const float3 dtu = make_float3(ku * D.x, ku * D.y, ku * D.z);
    const float3 dtv = make_float3(kv * D.x, kv * D.y, kv * D.z);
    float3 dn = make_float3(-gDd * D.x, -gDd * D.y, -gDd * D.z);
    if (kDirect) { dn.x += dnx.x; dn.y += dnx.y; dn.z += dnx.z; }
    // d(columns of R)/d(unit quaternion)
    float dqw = 2.f * (dtu.y * qz - dtu.z * qy - dtv.x * qz + dtv.z * qx + dn.x * qy - dn.y * qx);
    float dqx = 2.f * (dtu.y * qy + dtu.z * qz + dtv.x * qy - 2.f * dtv.y * qx + dtv.z * qw + dn.x * qz - dn.y * qw -
                       2.f * dn.z * qx);
    float dqy = 2.f * (-2.f * dtu.x * qy + dtu.y * qx - dtu.z * qw + dtv.x * qx + dtv.z * qz + dn.x * qw +
                       dn.y * qz - 2.f * dn.z * qy);
    float dqz = 2.f * (-2.f * dtu.x * qz + dtu.y * qw + dtu.z * qx - dtv.x * qw - 2.f * dtv.y * qz + dtv.z * qy +
                       dn.x * qx + dn.y * qy);
    const float proj = qw * dqw + qx * dqx + qy * dqy + qz * dqz;
    dqw = (dqw - qw * proj) * iq; dqx = (dqx - qx * proj) * iq;
    dqy = (dqy - qy * proj) * iq; dqz = (dqz - qz * proj) * iq;
    out[0] = dmu.x; out[1] = dmu.y; out[2] = dmu.z;
    out[3] = dsu; out[4] = dsv;
    out[5] = dqw; out[6] = dqx; out[7] = dqy; out[8] = dqz;
    out[9] = G * dA;
}

// kOrigin: also sum the hits' mean terms per ray.  Every hit's geometry is a
// function of mu - o, so the loss's gradient with respect to the ray origin
// is minus that sum (kept in `gmu`).
template <bool kOrigin = false>
struct GradVisitT : VisitBase {
    static constexpr int kIn = 5;                   // alpha, canonical alpha, colour
    static constexpr int kOut = 2;                  // w, dL/dalpha
    static constexpr int kRay = 3;                  // gC
    static constexpr int kBack = kOrigin ? 3 : 0;   // dL/dmu
    struct Item {
        HitGeo hg;
        float4 r1, r2, r3;
        float3 d;
        float a, G, sv;
        uint32_t p, id;
    };
    float tcut;
    WaveStage *stage = nullptr;  // the wavefront's staging list
    float3 gC;
    float3 R;     // colour still ahead: the saved c_rt minus the hits composited so far
    float gTf;    // dL/dT times the saved transmittance
    float T, Td;
    float3 gmu;

    __device__ GradVisitT() {}
    __device__ explicit GradVisitT(float t_cut) : tcut(t_cut) {}

    __device__ __forceinline__ void reset(float3 gC_, float gT_, float3 Cf_, float Tf_)
    {
        gC = gC_;
        R = Cf_;
        gTf = gT_ * Tf_;
        T = 1.0f;
        Td = 1.0f;
        gmu = make_float3(0.f, 0.f, 0.f);
    }

    static __device__ __forceinline__ void item(const SceneDev &S, NoTables, uint32_t p, const float4 r0,
                                                const float4 r1, const float4 r2, const float4 r3, float crho2,
                                                const float3 o, const float3 d, Item &it, float *in)
    {
        const float4 c = S.col[p];
        value_geo(r0, r1, r2, r3, o, d, it.hg);
        it.G = expf(-0.5f * it.hg.rho2);
        it.a = r1.w * it.G;
        it.r1 = r1; it.r2 = r2; it.r3 = r3;
        it.d = d;
        it.sv = c.w;
        it.p = p;
        it.id = __float_as_uint(r2.w);
        in[0] = it.a;
        in[1] = hit_alpha(r1.w, crho2);
        in[2] = c.x; in[3] = c.y; in[4] = c.z;
    }

    __device__ __forceinline__ bool step(const float *in, uint32_t, uint32_t, float, float *out)
    {
        const float a = in[0], w = T * a;
        R.x -= w * in[2]; R.y -= w * in[3]; R.z -= w * in[4];
        float dA = T * (gC.x * in[2] + gC.y * in[3] + gC.z * in[4]);
        const float om = 1.0f - a;
        if (om >= 1e-6f) {
            float behind = gC.x * R.x + gC.y * R.y + gC.z * R.z + gTf;
            dA -= behind / om;
        }
        out[0] = w;
        out[1] = dA;
        T = T * (1.0f - a);
        Td = trans_step(Td, in[1]);
        return Td < tcut;
    }

    __device__ __forceinline__ void ray_terms(float *ray) const { ray[0] = gC.x; ray[1] = gC.y; ray[2] = gC.z; }

    __device__ __forceinline__ void emit(const SceneDev &S, const Item &it, const float *out, const float *ray, float *ret)
    {
        const float w = out[0], dA = out[1];
        float terms[13];
        hit_param_grads<false>(it.hg, it.r1, it.r2, it.r3, it.d, it.a, it.G, dA, 0.0f, make_float3(0.f, 0.f, 0.f),
                               S.quat[it.p], it.r3.w, it.sv, terms);
        terms[10] = w * ray[0]; terms[11] = w * ray[1]; terms[12] = w * ray[2];
        stage_add(stage, it.id, terms);
        if constexpr (kOrigin) { ret[0] = terms[0]; ret[1] = terms[1]; ret[2] = terms[2]; }
    }

    __device__ __forceinline__ void collect(const float *x) { gmu.x += x[0]; gmu.y += x[1]; gmu.z += x[2]; }
};

using GradVisit = GradVisitT<false>;

// Backward of the primary-ray G-buffer (Eq. deferred_maps on traced camera
// rays).  Every map is a ratio S_f / W of blended sums S_f = sum_k w_k f_k,
// W = sum_k w_k, w_k = T_k alpha_k, and the normal map is N / |N| with
// N = sum_k w_k s_k n_k.  Holding the hits' values fixed, dL/dw_k is
//   e_k = sum_f g_f (f_k - F_f) / W + s_k n_k . (I - n n^T) g_n / |N|,
// and sum_k w_k e_k = 0 (every map is invariant to a common scale of the
// weights), so the part of the loss behind hit k is -(e_1 w_1 + ... + e_k w_k).
// The per-ray constants come from the forward's maps, W and |N| / W.
struct GBufGradVisit : VisitBase {
    // alpha, canonical alpha, albedo, roughness, metallic, normal toward the camera, colour
    static constexpr int kIn = 13;
    static constexpr int kOut = 2;   // w, dL/dalpha
    static constexpr int kRay = 12;  // kD, kR, kM, kA, kC, kN
    struct Item {
        HitGeo hg;
        float4 r1, r2, r3;
        float3 d;
        float a, G, sv;
        uint32_t p, id;
    };
    AttrTables t;
    float *ga_albedo, *ga_rough, *ga_metal;  // attribute gradients (NULL: skipped)
    float tcut;
    WaveStage *stage = nullptr;
    float kD, kR, kM, e0;  // upstream gradients over W, and sum_f g_f F_f / W
    float3 kA, kC, kN;
    float T, Td, P;

    __device__ GBufGradVisit() {}
    __device__ explicit GBufGradVisit(float t_cut) : tcut(t_cut) {}

    __device__ __forceinline__ AttrTables tables(int) const { return t; }

    __device__ __forceinline__ void reset()
    {
        T = 1.0f;
        Td = 1.0f;
        P = 0.0f;
    }

    static __device__ __forceinline__ void item(const SceneDev &S, const AttrTables &t, uint32_t p, const float4 r0,
                                                const float4 r1, const float4 r2, const float4 r3, float crho2,
                                                const float3 o, const float3 d, Item &it, float *in)
    {
        const float4 c = S.col[p];
        const size_t i = __float_as_uint(r2.w);
        in[2] = t.albedo[3 * i]; in[3] = t.albedo[3 * i + 1]; in[4] = t.albedo[3 * i + 2];
        in[5] = t.rough[i];
        in[6] = t.metal[i];
        value_geo(r0, r1, r2, r3, o, d, it.hg);
        it.G = expf(-0.5f * it.hg.rho2);
        it.a = r1.w * it.G;
        it.r1 = r1; it.r2 = r2; it.r3 = r3;
        it.d = d;
        it.sv = c.w;
        it.p = p;
        it.id = __float_as_uint(r2.w);
        in[0] = it.a;
        in[1] = hit_alpha(r1.w, crho2);
        const bool away = it.hg.den > 0.0f;  // normal toward the camera
        in[7] = away ? -r1.x : r1.x; in[8] = away ? -r1.y : r1.y; in[9] = away ? -r1.z : r1.z;
        in[10] = c.x; in[11] = c.y; in[12] = c.z;
    }

    __device__ __forceinline__ bool step(const float *in, uint32_t, uint32_t, float tau, float *out)
    {
        const float a = in[0], w = T * a;
        const float e = kD * tau + kA.x * in[2] + kA.y * in[3] + kA.z * in[4] + kR * in[5] + kM * in[6] +
                        kC.x * in[10] + kC.y * in[11] + kC.z * in[12] - e0 +
                        (in[7] * kN.x + in[8] * kN.y + in[9] * kN.z);
        P += w * e;
        float dA = T * e;
        const float om = 1.0f - a;
        if (om >= 1e-6f) dA += P / om;
        out[0] = w;
        out[1] = dA;
        T = T * (1.0f - a);
        Td = trans_step(Td, in[1]);
        return Td < tcut;
    }

    __device__ __forceinline__ void ray_terms(float *ray) const
    {
        ray[0] = kD; ray[1] = kR; ray[2] = kM;
        ray[3] = kA.x; ray[4] = kA.y; ray[5] = kA.z;
        ray[6] = kC.x; ray[7] = kC.y; ray[8] = kC.z;
        ray[9] = kN.x; ray[10] = kN.y; ray[11] = kN.z;
    }

    __device__ __forceinline__ void emit(const SceneDev &S, const Item &it, const float *out, const float *ray, float *)
    {
        const float w = out[0], dA = out[1], sw = it.hg.den > 0.0f ? -w : w;
        const size_t i = it.id;
        float terms[13];
        hit_param_grads<true>(it.hg, it.r1, it.r2, it.r3, it.d, it.a, it.G, dA, w * ray[0],
                              make_float3(sw * ray[9], sw * ray[10], sw * ray[11]), S.quat[it.p], it.r3.w, it.sv,
                              terms);
        terms[10] = w * ray[6]; terms[11] = w * ray[7]; terms[12] = w * ray[8];
        stage_add(stage, it.id, terms);
        if (ga_albedo) {
            atomicAdd(ga_albedo + 3 * i, w * ray[3]);
            atomicAdd(ga_albedo + 3 * i + 1, w * ray[4]);
            atomicAdd(ga_albedo + 3 * i + 2, w * ray[5]);
        }
        if (ga_rough) atomicAdd(ga_rough + i, w * ray[1]);
        if (ga_metal) atomicAdd(ga_metal + i, w * ray[2]);
    }
};

// Hand hit p of the lane's own ray to `visit`, all its parts: for callers that
// hold the record positions of a ray's hits.
template <class Visit>
__device__ __forceinline__ bool visit_hit(Visit &visit, const SceneDev &S, uint32_t p, float3 o, float3 d)
{
    const float4 *r = S.rec + 4 * (size_t)p;
    const float4 r0 = r[0], r1 = r[1], r2 = r[2], r3 = r[3];
    float den, tau, rho2;
    canon_geo(r0, r1, r2, r3, o, d, den, tau, rho2);
    typename Visit::Item item;
    float in[Visit::kIn], out[Visit::kOut], ray[Visit::kRay], ret[Visit::kBack + 1];
    Visit::item(S, visit.tables(0), p, r0, r1, r2, r3, rho2, o, d, item, in);
    const bool stop = visit.step(in, p, __float_as_uint(r2.w), tau, out);
    visit.ray_terms(ray);
    visit.emit(S, item, out, ray, ret);
    if constexpr (Visit::kBack > 0) visit.collect(ret);
    return stop;
}

}  // namespace grt
