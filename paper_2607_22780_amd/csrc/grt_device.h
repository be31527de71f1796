// grt_device.h -- device-side data layout and the shared traversal of libgrt.
//
// Scene layout in the caller's workspace (all in Morton order of the surfel
// bounding-box centres, so neighbouring surfels sit in neighbouring lines):
//   rec  [n][4] float4   r0 = (mu.xyz, r2max)      r1 = (n.xyz, opacity)
//                        r2 = (a_u.xyz, id bits)   r3 = (a_v.xyz, s_u)
//                        with a_u = t_u / s_u, a_v = t_v / s_v      (64 B)
//   col  [n]    float4   (rgb, s_v)                                  (16 B)
//   quat [n]    float4   the stored quaternion (w, x, y, z)          (16 B)
// The backward's chain rule reads the stored scales and quaternion of each
// composited hit from these, by record position, not from the caller's arrays
// by surfel id, which would cost a random line per hit.
//   node [n-1]  Node     both child boxes + child references        (64 B)
// A child reference >= 0 is an internal node, < 0 is leaf -(pos+1).
//   node4 [<= n-1] Node4 the same hierarchy collapsed to 4 children per
//                        node (boxes as structure of arrays, references as
//                        above, >= 0 now a 4-wide node)           (128 B)
//   nodeq [<= n-1] NodeQ the 4-wide nodes with their child boxes in 8 bits a
//                        plane, rounded outward                    (64 B)
// The traversal walks the NodeQ: half the node steps of the binary tree, each
// testing up to four boxes from one 64-byte line.
#pragma once

#include <type_traits>

#include <hip/hip_runtime.h>
#include <stdint.h>

#include "grt_nodeq.h"

namespace grt {

constexpr float kGrazing = 1e-6f; // |n . d| below this is no intersection
constexpr float kPad = 1e-5f;     // absolute padding of surfel boxes (scene units)

struct alignas(16) Node {
    float4 a;  // L.lo.x L.lo.y L.lo.z L.hi.x
    float4 b;  // L.hi.y L.hi.z R.lo.x R.lo.y
    float4 c;  // R.lo.z R.hi.x R.hi.y R.hi.z
    int4 d;    // left, right, leaves below (the collapse places its queue by them), unused
};

struct alignas(16) Node4 {
    float4 lx, ly, lz;  // lower corners of the four child boxes
    float4 hx, hy, hz;  // upper corners
    int4 ch;            // child references (kNoChild: unused slot)
    int4 pad;
};

struct SceneDev {
    const float4 *rec;
    const float4 *col;
    const Node *nodes;
    const float4 *quat;  // stored quaternions in record order
    const NodeQ *nodesq;
    int32_t n;
};

// Wavefronts per SIMD that a persistent kernel is held to (128 VGPRs at 4, 168
// at 3); the windows of the stacks take what LDS that leaves (20 entries at 4,
// 24 at 3).  At K = 16 a kernel held to 4 spills a few registers, which may cost
// less than the fourth wavefront gives.  Room of 1M surfels: the radiance
// forward (2 spilled) runs 512 x 512 x 32 rays in 33.4 ms at 4 and 37.3 at 3, the
// relighting query (8) 21.6 and 22.0; the attribute query (5) is the same at
// both; the plain trace (7) is the faster at 3.  Kernels that carry more per
// lane keep 3: primary-ray maps 11.0 against 11.6 ms at 4 (200k surfels, forward
// and backward), a server epoch of several requests 39.3 against 42.0 (both with
// hits still composited a lane at a time), and the backwards, whose LDS also
// holds gradient lines.
constexpr int kWindow4 = 20, kWindow3 = 24;
constexpr int waves_for(int k, int waves) { return k <= 16 ? waves : 1; }
#define GRT_WAVES(K, W) __attribute__((amdgpu_waves_per_eu(waves_for(K, W))))

// ---------------------------------------------------------------------------
// Canonical single-precision arithmetic of the hit decision.  The operation
// order is fixed and contraction is off, so the decision, the depth and the
// (depth, id) order are reproducible bit for bit by any IEEE implementation
// of the same sequence.
// ---------------------------------------------------------------------------

// Frame of a surfel: t_u, t_v, n are the columns of R(q/|q|) (Hamilton, w first).
__device__ __forceinline__ void frame32(float w, float x, float y, float z, float3 &tu, float3 &tv, float3 &n)
{
#pragma clang fp contract(off)
    float l = sqrtf(w * w + x * x + y * y + z * z);
    w = w / l; x = x / l; y = y / l; z = z / l;
    float xx = x * x, yy = y * y, zz = z * z;
    float xy = x * y, xz = x * z, yz = y * z;
    float wx = w * x, wy = w * y, wz = w * z;
    tu = make_float3(1.0f - 2.0f * (yy + zz), 2.0f * (xy + wz), 2.0f * (xz - wy));
    tv = make_float3(2.0f * (xy - wz), 1.0f - 2.0f * (xx + zz), 2.0f * (yz + wx));
    n = make_float3(2.0f * (xz + wy), 2.0f * (yz - wx), 1.0f - 2.0f * (xx + yy));
}

// Canonical crossing: m = mu - o, den = n.d, tau = n.m / den, D = tau d - m,
// u = a_u.D, v = a_v.D, rho^2 = u^2 + v^2 (fixed order, no contraction).
__device__ __forceinline__ void canon_geo(const float4 r0, const float4 r1, const float4 r2, const float4 r3,
                                          const float3 o, const float3 d, float &den, float &tau, float &rho2)
{
#pragma clang fp contract(off)
    float m0 = r0.x - o.x, m1 = r0.y - o.y, m2 = r0.z - o.z;
    den = r1.x * d.x + r1.y * d.y + r1.z * d.z;
    float num = r1.x * m0 + r1.y * m1 + r1.z * m2;
    tau = num / den;
    float dx = tau * d.x - m0, dy = tau * d.y - m1, dz = tau * d.z - m2;
    float u = r2.x * dx + r2.y * dy + r2.z * dz;
    float v = r3.x * dx + r3.y * dy + r3.z * dz;
    rho2 = u * u + v * v;
}

// Value geometry of a hit: the same crossing evaluated in double from the
// single-precision record (the in-plane offset D = tau d - m cancels badly in
// single precision for small surfels seen from afar).
struct HitGeo {
    float u, v, rho2, den;
    float3 D;
};

__device__ __forceinline__ void value_geo(const float4 r0, const float4 r1, const float4 r2, const float4 r3,
                                          const float3 o, const float3 d, HitGeo &g)
{
    // with num = n.m and den = n.d:  den * u = num (a_u.d) - den (a_u.m), the
    // cancelling terms taken in double; one single-precision reciprocal
    const double mx = (double)r0.x - (double)o.x, my = (double)r0.y - (double)o.y, mz = (double)r0.z - (double)o.z;
    const double dx = d.x, dy = d.y, dz = d.z;
    const double nx = r1.x, ny = r1.y, nz = r1.z;
    const double den = nx * dx + ny * dy + nz * dz;
    const double num = nx * mx + ny * my + nz * mz;
    const double U = num * ((double)r2.x * dx + (double)r2.y * dy + (double)r2.z * dz) -
                     den * ((double)r2.x * mx + (double)r2.y * my + (double)r2.z * mz);
    const double V = num * ((double)r3.x * dx + (double)r3.y * dy + (double)r3.z * dz) -
                     den * ((double)r3.x * mx + (double)r3.y * my + (double)r3.z * mz);
    const float fden = (float)den;
    const float rden = 1.0f / fden;
    g.u = (float)U * rden;
    g.v = (float)V * rden;
    g.rho2 = g.u * g.u + g.v * g.v;
    g.den = fden;
    g.D = make_float3((float)(num * dx - den * mx) * rden, (float)(num * dy - den * my) * rden,
                      (float)(num * dz - den * mz) * rden);
}

// Opacity contribution of a hit, alpha = o exp(-rho^2 / 2), and the
// single-precision transmittance step that decides where compositing stops.
__device__ __forceinline__ float hit_alpha(float op, float rho2)
{
#pragma clang fp contract(off)
    return op * expf(-0.5f * rho2);
}

__device__ __forceinline__ float trans_step(float T, float a)
{
#pragma clang fp contract(off)
    return T * (1.0f - a);
}

// order-preserving float <-> int maps (atomic min/max of floats)
__device__ __forceinline__ int f2o(float f)
{
    int i = __float_as_int(f);
    return i >= 0 ? i : i ^ 0x7fffffff;
}
__device__ __forceinline__ float o2f(int i) { return __int_as_float(i >= 0 ? i : i ^ 0x7fffffff); }

// One exchange of a sorting network: (sa, ca) takes the nearer of two children.
__device__ __forceinline__ void exchange(float &sa, int &ca, float &sb, int &cb)
{
    const bool sw = sb < sa;
    const float ts = sw ? sb : sa;
    const int tc = sw ? cb : ca;
    sb = sw ? sa : sb;
    cb = sw ? ca : cb;
    sa = ts;
    ca = tc;
}

// The sort key of a hit, (bits(tau), id), held as the double with those bits:
// a non-negative depth's bits order as its value does, tau is finite, so the
// key is a finite non-negative double, and doubles of one sign order as their
// bits do.  v_min_f64 / v_max_f64 then order keys at one instruction each.
__device__ __forceinline__ double make_key(float tau, uint32_t id)
{
    return __hiloint2double(__float_as_int(tau), (int)id);
}
__device__ __forceinline__ float key_tau(double k) { return __int_as_float(__double2hiint(k)); }

// An empty slot of the k-buffer: +infinity, above every key; its depth word
// reads as a quiet NaN, which fminf passes over.
__device__ __forceinline__ double empty_key() { return __hiloint2double(0x7ff00000, 0); }

__device__ __forceinline__ bool is_empty(double k) { return __double2hiint(k) == 0x7ff00000; }

// min / max of keys (never NaN), as the bare instructions: fmin and fmax put a
// canonicalizing instruction before each operand.
__device__ __forceinline__ double key_min(double a, double b)
{
    double r;
    asm("v_min_f64 %0, %1, %2" : "=v"(r) : "v"(a), "v"(b));
    return r;
}
__device__ __forceinline__ double key_max(double a, double b)
{
    double r;
    asm("v_max_f64 %0, %1, %2" : "=v"(r) : "v"(a), "v"(b));
    return r;
}

// ---------------------------------------------------------------------------
// Ordered traversal with a k-nearest hit buffer, in rounds that resume from a
// deferred frontier, as a per-lane state machine.
//
// A round walks the BVH keeping the K smallest keys (bits(tau), id) strictly
// greater than the last key composited in the previous round (registers,
// sorted by unrolled insertion).  Once the buffer is full its largest depth
// thi bounds the walk.  Everything the bound excludes is not dropped but
// deferred to the next round: subtrees whose box is entered beyond thi, hits
// rejected by the full buffer and hits evicted from it.  The buffered hits
// are then handed to `visit` (record position, surfel id, depth) in order;
// `visit` returns true to stop (transmittance cutoff).  The next round starts
// from the deferred items instead of the root, so a ray's hits cost about one
// walk whatever K is; a round that defers nothing ends the ray.  Keys are
// unique, so hits of equal depth are neither lost nor repeated, and results
// do not depend on K.
//
// If the deferred list grows too long it is dropped and the next round
// restarts from the root, which re-finds every hit beyond the last composited
// key.
//
// What bounds the walk is VALU issue: lanes of a wavefront take the node step
// and the leaf test in turns (29 of 64 lanes active per VALU instruction), at
// 75% of the issue peak.  So each of these blocks is kept short: pushes
// without branches into ring windows, one merged push for kept and deferred
// children, keys moved by min and max.  Node step 430 to 230 VALU
// instructions, insertion at K = 16 121 to 81; room of 1M surfels: forward
// K = 16 (512 x 512, 32 spp) 53.0 to 43.7 ms, backward K = 13 (1024 x 1024,
// 16 spp) 122.8 to 115.5 ms, relighting K = 12 31.9 to 28.1 ms.
//
// advance() does one node or one leaf and composite() a few hits, so a wavefront
// can hold rays at different rounds and refill lanes whose ray has finished (run_persistent).
// ---------------------------------------------------------------------------
// ---------------------------------------------------------------------------
// A lane's two stacks (walk and deferred): the newest entries of each are a
// window in LDS, a ring of D slots (lane-interleaved, so a wavefront's
// accesses are conflict-free); older ones lie in a private array.  Room is
// made once per walking step (the oldest entries of a window that the step
// could fill move out, and some come back when a pop finds its window empty),
// so pushing is one LDS store and a wrapped increment, without branches.
// ---------------------------------------------------------------------------
constexpr int kBwdLdsDepth = 16;  // backward kernels: their LDS also holds gradient tables
// Surfel steps run when at least kSurfelShare8 / 8 of a wavefront's walking
// lanes wait for one, and buffered hits are composited once kCompShare16 / 16
// of the lanes with a ray have a round's buffer to composite: shares, so that
// the last rays of a launch wait for few others (with 8 lanes as the rule,
// primary-ray maps took 10.6 ms, with 3 / 16 9.2).  Training step of 16.8M
// rays, 1M surfels: 1 / 16 154 ms, 2 142, 3 139, 4 142, 5 151; surfel shares
// 2 / 8 to 5 / 8 lie within 1%, but 50k surfels' forward and backward within
// 8% (3 / 8: 1.80 ms, 5 / 8: 1.96).
constexpr int kSurfelShare8 = 3, kCompShare16 = 3;
constexpr int kStackCap = 384;  // private entries of a stack
constexpr int kNone = 0x7fffffff;

// The roles of the two stacks swap each round (the deferred list becomes the
// next round's walk stack).  A round's stack starts with at most kMaxDeferred
// items; below them, a node step pops one item and pushes at most three, so
// the stack holds at most three siblings for each 4-wide level of the current
// path.  The 4-wide tree is no deeper than the binary one (each of its edges
// spans at least one binary edge), whose build keeps it within 63 levels, so
// the stack stays within kMaxDeferred + 3 * 63 <= kStackCap.
constexpr int kMaxDeferred = 192;
static_assert(kMaxDeferred + 3 * 63 <= kStackCap, "walk stack bound");

typedef __attribute__((address_space(3))) int LdsInt;
__device__ __forceinline__ uint32_t lds_addr(const int *p) { return (uint32_t)(uintptr_t)(LdsInt *)p; }
__device__ __forceinline__ int lds_load(uint32_t a) { return *(const LdsInt *)(uintptr_t)a; }
__device__ __forceinline__ void lds_store(uint32_t a, int x) { *(LdsInt *)(uintptr_t)a = x; }

// What the lanes of a wavefront wrote, before others of them read it (all
// lanes, wavefront-uniform point).  The barrier emits nothing: a fence alone
// orders the accesses of one path, but the compiler may copy it into both arms
// of a branch on the lane and run the readers' arm first.
__device__ __forceinline__ void wave_sync(bool global = false)
{
    if (global) __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup");
    else __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    if (global) __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "workgroup");
    else __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

// x of the lane at byte address 4 * lane (all lanes).
__device__ __forceinline__ float lane_pull(int address, float x)
{
    return __int_as_float(__builtin_amdgcn_ds_bpermute(address, __float_as_int(x)));
}

template <int D>
struct Frontier {
    static constexpr uint32_t kStride = 256;            // a slot of the wavefront: 64 lanes x 4 bytes
    static constexpr uint32_t kWindow = D * kStride;
    // Entries moved between a window and the private array at a time.  It
    // divides D, and a window's oldest entry always sits at a multiple of it,
    // so the entries of a move are consecutive slots (immediate offsets).
    static constexpr int kSpill = D % 8 == 0 ? 8 : 4;
    // Pushes between two calls of make_room, at most: 3 on the walk stack, 4 on
    // the deferred list.  A node step defers up to 4 children, and the leaf
    // test one hit more; but a node that yields a leaf has kept its nearest
    // child (walk_node), so it defers 3 before that test.  One slot of the
    // deferred window stays free beyond them, since push stores to it always.
    static constexpr int kWalkPush = 3, kDeferPush = 4;
    static constexpr int kWalkFull = D - kWalkPush, kDeferFull = D - kDeferPush - 1;  // most entries to leave
    static_assert(D % kSpill == 0 && kSpill >= kWalkPush && kSpill >= kDeferPush,
                  "a move out of a window makes the room of a step");
    static_assert(kDeferFull >= 0 && kSpill + kWalkPush <= D, "a refilled window takes a step");
    uint32_t base;        // LDS address of this lane's slot 0 of window 0; window 1 follows
    uint32_t woff;        // the window that holds the walk: 0 or kWindow (the other one defers)
    uint32_t wtop, dtop;  // LDS address of the next free slot of the walk / deferred window
    int wn, dn;           // entries in the windows
    int wold, dold;       // entries in the private arrays, below the windows'
    int *mem;             // [2][kStackCap] private arrays

    __device__ __forceinline__ uint32_t wlo() const { return base + woff; }
    __device__ __forceinline__ uint32_t dlo() const { return base + (kWindow - woff); }
    __device__ __forceinline__ int *mem_of(uint32_t off) const { return mem + (off ? kStackCap : 0); }
    static __device__ __forceinline__ uint32_t next(uint32_t a, uint32_t lo)
    {
        a += kStride;
        return a == lo + kWindow ? lo : a;
    }

    __device__ __forceinline__ void clear_def()
    {
        dtop = dlo();
        dn = 0;
        dold = 0;
    }
    __device__ __forceinline__ void reset()
    {
        wtop = wlo();
        wn = 0;
        wold = 0;
        clear_def();
    }

    static __device__ __forceinline__ void spill(uint32_t top, uint32_t lo, int &n, int &old, int *m)
    {
        uint32_t b = top - kStride * (uint32_t)n;  // the oldest entry of the window
        b = (int)(b - lo) < 0 ? b + kWindow : b;
#pragma unroll
        for (int j = 0; j < kSpill; ++j) m[old + j] = lds_load(b + kStride * j);
        n -= kSpill;
        old += kSpill;
    }

    // Before a walking step and the leaf test after it.  A deferred list too
    // long is dropped (lost); while it is, what is pushed on it goes the same
    // way.
    __device__ __forceinline__ void make_room(bool &lost)
    {
        if (wn <= kWalkFull && dn <= kDeferFull) return;
        if (wn > kWalkFull) spill(wtop, wlo(), wn, wold, mem_of(woff));
        if (dn > kDeferFull) {
            if (lost || dold + kSpill > kMaxDeferred - D) {
                lost = true;
                clear_def();
            } else {
                spill(dtop, dlo(), dn, dold, mem_of(kWindow - woff));
            }
        }
    }

    __device__ __forceinline__ bool walk_empty() const { return (wn | wold) == 0; }

    // the walk stack is not empty
    __device__ __forceinline__ int pop_walk()
    {
        const uint32_t lo = wlo();
        if (wn == 0) {
            const int *m = mem_of(woff) + (wold - kSpill);
#pragma unroll
            for (int j = 0; j < kSpill; ++j) lds_store(lo + kStride * j, m[j]);
            wtop = lo + kStride * kSpill;
            wn = kSpill;
            wold -= kSpill;
        }
        wtop = (wtop == lo ? lo + kWindow : wtop) - kStride;
        --wn;
        return lds_load(wtop);
    }

    __device__ __forceinline__ void push_def(int x)
    {
        lds_store(dtop, x);
        dtop = next(dtop, dlo());
        ++dn;
    }

    // x goes on the walk stack (w), on the deferred list (d) or nowhere; the
    // store is unconditional, since the slot it hits is free
    __device__ __forceinline__ void push(int x, bool w, bool d)
    {
        const uint32_t a = w ? wtop : dtop;
        lds_store(a, x);
        const uint32_t n = next(a, w ? wlo() : dlo());
        wtop = w ? n : wtop;
        dtop = d ? n : dtop;
        wn += (int)w;
        dn += (int)d;
    }

    // the deferred list becomes the walk stack, which is empty
    __device__ __forceinline__ void swap_roles()
    {
        wtop = dtop;
        wn = dn;
        wold = dold;
        woff = kWindow - woff;
        clear_def();
    }
};

template <int K, int D = kWindow4>
struct Walker {
    static constexpr int kDepth = D;  // LDS entries per lane and stack
    float3 o, d;
    float tmin, tmax;
    double last;          // start key of the round; while compositing, the last composited hit
    double key[K];
    uint32_t pos[K];
    int cur;              // item in hand: node >= 0, leaf -(pos+1), or kNone
    bool lost;            // deferred list dropped: next round restarts at the root
    Frontier<D> F;        // walk stack and deferred list (LDS + private spill)
    int st;               // kNone: walking; >= 0: record of a leaf that waits for the next surfel
                          // step; kMore, kFinal: compositing a full buffer, the last one
    static constexpr int kMore = -1, kFinal = -2;
#ifdef GRT_STATS
    int st_nodes, st_leaves, st_comps, st_rounds, st_lost, st_deferred;
#endif

    __device__ __forceinline__ void clear_buffer()
    {
#pragma unroll
        for (int i = 0; i < K; ++i) { key[i] = empty_key(); pos[i] = 0; }
    }

    // The round's walk covers [lo_bound, hi_bound]: from the last composited
    // key's depth (tmin in the first round) to the full buffer's largest
    // depth (tmax while it is not full: the empty key's depth word is a NaN).
    // Derived when needed rather than held, to keep two registers free.
    __device__ __forceinline__ float lo_bound() const { return fmaxf(tmin, key_tau(last)); }
    __device__ __forceinline__ float hi_bound() const { return fminf(tmax, key_tau(key[K - 1])); }

    // (tmin and tmax are the caller's to set: a job whose rays share them sets
    // them once, which keeps them out of the lanes' registers)
    __device__ __forceinline__ void start(const SceneDev &S, float3 o_, float3 d_)
    {
        o = o_;
        d = d_;
        last = 0.0;
        st = kNone;
        F.reset();
        lost = false;
        cur = S.n > 1 ? 0 : S.n == 1 ? -1 : kNone;  // no surfels: the first step ends the ray
        clear_buffer();
#ifdef GRT_STATS
        st_nodes = st_leaves = st_comps = st_lost = st_deferred = 0;
        st_rounds = 1;
#endif
    }

    // Leaf test from the canonical crossing of surfel record p (den, tau,
    // rho^2 as canon_geo computes them; r0.w is the bound r2max, r2.w the id):
    // a hit goes into the k-buffer, or is deferred when beyond it.
    __device__ __forceinline__ void test_leaf(uint32_t p, float den, float tau, float rho2, float r2max, float idbits)
    {
#ifdef GRT_STATS
        ++st_leaves;
#endif
        if (fabsf(den) < kGrazing || !(tau > tmin && tau <= tmax) || !(rho2 <= r2max)) return;
        const double k = make_key(tau, __float_as_uint(idbits));
        if (k <= last) return;
        // beyond a full buffer, or the largest key drops out of it: to the next round
        const bool beyond = k >= key[K - 1];
        if (!is_empty(key[K - 1])) {
            F.push_def(-(int)(beyond ? p : pos[K - 1]) - 1);
#ifdef GRT_STATS
            if (!lost) ++st_deferred;
#endif
        }
        if (beyond) return;
        // Sorted insertion: slot i takes the middle of (slot i - 1, k, itself),
        // which for keys is a min and a max, and for positions two selects.
        bool above = key[K - 1] > k;
#pragma unroll
        for (int i = K - 1; i > 0; --i) {
            const bool below = key[i - 1] > k;  // slot i - 1 moves up
            pos[i] = above ? (below ? pos[i - 1] : p) : pos[i];
            key[i] = key_max(key[i - 1], key_min(key[i], k));
            above = below;
        }
        pos[0] = above ? p : pos[0];
        key[0] = key_min(key[0], k);
    }

    // Test the children of 4-wide node `cur`; sets the next item and at most
    // one leaf to test.  The children met in [tlo, tmax] are sorted by entry
    // depth; those entered beyond thi (the full buffer's largest depth) are
    // deferred to the next round.  Of the others the nearest becomes the item
    // in hand, except that a leaf among the first two goes to the single
    // surfel site in advance() (a wavefront then runs it once per step however
    // its lanes' children are mixed); the rest go on the walk stack, farthest
    // first.  All of it is selects: with branches per child, lanes that defer,
    // push and skip took turns.
    __device__ __forceinline__ void walk_node(const SceneDev &S, int &leaf)
    {
#ifdef GRT_STATS
        ++st_nodes;
#endif
        const float4 *nd = reinterpret_cast<const float4 *>(S.nodesq + cur);
        const float4 w0 = nd[0], w1 = nd[1], w2 = nd[2];
        const int4 ch = *reinterpret_cast<const int4 *>(nd + 3);
        const float tlo = lo_bound();
        const float thi = fminf(hi_bound() * 1.0000005f, 3.402823466e+38f);
        const float tend = fminf(tmax * 1.0000005f + 1e-30f, 3.402823466e+38f);
        const float3 inv = make_float3(fast_inv(d.x), fast_inv(d.y), fast_inv(d.z));
        const float3 start = make_float3((w0.x - o.x) * inv.x, (w0.y - o.y) * inv.y, (w0.z - o.z) * inv.z);
        const float3 step = make_float3(w0.w * inv.x, w1.x * inv.y, w1.y * inv.z);
        const uint32_t lx = __float_as_uint(w1.z), ly = __float_as_uint(w1.w), lz = __float_as_uint(w2.x);
        const uint32_t hx = __float_as_uint(w2.y), hy = __float_as_uint(w2.z), hz = __float_as_uint(w2.w);
        const bool gx = __float_as_int(d.x) < 0, gy = __float_as_int(d.y) < 0, gz = __float_as_int(d.z) < 0;
        const uint32_t nx = gx ? hx : lx, fx = gx ? lx : hx;
        const uint32_t ny = gy ? hy : ly, fy = gy ? ly : hy;
        const uint32_t nz = gz ? hz : lz, fz = gz ? lz : hz;
        // an unused slot is masked by its reference
        float t0, t1, t2, t3;
        const bool k0 = slab_q<0>(nx, ny, nz, fx, fy, fz, step, start, tlo, t0) & (ch.x != kNoChild);
        const bool k1 = slab_q<1>(nx, ny, nz, fx, fy, fz, step, start, tlo, t1) & (ch.y != kNoChild);
        const bool k2 = slab_q<2>(nx, ny, nz, fx, fy, fz, step, start, tlo, t2) & (ch.z != kNoChild);
        const bool k3 = slab_q<3>(nx, ny, nz, fx, fy, fz, step, start, tlo, t3) & (ch.w != kNoChild);
        // by entry depth, missed children last (a five-exchange sorting network)
        float s0 = k0 ? t0 : INFINITY, s1 = k1 ? t1 : INFINITY, s2 = k2 ? t2 : INFINITY, s3 = k3 ? t3 : INFINITY;
        int c0 = ch.x, c1 = ch.y, c2 = ch.z, c3 = ch.w;
        exchange(s0, c0, s1, c1);
        exchange(s2, c2, s3, c3);
        exchange(s0, c0, s2, c2);
        exchange(s1, c1, s3, c3);
        exchange(s1, c1, s2, c2);
        const bool n0 = s0 <= thi, n1 = s1 <= thi, n2 = s2 <= thi, n3 = s3 <= thi;  // kept in this round
        const bool h0 = s0 <= tend, h1 = s1 <= tend, h2 = s2 <= tend, h3 = s3 <= tend;         // met by the ray
#ifdef GRT_STATS
        if (!lost) st_deferred += (int)(h0 & !n0) + (int)(h1 & !n1) + (int)(h2 & !n2) + (int)(h3 & !n3);
#endif
        const bool f0 = n0 & (c0 < 0), f1 = n1 & !f0 & (c1 < 0);
        F.push(c3, n3, h3 & !n3);
        F.push(c2, n2, h2 & !n2);
        F.push(c1, n1 & !f0 & !f1, h1 & !n1);
        F.push(c0, false, h0 & !n0);
        leaf = f0 ? c0 : f1 ? c1 : kNone;
        cur = f0 ? (n1 ? c1 : kNone) : n0 ? c0 : kNone;
    }

    // Set up the next round from the deferred frontier (or the root).  A next
    // round follows only a full buffer whose K hits were all composited, so
    // `last` already holds the round's largest key, where the next one starts.
    __device__ __forceinline__ void next_round(const SceneDev &S)
    {
        // The buffer is empty already (every composite shifted an empty key in
        // at its end, and the round composited all its hits): rewriting the
        // keys would give the registers a second version to reconcile at
        // every exit of the surfel step.
#ifdef GRT_STATS
        ++st_rounds;
        st_lost += lost ? 1 : 0;
#endif
        if (lost) {
            F.clear_def();
            lost = false;
            cur = S.n == 1 ? -1 : 0;
        } else {
            F.swap_roles();
            cur = kNone;
        }
    }

    // Depth of the last composited hit once the ray is finished (0 when none
    // was): a re-traversal bounded there meets the same composited hits.
    __device__ __forceinline__ float stop_depth() const { return key_tau(last); }

    __device__ __forceinline__ bool deferred_empty() const
    {
        return !lost && (F.dn | F.dold) == 0;
    }

    // A step of a walking lane (st >= 0): a node or a leaf of the walk.  A
    // leaf that a node step finds waits (st) for a surfel step: the record,
    // its canonical crossing and the k-buffer insertion run for the wavefront
    // at once, when enough of its walking lanes wait for it, so that block
    // runs with many lanes (leaf tests postponed as in speculative while-while
    // traversal).  A lane whose round's walk is complete then waits for
    // composite() (st < 0).  Returns true when the ray is finished.  Every
    // walking lane of the wavefront calls it in the same step (the decision
    // is a ballot over them).
    __device__ __forceinline__ bool advance(const SceneDev &S)
    {
        if (st == kNone) {
            F.make_room(lost);
            if (cur == kNone && F.walk_empty()) {  // the round's walk is complete
                if (is_empty(key[0])) return true;
                st = is_empty(key[K - 1]) ? kFinal : kMore;
            } else {
                if (cur == kNone) cur = F.pop_walk();
                int leaf = cur;
                if (cur < 0) cur = kNone;
                else walk_node(S, leaf);
                st = leaf != kNone ? -leaf - 1 : kNone;
            }
        }
        const bool want = st >= 0 && st != kNone;
        const int nwant = __popcll(__ballot(want)), nwalk = __popcll(__ballot(st == kNone));
        if (!want || 8 * nwant < kSurfelShare8 * (nwant + nwalk)) return false;
        const float4 *r = S.rec + 4 * (size_t)(uint32_t)st;
        const float4 r0 = r[0], r1 = r[1], r2 = r[2], r3 = r[3];
        float den, tau, rho2;
        canon_geo(r0, r1, r2, r3, o, d, den, tau, rho2);
        test_leaf((uint32_t)st, den, tau, rho2, r0.w, r2.w);
        st = kNone;
        return false;
    }

    // Composite the next hits of lanes whose buffers wait (lanes of `comps`),
    // at a wavefront-uniform point, all lanes.
    //
    // A hit's share of the work that does not depend on the hits before it --
    // record, crossing, value geometry in double, alpha, and the gradient's
    // chain rule behind the running sums -- is done by a helper lane,
    // whichever ray the helper holds itself; the compositing lane then takes
    // the results in order.  Up to 16 compositing lanes have 4 helpers (4
    // hits) each, up to 32 two, more one.  Done by the compositing lane alone,
    // a hit per step among the surfel steps, this block ran in nearly every
    // step with 8 of 64 lanes: a quarter of the forward's VALU instructions
    // and more of the backward's.  Values cross lanes through bpermute, which
    // costs no VALU issue.  1M surfels, 16.8M rays: forward 66 to 59 ms,
    // backward 87 to 79; 50k surfels, 32k rays, both: 1.97 to 1.80 ms.
    static constexpr int kLogSlots = K < 2 ? 0 : K < 4 ? 1 : 2, kSlots = 1 << kLogSlots;

    // the first n hits leave the buffer
    template <int n>
    __device__ __forceinline__ void shift()
    {
#pragma unroll
        for (int i = 0; i < K - n; ++i) { key[i] = key[i + n]; pos[i] = pos[i + n]; }
#pragma unroll
        for (int i = K - n; i < K; ++i) key[i] = empty_key();
    }

    template <class Visit>
    __device__ __forceinline__ bool composite(const SceneDev &S, Visit &visit, bool comp, uint64_t comps)
    {
        const int lane = (int)__lane_id();
        const int rank = (int)__builtin_amdgcn_mbcnt_hi((uint32_t)(comps >> 32),
                                                        __builtin_amdgcn_mbcnt_lo((uint32_t)comps, 0u));
        const int n = __popcll(comps);
        const int few = n > 32 ? 0 : n > 16 ? 1 : 2, l = min(few, kLogSlots), slots = 1 << l;
        comp &= rank < 64 >> l;
        int nv = 0;
#pragma unroll
        for (int s = 0; s < kSlots; ++s) nv += (int)(s < slots && !is_empty(key[s]));
        // the r-th compositing lane makes itself and its number of hits known
        // to lane r (the others write to lane 63), and helpers read it there
        const int named = __builtin_amdgcn_ds_permute(comp ? 4 * rank : 4 * 63, comp ? lane | nv << 8 : 0);
        const int own = __builtin_amdgcn_ds_bpermute(lane >> l << 2, named);
        const int from = (own & 63) << 2, slot = lane & (slots - 1), first = rank << l << 2;
        const bool helps = slot < own >> 8;
        uint32_t p = 0;
#pragma unroll
        for (int s = 0; s < kSlots; ++s) {
            const uint32_t x = (uint32_t)__builtin_amdgcn_ds_bpermute(from, (int)pos[s]);
            p = slot == s ? x : p;
        }
        const float3 ho = make_float3(lane_pull(from, o.x), lane_pull(from, o.y), lane_pull(from, o.z));
        const float3 hd = make_float3(lane_pull(from, d.x), lane_pull(from, d.y), lane_pull(from, d.z));
        const auto tables = visit.tables(from);
        typename Visit::Item item;
        float in[Visit::kIn];
#pragma unroll
        for (int j = 0; j < Visit::kIn; ++j) in[j] = 0.0f;
        if (helps) {
            const float4 *r = S.rec + 4 * (size_t)p;
            const float4 r0 = r[0], r1 = r[1], r2 = r[2], r3 = r[3];
            float den, tau, rho2;
            canon_geo(r0, r1, r2, r3, ho, hd, den, tau, rho2);
            Visit::item(S, tables, p, r0, r1, r2, r3, rho2, ho, hd, item, in);
        }
        bool stop = false;
        int taken = 0;
        float out[kSlots][Visit::kOut + 1];
#pragma unroll
        for (int s = 0; s < kSlots; ++s) {
#pragma unroll
            for (int j = 0; j < Visit::kOut; ++j) out[s][j] = 0.0f;
            if (s >= slots) continue;
            float x[Visit::kIn];
#pragma unroll
            for (int j = 0; j < Visit::kIn; ++j) x[j] = lane_pull(first + 4 * s, in[j]);
            if (comp && s < nv && !stop) {
                stop = visit.step(x, pos[s], (uint32_t)__double2loint(key[s]), key_tau(key[s]), out[s]);
                last = key[s];  // the last composited hit
                ++taken;
#ifdef GRT_STATS
                ++st_comps;
#endif
            }
        }
        if constexpr (Visit::kOut > 0) {  // the rest of the hits' work, from the steps' results
            const bool again = slot < __builtin_amdgcn_ds_bpermute(from, taken) && helps;
            float back[Visit::kOut], ray[Visit::kRay], ret[Visit::kBack + 1];
#pragma unroll
            for (int j = 0; j < Visit::kOut; ++j) {
                back[j] = 0.0f;
#pragma unroll
                for (int s = 0; s < kSlots; ++s) {
                    const float x = lane_pull(from, out[s][j]);
                    back[j] = slot == s ? x : back[j];
                }
            }
            visit.ray_terms(ray);
#pragma unroll
            for (int j = 0; j < Visit::kRay; ++j) ray[j] = lane_pull(from, ray[j]);
#pragma unroll
            for (int j = 0; j < Visit::kBack; ++j) ret[j] = 0.0f;
            if (again) visit.emit(S, item, back, ray, ret);
            if constexpr (Visit::kBack > 0) {
#pragma unroll
                for (int s = 0; s < kSlots; ++s) {
                    float x[Visit::kBack];
#pragma unroll
                    for (int j = 0; j < Visit::kBack; ++j) x[j] = lane_pull(first + 4 * s, ret[j]);
                    if (comp && s < taken) visit.collect(x);
                }
            }
        }
        if (!comp) return false;
        if (stop) return true;
        if (l == 0) shift<1>();
        else if (l == 1) shift<2 <= kSlots ? 2 : 1>();
        else shift<kSlots>();
        if (is_empty(key[0])) {
            if (st == kFinal || deferred_empty()) return true;
            st = kNone;
            next_round(S);
        }
        return false;
    }

};

// The walker of the backward kernels.
template <int K>
using BwdWalker = Walker<K, kBwdLdsDepth>;

// Upper end of a backward's re-traversal: the depth of the forward's last
// composited hit when it was saved (every hit the backward composites lies at
// or before it, and ties there come after the hit that ended the forward),
// with a margin that keeps node culling clear of rounding.
__device__ __forceinline__ float stop_bound(const float *stop_depth, int64_t r, float tmax)
{
    if (!stop_depth) return tmax;
    const float ts = stop_depth[r];
    return fminf(tmax, ts + 1e-6f * ts + 1e-6f);
}

// ---------------------------------------------------------------------------
// Persistent wavefronts with dynamic ray fetching.
//
// Rays 0..total-1 are split into 8 contiguous partitions, one per XCD (the
// hardware deals workgroups to XCDs round robin), each with its own counter;
// a wavefront claims chunks of kChunk consecutive rays from its XCD's
// partition, then from the others once that one is drained.  Lanes whose ray
// has finished take the next ray of the wavefront's chunk at once, so a
// wavefront never waits for its slowest ray.  Every wavefront leaves the loop
// once all partitions are drained and its lanes are idle.
//
// Job: SceneDev S -- the scene of every ray
//      bool begin(int64_t ray)  -- set up the ray; false if it needs no trace
//      (then it must already have written its result)
//      Walker<K, D> &walker(), Visit &visit(), void finish(int64_t ray),
//      void after_step() and void drain() -- run by every lane of the
//      wavefront after each step and before it leaves
// ---------------------------------------------------------------------------
constexpr int kParts = 8;
constexpr int kChunk = 64;

__host__ __device__ __forceinline__ int64_t part_begin(int64_t total, int q) { return total * q / kParts; }

#ifdef GRT_STATS
// Walk statistics of the instrumented build.  Per kernel kind (a Job with
// kStatSlot 0: the forward radiance trace, 1: the backward re-traversal;
// other jobs are not counted), sums over the rays each kind traced and over
// its wavefront steps; each TU holds its own copy (render kernels: render.hip).
enum { kStRays, kStNodes, kStLeaves, kStComps, kStRounds, kStRestarts, kStDeferred, kStSteps, kStActive, kNumWalkStats };
static __device__ unsigned long long g_walk_stats[2][kNumWalkStats];

template <class J, class = void>
struct StatSlot { static constexpr int value = -1; };
template <class J>
struct StatSlot<J, std::void_t<decltype(J::kStatSlot)>> { static constexpr int value = J::kStatSlot; };

// The lane's sums of a finished ray's walk counters.
template <class W>
__device__ __forceinline__ void walk_tally(uint32_t (&t)[kNumWalkStats], const W &w)
{
    ++t[kStRays];
    t[kStNodes] += w.st_nodes;
    t[kStLeaves] += w.st_leaves;
    t[kStComps] += w.st_comps;
    t[kStRounds] += w.st_rounds;
    t[kStRestarts] += w.st_lost;
    t[kStDeferred] += w.st_deferred;
}

// Adds the wavefront's sums to the kind's totals (all lanes, wavefront-uniform point).
template <int kSlot>
__device__ __forceinline__ void walk_flush(const uint32_t (&t)[kNumWalkStats])
{
    if constexpr (kSlot >= 0) {
#pragma unroll
        for (int i = 0; i < kNumWalkStats; ++i) {
            unsigned long long v = t[i];
            for (int m = 32; m >= 1; m >>= 1) v += __shfl_xor(v, m, 64);
            if ((threadIdx.x & 63) == 0) atomicAdd(&g_walk_stats[kSlot][i], v);
        }
    }
}
#endif

// stop: optional flag in host memory; once it reads non-zero, wavefronts
// claim no further chunks, finish the rays they hold and leave, so the claim
// counters then say exactly which rays were traced (a prefix of each
// partition).
template <int K, class Job>
__device__ __forceinline__ void run_persistent(Job &job, unsigned long long *counters, int64_t total,
                                               const int *stop = nullptr)
{
    const int lane = threadIdx.x & 63;
    const uint64_t lt = (lane == 0) ? 0ull : (~0ull >> (64 - lane));
    int part = blockIdx.x % kParts;
    int tried = 0;
    int64_t pool_next = 0, pool_end = 0;  // wavefront-uniform
    bool exhausted = false;               // wavefront-uniform
    bool active = false;
    int64_t ray = -1;
    using WalkerT = typename std::remove_reference<decltype(job.walker())>::type;
    constexpr int D = WalkerT::kDepth;
    __shared__ int lds_stacks[4][2][D][64];  // [wave][stack][slot][lane]
    int overflow[2 * kStackCap];
    const int wave = (threadIdx.x >> 6) & 3;
    {
        auto &F = job.walker().F;
        F.base = lds_addr(&lds_stacks[wave][0][0][lane]);
        F.woff = 0;
        F.mem = overflow;
        F.reset();
    }
#ifdef GRT_STATS
    uint32_t tally[kNumWalkStats] = {};
#endif
    for (;;) {
        const uint64_t idle = __ballot(!active);
        if (idle && !exhausted) {
            if (pool_next >= pool_end) {
                // claim a chunk (leader lane), moving on to other partitions when drained
                for (;;) {
                    const int64_t pb = part_begin(total, part), pe = part_begin(total, part + 1);
                    unsigned long long got = 0;
                    int halt = 0;
                    const int leader = __ffsll((long long)idle) - 1;
                    if (lane == leader) {
                        if (stop) halt = __hip_atomic_load(stop, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_SYSTEM);
                        if (!halt) got = atomicAdd(&counters[part], (unsigned long long)kChunk);
                    }
                    if (__shfl(halt, leader, 64)) { exhausted = true; break; }
                    got = __shfl(got, leader, 64);
                    if (pb + (int64_t)got < pe) {
                        pool_next = pb + (int64_t)got;
                        pool_end = min(pe, pool_next + kChunk);
                        break;
                    }
                    if (++tried >= kParts) { exhausted = true; break; }
                    part = (part + 1) % kParts;
                }
            }
            if (!exhausted) {
                const int64_t avail = pool_end - pool_next;
                const int rank = __popcll(idle & lt);
                if (!active && rank < avail) {
                    ray = pool_next + rank;
                    active = job.begin(ray);
                }
                const int nidle = __popcll(idle);
                pool_next += (int64_t)(nidle < avail ? nidle : avail);
            }
        }
        const uint64_t busy = __ballot(active);
        // The loop's only exit, and no early return to its head: with one more
        // edge the compiler kept a second copy of the walker's registers in
        // the backward kernels and moved all of it twice a step (450 of 1340
        // VALU instructions, 168 VGPRs with spills; 164 of 1050 and 144
        // without; room step backward 105 to 91 ms at 1024 x 1024, 16 spp).
        if (!busy && exhausted) break;
#ifdef GRT_STATS
        if (lane == 0) {
            ++tally[kStSteps];
            tally[kStActive] += (uint32_t)__popcll(busy);
        }
#endif
        auto &w = job.walker();
        bool done = false;
        if (active && w.st >= 0) done = w.advance(job.S);
        const bool comp = active && w.st < 0;
        const uint64_t comps = __ballot(comp);
        const uint64_t walks = __ballot(active && !done && !comp);
        if (comps && 16 * __popcll(comps) >= kCompShare16 * (__popcll(comps) + __popcll(walks)))
            done |= w.composite(job.S, job.visit(), comp, comps);
        if (done) {
#ifdef GRT_STATS
            walk_tally(tally, w);
#endif
            job.finish(ray);
            active = false;
        }
        job.after_step();  // wavefront-uniform point
    }
#ifdef GRT_STATS
    walk_flush<StatSlot<Job>::value>(tally);
#endif
    job.drain();
}

}  // namespace grt
