// grt_nodeq.h -- the quantized 4-wide node of the traversals: its layout, how
// it is made from child boxes, and the test of a ray against it.  What the
// test rounds and what the planes allow for it belong together; the header
// needs no other of the library, so that the pair is also run on the CPU.
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

namespace grt {

// Unused child slots of a 4-wide node hold this reference (and a zero box).
constexpr int kNoChild = 0x7fffffff;

// The node a walk loads: child j spans org + scale * [lo_j, hi_j] on each
// axis, with byte j of the axis' lo and hi words (conservative, see
// quantize_node).  The vector L1 bounds the walk as much as VALU issue does (a
// divergent load is one tag access per lane and 16 bytes: 97% of its cycles
// were busy or stalled with the seven loads of a 128-byte node), so a node is
// four loads.
struct alignas(16) NodeQ {
    float org[3];
    float scale[3];
    uint32_t lo[3], hi[3];
    int4 ch;  // child references (kNoChild: unused slot)
};
static_assert(sizeof(NodeQ) == 64, "four 16-byte loads");

// The walk's inverse direction, formed at each node step rather than held (3
// registers), by the hardware reciprocal (1 ulp, which the slab test's slack
// counts).  Components below 1e-18 are taken as that, so that plane * inverse
// stays finite; the sign is kept.
__device__ __forceinline__ float fast_inv(float d)
{
    return __builtin_amdgcn_rcpf(fabsf(d) > 1e-18f ? d : copysignf(1e-18f, d));
}

// Byte j of a word as a float (one instruction).
template <int j>
__device__ __forceinline__ float byte_f(uint32_t w)
{
    return (float)((w >> (8 * j)) & 255u);
}

// Child j of a node from the words of its near and far planes (chosen by the
// sign of the direction): the depth of plane q of an axis is q * step + start,
// one fused multiply-add, with no min or max of the pair.  Where start and step
// cancel, rounding moves a plane by less than the margin the node was quantized
// with.  The rest is relative to the depth: with u = 2^-24, 2 u of the
// reciprocal and u each of the difference to the origin, its product and the
// sum, so 5 u a plane; planes of two axes 10 u and the comparison's product 1,
// for which it allows 16.  (With 8 u a ray through an edge of a box was lost
// where all of them met.)  A NaN keeps the child.
template <int j>
__device__ __forceinline__ bool slab_q(uint32_t nx, uint32_t ny, uint32_t nz, uint32_t fx, uint32_t fy, uint32_t fz,
                                       const float3 step, const float3 start, float t0, float &tnear)
{
    const float ax = fmaf(byte_f<j>(nx), step.x, start.x), bx = fmaf(byte_f<j>(fx), step.x, start.x);
    const float ay = fmaf(byte_f<j>(ny), step.y, start.y), by = fmaf(byte_f<j>(fy), step.y, start.y);
    const float az = fmaf(byte_f<j>(nz), step.z, start.z), bz = fmaf(byte_f<j>(fz), step.z, start.z);
    const float tn = fmaxf(fmaxf(ax, ay), fmaxf(az, t0));
    const float tf = fminf(fminf(bx, by), bz);
    tnear = tn;
    return !(tn > tf * 1.000001f + 1e-30f);
}

// The NodeQ of m child boxes (lo xyz, hi xyz).  Per axis, a grid of 256 planes
// over the children's union; each child takes the grid planes just outside its
// own.  All of it is done on offsets from the grid's origin: far from the
// scene's origin coordinates are coarser than the margin, and a plane compared
// there could end up inside its box by half of their spacing.  With u = 2^-24
// and E the grid's length, an offset, its margin and a plane's product are off
// by 3 u E together, and the walk's depth of a plane by 3 u E more (start and
// step, where they cancel) beside a part relative to the depth; the margin is
// 16 u times the union's extent.
__device__ __forceinline__ NodeQ quantize_node(const float (&box)[4][6], const int (&ref)[4], int m)
{
    NodeQ q;
#pragma unroll
    for (int a = 0; a < 3; ++a) {
        float lo = box[0][a], hi = box[0][3 + a];
#pragma unroll
        for (int j = 1; j < 4; ++j)
            if (j < m) {
                lo = fminf(lo, box[j][a]);
                hi = fmaxf(hi, box[j][3 + a]);
            }
        const float margin = (hi - lo) * 9.5367431640625e-07f;
        float org = lo - 2.0f * margin;
        if (lo - org < margin) org = nextafterf(lo, -INFINITY);  // the margin is below the coordinate's spacing
        const float len = (hi - org) + margin;
        float scale = len * (1.0f / 255.0f) * 1.000001f;
        if (255.0f * scale < len) scale *= 1.00001f;
        q.org[a] = org;
        q.scale[a] = scale;
        uint32_t wl = 0, wh = 0;
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            if (j >= m) continue;
            const float l = (box[j][a] - org) - margin, h = (box[j][3 + a] - org) + margin;
            // (a NaN plane, of a surfel with NaN parameters, keeps the whole span)
            int ql = (int)fminf(fmaxf(floorf(l / scale), 0.0f), 255.0f);
            int qh = (int)fminf(fmaxf(ceilf(h / scale), 0.0f), 255.0f);
            if (ql > 0 && !((float)ql * scale <= l)) --ql;
            if (qh < 255 && !((float)qh * scale >= h)) ++qh;
            if (!(scale > 0.0f && l <= h)) { ql = 0; qh = 255; }
            wl |= (uint32_t)ql << (8 * j);
            wh |= (uint32_t)qh << (8 * j);
        }
        q.lo[a] = wl;
        q.hi[a] = wh;
    }
    q.ch = make_int4(ref[0], ref[1], ref[2], ref[3]);
    return q;
}

}  // namespace grt
