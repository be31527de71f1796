// denoise.hip -- cross-bilateral denoiser for low-sample renders (Sec. 3.4.2,
// "Denoising"; SVGF-style spatial filtering guided by depth and normal).
//
// For each valid pixel p, over the valid pixels p' of the (2R+1)^2 window:
//   B(p,p') = exp(-|p-p'|^2 / (2 sigma_s^2))
//           * exp(-|D(p)-D(p')| / (sigma_d |grad D(p) . (p-p')| + eps_d))
//           * max(0, N(p).N(p'))^sigma_n
//   out(p)  = sum B c(p') / sum B
// N is normalized per pixel; grad D is the screen-space depth gradient by
// central differences (one-sided where a neighbour is outside the image or
// invalid, 0 where both are).  Invalid pixels pass through unchanged.
//
// Image-space stencil: a workgroup stages its 16x16 pixels and an R-pixel
// halo (colour, depth, unit normal, validity) in LDS once, so each input is
// read from HBM about (16+2R)^2/256 times instead of (2R+1)^2 times.
//
// Bound by VALU issue: (2R+1)^2 weights a pixel.  So a weight's three factors
// are one exponential of a summed base-2 exponent, with a hardware reciprocal
// in the depth term; the normal term's logarithm is a short series near 1,
// where sigma_n multiplies its error (two expf, a powf and a division per
// weight took 3.5 times as long).
#include <type_traits>

#include "grt_internal.h"

namespace grt {

constexpr int kDnTile = 16;
constexpr int kDnSpan = kDnTile + 2 * kDenoiseMaxRadius;

// log2 of the cosine between two unit normals (0 where it is not positive).
// Near 1 the hardware logarithm's absolute error is about that of its result
// at 2, and sigma_n multiplies it; there 2 atanh(s), s = (c - 1) / (c + 1),
// with terms up to s^7 (|s| <= 1/7: the next is below 2^-25 of the sum).
// The hardware logarithm takes subnormal cosines for 0; kTiny scales them first.
template <bool kTiny>
__device__ __forceinline__ float log2_cos(float c)
{
    const float s = (c - 1.0f) * __builtin_amdgcn_rcpf(c + 1.0f), s2 = s * s;
    const float near1 = s * fmaf(s2, fmaf(s2, fmaf(s2, 2.8853901f / 7.0f, 2.8853901f / 5.0f), 2.8853901f / 3.0f), 2.8853901f);
    float l;
    if (kTiny) {
        const bool sub = c < 1.17549435e-38f;
        l = __builtin_amdgcn_logf(sub ? c * 4294967296.0f : c) - (sub ? 32.0f : 0.0f);
    } else {
        l = __builtin_amdgcn_logf(c);
    }
    l = c >= 0.75f ? near1 : l;
    return c > 0.0f ? l : 0.0f;
}

// A component that may make a cosine subnormal.  Where no unit normal of a
// tile has one, the products of its normals are multiples of 2^-126 (two
// components of 2^-40 and 24 bits), and so are their sums: a workgroup then
// runs the weights without kTiny, which costs 5 instructions a weight (1024 x
// 1024, radius 3: 59 us with it, 56 without).
__device__ __forceinline__ bool tiny(float x) { return x != 0.0f && fabsf(x) < 9.0949470e-13f; }

__global__ void __launch_bounds__(256) k_denoise(DenoiseArgs a)
{
    __shared__ float4 lc[kDnSpan * kDnSpan];  // rgb, depth
    __shared__ float4 ln[kDnSpan * kDnSpan];  // unit normal, valid (>= 1, or below)
    const int R = a.radius, span = kDnTile + 2 * R;
    const int x0 = blockIdx.x * kDnTile - R, y0 = blockIdx.y * kDnTile - R;
    bool small = false;
    for (int i = threadIdx.x; i < span * span; i += blockDim.x) {
        const int ty = i / span, tx = i - ty * span;
        const int gx = x0 + tx, gy = y0 + ty;
        float4 c = make_float4(0.f, 0.f, 0.f, 0.f), n = c;
        if (gx >= 0 && gx < a.W && gy >= 0 && gy < a.H) {
            const int64_t p = (int64_t)gy * a.W + gx;
            if (a.valid[p]) {
                const float nx = a.normal[3 * p], ny = a.normal[3 * p + 1], nz = a.normal[3 * p + 2];
                const float l = sqrtf(nx * nx + ny * ny + nz * nz);
                const float il = l > 0.0f ? 1.0f / l : 0.0f;
                c = make_float4(a.rgb[3 * p], a.rgb[3 * p + 1], a.rgb[3 * p + 2], a.depth[p]);
                n = make_float4(nx * il, ny * il, nz * il, 1.0f);
                small |= tiny(n.x) | tiny(n.y) | tiny(n.z);
            }
        }
        lc[ty * span + tx] = c;
        ln[ty * span + tx] = n;
    }
    __syncthreads();
    // (the flag is the lowest bit of a word that is there: one more word, and
    // a compute unit takes four workgroups instead of five)
    uint32_t *flag = reinterpret_cast<uint32_t *>(&ln[0].w);
    if (small) atomicOr(flag, 1u);
    __syncthreads();
    const bool any_tiny = *flag & 1u;
    const int tx = threadIdx.x % kDnTile, ty = threadIdx.x / kDnTile;
    const int px = blockIdx.x * kDnTile + tx, py = blockIdx.y * kDnTile + ty;
    if (px >= a.W || py >= a.H) return;
    const int64_t p = (int64_t)py * a.W + px;
    const int lx = tx + R, ly = ty + R;
    const float4 cc = lc[ly * span + lx], cn = ln[ly * span + lx];
    if (cn.w < 1.0f) {  // invalid: unchanged
        a.out[3 * p] = a.rgb[3 * p]; a.out[3 * p + 1] = a.rgb[3 * p + 1]; a.out[3 * p + 2] = a.rgb[3 * p + 2];
        return;
    }
    // depth gradient (R >= 1, so the four neighbours are staged)
    auto grad = [&](int ox, int oy) {
        const float4 pc = lc[(ly + oy) * span + lx + ox], mc = lc[(ly - oy) * span + lx - ox];
        const bool hp = ln[(ly + oy) * span + lx + ox].w >= 1.0f, hm = ln[(ly - oy) * span + lx - ox].w >= 1.0f;
        if (hp && hm) return (pc.w - mc.w) * 0.5f;
        if (hp) return pc.w - cc.w;
        if (hm) return cc.w - mc.w;
        return 0.0f;
    };
    const float gx = grad(1, 0), gy = grad(0, 1);
    constexpr float kLog2e = 1.44269504f;
    const float inv2s2 = kLog2e / (2.0f * a.sigma_s * a.sigma_s);
    const float sigma_n = fminf(a.sigma_n, 3.402823466e+38f);  // (infinity times log2 1 is no weight)
    float sr = 0.0f, sg = 0.0f, sb = 0.0f, sw = 0.0f;
    const auto sums = [&](auto tiny_cosines) {
        for (int dy = -R; dy <= R; ++dy)
            for (int dx = -R; dx <= R; ++dx) {
                const int q = (ly + dy) * span + lx + dx;
                const float4 qn = ln[q], qc = lc[q];
                const float c = cn.x * qn.x + cn.y * qn.y + cn.z * qn.z;
                // (kept above what the reciprocal can take)
                const float scale = fmaxf(a.sigma_d * fabsf(gx * (float)dx + gy * (float)dy) + a.eps_d, 1e-37f);
                float x = -(float)(dx * dx + dy * dy) * inv2s2;
                x = fmaf(-kLog2e * fabsf(cc.w - qc.w), __builtin_amdgcn_rcpf(scale), x);
                x = fmaf(sigma_n, log2_cos<decltype(tiny_cosines)::value>(c), x);
                // (an invalid neighbour's normal is 0; a zero base to the power 0 is 1)
                const bool on = (c > 0.0f) | ((sigma_n == 0.0f) & (qn.w >= 1.0f));
                const float B = on ? __builtin_amdgcn_exp2f(x) : 0.0f;
                sr += B * qc.x; sg += B * qc.y; sb += B * qc.z; sw += B;
            }
    };
    if (any_tiny) sums(std::true_type{});
    else sums(std::false_type{});
    const float inv = sw > 0.0f ? 1.0f / sw : 1.0f;
    a.out[3 * p] = sr * inv; a.out[3 * p + 1] = sg * inv; a.out[3 * p + 2] = sb * inv;
}

hipError_t launch_denoise(const DenoiseArgs &a, hipStream_t st)
{
    if (a.H <= 0 || a.W <= 0) return hipSuccess;
    const dim3 grid((unsigned)((a.W + kDnTile - 1) / kDnTile), (unsigned)((a.H + kDnTile - 1) / kDnTile));
    hipLaunchKernelGGL(k_denoise, grid, dim3(kDnTile * kDnTile), 0, st, a);
    return hipGetLastError();
}

}  // namespace grt
