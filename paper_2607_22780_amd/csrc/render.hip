// render.hip -- environment tables and the fused MIS render (forward and
// backward by re-traversal).
//
// One ray per (pixel, sample): a generation kernel draws every sample and
// writes its ray record, persistent wavefronts trace them (fetching rays
// dynamically), and a reduction sums each pixel.  Per sample (Sec. 3.3 Eq.
// montecarlo, Sec. 3.4.1 Eq. mis):
//   u1,u2  <- Philox-4x32-10(key = seed, counter = (pixel, j, job, 0))
//   w      <- cosine (j < N_c) | GGX visible normal (j < N_c+N_g) | env texel
//   q      =  (N_c p_c + N_g p_g + N_e p_e) / N_r          (balance heuristic)
//   if w.n > 0:  (C, T) <- Trace(x, w);  L_i = C + T L_env(w)   (Eqs. incident_trace, lighting_decompose)
//                g/q = f(wo, w) L_i (w.n) / q              (Eqs. brdf_decompose, brdf_specular)
// is written per sample; a second kernel sums each pixel's samples in sample
// order, so the estimate (1/N_r) sum g/q is reproducible run to run and does
// not depend on other pixels or on the scheduling.
#include "grt_render.h"

namespace grt {

// ---------------------------------------------------------------------------
// Environment proposal tables: texel weight = luminance x sin(theta_centre);
// cumulative sums in double, left to right, rounded to float at the end.
// ---------------------------------------------------------------------------
// The sums are a serial chain by definition (left to right), so what surrounds
// the chain is taken off it (93 to 7 us for 128 x 256 with a thread per row, the
// marginal 21 to 4): a block loads and weights a chunk in parallel,
// one thread adds it up in LDS, and the block divides and stores.  Rows longer
// than a chunk go over it twice, since the quotients need the row's total.
constexpr int kCdfChunk = 1024;

// x[0..m) in LDS to its running sums, left to right, from acc on; returns the
// last.  One thread; eight loads are in flight ahead of the additions.
__device__ __forceinline__ double run_sums(double *x, int m, double acc)
{
#pragma clang fp contract(off)
    int j = 0;
    for (; j + 8 <= m; j += 8) {
        double v[8];
#pragma unroll
        for (int k = 0; k < 8; ++k) v[k] = x[j + k];
#pragma unroll
        for (int k = 0; k < 8; ++k) {
            acc += v[k];
            x[j + k] = acc;
        }
    }
    for (; j < m; ++j) {
        acc += x[j];
        x[j] = acc;
    }
    return acc;
}

// cdf[1..n] = running sums of val over their total (uniform steps where that
// is 0), cdf[0] = 0, cdf[n] = 1; returns the total.  A block of 256.
template <class Val>
__device__ __forceinline__ double block_cdf(int n, Val val, double *x, double *carry, float *__restrict__ cdf)
{
#pragma clang fp contract(off)
    const bool once = n <= kCdfChunk;
    double total = 0.0;
    for (int pass = once ? 1 : 0; pass < 2; ++pass) {
        if (threadIdx.x == 0) *carry = 0.0;
        for (int base = 0; base < n; base += kCdfChunk) {
            const int m = min(kCdfChunk, n - base);
            for (int j = threadIdx.x; j < m; j += 256) x[j] = val(base + j);
            __syncthreads();
            if (threadIdx.x == 0) *carry = run_sums(x, m, *carry);
            __syncthreads();
            if (once) total = *carry;
            if (pass == 1)
                for (int j = threadIdx.x; j < m; j += 256)
                    cdf[base + j + 1] = base + j + 1 == n ? 1.0f
                                        : total > 0.0     ? (float)(x[j] / total)
                                                          : (float)((double)(base + j + 1) / n);
            __syncthreads();
        }
        total = *carry;
        __syncthreads();
    }
    if (threadIdx.x == 0) cdf[0] = 0.0f;
    return total;
}

__global__ void __launch_bounds__(256) k_env_rows(int H, int W, const float *__restrict__ rgb, float *__restrict__ cond,
                                                  double *__restrict__ rows)
{
#pragma clang fp contract(off)
    __shared__ double x[kCdfChunk], carry;
    const int i = blockIdx.x;
    const double st = sin(3.14159265358979323846 * (i + 0.5) / H);
    const float *p = rgb + (size_t)i * W * 3;
    auto val = [&](int j) {
        const double lum = 0.2126 * (double)p[3 * j] + 0.7152 * (double)p[3 * j + 1] + 0.0722 * (double)p[3 * j + 2];
        return lum * st;
    };
    const double total = block_cdf(W, val, x, &carry, cond + (size_t)i * (W + 1));
    if (threadIdx.x == 0) rows[i] = total;
}

__global__ void __launch_bounds__(256) k_env_marginal(int H, const double *__restrict__ rows, float *__restrict__ marg)
{
    __shared__ double x[kCdfChunk], carry;
    block_cdf(H, [&](int i) { return rows[i]; }, x, &carry, marg);
}

hipError_t launch_env_build(const float *rgb, int H, int W, const EnvWS &w, hipStream_t st)
{
    hipLaunchKernelGGL(k_env_rows, dim3(H), dim3(256), 0, st, H, W, rgb, w.cond, w.rows);
    hipLaunchKernelGGL(k_env_marginal, dim3(1), dim3(256), 0, st, H, w.rows, w.marg);
    return hipGetLastError();
}

// ---------------------------------------------------------------------------
// Prefiltered environment for split-sum relighting (Eq. relight_splitsum).
// The environment is piecewise constant over its texels; each table entry is
// a ratio of sums over all texels (centre direction l, exact solid angle dW)
// accumulated in double:
//   E_d(n)    = sum L max(0, n.l) dW / sum max(0, n.l) dW
//   E_s(R, r) = sum L D(h) max(0, R.l) dW / sum D(h) max(0, R.l) dW,
//               h = normalize(R + l), GGX D with alpha = r^2.
// A ratio of sums does not see a common factor of its weights, and for unit
// vectors (n.h)^2 = (1 + n.l) / 2, so a level's weight is max(0, R.l) dW / t^2
// with t = (1 + n.l) / 2 (a2 - 1) + 1: no square root, and one reciprocal.
// Bound by double-precision issue.  The texels' angles come from a table per
// row and column (three trigonometric calls a texel and entry were most of the
// time), and a block of four wavefronts shares a table texel: 512 wavefronts
// left half of the chip's SIMDs idle.  128 x 256 map: 728 to 82 us.
// ---------------------------------------------------------------------------
// rows: sin and cos of the polar angle and the solid angle of a texel there;
// columns: cos and sin of the azimuth (at texel centres).
__global__ void __launch_bounds__(256) k_env_dirs(int H, int W, double *__restrict__ dirs)
{
#pragma clang fp contract(off)
    const int i = blockIdx.x * 256 + threadIdx.x;
    if (i < H) {
        const double th = kPiD * (i + 0.5) / H;
        dirs[i] = sin(th);
        dirs[H + i] = cos(th);
        dirs[2 * (size_t)H + i] = 2.0 * kPiD / W * (cos(kPiD * i / H) - cos(kPiD * (i + 1) / H));
    } else if (i - H < W) {
        const double ph = 2.0 * kPiD * (i - H + 0.5) / W;
        dirs[2 * (size_t)H + i] = cos(ph);
        dirs[2 * (size_t)H + W + i] = sin(ph);
    }
}

// 1 / x to the last bits: the hardware's estimate and two Newton steps.
__device__ __forceinline__ double fast_recip(double x)
{
    double r = __builtin_amdgcn_rcp(x);
    r = fma(fma(-x, r, 1.0), r, r);
    return fma(fma(-x, r, 1.0), r, r);
}

__global__ void __launch_bounds__(256) k_env_prefilter(int H, int W, const float *__restrict__ rgb,
                                                       const double *__restrict__ dirs, float *__restrict__ Ed,
                                                       float *__restrict__ Es)
{
    constexpr int kAcc = 4 + 4 * (kPfL - 1);  // diffuse (L, weight), then each level
    __shared__ double part[4][kAcc];
    const int t = blockIdx.x;
    const double tth = kPiD * ((t / kPfW) + 0.5) / kPfH, tph = 2.0 * kPiD * ((t % kPfW) + 0.5) / kPfW;
    const V3 nt = v3(sin(tth) * cos(tph), cos(tth), sin(tth) * sin(tph));
    double acc[kAcc];
#pragma unroll
    for (int q = 0; q < kAcc; ++q) acc[q] = 0.0;
    const double *st = dirs, *ct = dirs + H, *om = dirs + 2 * (size_t)H, *cp = dirs + 3 * (size_t)H, *sp = cp + W;
    const int total = H * W, rows = 256 / W, cols = 256 - rows * W;  // a step of 256 texels
    int i = (int)threadIdx.x / W, j = (int)threadIdx.x - i * W;
    for (int k = threadIdx.x; k < total; k += 256) {
        const double c = nt.x * (st[i] * cp[j]) + nt.y * ct[i] + nt.z * (st[i] * sp[j]);
        if (c > 0.0) {
            const float *L = rgb + (size_t)k * 3;
            const double Lx = L[0], Ly = L[1], Lz = L[2], w = c * om[i];
            acc[0] += w * Lx; acc[1] += w * Ly; acc[2] += w * Lz; acc[3] += w;
            const double nh2 = 0.5 + 0.5 * c;
#pragma unroll
            for (int lv = 1; lv < kPfL; ++lv) {
                const double r = (double)lv / (kPfL - 1), a2 = r * r * r * r;
                const double x = nh2 * (a2 - 1.0) + 1.0;
                const double wl = w * fast_recip(x * x);
                double *s = acc + 4 * lv;
                s[0] += wl * Lx; s[1] += wl * Ly; s[2] += wl * Lz; s[3] += wl;
            }
        }
        i += rows;
        j += cols;
        if (j >= W) { j -= W; ++i; }
    }
#pragma unroll
    for (int q = 0; q < kAcc; ++q) {
        for (int m = 32; m >= 1; m >>= 1) acc[q] += __shfl_xor(acc[q], m, 64);
        if ((threadIdx.x & 63) == 0) part[threadIdx.x >> 6][q] = acc[q];
    }
    __syncthreads();
    if (threadIdx.x < 3 * kPfL) {
        const int lv = threadIdx.x / 3, c = threadIdx.x - 3 * lv;
        double s = 0.0, w = 0.0;
        for (int k = 0; k < 4; ++k) {
            s += part[k][4 * lv + c];
            w += part[k][4 * lv + 3];
        }
        const float v = w > 0.0 ? (float)(s / w) : 0.0f;
        if (lv == 0) Ed[t * 3 + c] = v;
        else Es[((size_t)(lv - 1) * kPfH * kPfW + t) * 3 + c] = v;
    }
}

// DFG table: per cell (n.v = mu, roughness r at cell centres), the Schlick
// split of the specular directional albedo (F = 1),
//   A = E[g (1 - (1 - v.h)^5)],  B = E[g (1 - v.h)^5],  g = G (v.h) / (mu n.h),
// over half vectors h distributed as D(h) n.h (the inverse GGX distribution
// on a kLutQ x kLutQ midpoint grid of (xi, azimuth)), l = reflect(v, h) above
// the horizon.  v lies in the xz plane, so only the azimuth's cosine enters
// and the two halves of the circle are equal: a thread takes one xi and the
// 128 azimuths of one half, whose cosines the block keeps in LDS (a sine and a
// cosine per node took most of 417 us; 57 now).  Bound by double-precision
// issue.
__global__ void __launch_bounds__(256) k_dfg_lut(float *__restrict__ lut)
{
    static_assert(kLutQ == 256, "one thread per xi");
    __shared__ double cp[kLutQ / 2], part[4][2];
    const int cell = blockIdx.x, i = cell / kLutN, j = cell % kLutN, s = threadIdx.x;
    if (s < kLutQ / 2) cp[s] = cos(2.0 * kPiD * (s + 0.5) / kLutQ);
    __syncthreads();
    const double mu = (i + 0.5) / kLutN, r = (j + 0.5) / kLutN, al = r * r, a2 = al * al;
    const double xi = (s + 0.5) / kLutQ;
    const double c2 = (1.0 - xi) / (1.0 + (a2 - 1.0) * xi);
    const double ct = sqrt(c2), st = sqrt(1.0 - c2 > 0.0 ? 1.0 - c2 : 0.0);
    const double vx = sqrt(1.0 - mu * mu) * st, vz = mu * ct;
    double A = 0.0, B = 0.0;
    for (int t = 0; t < kLutQ / 2; ++t) {
        const double vh = vx * cp[t] + vz;
        const double nl = 2.0 * vh * ct - mu;
        if (vh > 0.0 && nl > 0.0) {
            // G1(n.l) (v.h) / 2, the rest of g being constant in the azimuth
            const double g = nl * vh * fast_recip(nl + sqrt(a2 + (1.0 - a2) * nl * nl));
            const double x = 1.0 - vh, x2 = x * x, fc = x2 * x2 * x;
            A += g * (1.0 - fc);
            B += g * fc;
        }
    }
    const double f = 2.0 * smith_G1(mu, a2) / (mu * ct);
    A *= f;
    B *= f;
    for (int m = 32; m >= 1; m >>= 1) {
        A += __shfl_xor(A, m, 64);
        B += __shfl_xor(B, m, 64);
    }
    if ((s & 63) == 0) {
        part[s >> 6][0] = A;
        part[s >> 6][1] = B;
    }
    __syncthreads();
    if (s < 2)  // both halves of the circle
        lut[2 * cell + s] = (float)(2.0 * ((part[0][s] + part[1][s]) + (part[2][s] + part[3][s])) /
                                    ((double)kLutQ * kLutQ));
}

hipError_t launch_env_prefilter(const float *rgb, int H, int W, const EnvWS &w, hipStream_t st, bool lut)
{
    hipLaunchKernelGGL(k_env_dirs, dim3((H + W + 255) / 256), dim3(256), 0, st, H, W, w.dirs);
    hipLaunchKernelGGL(k_env_prefilter, dim3(kPfH * kPfW), dim3(256), 0, st, H, W, rgb, w.dirs, w.Ed, w.Es);
    hipError_t e = hipGetLastError();
    if (e != hipSuccess || !lut) return e;
    return launch_dfg_lut(w.lut, st);
}

hipError_t launch_dfg_lut(float *lut, hipStream_t st)
{
    hipLaunchKernelGGL(k_dfg_lut, dim3(kLutN * kLutN), dim3(256), 0, st, lut);
    return hipGetLastError();
}

// A wavefront draws one sample index of 64 neighbouring pixels, so that it
// runs one proposal: with a pixel's samples side by side, every wavefront ran
// all three in turns.  Bound by double-precision issue.  An image of at most
// 32 pixels (probes with many samples) fills the lanes with 64 / 2^lp
// consecutive samples of each of 2^lp pixels instead, which costs turns only
// where a proposal begins (1 pixel x 65,536 samples: 163 us with one lane of
// each wavefront, 11 so; 63 x 1,024: 11 either way).
__global__ void __launch_bounds__(256) k_render_gen(RenderArgs a, int lp)
{
    const int spp = a.nc + a.ng + a.ne, lane = threadIdx.x & 63;
    const int64_t npix = (int64_t)a.H * a.W;
    const uint32_t runs = ((uint32_t)spp + (63u >> lp)) >> (6 - lp);  // of samples
    const uint32_t w = __builtin_amdgcn_readfirstlane(blockIdx.x * 4u + (threadIdx.x >> 6));
    const uint32_t group = w / runs;
    const int64_t p = ((int64_t)group << lp) + (lane & ((1 << lp) - 1));
    const int j = (int)((w - group * runs) << (6 - lp)) + (lane >> lp);
    if (p < npix && j < spp) gen_ray(a, p, j);
}

// ---------------------------------------------------------------------------
// Jobs for the persistent loop.  Ray index order keeps a wavefront's chunk on
// neighbouring pixels (shared origins, nearby surfaces).
// ---------------------------------------------------------------------------
template <int K, bool kHitList>
struct RenderJob {
    static constexpr int kStatSlot = 0;  // walk statistics (instrumented build)
    const RenderArgs &a;
    SceneDev S;
    ShadeTrace<K, kHitList> t;
    uint32_t r;  // sample index of the lane's ray

    __device__ RenderJob(const RenderArgs &a_) : a(a_), S(a_.S), r(0) { t.bind(a, S); }
    __device__ __forceinline__ Walker<K> &walker() { return t.w; }
    __device__ __forceinline__ decltype(t.v) &visit() { return t.v; }
    __device__ __forceinline__ bool begin(int64_t g)
    {
        r = a.order ? a.order[g] : (uint32_t)g;
        return t.begin(a, S, r);
    }
    __device__ __forceinline__ void finish(int64_t) { t.finish(a, r); }
    __device__ __forceinline__ void after_step() {}
    __device__ __forceinline__ void drain() {}
};

// Relighting (Sec. 3.5.1), first pass: the forward render's job with the
// attribute query instead of the radiance trace (RelightTrace parks each
// traced sample's query result for the shading pass).
template <int K>
struct RelightJob {
    const RenderArgs &a;
    SceneDev S;
    RelightTrace<K> t;
    uint32_t r;

    __device__ RelightJob(const RenderArgs &a_) : a(a_), S(a_.S), r(0) { t.bind(a, S); }
    __device__ __forceinline__ Walker<K> &walker() { return t.w; }
    __device__ __forceinline__ decltype(t.v) &visit() { return t.v; }
    __device__ __forceinline__ bool begin(int64_t g)
    {
        r = a.order ? a.order[g] : (uint32_t)g;
        return t.begin(a, S, r);
    }
    __device__ __forceinline__ void finish(int64_t) { t.finish(a, r); }
    __device__ __forceinline__ void after_step() {}
    __device__ __forceinline__ void drain() {}
};

// Relighting, second pass (one thread per sample): the incident radiance
// V L_env(w) + (1 - V) SplitSum(a, r, m, n, E) (Eq. relight_splitsum) of each
// traced sample from its parked query, weighted by f cos / q.
__global__ void __launch_bounds__(256) k_relight_shade(RenderArgs a, int64_t total)
{
    const int64_t r = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (r >= total) return;
    const float4 r0 = a.rays[3 * r];
    if (r0.w == 0.0f) return;  // untraced: its contribution is already 0
    const float4 r1 = a.rays[3 * r + 1], r2 = a.rays[3 * r + 2], q = a.contrib[r];
    const double V = q.x;
    V3 L = v3((double)r1.w * V, (double)r2.x * V, (double)r2.y * V);
    if (V < 1.0) {
        const V3 ss = split_sum(a.E, v3(q.y, q.z, q.w), r2.z, r2.w, v3(a.rl_nx[r], a.rl_ny[r], a.rl_nz[r]),
                                v3(r0.x, r0.y, r0.z));
        L = v3(L.x + (1.0 - V) * ss.x, L.y + (1.0 - V) * ss.y, L.z + (1.0 - V) * ss.z);
    }
    a.contrib[r] = make_float4((float)(r1.x * L.x), (float)(r1.y * L.y), (float)(r1.z * L.z), 0.0f);
    if (a.dump) {
        float *dp = a.dump + r * 10;
        dp[7] = (float)L.x; dp[8] = (float)L.y; dp[9] = (float)L.z;
    }
}

// kOrigin: also write each sample's origin gradient to a.gorig (zero for a
// sample that contributes nothing; samples done from stored hit lists are
// left to that kernel).
template <int K, bool kOrigin>
struct RenderBwdJob {
    static constexpr int kStatSlot = 1;  // walk statistics (instrumented build)
    const RenderArgs &a;
    SceneDev S;
    BwdWalker<K> w;
    GradVisitT<kOrigin> v;
    int spp;

    __device__ RenderBwdJob(const RenderArgs &a_, WaveStage *t)
        : a(a_), S(a_.S), v(a_.tcut), spp(a_.nc + a_.ng + a_.ne)
    {
        v.stage = t;
        stage_init(t);
        w.tmin = a.tmin;
    }
    __device__ __forceinline__ BwdWalker<K> &walker() { return w; }
    __device__ __forceinline__ GradVisitT<kOrigin> &visit() { return v; }

    __device__ __forceinline__ bool skip(int64_t r)
    {
        if constexpr (kOrigin) a.gorig[r] = make_float4(0.f, 0.f, 0.f, 0.f);
        return false;
    }

    __device__ __forceinline__ bool begin(int64_t g)
    {
        const int64_t r = a.order ? (int64_t)a.order[g] : g;
        if (S.n <= 0) return skip(r);
        const float4 r0 = a.rays[3 * r];
        if (r0.w == 0.0f) return skip(r);
        if (a.hits && a.hits[r] <= (uint32_t)a.hcap) return false;  // done from its stored list
        const int64_t p = (uint32_t)r / (uint32_t)spp;  // fewer than 2^31 samples
        const float inv = 1.0f / (float)spp;
        const float3 gp = make_float3(a.grad[3 * p] * inv, a.grad[3 * p + 1] * inv, a.grad[3 * p + 2] * inv);
        if (gp.x == 0.0f && gp.y == 0.0f && gp.z == 0.0f) return skip(r);
        const float4 r1 = a.rays[3 * r + 1], r2 = a.rays[3 * r + 2];
        const float3 gC = make_float3(r1.x * gp.x, r1.y * gp.y, r1.z * gp.z);
        const float gT = gC.x * r1.w + gC.y * r2.x + gC.z * r2.y;
        const float4 sv = a.saved[r];
        const float3 x = make_float3(a.x[3 * p], a.x[3 * p + 1], a.x[3 * p + 2]);
        const float3 d = make_float3(r0.x, r0.y, r0.z);
        v.reset(gC, gT, make_float3(sv.x, sv.y, sv.z), sv.w);
        w.tmax = stop_bound(a.saved_t, r, INFINITY);
        w.start(S, x, d);
        if constexpr (kOrigin) cur = (uint32_t)r;
        return true;
    }

    __device__ __forceinline__ void finish(int64_t)
    {
        if constexpr (kOrigin) a.gorig[cur] = make_float4(-v.gmu.x, -v.gmu.y, -v.gmu.z, 0.0f);
    }
    __device__ __forceinline__ void after_step() { stage_sync(a.g.acc, v.stage, false); }
    __device__ __forceinline__ void drain() { stage_sync(a.g.acc, v.stage, true); }

    uint32_t cur = 0;  // the lane's sample (kOrigin)
};

// kHitList: the launch stores hit lists (a.hits set); a separate kernel, so
// that the plain forward carries no list pointer in its registers.
template <int K, bool kHitList>
__global__ void __launch_bounds__(256) GRT_WAVES(K, 4) k_render(RenderArgs a)
{
    RenderJob<K, kHitList> job(a);
    run_persistent<K>(job, a.counters, (int64_t)a.H * a.W * (a.nc + a.ng + a.ne));
}

template <int K>
__global__ void __launch_bounds__(256) GRT_WAVES(K, 4) k_render_relight(RenderArgs a)
{
    RelightJob<K> job(a);
    run_persistent<K>(job, a.counters, (int64_t)a.H * a.W * (a.nc + a.ng + a.ne));
}

// Word of a launch's counters, behind the claim counters: set when a sample's
// hit list overflowed.
constexpr int kOverflowed = kParts;
static_assert((kOverflowed + 1) * sizeof(unsigned long long) <= kCounterBytes, "counters of a launch");

template <int K, bool kOrigin>
__global__ void __launch_bounds__(256) GRT_WAVES(K, kOrigin && K > 8 ? 2 : 3) k_render_bwd(RenderArgs a)
{
    // From lists none of which overflowed there is nothing to trace, and to
    // claim every ray only to find its list would cost as much as a third of the
    // lists' pass (180k samples: 306 us, most of it the claim counters).
    if (a.hits && !a.counters[kOverflowed]) return;
    __shared__ WaveStage stages[4];
    RenderBwdJob<K, kOrigin> job(a, &stages[(threadIdx.x >> 6) & 3]);
    run_persistent<K>(job, a.counters, (int64_t)a.H * a.W * (a.nc + a.ng + a.ne));
}

// Backward from stored hit lists: one thread per sample runs the gradient of
// its composited hits in order (no traversal).  Samples whose list
// overflowed are left to the re-traversal kernel.  The wavefront steps
// through the lists together, one hit per lane per step, so that its staged
// terms are flushed at wavefront-uniform points.  kOrigin: also writes each
// sample's origin gradient (overflowed samples: by the re-traversal).
template <bool kOrigin>
__global__ void __launch_bounds__(256) k_render_bwd_stored(RenderArgs a)
{
    __shared__ WaveStage stages[4];
    WaveStage *stage = &stages[(threadIdx.x >> 6) & 3];
    stage_init(stage);
    const int spp = a.nc + a.ng + a.ne;
    const int64_t nray = (int64_t)a.H * a.W * spp;
    const int64_t g = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    // samples in traversal order: a wavefront's rays are neighbours and share surfels
    const int64_t r = g < nray ? (a.order ? (int64_t)a.order[g] : g) : 0;
    const uint32_t nh = g < nray && a.S.n > 0 ? a.hits[r] : 0u;
    const float4 r0 = nh ? a.rays[3 * r] : make_float4(0.f, 0.f, 0.f, 0.f);
    const bool over = nh > (uint32_t)a.hcap && r0.w != 0.0f;  // left to the re-traversal
    if (__ballot(over) && (threadIdx.x & 63) == 0) a.counters[kOverflowed] = 1ull;
    GradVisitT<kOrigin> v(a.tcut);
    v.stage = stage;
    v.gmu = make_float3(0.f, 0.f, 0.f);
    uint32_t cnt = 0;
    float3 x = make_float3(0.f, 0.f, 0.f), d = x;
    const uint32_t *list = a.hits + nray + r * a.hcap;
    if (nh > 0u && nh <= (uint32_t)a.hcap && r0.w != 0.0f) {
        const int64_t p = r / spp;
        const float inv = 1.0f / (float)spp;
        const float3 gp = make_float3(a.grad[3 * p] * inv, a.grad[3 * p + 1] * inv, a.grad[3 * p + 2] * inv);
        if (gp.x != 0.0f || gp.y != 0.0f || gp.z != 0.0f) {
            const float4 r1 = a.rays[3 * r + 1], r2 = a.rays[3 * r + 2];
            const float3 gC = make_float3(r1.x * gp.x, r1.y * gp.y, r1.z * gp.z);
            const float gT = gC.x * r1.w + gC.y * r2.x + gC.z * r2.y;
            const float4 sv = a.saved[r];
            x = make_float3(a.x[3 * p], a.x[3 * p + 1], a.x[3 * p + 2]);
            d = make_float3(r0.x, r0.y, r0.z);
            v.reset(gC, gT, make_float3(sv.x, sv.y, sv.z), sv.w);
            cnt = nh;
        }
    }
    for (uint32_t i = 0; __ballot(i < cnt); ++i) {
        if (i < cnt) visit_hit(v, a.S, list[i], x, d);
        stage_sync(a.g.acc, stage, false);
    }
    stage_sync(a.g.acc, stage, true);
    if constexpr (kOrigin) {
        if (g < nray && !over)
            a.gorig[r] = make_float4(-v.gmu.x, -v.gmu.y, -v.gmu.z, 0.0f);
    }
}

// Gradients of the loss with respect to each pixel's shading state (x, the
// stored normal and view direction, albedo, roughness, metallic), each
// sample's direction and mixture pdf held fixed; one thread per pixel, its
// samples in order.  The sample's weight f (n.w) / q is differentiated from
// the regenerated direction and pdf (in double), its incident radiance L_i =
// c_rt + T L_env comes from the forward's saved state, and x moves every
// secondary ray's origin (the per-sample origin gradients of the backward
// pass, a.gorig).  Unit n and wo are the stored vectors over their lengths,
// so their gradients are projected off the unit vector and divided by them.
__global__ void __launch_bounds__(256) k_render_shade_grad(RenderArgs a, ShadeGradOut o)
{
    const int64_t p = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (p >= (int64_t)a.H * a.W) return;
    const int spp = a.nc + a.ng + a.ne;
    ShadeGrad g{};
    double gx[3] = {0.0, 0.0, 0.0};
    Shade s;
    const bool lit = load_pixel(a, p, s);
    if (lit) {
        const double gp[3] = {a.grad[3 * p], a.grad[3 * p + 1], a.grad[3 * p + 2]};
        for (int j = 0; j < spp; ++j) {
            const int64_t r = p * spp + j;
            if (a.rays[3 * r].w == 0.0f) continue;  // below the horizon: not traced
            const float4 go = a.gorig[r];
            gx[0] += go.x; gx[1] += go.y; gx[2] += go.z;
            V3 w;
            EnvTexel tx = {0, 0, 0.0};
            float3 wf, wt;
            double q;
            draw<false>(a, s, p, j, w, wf, tx, q, wt);
            if (!(q > 0.0)) continue;
            const float4 sv = a.saved[r], r1 = a.rays[3 * r + 1], r2 = a.rays[3 * r + 2];
            const float Li[3] = {sv.x + sv.w * r1.w, sv.y + sv.w * r2.x, sv.z + sv.w * r2.y};
            double u[3];
            for (int c = 0; c < 3; ++c) u[c] = gp[c] * (double)Li[c] / ((double)spp * q);
            brdf_cos_backward(s.n, s.wo, w, s.alb, s.rough, s.metal, u, g);
        }
    }
    V3 gn = v3(0.0, 0.0, 0.0), gw = gn;
    if (lit) {
        const double ln = sqrt((double)a.n[3 * p] * a.n[3 * p] + (double)a.n[3 * p + 1] * a.n[3 * p + 1] +
                               (double)a.n[3 * p + 2] * a.n[3 * p + 2]);
        const double lo = sqrt((double)a.wo[3 * p] * a.wo[3 * p] + (double)a.wo[3 * p + 1] * a.wo[3 * p + 1] +
                               (double)a.wo[3 * p + 2] * a.wo[3 * p + 2]);
        const double pn = dot(s.n, g.n), po = dot(s.wo, g.wo);
        gn = v3((g.n.x - s.n.x * pn) / ln, (g.n.y - s.n.y * pn) / ln, (g.n.z - s.n.z * pn) / ln);
        gw = v3((g.wo.x - s.wo.x * po) / lo, (g.wo.y - s.wo.y * po) / lo, (g.wo.z - s.wo.z * po) / lo);
    }
    auto put3 = [&](float *dst, double x, double y, double z) {
        if (dst) { dst[3 * p] = (float)x; dst[3 * p + 1] = (float)y; dst[3 * p + 2] = (float)z; }
    };
    put3(o.x, gx[0], gx[1], gx[2]);
    put3(o.n, gn.x, gn.y, gn.z);
    put3(o.wo, gw.x, gw.y, gw.z);
    put3(o.alb, g.alb.x, g.alb.y, g.alb.z);
    if (o.rough) o.rough[p] = (float)g.rough;
    if (o.metal) o.metal[p] = (float)g.metal;
}

hipError_t launch_render_shade_grad(const RenderArgs &a, const ShadeGradOut &o, hipStream_t st)
{
    const int64_t npix = (int64_t)a.H * a.W;
    if (npix <= 0) return hipSuccess;
    hipLaunchKernelGGL(k_render_shade_grad, dim3((unsigned)((npix + 255) / 256)), dim3(256), 0, st, a, o);
    return hipGetLastError();
}

template <int kLog>
__global__ void __launch_bounds__(256) k_render_reduce(int64_t npix, int spp, const float4 *__restrict__ contrib,
                                                       float *__restrict__ out)
{
    __shared__ ReduceTile<kLog> tile;
    reduce_pixels<kLog>(npix, spp, contrib, out, tile);
}

template <int kLog>
static void go_reduce(int64_t npix, int spp, const RenderArgs &a, hipStream_t st)
{
    const unsigned nb = (unsigned)((npix + kReducePixels<kLog> - 1) / kReducePixels<kLog>);
    hipLaunchKernelGGL(k_render_reduce<kLog>, dim3(nb), dim3(256), 0, st, npix, spp, a.contrib, a.out);
}

static hipError_t launch_reduce(const RenderArgs &a, hipStream_t st)
{
    const int64_t npix = (int64_t)a.H * a.W;
    const int spp = a.nc + a.ng + a.ne;
    switch (reduce_shape(npix, spp)) {
    case 0: go_reduce<0>(npix, spp, a, st); break;
    case 2: go_reduce<2>(npix, spp, a, st); break;
    default: go_reduce<kReduceOwn>(npix, spp, a, st);
    }
    return hipGetLastError();
}

template <int K, bool kHitList>
static hipError_t go_render_as(const RenderArgs &a, int num_cu, hipStream_t st)
{
    const int64_t total = (int64_t)a.H * a.W * (a.nc + a.ng + a.ne);
    const int nb = persistent_blocks(k_render<K, kHitList>, num_cu, total);
    hipLaunchKernelGGL((k_render<K, kHitList>), dim3(nb), dim3(256), 0, st, a);
    return hipGetLastError();
}

template <int K>
static hipError_t go_render(const RenderArgs &a, int num_cu, hipStream_t st)
{
    return a.hits ? go_render_as<K, true>(a, num_cu, st) : go_render_as<K, false>(a, num_cu, st);
}

template <int K, bool kOrigin>
static hipError_t go_render_bwd_as(const RenderArgs &a, int num_cu, hipStream_t st)
{
    const int64_t total = (int64_t)a.H * a.W * (a.nc + a.ng + a.ne);
    const int nb = persistent_blocks(k_render_bwd<K, kOrigin>, num_cu, total);
    hipLaunchKernelGGL((k_render_bwd<K, kOrigin>), dim3(nb), dim3(256), 0, st, a);
    return hipGetLastError();
}

// With origin gradients (the shading state's) 8 hits are the most that 3
// wavefronts per SIMD hold without spilling (164 VGPRs; 12 hits spill 9, 16
// hits 94), so larger buffers run 8: re-traversal alone, 500k surfels of a
// room, 320 x 320 x 16, 7.7 ms, with 12 hits 7.9, with 16 9.2 and with 16 at 2
// wavefronts, which do not spill, 8.6.  The last are the better only where a
// launch traces no more than the samples that overflowed long hit lists, so
// that few rays with many hits set its time: lists of 64 4.8 against 5.1, lists
// of 16 7.7 against 6.9.
constexpr int kLongList = 32;

template <int K>
static hipError_t go_render_bwd(const RenderArgs &a, int num_cu, hipStream_t st)
{
    if (!a.gorig) return go_render_bwd_as<K, false>(a, num_cu, st);
    if (K == 16 && !(a.hits && a.hcap >= kLongList)) return go_render_bwd_as<8, true>(a, num_cu, st);
    return go_render_bwd_as<K, true>(a, num_cu, st);
}

static hipError_t timer_mark(const KernelTimer *tm, bool end, hipStream_t st)
{
    return tm ? hipEventRecord(end ? tm->end : tm->begin, st) : hipSuccess;
}

hipError_t launch_render_backward_stored(const RenderArgs &a, const RenderWS &w, int k, int num_cu, hipStream_t st,
                                         const KernelTimer *tm)
{
    const int64_t nray = (int64_t)a.H * a.W * (a.nc + a.ng + a.ne);
    if (nray <= 0) return hipSuccess;
    hipError_t e = launch_zero_counters(a.counters, st);
    if (e != hipSuccess) return e;
    if ((e = launch_render_gen(a, st)) != hipSuccess) return e;
    if (a.order && (e = launch_ray_order(a, w, st)) != hipSuccess) return e;
    if ((e = timer_mark(tm, false, st)) != hipSuccess) return e;
    if (a.gorig)
        hipLaunchKernelGGL(k_render_bwd_stored<true>, dim3((unsigned)((nray + 255) / 256)), dim3(256), 0, st, a);
    else
        hipLaunchKernelGGL(k_render_bwd_stored<false>, dim3((unsigned)((nray + 255) / 256)), dim3(256), 0, st, a);
    if ((e = hipGetLastError()) != hipSuccess) return e;
    // samples whose list overflowed: re-traverse (the others return at once)
    RenderArgs b = a;
    b.order = nullptr;
    switch (k) {
    case 1: e = go_render_bwd<1>(b, num_cu, st); break;
    case 2: e = go_render_bwd<2>(b, num_cu, st); break;
    case 4: e = go_render_bwd<4>(b, num_cu, st); break;
    case 8: e = go_render_bwd<8>(b, num_cu, st); break;
    case 12:
    case 13:  // as 16, which fits the same registers: 143.3 to 139.0 ms with the forward (1M, 1024 x 1024 x 16)
    case 16: e = go_render_bwd<16>(b, num_cu, st); break;
    case 32: e = go_render_bwd<32>(b, num_cu, st); break;
    default: return hipErrorInvalidValue;
    }
    if (e != hipSuccess) return e;
    return timer_mark(tm, true, st);
}

hipError_t launch_render_gen(const RenderArgs &a, hipStream_t st)
{
    // (fewer than 2^31 samples: at most 2^25 + 65536 wavefronts)
    const int64_t npix = (int64_t)a.H * a.W;
    const int spp = a.nc + a.ng + a.ne;
    int lp = 0;
    while (lp < 6 && npix > (int64_t)1 << lp) ++lp;
    const int64_t waves = ((npix + (1 << lp) - 1) >> lp) * ((spp + (63 >> lp)) >> (6 - lp));
    hipLaunchKernelGGL(k_render_gen, dim3((unsigned)((waves + 3) / 4)), dim3(256), 0, st, a, lp);
    return hipGetLastError();
}

// ---- coherent traversal order ------------------------------------------------
// Samples of one pixel leave in all directions, so index order hands a
// wavefront 64 unrelated rays.  Sorting by (direction bin, origin cell) gives
// each wavefront rays that walk nearly the same nodes, which the per-XCD L2
// then serves.  The order changes only which lane traces which ray: every
// result is written at its sample index.

__device__ __forceinline__ uint32_t spread3(uint32_t x)  // 6 bits -> every third bit
{
    x &= 63u;
    x = (x | (x << 8)) & 0x0000F00Fu;
    x = (x | (x << 4)) & 0x000C30C3u;
    x = (x | (x << 2)) & 0x00249249u;
    return x;
}

__global__ void __launch_bounds__(256) k_ray_keys(RenderArgs a, int n, uint32_t *__restrict__ keys,
                                                  uint32_t *__restrict__ vals, uint32_t tag)
{
    const int r = blockIdx.x * blockDim.x + threadIdx.x;
    if (r >= n) return;
    const float4 r0 = a.rays[3 * (int64_t)r];
    uint32_t key = 0xFFFFFFu;  // untraced samples go last
    if (r0.w != 0.0f) {
        // scene root box from the two child boxes of node 0
        const Node nd = a.S.nodes[0];
        const float lx = fminf(nd.a.x, nd.b.z), ly = fminf(nd.a.y, nd.b.w), lz = fminf(nd.a.z, nd.c.x);
        const float hx = fmaxf(nd.a.w, nd.c.y), hy = fmaxf(nd.b.x, nd.c.z), hz = fmaxf(nd.b.y, nd.c.w);
        const int spp = a.nc + a.ng + a.ne;
        const int64_t p = (int64_t)r / spp;
        auto cell = [](float v, float lo, float hi) -> uint32_t {
            const float t = (v - lo) / fmaxf(hi - lo, 1e-20f) * 64.0f;
            return (uint32_t)fminf(fmaxf(t, 0.0f), 63.0f);
        };
        const uint32_t m = (spread3(cell(a.x[3 * p], lx, hx)) << 2) | (spread3(cell(a.x[3 * p + 1], ly, hy)) << 1) |
                           spread3(cell(a.x[3 * p + 2], lz, hz));
        // octahedral direction bin, 8 x 8
        const float s = fabsf(r0.x) + fabsf(r0.y) + fabsf(r0.z);
        float u = r0.x / s, v = r0.z / s;
        if (r0.y < 0.0f) {
            const float uu = (1.0f - fabsf(v)) * (u >= 0.0f ? 1.0f : -1.0f);
            const float vv = (1.0f - fabsf(u)) * (v >= 0.0f ? 1.0f : -1.0f);
            u = uu;
            v = vv;
        }
        const uint32_t iu = (uint32_t)fminf(fmaxf((u * 0.5f + 0.5f) * 8.0f, 0.0f), 7.0f);
        const uint32_t iv = (uint32_t)fminf(fmaxf((v * 0.5f + 0.5f) * 8.0f, 0.0f), 7.0f);
        key = ((iv * 8u + iu) << 18) | m;
    }
    keys[r] = key;
    vals[r] = tag | (uint32_t)r;
}

hipError_t launch_ray_keys(const RenderArgs &a, int n, uint32_t *keys, uint32_t *vals, uint32_t tag, hipStream_t st)
{
    if (n <= 0) return hipSuccess;
    hipLaunchKernelGGL(k_ray_keys, dim3((unsigned)((n + 255) / 256)), dim3(256), 0, st, a, n, keys, vals, tag);
    return hipGetLastError();
}

hipError_t launch_ray_order(const RenderArgs &a, const RenderWS &w, hipStream_t st)
{
    const int64_t n = (int64_t)a.H * a.W * (a.nc + a.ng + a.ne);
    if (n <= 0 || a.S.n < 2) return hipSuccess;
    hipLaunchKernelGGL(k_ray_keys, dim3((unsigned)((n + 255) / 256)), dim3(256), 0, st, a, (int)n, w.k0, w.v0, 0u);
    // 24-bit keys: three passes leave the order in (k1, v1)
    launch_radix_sort((int)n, 3, w.k0, w.v0, w.k1, w.v1, w.hist, st);
    return hipGetLastError();
}

hipError_t launch_render(const RenderArgs &a, const RenderWS &w, int k, int num_cu, hipStream_t st,
                         const KernelTimer *tm)
{
    const int64_t npix = (int64_t)a.H * a.W;
    if (npix <= 0) return hipSuccess;
    hipError_t e = launch_zero_counters(a.counters, st);
    if (e != hipSuccess) return e;
    if ((e = launch_render_gen(a, st)) != hipSuccess) return e;
    if (a.order && (e = launch_ray_order(a, w, st)) != hipSuccess) return e;
    if ((e = timer_mark(tm, false, st)) != hipSuccess) return e;
    switch (k) {
    case 1: e = go_render<1>(a, num_cu, st); break;
    case 2: e = go_render<2>(a, num_cu, st); break;
    case 4: e = go_render<4>(a, num_cu, st); break;
    case 8: e = go_render<8>(a, num_cu, st); break;
    case 12:  // 16 hits fit the same registers and take fewer rounds: 37.1 to 32.3 ms (1M, 512 x 512 x 32)
    case 16: e = go_render<16>(a, num_cu, st); break;
    case 32: e = go_render<32>(a, num_cu, st); break;
    default: return hipErrorInvalidValue;
    }
    if (e != hipSuccess) return e;
    if ((e = timer_mark(tm, true, st)) != hipSuccess) return e;
    return launch_reduce(a, st);
}

template <int K>
static hipError_t go_relight(const RenderArgs &a, int num_cu, hipStream_t st)
{
    const int64_t total = (int64_t)a.H * a.W * (a.nc + a.ng + a.ne);
    const int nb = persistent_blocks(k_render_relight<K>, num_cu, total);
    hipLaunchKernelGGL(k_render_relight<K>, dim3(nb), dim3(256), 0, st, a);
    return hipGetLastError();
}

hipError_t launch_render_relight(const RenderArgs &a, const RenderWS &w, int k, int num_cu, hipStream_t st)
{
    const int64_t npix = (int64_t)a.H * a.W;
    if (npix <= 0) return hipSuccess;
    hipError_t e = launch_zero_counters(a.counters, st);
    if (e != hipSuccess) return e;
    if ((e = launch_render_gen(a, st)) != hipSuccess) return e;
    if (a.order && (e = launch_ray_order(a, w, st)) != hipSuccess) return e;
    switch (k) {
    case 1: e = go_relight<1>(a, num_cu, st); break;
    case 2: e = go_relight<2>(a, num_cu, st); break;
    case 4: e = go_relight<4>(a, num_cu, st); break;
    case 8: e = go_relight<8>(a, num_cu, st); break;
    case 12:  // 16 hits fit the same registers and take fewer rounds: 26.7 to 23.9 ms (1M, 512 x 512 x 16)
    case 16: e = go_relight<16>(a, num_cu, st); break;
    case 32: e = go_relight<32>(a, num_cu, st); break;
    default: return hipErrorInvalidValue;
    }
    if (e != hipSuccess) return e;
    const int64_t total = npix * (a.nc + a.ng + a.ne);
    hipLaunchKernelGGL(k_relight_shade, dim3((unsigned)((total + 255) / 256)), dim3(256), 0, st, a, total);
    return launch_reduce(a, st);
}

hipError_t launch_relight_shade(const RenderArgs &a, hipStream_t st)
{
    const int64_t total = (int64_t)a.H * a.W * (a.nc + a.ng + a.ne);
    if (total <= 0) return hipSuccess;
    hipLaunchKernelGGL(k_relight_shade, dim3((unsigned)((total + 255) / 256)), dim3(256), 0, st, a, total);
    return hipGetLastError();
}

hipError_t launch_render_relight_mesh(const RenderArgs &a, const MeshTraceArgs &m, hipStream_t st)
{
    const int64_t npix = (int64_t)a.H * a.W;
    if (npix <= 0) return hipSuccess;
    hipError_t e = launch_render_gen(a, st);
    if (e != hipSuccess) return e;
    if ((e = launch_mesh_relight_query(a, m, st)) != hipSuccess) return e;
    const int64_t total = npix * (a.nc + a.ng + a.ne);
    hipLaunchKernelGGL(k_relight_shade, dim3((unsigned)((total + 255) / 256)), dim3(256), 0, st, a, total);
    return launch_reduce(a, st);
}

hipError_t launch_render_backward(const RenderArgs &a, const RenderWS &w, int k, int num_cu, hipStream_t st,
                                  const KernelTimer *tm)
{
    if ((int64_t)a.H * a.W <= 0) return hipSuccess;
    hipError_t e = launch_zero_counters(a.counters, st);
    if (e != hipSuccess) return e;
    if ((e = launch_render_gen(a, st)) != hipSuccess) return e;
    if (a.order && (e = launch_ray_order(a, w, st)) != hipSuccess) return e;
    if ((e = timer_mark(tm, false, st)) != hipSuccess) return e;
    switch (k) {
    case 1: e = go_render_bwd<1>(a, num_cu, st); break;
    case 2: e = go_render_bwd<2>(a, num_cu, st); break;
    case 4: e = go_render_bwd<4>(a, num_cu, st); break;
    case 8: e = go_render_bwd<8>(a, num_cu, st); break;
    case 12:
    case 13:  // as 16, which fits the same registers: 143.3 to 139.0 ms with the forward (1M, 1024 x 1024 x 16)
    case 16: e = go_render_bwd<16>(a, num_cu, st); break;
    case 32: e = go_render_bwd<32>(a, num_cu, st); break;
    default: return hipErrorInvalidValue;
    }
    if (e != hipSuccess) return e;
    return timer_mark(tm, true, st);
}

bool walk_stats_built()
{
#ifdef GRT_STATS
    return true;
#else
    return false;
#endif
}

hipError_t walk_stats_read(unsigned long long *out, bool reset)
{
#ifdef GRT_STATS
    hipError_t e = hipMemcpyFromSymbol(out, HIP_SYMBOL(g_walk_stats), sizeof(g_walk_stats));
    if (e == hipSuccess && reset) {
        unsigned long long zero[2][kNumWalkStats] = {};
        e = hipMemcpyToSymbol(HIP_SYMBOL(g_walk_stats), zero, sizeof(zero));
    }
    return e;
#else
    (void)out;
    (void)reset;
    return hipErrorNotSupported;
#endif
}

}  // namespace grt
