// scene.hip -- surfel records and BVH construction on the GPU.
//
// The paper bounds each 2D Gaussian by an adaptive icosahedron whose radius
// sqrt(2 ln(o / alpha_min)) shrinks with opacity, and indexes the proxies with
// a BVH (Sec. 3.2, Eq. icosahedron_transform).  Here the proxy is the
// axis-aligned box of the ellipse rho <= min(3, sqrt(2 ln(o / alpha_min))), and
// the BVH is built over the Morton order in five steps, all on the caller's stream:
//   1. scene bounds of the box centres         (k_bounds, ordered-int atomics)
//   2. 30-bit Morton codes of the centres      (k_morton)
//   3. stable LSD radix sort, 4 passes x 8 bit (k_radix_hist/scan/scatter)
//   4. records and boxes in sorted order       (k_records)
//   5. binary hierarchy by clustering          (k_cluster)
// and collapsed to the 4-wide nodes the traversal walks (k_collapse_*).
#include <algorithm>

#include "grt_internal.h"

namespace grt {


// support bound rho^2 <= min(9, 2 ln(o / alpha_min)), evaluated in double and
// rounded once, so it does not depend on the math library's last ulp
__device__ __forceinline__ float support_r2(float op, float alpha_min)
{
    if (!(alpha_min > 0.0f)) return 9.0f;
    double b = 2.0 * log((double)op / (double)alpha_min);
    return (float)(b < 9.0 ? b : 9.0);
}

__global__ void k_init(int32_t *bounds)
{
    if (threadIdx.x < 3) bounds[threadIdx.x] = 0x7fffffff;            // min of centres
    else if (threadIdx.x < 6) bounds[threadIdx.x] = (int32_t)0x80000000;  // max of centres
}

// Bounds of the surfel centres: at most 512 blocks, so that few atomics meet
// on the six words.
__global__ void __launch_bounds__(256) k_bounds(int n, const float *__restrict__ means, int32_t *__restrict__ bounds)
{
    float c[3] = {INFINITY, INFINITY, INFINITY}, C[3] = {-INFINITY, -INFINITY, -INFINITY};
    for (int i = blockIdx.x * blockDim.x + threadIdx.x; i < n; i += (int)(gridDim.x * blockDim.x))
#pragma unroll
        for (int a = 0; a < 3; ++a) {
            const float mu = means[3 * (size_t)i + a];
            c[a] = fminf(c[a], mu);
            C[a] = fmaxf(C[a], mu);
        }
    __shared__ float red[4][6];
#pragma unroll
    for (int a = 0; a < 3; ++a)
        for (int m = 32; m >= 1; m >>= 1) {
            c[a] = fminf(c[a], __shfl_xor(c[a], m, 64));
            C[a] = fmaxf(C[a], __shfl_xor(C[a], m, 64));
        }
    if ((threadIdx.x & 63) == 0)
#pragma unroll
        for (int a = 0; a < 3; ++a) {
            red[threadIdx.x >> 6][a] = c[a];
            red[threadIdx.x >> 6][3 + a] = C[a];
        }
    __syncthreads();
    const int t = threadIdx.x;
    if (t < 3) atomicMin(&bounds[t], f2o(fminf(fminf(red[0][t], red[1][t]), fminf(red[2][t], red[3][t]))));
    else if (t < 6) atomicMax(&bounds[t], f2o(fmaxf(fmaxf(red[0][t], red[1][t]), fmaxf(red[2][t], red[3][t]))));
}

// Padded box of a surfel's support ellipse.
__device__ __forceinline__ void surfel_box(float3 tu, float3 tv, float su, float sv, float r2, const float *mean,
                                           float *box)
{
    const float r = r2 > 0.0f ? sqrtf(r2) * 1.00001f : 0.0f;
    const float tuv[3][2] = {{tu.x, tv.x}, {tu.y, tv.y}, {tu.z, tv.z}};
#pragma unroll
    for (int a = 0; a < 3; ++a) {
        const float x = su * tuv[a][0], y = sv * tuv[a][1];
        const float e = r * sqrtf(x * x + y * y) + kPad;
        box[a] = mean[a] - e;
        box[3 + a] = mean[a] + e;
    }
}

__device__ __forceinline__ uint32_t spread_bits(uint32_t v)
{
    v &= 0x3ffu;
    v = (v | (v << 16)) & 0x030000FFu;
    v = (v | (v << 8)) & 0x0300F00Fu;
    v = (v | (v << 4)) & 0x030C30C3u;
    v = (v | (v << 2)) & 0x09249249u;
    return v;
}

__global__ void k_morton(int n, const float *__restrict__ means, const int32_t *__restrict__ bounds,
                         uint32_t *__restrict__ keys, uint32_t *__restrict__ vals)
{
    int i = blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= n) return;
    uint32_t q[3];
#pragma unroll
    for (int a = 0; a < 3; ++a) {
        float lo = o2f(bounds[a]), hi = o2f(bounds[3 + a]);
        float ext = hi - lo;
        float f = ext > 0.0f ? (means[3 * i + a] - lo) / ext : 0.0f;
        int v = (int)floorf(f * 1024.0f);
        q[a] = (uint32_t)min(max(v, 0), 1023);
    }
    keys[i] = (spread_bits(q[0]) << 2) | (spread_bits(q[1]) << 1) | spread_bits(q[2]);
    vals[i] = (uint32_t)i;
}

// ---- stable LSD radix sort, 8-bit digits -----------------------------------

// Per-tile digit counts, stored digit-major: hist[digit * blocks + tile].
__global__ void __launch_bounds__(kSortThreads) k_radix_hist(int n, const uint32_t *__restrict__ keys, int shift,
                                                             uint32_t *__restrict__ hist)
{
    __shared__ uint32_t h[256];
    h[threadIdx.x] = 0;
    __syncthreads();
    int base = blockIdx.x * kSortTile;
#pragma unroll 4
    for (int r = 0; r < kSortItems; ++r) {
        int i = base + r * kSortThreads + threadIdx.x;
        if (i < n) atomicAdd(&h[(keys[i] >> shift) & 255u], 1u);
    }
    __syncthreads();
    hist[threadIdx.x * gridDim.x + blockIdx.x] = h[threadIdx.x];
}

// Exclusive prefix sum over the digit-major histogram (one block): tiles of
// four words a thread, read and written in order, the running total carried
// from tile to tile.
__global__ void __launch_bounds__(1024) k_radix_scan(int total, uint32_t *__restrict__ hist)
{
    __shared__ uint32_t wsum[16];
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    uint32_t carry = 0;
    for (int base = 0; base < total; base += 4096) {
        const int i = base + 4 * (int)threadIdx.x;
        uint32_t v[4];
#pragma unroll
        for (int j = 0; j < 4; ++j) v[j] = i + j < total ? hist[i + j] : 0u;
        const uint32_t own = v[0] + v[1] + v[2] + v[3];
        uint32_t x = own;  // inclusive over the wavefront
#pragma unroll
        for (int off = 1; off < 64; off <<= 1) {
            const uint32_t y = __shfl_up(x, off, 64);
            if (lane >= off) x += y;
        }
        if (lane == 63) wsum[wave] = x;
        __syncthreads();
        uint32_t before = carry, all = carry;
#pragma unroll
        for (int w = 0; w < 16; ++w) {
            const uint32_t t = wsum[w];
            before += w < wave ? t : 0u;
            all += t;
        }
        uint32_t run = before + x - own;
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            if (i + j < total) hist[i + j] = run;
            run += v[j];
        }
        carry = all;
        __syncthreads();
    }
}

// The same exclusive prefix sum for long histograms (the sort of a frame's
// samples): per-chunk sums, a scan of the sums, then each chunk rescanned
// from its offset.  kScanChunk entries per block, 16 per thread.
constexpr int kScanChunk = 4096;
// Up to this many chunks one block scans them in turn (about 1.5 us each),
// beyond it three launches of about 5 us do.
constexpr int kScanOneBlock = 6;

__global__ void __launch_bounds__(256) k_scan_sums(int total, const uint32_t *__restrict__ hist,
                                                   uint32_t *__restrict__ sums)
{
    __shared__ uint32_t part[256];
    const int base = blockIdx.x * kScanChunk + threadIdx.x * 16;
    uint32_t acc = 0;
#pragma unroll
    for (int i = 0; i < 16; ++i)
        if (base + i < total) acc += hist[base + i];
    part[threadIdx.x] = acc;
    __syncthreads();
    for (int off = 128; off > 0; off >>= 1) {
        if (threadIdx.x < off) part[threadIdx.x] += part[threadIdx.x + off];
        __syncthreads();
    }
    if (threadIdx.x == 0) sums[blockIdx.x] = part[0];
}

__global__ void __launch_bounds__(256) k_scan_apply(int total, uint32_t *__restrict__ hist,
                                                    const uint32_t *__restrict__ sums)
{
    __shared__ uint32_t part[256];
    const int base = blockIdx.x * kScanChunk + threadIdx.x * 16;
    uint32_t v[16], acc = 0;
#pragma unroll
    for (int i = 0; i < 16; ++i) {
        v[i] = base + i < total ? hist[base + i] : 0u;
        acc += v[i];
    }
    part[threadIdx.x] = acc;
    __syncthreads();
    for (int off = 1; off < 256; off <<= 1) {  // inclusive scan of the thread sums
        const uint32_t x = threadIdx.x >= off ? part[threadIdx.x - off] : 0u;
        __syncthreads();
        part[threadIdx.x] += x;
        __syncthreads();
    }
    uint32_t run = sums[blockIdx.x] + part[threadIdx.x] - acc;
#pragma unroll
    for (int i = 0; i < 16; ++i) {
        if (base + i < total) hist[base + i] = run;
        run += v[i];
    }
}

// Scatter with ranks that follow the input order inside the tile: each round
// of 256 keys is ranked per wavefront by matching digits bit by bit with
// ballots, then across the four wavefronts of the block through LDS.
__global__ void __launch_bounds__(kSortThreads) k_radix_scatter(int n, const uint32_t *__restrict__ kin,
                                                                const uint32_t *__restrict__ vin,
                                                                uint32_t *__restrict__ kout,
                                                                uint32_t *__restrict__ vout, int shift,
                                                                const uint32_t *__restrict__ hist)
{
    __shared__ uint32_t run[256];
    __shared__ uint32_t wcnt[4][256];
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    run[tid] = hist[tid * gridDim.x + blockIdx.x];
    const uint64_t lt = (lane == 0) ? 0ull : (~0ull >> (64 - lane));
    const int base = blockIdx.x * kSortTile;
    for (int r = 0; r < kSortItems; ++r) {
        int i = base + r * kSortThreads + tid;
        bool valid = i < n;
        uint32_t key = valid ? kin[i] : 0u;
        uint32_t val = valid ? vin[i] : 0u;
        uint32_t dig = (key >> shift) & 255u;
        uint64_t peers = __ballot(valid);
#pragma unroll
        for (int b = 0; b < 8; ++b) {
            bool bit = (dig >> b) & 1u;
            uint64_t m = __ballot(bit);
            peers &= bit ? m : ~m;
        }
        uint32_t rank = (uint32_t)__popcll(peers & lt);
#pragma unroll
        for (int w = 0; w < 4; ++w) wcnt[w][tid] = 0u;
        __syncthreads();
        if (valid && rank == 0) wcnt[wave][dig] = (uint32_t)__popcll(peers);
        __syncthreads();
        if (valid) {
            uint32_t p = run[dig] + rank;
            for (int w = 0; w < wave; ++w) p += wcnt[w][dig];
            kout[p] = key;
            vout[p] = val;
        }
        __syncthreads();
        run[tid] += wcnt[0][tid] + wcnt[1][tid] + wcnt[2][tid] + wcnt[3][tid];
        __syncthreads();
    }
}

// ---- records in sorted order ---------------------------------------------------

__global__ void k_records(int n, const uint32_t *__restrict__ order, const float *__restrict__ means,
                          const float *__restrict__ scales, const float *__restrict__ quats,
                          const float *__restrict__ opacity, const float *__restrict__ rgb, float alpha_min,
                          float4 *__restrict__ rec, float4 *__restrict__ col, float *__restrict__ leaf_box,
                          float4 *__restrict__ qrec)
{
#pragma clang fp contract(off)
    int p = blockIdx.x * blockDim.x + threadIdx.x;
    if (p >= n) return;
    uint32_t id = order[p];
    float3 tu, tv, nn;
    const float4 q = reinterpret_cast<const float4 *>(quats)[id];  // (16-byte aligned, checked at creation)
    frame32(q.x, q.y, q.z, q.w, tu, tv, nn);
    float su = scales[2 * id], sv = scales[2 * id + 1];
    float op = opacity[id];
    const float mu[3] = {means[3 * id], means[3 * id + 1], means[3 * id + 2]};
    const float r2 = support_r2(op, alpha_min);
    rec[4 * (size_t)p + 0] = make_float4(mu[0], mu[1], mu[2], r2);
    rec[4 * (size_t)p + 1] = make_float4(nn.x, nn.y, nn.z, op);
    rec[4 * (size_t)p + 2] = make_float4(tu.x / su, tu.y / su, tu.z / su, __uint_as_float(id));
    rec[4 * (size_t)p + 3] = make_float4(tv.x / sv, tv.y / sv, tv.z / sv, su);
    col[p] = make_float4(rgb[3 * id], rgb[3 * id + 1], rgb[3 * id + 2], sv);
    qrec[p] = q;
    surfel_box(tu, tv, su, sv, r2, mu, leaf_box + 6 * (size_t)p);
}

// ---- hierarchy ----------------------------------------------------------------

__device__ __forceinline__ float box_area(const float *b)
{
    const float dx = b[3] - b[0], dy = b[4] - b[1], dz = b[5] - b[2];
    return dx * dy + dy * dz + dz * dx;
}

// Binary hierarchy by parallel locally-ordered clustering (Meister and Bittner,
// TVCG 2018): in the Morton order, each cluster names the neighbour within
// kClusterRadius places with which it has the smallest common box, and pairs
// that name each other become a node, which takes the place of the first.
//
// A block keeps kClusterBlock consecutive clusters in LDS and repeats that
// until an eighth is left, so one launch takes the whole array three levels
// up; the last launch, of one block, goes on to the root.  Clusters at a
// block's edge find fewer partners, but an eighth of a block need find none:
// counted on 1M surfels, rays visit as many nodes as with clustering over the
// whole array.  A block's merges are as many as it has clusters to lose, so
// the place of every node is known beforehand: nodes are numbered down from
// n - 2 in the order they are made, and the root is 0.
//
// Height: the walks' stacks take 63 levels.  Free merges stay within `cap`;
// when a pass made no merge, or after kClusterIters passes, each cluster is
// joined with its neighbour, which halves their number: at most 3 such passes
// (kClusterForced in the last launch), so the caps of the launches are 3 apart
// and end at 63 - kClusterForced.  (A room of 1M surfels: 36 levels, about 13
// passes a launch.)
//
// In that room a ray visits 28% fewer nodes than in the hierarchy of the
// codes' common prefixes (164 -> 118; up to the stop depth 128 -> 92), with
// which a training step of 16.8M rays took 170 ms and takes 157, a relit frame
// of 4.2M 23.4 and 21.8, the mesh query of 33.5M 9.9 and 9.3; scattered
// surfels gain nothing.  The build is 0.72 ms instead of 0.57.  Bound by the
// latency of a pass (barriers, LDS): blocks of 1024 0.88, of 256 0.77; radius
// 4 0.73 with 1-2% slower walks, 7 0.83 and 10 1.0 with none faster.
constexpr int kClusterRadius = 5, kClusterIters = 40;
constexpr int kClusterForced = 9;  // passes that halve the clusters of a block to one
static_assert(kClusterShrink == 8 && (1 << kClusterForced) == kClusterBlock, "forced passes of a launch");

// Clusters of one launch's input or output: the box and, after the first
// launch, the node, its number of leaves and its height.
struct ClusterList {
    float *box;     // [6 c]
    int2 *ref;      // [c] node, leaves (null: leaf i, 1 leaf)
    uint8_t *high;  // [c]
};

__global__ void __launch_bounds__(kClusterBlock) k_cluster(int n, int count, ClusterList in, ClusterList out, int cap,
                                                           Node *__restrict__ nodes, uint32_t *__restrict__ mark)
{
    __shared__ float4 box0[kClusterBlock];  // lo xyz, hi x
    __shared__ float2 box1[kClusterBlock];  // hi yz
    __shared__ int ref[kClusterBlock], leaves[kClusterBlock], high[kClusterBlock], near[kClusterBlock];
    __shared__ uint32_t wsum[kClusterBlock / 64];
    const int t = threadIdx.x, lane = t & 63, wave = __builtin_amdgcn_readfirstlane(t >> 6);
    const uint64_t below = lane ? ~0ull >> (64 - lane) : 0ull;
    const int64_t at = (int64_t)blockIdx.x * kClusterBlock;
    int m = (int)(count - at < kClusterBlock ? count - at : kClusterBlock);  // clusters left
    const int target = count <= kClusterBlock ? 1 : (m + kClusterShrink - 1) / kClusterShrink;
    // number of the block's first node: the merges of earlier launches, then of earlier blocks
    int id = n - 2 - (n - count) - (int)blockIdx.x * (kClusterBlock - kClusterBlock / kClusterShrink);
    if (t < m) {
        const float *b = in.box + 6 * (at + t);
        box0[t] = make_float4(b[0], b[1], b[2], b[3]);
        box1[t] = make_float2(b[4], b[5]);
        const int2 r = in.ref ? in.ref[at + t] : make_int2(-(int)(at + t) - 1, 1);
        ref[t] = r.x;
        leaves[t] = r.y;
        high[t] = in.ref ? in.high[at + t] : 0;
    }
    __syncthreads();
    bool stuck = false;
    for (int pass = 0; m > target; ++pass) {
        // a single wavefront's clusters need no barrier (the others wait below)
        const bool alone = m <= 64;
        if (alone && wave) break;
        const auto sync = [&]() {
            if (alone) wave_sync();
            else __syncthreads();
        };
        // number of the pairs and (upper half) of the merged clusters before
        // this one, and in all
        const auto before = [&](uint64_t pairs, uint64_t lost, uint32_t &all) {
            if (lane == 0) wsum[wave] = __popcll(pairs) | __popcll(lost) << 16;
            sync();
            uint32_t x = __popcll(pairs & below) | __popcll(lost & below) << 16;
            all = wsum[0];
            if (alone) return x;
#pragma unroll
            for (int w = 1; w < kClusterBlock / 64; ++w) {
                x += wave >= w ? wsum[w - 1] : 0u;
                all += wsum[w];
            }
            return x;
        };
        const bool force = stuck || pass >= kClusterIters;
        const bool on = t < m;
        int best = -1;
        float4 b0 = make_float4(0.f, 0.f, 0.f, 0.f);
        float2 b1 = make_float2(0.f, 0.f);
        if (on) {
            b0 = box0[t];
            b1 = box1[t];
            if (force) {
                best = (t ^ 1) < m ? t ^ 1 : -1;
            } else {
                // equal areas go to the neighbour t ^ 1, then to the lowest: of
                // the closest pairs of all, one is mutual
                float least = INFINITY;
#pragma unroll
                for (int k = 0; k < 2 * kClusterRadius; ++k) {
                    const int j = t + (k < kClusterRadius ? k - kClusterRadius : k - kClusterRadius + 1);
                    const int jj = min(max(j, 0), m - 1);
                    const float4 v0 = box0[jj];
                    const float2 v1 = box1[jj];
                    const float u[6] = {fminf(b0.x, v0.x), fminf(b0.y, v0.y), fminf(b0.z, v0.z),
                                        fmaxf(b0.w, v0.w), fmaxf(b1.x, v1.x), fmaxf(b1.y, v1.y)};
                    const float area = box_area(u);
                    if (j == jj && (area < least || (area == least && j == (t ^ 1)))) {
                        least = area;
                        best = j;
                    }
                }
            }
            near[t] = best;
        }
        sync();
        int r = 0, l = 0, h = 0, pl = 0, pr = 0;
        float4 v0 = b0;
        float2 v1 = b1;
        bool pair = false, gone = false;
        if (on) {
            r = ref[t];
            l = leaves[t];
            h = high[t];
            if (best >= 0 && near[best] == t && (force || max(h, high[best]) < cap)) {
                pair = best > t;
                gone = !pair;
                v0 = box0[best];
                v1 = box1[best];
                pr = ref[best];
                pl = leaves[best];
                h = max(h, high[best]) + 1;
            }
        }
        uint32_t all;
        uint32_t x = before(__ballot(pair), __ballot(gone), all);
        const int npairs = (int)(all & 0xffffu), rank = (int)(x & 0xffffu), made = min(npairs, m - target);
        if (made < npairs) {  // more pairs than the block may lose: the first of them
            if (pair && rank >= made) {
                near[best] = -2;
                pair = false;
                h = high[t];
            }
            sync();
            if (gone && near[t] == -2) {
                gone = false;
                h = high[t];
            }
            x = before(0, __ballot(gone), all);
        }
        const int to = t - (int)(x >> 16);
        if (pair) {
            Node nd;
            nd.a = make_float4(b0.x, b0.y, b0.z, b0.w);
            nd.b = make_float4(b1.x, b1.y, v0.x, v0.y);
            nd.c = make_float4(v0.z, v0.w, v1.x, v1.y);
            l += pl;
            nd.d = make_int4(r, pr, l, 0);
            r = id - rank;
            nodes[r] = nd;
            if (mark) mark[r] = 0u;  // of the collapse to 4-wide nodes
            b0 = make_float4(fminf(b0.x, v0.x), fminf(b0.y, v0.y), fminf(b0.z, v0.z), fmaxf(b0.w, v0.w));
            b1 = make_float2(fmaxf(b1.x, v1.x), fmaxf(b1.y, v1.y));
        }
        if (on && !gone) {
            box0[to] = b0;
            box1[to] = b1;
            ref[to] = r;
            leaves[to] = l;
            high[to] = h;
        }
        id -= made;
        m -= made;
        stuck = made == 0;
        sync();
    }
    __syncthreads();
    if (count > kClusterBlock && t < target) {
        const int64_t o = (int64_t)blockIdx.x * (kClusterBlock / kClusterShrink) + t;
        const float4 b0 = box0[t];
        const float2 b1 = box1[t];
        const float b[6] = {b0.x, b0.y, b0.z, b0.w, b1.x, b1.y};
#pragma unroll
        for (int a = 0; a < 6; ++a) out.box[6 * o + a] = b[a];
        out.ref[o] = make_int2(ref[t], leaves[t]);
        out.high[o] = (uint8_t)high[t];
    }
    if (count <= kClusterBlock && t == 0 && mark) mark[n - 1] = 0u;  // the word past the nodes' (the scan takes n)
}

// ---------------------------------------------------------------------------
// The 4-wide hierarchy the traversal walks, collapsed top down from the
// binary one.  A 4-wide node starts from a binary node's two children and
// twice opens the internal child of largest surface area (replacing it by its
// two children), so it has 2..4 children; its internal children are the binary
// nodes that further 4-wide nodes start from.  Which binary nodes those are is
// decided from the root down and marked: one block expands the top level by
// level until a level is wide enough to give every wavefront of the second
// launch a part of it, and those mark the subtrees below, each in a part of
// the queue as long as its subtree, so no wavefront waits for another.  A
// prefix sum over the marks then numbers the 4-wide nodes in the order of
// their binary nodes (neighbours stay neighbours; the root is number 0), and
// every node is written at once.  1M surfels: 0.92 ms with a launch per level
// and 64 more to advance the level's range, 0.33 ms with nodes numbered by one
// counter (4,096 wavefronts met on it).
// ---------------------------------------------------------------------------
constexpr int kCollapseTop = 1024;   // threads of the first launch
constexpr int kCollapseWide = 2048;  // level width handed to the second
constexpr int kCollapseWaves = 4096;

struct Collapsed {
    float box[4][6];
    int ref[4];  // binary node >= 0, leaf -(pos+1)
    int m;       // children
};

__device__ __forceinline__ Collapsed collapse_node(const Node *__restrict__ bin, int node)
{
    Collapsed c;
    const float *w = reinterpret_cast<const float *>(&bin[node]);
    const int4 ch = bin[node].d;
#pragma unroll
    for (int a = 0; a < 6; ++a) {
        c.box[0][a] = w[a];
        c.box[1][a] = w[6 + a];
        c.box[2][a] = c.box[3][a] = 0.0f;
    }
    c.ref[0] = ch.x;
    c.ref[1] = ch.y;
    c.ref[2] = c.ref[3] = kNoChild;
    c.m = 2;
#pragma unroll
    for (int e = 0; e < 2; ++e) {
        int best = -1;
        float ba = -1.0f;
#pragma unroll
        for (int j = 0; j < 3; ++j)
            if (j < c.m && c.ref[j] >= 0) {
                const float ar = box_area(c.box[j]);
                if (best < 0 || ar > ba) { ba = ar; best = j; }
            }
        if (best < 0) break;
        const int open = best == 0 ? c.ref[0] : best == 1 ? c.ref[1] : c.ref[2];
        const float *v = reinterpret_cast<const float *>(&bin[open]);
        const int4 d = bin[open].d;
        float l[6], r[6];
#pragma unroll
        for (int a = 0; a < 6; ++a) { l[a] = v[a]; r[a] = v[6 + a]; }
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            const bool first = j == best, second = j == c.m;
            c.ref[j] = first ? d.x : second ? d.y : c.ref[j];
#pragma unroll
            for (int a = 0; a < 6; ++a) c.box[j][a] = first ? l[a] : second ? r[a] : c.box[j][a];
        }
        ++c.m;
    }
    return c;
}

__device__ __forceinline__ int internal_children(const Collapsed &c)
{
    int k = 0;
#pragma unroll
    for (int j = 0; j < 4; ++j) k += (j < c.m && c.ref[j] >= 0) ? 1 : 0;
    return k;
}

// Queues and marks the internal children of a 4-wide node.
__device__ __forceinline__ void queue_children(const Collapsed &c, int32_t *q, uint32_t *mark)
{
#pragma unroll
    for (int j = 0; j < 4; ++j)
        if (j < c.m && c.ref[j] >= 0) {
            *q++ = c.ref[j];
            mark[c.ref[j]] = 1u;
        }
}

// Writes the 4-wide nodes; num: the marks' exclusive prefix sum, so binary
// node i is marked where it steps up behind i.
__global__ void __launch_bounds__(256) k_collapse_write(int n, const Node *__restrict__ bin,
                                                        const uint32_t *__restrict__ num, int32_t *__restrict__ ctl,
                                                        Node4 *out, NodeQ *__restrict__ outq)
{
    const int i = blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= n - 1) return;
    const uint32_t at = num[i], behind = num[i + 1];
    if (i == n - 2) ctl[2] = (int32_t)behind;
    if (at == behind) return;
    Collapsed c = collapse_node(bin, i);
#pragma unroll
    for (int j = 0; j < 4; ++j)
        if (j < c.m && c.ref[j] >= 0) c.ref[j] = (int)num[c.ref[j]];
    Node4 o;
    o.lx = make_float4(c.box[0][0], c.box[1][0], c.box[2][0], c.box[3][0]);
    o.ly = make_float4(c.box[0][1], c.box[1][1], c.box[2][1], c.box[3][1]);
    o.lz = make_float4(c.box[0][2], c.box[1][2], c.box[2][2], c.box[3][2]);
    o.hx = make_float4(c.box[0][3], c.box[1][3], c.box[2][3], c.box[3][3]);
    o.hy = make_float4(c.box[0][4], c.box[1][4], c.box[2][4], c.box[3][4]);
    o.hz = make_float4(c.box[0][5], c.box[1][5], c.box[2][5], c.box[3][5]);
    o.ch = make_int4(c.ref[0], c.ref[1], c.ref[2], c.ref[3]);
    o.pad = make_int4(c.m, 0, 0, 0);
    if (out) out[at] = o;
    outq[at] = quantize_node(c.box, c.ref, c.m);
}

// inclusive prefix sum over the wavefront
__device__ __forceinline__ int wave_scan(int x)
{
    const int lane = threadIdx.x & 63;
#pragma unroll
    for (int off = 1; off < 64; off <<= 1) {
        const int y = __shfl_up(x, off, 64);
        if (lane >= off) x += y;
    }
    return x;
}

// Sum of x over the block's threads before this one; the block's total in all.
__device__ __forceinline__ int block_before(int x, int *wsum, int &all)
{
    const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63;
    const int incl = wave_scan(x);
    if (lane == 63) wsum[wave] = incl;
    __syncthreads();
    int before = 0;
    all = 0;
    for (int w = 0; w < kCollapseTop / 64; ++w) {
        before += w < wave ? wsum[w] : 0;
        all += wsum[w];
    }
    __syncthreads();
    return before + incl - x;
}

// queue: the levels one after the other.  part: for each node of the level
// handed on, where its subtree's part of the queue begins (the internal nodes
// below it, one fewer than its leaves less itself; with the queue's levels, at
// most the n - 1 binary nodes).  ctl: that level's range.
__global__ void __launch_bounds__(kCollapseTop) k_collapse_top(const Node *__restrict__ bin, int32_t *queue,
                                                               uint32_t *mark, uint32_t *part, int32_t *ctl)
{
    __shared__ int wsum[kCollapseTop / 64];
    if (threadIdx.x == 0) {
        queue[0] = 0;
        mark[0] = 1u;
    }
    int lo = 0, hi = 1, next = 1;  // the level's range, nodes queued so far
    __syncthreads();
    while (lo < hi && hi - lo < kCollapseWide) {
        for (int base = lo; base < hi; base += kCollapseTop) {
            const int i = base + (int)threadIdx.x;
            Collapsed c;
            int k = 0, all;
            if (i < hi) {
                c = collapse_node(bin, queue[i]);
                k = internal_children(c);
            }
            const int before = block_before(k, wsum, all);
            if (i < hi) queue_children(c, queue + next + before, mark);
            next += all;
        }
        lo = hi;
        hi = next;
        __syncthreads();  // the level's entries, before they are read
    }
    for (int base = lo; base < hi; base += kCollapseTop) {
        const int i = base + (int)threadIdx.x;
        int all;
        const int before = block_before(i < hi ? bin[queue[i]].d.z - 2 : 0, wsum, all);
        if (i < hi) part[i - lo] = (uint32_t)(next + before);
        next += all;
    }
    if (threadIdx.x == 0) {
        ctl[0] = lo;
        ctl[1] = hi;
    }
}

// One wavefront per piece of the level that the top left: it keeps the ranges
// of queued nodes still to expand on a stack, takes up to 64 of the topmost at
// a time and queues their children.  The rest of a range stays below its
// children's, so the stack holds at most one range for each 4-wide level
// below, fewer than 64.
__global__ void __launch_bounds__(256) k_collapse_subtrees(const Node *__restrict__ bin, int32_t *queue, uint32_t *mark,
                                                           const uint32_t *__restrict__ part,
                                                           const int32_t *__restrict__ ctl)
{
    __shared__ int2 stacks[4][72];
    const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63;
    int2 *stack = stacks[wave];
    const int64_t w = (int64_t)blockIdx.x * 4 + wave;
    const int lo = ctl[0], width = ctl[1] - lo;
    const int beg = (int)(width * w / kCollapseWaves), end = (int)(width * (w + 1) / kCollapseWaves);
    if (beg >= end) return;
    int next = (int)part[beg], sp = 0;
    int2 cur = make_int2(lo + beg, lo + end);  // wavefront-uniform
    while (cur.x < cur.y || sp > 0) {
        if (cur.x >= cur.y) {
            cur = stack[--sp];
            continue;
        }
        const int i = cur.x + lane;
        const bool on = i < cur.y;
        Collapsed c;
        int k = 0;
        if (on) {
            c = collapse_node(bin, queue[i]);
            k = internal_children(c);
        }
        const int incl = wave_scan(k);
        const int all = __shfl(incl, 63, 64);
        if (on) queue_children(c, queue + next + incl - k, mark);
        if (cur.x + 64 < cur.y) {
            if (lane == 0) stack[sp] = make_int2(cur.x + 64, cur.y);
            ++sp;
        }
        cur = make_int2(next, next + all);
        next += all;
        // the lanes' entries of the queue and the stack, before another lane reads them
        wave_sync(true);
    }
}

// Exclusive prefix sum of a long array in place; sums: one word per 4096.
static void launch_scan(int total, uint32_t *x, uint32_t *sums, hipStream_t st)
{
    const int chunks = (total + kScanChunk - 1) / kScanChunk;
    if (chunks > kScanOneBlock) {
        hipLaunchKernelGGL(k_scan_sums, dim3(chunks), dim3(256), 0, st, total, x, sums);
        hipLaunchKernelGGL(k_radix_scan, dim3(1), dim3(1024), 0, st, chunks, sums);
        hipLaunchKernelGGL(k_scan_apply, dim3(chunks), dim3(256), 0, st, total, x, sums);
    } else {
        hipLaunchKernelGGL(k_radix_scan, dim3(1), dim3(1024), 0, st, total, x);
    }
}

hipError_t launch_collapse4(int n, const Node *nodes, Node4 *nodes4, NodeQ *nodesq, int32_t *queue, uint32_t *mark,
                            uint32_t *part, uint32_t *sums, int32_t *ctl, hipStream_t st)
{
    if (n <= 1) return hipSuccess;
    hipLaunchKernelGGL(k_collapse_top, dim3(1), dim3(kCollapseTop), 0, st, nodes, queue, mark, part, ctl);
    // fewer leaves have no level that wide
    if (n > kCollapseWide)
        hipLaunchKernelGGL(k_collapse_subtrees, dim3(kCollapseWaves / 4), dim3(256), 0, st, nodes, queue, mark, part,
                           ctl);
    launch_scan(n, mark, sums, st);
    hipLaunchKernelGGL(k_collapse_write, dim3((n - 1 + 255) / 256), dim3(256), 0, st, n, nodes, mark, ctl, nodes4,
                       nodesq);
    return hipGetLastError();
}

void launch_radix_sort(int n, int passes, uint32_t *k0, uint32_t *v0, uint32_t *k1, uint32_t *v1, uint32_t *hist,
                       hipStream_t st)
{
    const int sb = (int)sort_blocks(n);
    const int total = 256 * sb;
    // long histograms: chunk sums live after the histogram (scan_sum_words)
    uint32_t *sums = hist + total;
    uint32_t *ki = k0, *vi = v0, *ko = k1, *vo = v1;
    for (int pass = 0; pass < passes; ++pass) {
        const int shift = 8 * pass;
        hipLaunchKernelGGL(k_radix_hist, dim3(sb), dim3(kSortThreads), 0, st, n, ki, shift, hist);
        launch_scan(total, hist, sums, st);
        hipLaunchKernelGGL(k_radix_scatter, dim3(sb), dim3(kSortThreads), 0, st, n, ki, vi, ko, vo, shift, hist);
        uint32_t *t0 = ki, *t1 = vi;
        ki = ko; vi = vo; ko = t0; vo = t1;
    }
}

// Pieces of the BVH build shared with the triangle mesh: reset the centre
// bounds; Morton codes of centres [n,3] within the bounds and their sort
// (sorted codes / original indices back in keys0 / vals0); the binary
// hierarchy, from leaf boxes in sorted order.
hipError_t launch_bounds_reset(int32_t *bounds, hipStream_t st)
{
    hipLaunchKernelGGL(k_init, dim3(1), dim3(64), 0, st, bounds);
    return hipGetLastError();
}

hipError_t launch_morton_sort(int n, const float *centres, const int32_t *bounds, uint32_t *keys0, uint32_t *vals0,
                              uint32_t *keys1, uint32_t *vals1, uint32_t *hist, hipStream_t st)
{
    const int tb = 256, gb = (n + tb - 1) / tb;
    hipLaunchKernelGGL(k_morton, dim3(gb), dim3(tb), 0, st, n, centres, bounds, keys0, vals0);
    launch_radix_sort(n, 4, keys0, vals0, keys1, vals1, hist, st);
    return hipGetLastError();
}

hipError_t launch_hierarchy(int n, const float *leaf_box, void *scratch, Node *nodes, uint32_t *mark, hipStream_t st)
{
    if (n <= 1) return hipSuccess;
    const auto list = [](void *p, size_t c) {
        ClusterList v;
        v.ref = (int2 *)p;
        v.box = (float *)(v.ref + c);
        v.high = (uint8_t *)(v.box + 6 * c);
        return v;
    };
    const auto blocks = [](int64_t c) { return (int)((c + kClusterBlock - 1) / kClusterBlock); };
    int launches = 0;
    for (int64_t c = n; c > kClusterBlock; c = (c + kClusterShrink - 1) / kClusterShrink) ++launches;
    const size_t c1 = cluster_words(n), c2 = cluster_words((int64_t)c1);
    const ClusterList lists[2] = {list(scratch, c1), list((char *)scratch + align256(33 * c1), c2)};
    ClusterList in{const_cast<float *>(leaf_box), nullptr, nullptr};
    int count = n;
    for (int k = 0; k <= launches; ++k) {
        const ClusterList out = lists[k & 1];
        const int cap = 63 - kClusterForced - 3 * (launches - k);
        hipLaunchKernelGGL(k_cluster, dim3(blocks(count)), dim3(kClusterBlock), 0, st, n, count, in, out, cap, nodes,
                           mark);
        count = (count + kClusterShrink - 1) / kClusterShrink;
        in = out;
    }
    return hipGetLastError();
}

hipError_t launch_scene_build(const grt_surfels &s, float alpha_min, const SceneWS &w, hipStream_t st)
{
    const int n = (int)s.n;
    if (n <= 0) return hipSuccess;
    const int tb = 256, gb = (n + tb - 1) / tb;
    hipError_t e = launch_bounds_reset(w.bounds, st);
    if (e != hipSuccess) return e;
    hipLaunchKernelGGL(k_bounds, dim3(std::min(gb, 512)), dim3(tb), 0, st, n, s.means, w.bounds);
    // (sorted codes / ids are back in keys0 / vals0)
    if ((e = launch_morton_sort(n, s.means, w.bounds, w.keys0, w.vals0, w.keys1, w.vals1, w.hist, st)) != hipSuccess)
        return e;
    hipLaunchKernelGGL(k_records, dim3(gb), dim3(tb), 0, st, n, w.vals0, s.means, s.scales, s.quats, s.opacity, s.rgb,
                       alpha_min, w.rec, w.col, w.leaf_box, w.quat);
    if ((e = hipGetLastError()) != hipSuccess) return e;
    if ((e = launch_hierarchy(n, w.leaf_box, w.clusters, w.nodes, w.mark, st)) != hipSuccess) return e;
    // (the sort's other keys and its histogram are free again)
    return launch_collapse4(n, w.nodes, w.nodes4, w.nodesq, w.queue, w.mark, w.keys1, w.hist, w.ctl4, st);
}

}  // namespace grt
