// mesh.hip -- mesh backend of the attribute query (Sec. 3.5.2, "Mesh-based
// ray tracing"): a triangle mesh with per-vertex albedo, roughness, metallic
// and normal answers Trace_attr by one closest-hit ray-triangle query per ray
// instead of ordered ray-splat evaluation.  A miss sets V = 1 (the ray sees
// the environment); a hit sets V = 0 and interpolates the vertex attributes
// with the hit's barycentric weights.
//
// MI355X has no ray-tracing units, so the query is software: a BVH over the
// triangles' boxes, built and collapsed to 4-wide quantized nodes with the
// surfel scene's kernels, and a closest-hit traversal, one thread per ray,
// nearer child first, pruned by the closest hit so far.
#include "grt_internal.h"

namespace grt {

// Box (exact, padded by kPad) and centre of each triangle; the centres'
// bounds by block reduction and one atomic per block and axis.  A triangle
// with a vertex index outside [0, nv) is made degenerate: an empty box that
// no ray enters.
__global__ void k_tri_boxes(int nv, const float *__restrict__ verts, int nf, const int32_t *__restrict__ tris,
                            float *__restrict__ box, float *__restrict__ centre, int32_t *__restrict__ bounds)
{
    const int i = blockIdx.x * blockDim.x + threadIdx.x;
    float c[3] = {INFINITY, INFINITY, INFINITY}, C[3] = {-INFINITY, -INFINITY, -INFINITY};
    if (i < nf) {
        const int ia = tris[3 * i], ib = tris[3 * i + 1], ic = tris[3 * i + 2];
        const bool ok = ia >= 0 && ia < nv && ib >= 0 && ib < nv && ic >= 0 && ic < nv;
#pragma unroll
        for (int a = 0; a < 3; ++a) {
            float lo = INFINITY, hi = -INFINITY, m = 0.0f;
            if (ok) {
                const float x = verts[3 * ia + a], y = verts[3 * ib + a], z = verts[3 * ic + a];
                lo = fminf(fminf(x, y), z) - kPad;
                hi = fmaxf(fmaxf(x, y), z) + kPad;
                m = (x + y + z) * (1.0f / 3.0f);
                c[a] = C[a] = m;
            }
            box[6 * (size_t)i + a] = lo;
            box[6 * (size_t)i + 3 + a] = hi;
            centre[3 * (size_t)i + a] = m;
        }
    }
    __shared__ float red[6][256];
#pragma unroll
    for (int a = 0; a < 3; ++a) { red[a][threadIdx.x] = c[a]; red[3 + a][threadIdx.x] = C[a]; }
    __syncthreads();
    for (int s = blockDim.x / 2; s > 0; s >>= 1) {
        if (threadIdx.x < s) {
#pragma unroll
            for (int a = 0; a < 3; ++a) {
                red[a][threadIdx.x] = fminf(red[a][threadIdx.x], red[a][threadIdx.x + s]);
                red[3 + a][threadIdx.x] = fmaxf(red[3 + a][threadIdx.x], red[3 + a][threadIdx.x + s]);
            }
        }
        __syncthreads();
    }
    if (threadIdx.x < 3 && red[threadIdx.x][0] <= red[3 + threadIdx.x][0]) {
        atomicMin(&bounds[threadIdx.x], f2o(red[threadIdx.x][0]));
        atomicMax(&bounds[3 + threadIdx.x], f2o(red[3 + threadIdx.x][0]));
    }
}

// Records and leaf boxes in Morton order.
__global__ void k_tri_records(int nv, const float *__restrict__ verts, int nf, const int32_t *__restrict__ tris,
                              const uint32_t *__restrict__ order, const float *__restrict__ box_tmp,
                              float4 *__restrict__ rec, float *__restrict__ leaf_box)
{
    const int p = blockIdx.x * blockDim.x + threadIdx.x;
    if (p >= nf) return;
    const uint32_t id = order[p];
    const int ia = tris[3 * id], ib = tris[3 * id + 1], ic = tris[3 * id + 2];
    const bool ok = ia >= 0 && ia < nv && ib >= 0 && ib < nv && ic >= 0 && ic < nv;
    float3 v0 = make_float3(0.f, 0.f, 0.f), e1 = v0, e2 = v0;
    if (ok) {
        v0 = make_float3(verts[3 * ia], verts[3 * ia + 1], verts[3 * ia + 2]);
        e1 = make_float3(verts[3 * ib] - v0.x, verts[3 * ib + 1] - v0.y, verts[3 * ib + 2] - v0.z);
        e2 = make_float3(verts[3 * ic] - v0.x, verts[3 * ic + 1] - v0.y, verts[3 * ic + 2] - v0.z);
    }
    rec[3 * (size_t)p] = make_float4(v0.x, v0.y, v0.z, __uint_as_float(id));
    rec[3 * (size_t)p + 1] = make_float4(e1.x, e1.y, e1.z, 0.0f);
    rec[3 * (size_t)p + 2] = make_float4(e2.x, e2.y, e2.z, 0.0f);
#pragma unroll
    for (int a = 0; a < 6; ++a) leaf_box[6 * (size_t)p + a] = box_tmp[6 * (size_t)id + a];
}

hipError_t launch_mesh_build(int nv, const float *verts, int nf, const int32_t *tris, const MeshWS &w, hipStream_t st)
{
    if (nf <= 0) return hipSuccess;
    const int tb = 256, gb = (nf + tb - 1) / tb;
    hipError_t e = launch_bounds_reset(w.bounds, st);
    if (e != hipSuccess) return e;
    hipLaunchKernelGGL(k_tri_boxes, dim3(gb), dim3(tb), 0, st, nv, verts, nf, tris, w.box_tmp, w.centre, w.bounds);
    if ((e = launch_morton_sort(nf, w.centre, w.bounds, w.keys0, w.vals0, w.keys1, w.vals1, w.hist, st)) != hipSuccess)
        return e;
    hipLaunchKernelGGL(k_tri_records, dim3(gb), dim3(tb), 0, st, nv, verts, nf, tris, w.vals0, w.box_tmp, w.rec,
                       w.leaf_box);
    if ((e = launch_hierarchy(nf, w.leaf_box, w.box_tmp, w.nodes, w.mark, st)) != hipSuccess) return e;
    // (the sort's other keys and its histogram are free again)
    return launch_collapse4(nf, w.nodes, nullptr, w.nodesq, w.queue, w.mark, w.keys1, w.hist, w.ctl4, st);
}

// Moller-Trumbore (two-sided) with a fixed operation order; true on a hit
// with t in (tmin, tbest], or at t == tbest with a lower triangle id.
__device__ __forceinline__ bool tri_hit(const float4 r0, const float4 r1, const float4 r2, float3 o, float3 d,
                                        float tmin, float tbest, uint32_t best_id, float &t, float &u, float &v)
{
#pragma clang fp contract(off)
    const float3 e1 = make_float3(r1.x, r1.y, r1.z), e2 = make_float3(r2.x, r2.y, r2.z);
    const float px = d.y * e2.z - d.z * e2.y, py = d.z * e2.x - d.x * e2.z, pz = d.x * e2.y - d.y * e2.x;
    const float det = e1.x * px + e1.y * py + e1.z * pz;
    if (fabsf(det) < 1e-20f) return false;
    const float inv = 1.0f / det;
    const float sx = o.x - r0.x, sy = o.y - r0.y, sz = o.z - r0.z;
    u = (sx * px + sy * py + sz * pz) * inv;
    if (u < 0.0f || u > 1.0f) return false;
    const float qx = sy * e1.z - sz * e1.y, qy = sz * e1.x - sx * e1.z, qz = sx * e1.y - sy * e1.x;
    v = (d.x * qx + d.y * qy + d.z * qz) * inv;
    if (v < 0.0f || u + v > 1.0f) return false;
    t = (e2.x * qx + e2.y * qy + e2.z * qz) * inv;
    if (!(t > tmin && t <= tbest)) return false;
    return t < tbest || __float_as_uint(r0.w) < best_id;
}

// A ray's stack: entries (4-wide node or leaf, entry depth), the first
// kMeshLds in LDS (lane-interleaved), deeper ones in a private array.  A node
// leaves at most three siblings behind, on at most 63 levels.
constexpr int kMeshLds = 8, kMeshDeep = 3 * 63 - kMeshLds;

struct MeshStack {
    int2 *lds;  // the thread's slot 0; slot i at lds[256 * i]
    int2 *deep;
    int sp;

    __device__ __forceinline__ void push(int ref, float t)
    {
        const int2 e = make_int2(ref, __float_as_int(t));
        if (sp < kMeshLds) lds[256 * sp] = e;
        else deep[sp - kMeshLds] = e;
        ++sp;
    }
    // the topmost entry not beyond `best`; kNone when there is none
    __device__ __forceinline__ int pop(float best)
    {
        while (sp > 0) {
            --sp;
            const int2 e = sp < kMeshLds ? lds[256 * sp] : deep[sp - kMeshLds];
            if (__int_as_float(e.y) <= best) return e.x;
        }
        return kNone;
    }
};

// Closest hit of one ray: triangle id (0xffffffff: miss) and barycentrics.
// Bound by VALU issue (84% of the peak, 26 of 64 lanes in an instruction) and
// by the vector L1 (one tag access per lane and 16 bytes of a divergent load):
// a 4-wide quantized node is four loads, as a binary one was, for half the node
// steps.  (Lanes that take new rays as theirs end: 9.5 against 9.3 ms for a
// relit frame of 33.5M rays, since results are then gathered by few lanes.)
__device__ __forceinline__ void mesh_closest(const float4 *__restrict__ rec, const NodeQ *__restrict__ nodes, int nf,
                                             float3 o, float3 d, float tmin, float tmax, MeshStack &stack,
                                             uint32_t &bid, float &bu, float &bv)
{
    const float3 inv = make_float3(fast_inv(d.x), fast_inv(d.y), fast_inv(d.z));
    const bool gx = __float_as_int(d.x) < 0, gy = __float_as_int(d.y) < 0, gz = __float_as_int(d.z) < 0;
    float best = tmax;
    bu = 0.0f; bv = 0.0f;
    bid = 0xffffffffu;
    stack.sp = 0;
    int cur = nf <= 0 ? kNone : (nf == 1 ? -1 : 0);
    while (cur != kNone) {
        // (entry depths carry rounding: prune with some slack)
        if (cur >= 0) {
            const float bound = best * 1.0000005f;
            const float4 *nd = reinterpret_cast<const float4 *>(nodes + cur);
            const float4 w0 = nd[0], w1 = nd[1], w2 = nd[2];
            const int4 ch = *reinterpret_cast<const int4 *>(nd + 3);
            const float3 start = make_float3((w0.x - o.x) * inv.x, (w0.y - o.y) * inv.y, (w0.z - o.z) * inv.z);
            const float3 step = make_float3(w0.w * inv.x, w1.x * inv.y, w1.y * inv.z);
            const uint32_t lx = __float_as_uint(w1.z), ly = __float_as_uint(w1.w), lz = __float_as_uint(w2.x);
            const uint32_t hx = __float_as_uint(w2.y), hy = __float_as_uint(w2.z), hz = __float_as_uint(w2.w);
            const uint32_t nx = gx ? hx : lx, fx = gx ? lx : hx;
            const uint32_t ny = gy ? hy : ly, fy = gy ? ly : hy;
            const uint32_t nz = gz ? hz : lz, fz = gz ? lz : hz;
            float t0, t1, t2, t3;
            const bool k0 = slab_q<0>(nx, ny, nz, fx, fy, fz, step, start, tmin, t0) & (t0 <= bound) & (ch.x != kNoChild);
            const bool k1 = slab_q<1>(nx, ny, nz, fx, fy, fz, step, start, tmin, t1) & (t1 <= bound) & (ch.y != kNoChild);
            const bool k2 = slab_q<2>(nx, ny, nz, fx, fy, fz, step, start, tmin, t2) & (t2 <= bound) & (ch.z != kNoChild);
            const bool k3 = slab_q<3>(nx, ny, nz, fx, fy, fz, step, start, tmin, t3) & (t3 <= bound) & (ch.w != kNoChild);
            const int m = (int)k0 + (int)k1 + (int)k2 + (int)k3;
            float s0 = k0 ? t0 : INFINITY, s1 = k1 ? t1 : INFINITY, s2 = k2 ? t2 : INFINITY, s3 = k3 ? t3 : INFINITY;
            int c0 = ch.x, c1 = ch.y, c2 = ch.z, c3 = ch.w;
            exchange(s0, c0, s1, c1);
            exchange(s2, c2, s3, c3);
            exchange(s0, c0, s2, c2);
            exchange(s1, c1, s3, c3);
            exchange(s1, c1, s2, c2);
            if (m > 3) stack.push(c3, s3);
            if (m > 2) stack.push(c2, s2);
            if (m > 1) stack.push(c1, s1);
            cur = m > 0 ? c0 : stack.pop(bound);
        }
        if (cur < 0) {  // leaf: triangle record -(cur + 1)
            const float4 *rr = rec + 3 * (size_t)(-cur - 1);
            const float4 r0 = rr[0], r1 = rr[1], r2 = rr[2];
            float t, u, v;
            if (tri_hit(r0, r1, r2, o, d, tmin, best, bid, t, u, v)) {
                best = t; bu = u; bv = v; bid = __float_as_uint(r0.w);
            }
            cur = stack.pop(best * 1.0000005f);
        }
    }
}

// Barycentric vertex attributes of the hit (the normal facing the ray
// origin); V = 1 and zeros on a miss.
struct MeshHitAttrs {
    float V, A[3], R, M, N[3];
};
__device__ __forceinline__ MeshHitAttrs mesh_attrs(const int32_t *__restrict__ tris, int nf, const float *albedo,
                                                   const float *rough, const float *metal, const float *vnormal,
                                                   uint32_t bid, float bu, float bv, float3 d)
{
    MeshHitAttrs h = {1.0f, {0.f, 0.f, 0.f}, 0.0f, 0.0f, {0.f, 0.f, 0.f}};
    if (bid == 0xffffffffu || bid >= (uint32_t)nf) return h;
    h.V = 0.0f;
    const float w[3] = {1.0f - bu - bv, bu, bv};
#pragma unroll
    for (int k = 0; k < 3; ++k) {
        const int vi = tris[3 * (size_t)bid + k];  // valid: degenerate triangles are never hit
#pragma unroll
        for (int c = 0; c < 3; ++c) {
            h.A[c] += w[k] * albedo[3 * (size_t)vi + c];
            h.N[c] += w[k] * vnormal[3 * (size_t)vi + c];
        }
        h.R += w[k] * rough[vi];
        h.M += w[k] * metal[vi];
    }
    if (h.N[0] * d.x + h.N[1] * d.y + h.N[2] * d.z > 0.0f) { h.N[0] = -h.N[0]; h.N[1] = -h.N[1]; h.N[2] = -h.N[2]; }
    return h;
}

__global__ void __launch_bounds__(256) k_mesh_trace_attr(MeshTraceArgs a)
{
    __shared__ int2 top[kMeshLds][256];
    int2 deep[kMeshDeep];
    const int64_t r = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (r >= a.n) return;
    const float3 o = make_float3(a.o[3 * r], a.o[3 * r + 1], a.o[3 * r + 2]);
    const float3 d = make_float3(a.d[3 * r], a.d[3 * r + 1], a.d[3 * r + 2]);
    MeshStack stack = {&top[0][threadIdx.x], deep, 0};
    uint32_t bid;
    float bu, bv;
    mesh_closest(a.rec, a.nodes, a.nf, o, d, a.tmin, a.tmax, stack, bid, bu, bv);
    const MeshHitAttrs h = mesh_attrs(a.tris, a.nf, a.albedo, a.rough, a.metal, a.vnormal, bid, bu, bv, d);
    a.out_V[r] = h.V;
#pragma unroll
    for (int c = 0; c < 3; ++c) { a.out_albedo[3 * r + c] = h.A[c]; a.out_normal[3 * r + c] = h.N[c]; }
    a.out_rough[r] = h.R;
    a.out_metal[r] = h.M;
}

// Relighting through the mesh, query pass: for every traced sample of the
// render's ray records, the mesh query parked for the shading pass as the
// surfel relight parks it ((V, albedo) in the contribution slot, (r, m) in
// the ray record's spare words, the normal in rl_n*).
// A block takes the samples of neighbouring pixels, kMeshTile of them, and
// traces them in the order of their directions' bins (a counting sort in LDS):
// a pixel's samples leave in all directions, and 64 of them in index order
// share few nodes.  Everything else stays within the tile's records, so no
// global sort and no scattered writes are paid for it.  (Relit frame of 1024 x
// 1024 x 32 through 46k triangles: tiles of 1,024 11.0 ms, 2,048 11.3, 4,096
// 11.8; 12 stack entries in LDS instead of 8, so fewer blocks, 12.0.)
// Tiles of 1,024 give a thread four rays in turn, so they wait for launches
// that fill the chip anyway: through 46k triangles 16 x 16 x 16 samples take 107
// us in tiles of 256 and 270 in tiles of 1,024, 256 x 256 x 4 159 and 370, 512 x
// 512 x 8 637 and 687, 512 x 512 x 16 1.29 ms both, 1024 x 1024 x 16 4.83 and 4.70.
constexpr int64_t kMeshWide = 1 << 22;  // samples
constexpr int kMeshBins = 257;  // 16 x 16 directions, then the untraced

// octahedral direction bin, 16 x 16, along a Morton curve
__device__ __forceinline__ int dir_bin(float4 d)
{
    const float s = fabsf(d.x) + fabsf(d.y) + fabsf(d.z);
    float u = d.x / s, v = d.z / s;
    if (d.y < 0.0f) {
        const float uu = (1.0f - fabsf(v)) * (u >= 0.0f ? 1.0f : -1.0f);
        const float vv = (1.0f - fabsf(u)) * (v >= 0.0f ? 1.0f : -1.0f);
        u = uu;
        v = vv;
    }
    const int iu = (int)fminf(fmaxf((u * 0.5f + 0.5f) * 16.0f, 0.0f), 15.0f);
    const int iv = (int)fminf(fmaxf((v * 0.5f + 0.5f) * 16.0f, 0.0f), 15.0f);
    auto spread = [](int x) { x = (x | (x << 2)) & 0x33; return (x | (x << 1)) & 0x55; };
    return spread(iu) | (spread(iv) << 1);
}

template <int kMeshTile>
__global__ void __launch_bounds__(256) k_mesh_relight_query(RenderArgs a, MeshTraceArgs m, int64_t total)
{
    __shared__ int2 top[kMeshLds][256];
    __shared__ uint16_t order[kMeshTile];
    __shared__ int count[kMeshBins], sums[4];
    int2 deep[kMeshDeep];
    const int64_t base = (int64_t)blockIdx.x * kMeshTile;
    const int tile = (int)(total - base < kMeshTile ? total - base : kMeshTile);
    constexpr int kPer = kMeshTile / 256;
    for (int b = threadIdx.x; b < kMeshBins; b += 256) count[b] = 0;
    __syncthreads();
    int bin[kPer], rank[kPer];
#pragma unroll
    for (int k = 0; k < kPer; ++k) {
        const int i = k * 256 + threadIdx.x;
        if (i < tile) {
            const float4 r0 = a.rays[3 * (base + i)];
            bin[k] = r0.w == 0.0f ? kMeshBins - 1 : dir_bin(r0);
            rank[k] = atomicAdd(&count[bin[k]], 1);
        }
    }
    __syncthreads();
    {   // exclusive prefix sum of the first 256 bins; the untraced come last
        const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
        const int own = count[threadIdx.x];
        int x = own;
#pragma unroll
        for (int off = 1; off < 64; off <<= 1) {
            const int y = __shfl_up(x, off, 64);
            if (lane >= off) x += y;
        }
        if (lane == 63) sums[wave] = x;
        __syncthreads();
        int before = x - own;
        for (int w = 0; w < wave; ++w) before += sums[w];
        count[threadIdx.x] = before;
        if (threadIdx.x == 255) count[256] = before + own;
    }
    __syncthreads();
#pragma unroll
    for (int k = 0; k < kPer; ++k)
        if (k * 256 + (int)threadIdx.x < tile) order[count[bin[k]] + rank[k]] = (uint16_t)(k * 256 + threadIdx.x);
    __syncthreads();
    MeshStack stack = {&top[0][threadIdx.x], deep, 0};
    for (int i = threadIdx.x; i < tile; i += 256) {
        const int64_t r = base + order[i];
        const float4 r0 = a.rays[3 * r];
        if (r0.w == 0.0f) {
            a.contrib[r] = make_float4(0.f, 0.f, 0.f, 0.f);
            continue;
        }
        const int64_t p = (uint32_t)r / (uint32_t)(a.nc + a.ng + a.ne);  // fewer than 2^31 samples
        const float3 x = make_float3(a.x[3 * p], a.x[3 * p + 1], a.x[3 * p + 2]);
        const float3 d = make_float3(r0.x, r0.y, r0.z);
        uint32_t bid;
        float bu, bv;
        mesh_closest(m.rec, m.nodes, m.nf, x, d, a.tmin, INFINITY, stack, bid, bu, bv);
        const MeshHitAttrs h = mesh_attrs(m.tris, m.nf, m.albedo, m.rough, m.metal, m.vnormal, bid, bu, bv, d);
        a.contrib[r] = make_float4(h.V, h.A[0], h.A[1], h.A[2]);
        float4 *r2 = a.rays + 3 * r + 2;
        r2->z = h.R;
        r2->w = h.M;
        a.rl_nx[r] = h.N[0];
        a.rl_ny[r] = h.N[1];
        a.rl_nz[r] = h.N[2];
    }
}

hipError_t launch_mesh_relight_query(const RenderArgs &a, const MeshTraceArgs &m, hipStream_t st)
{
    const int64_t total = (int64_t)a.H * a.W * (a.nc + a.ng + a.ne);
    if (total <= 0) return hipSuccess;
    if (total >= kMeshWide)
        hipLaunchKernelGGL(k_mesh_relight_query<1024>, dim3((unsigned)((total + 1023) / 1024)), dim3(256), 0, st, a, m,
                           total);
    else
        hipLaunchKernelGGL(k_mesh_relight_query<256>, dim3((unsigned)((total + 255) / 256)), dim3(256), 0, st, a, m,
                           total);
    return hipGetLastError();
}

hipError_t launch_mesh_trace_attr(const MeshTraceArgs &a, hipStream_t st)
{
    if (a.n <= 0) return hipSuccess;
    hipLaunchKernelGGL(k_mesh_trace_attr, dim3((unsigned)((a.n + 255) / 256)), dim3(256), 0, st, a);
    return hipGetLastError();
}

}  // namespace grt
