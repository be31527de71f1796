// The quantized node on the CPU: quantize_node and slab_q compiled for the
// host, checked in extended precision.  argv[1] names the check.  Prints the
// number of cases and of failures.
#include <algorithm>
#include <cmath>
#include <cstdint>
#include <cstdio>
#include <cstdlib>
#include <cstring>
#include <random>
#include <vector>

#define __device__
#define __forceinline__ inline
struct float3 { float x, y, z; };
struct int4 { int x, y, z, w; };
static int4 make_int4(int x, int y, int z, int w) { return {x, y, z, w}; }
static float __builtin_amdgcn_rcpf(float x) { return 1.0f / x; }
#include "grt_nodeq.h"
using namespace grt;

static std::mt19937_64 R(1);
static double U(double a, double b) { return a + (b - a) * (double)(R() >> 11) * 0x1p-53; }
static const long double kU = 0x1p-24L;  // half a unit in the last place, relative
static const int kRef[4] = {0, 1, 2, 3};

// child boxes of about `size` around `at`, some thin, some flat
static int draw_boxes(float (&box)[4][6], double size, double at)
{
    const int m = 2 + (int)(R() % 3);
    for (int j = 0; j < 4; ++j)
        for (int a = 0; a < 3; ++a) {
            const double x = at + U(-1, 1) * size, y = x + U(0, 1) * size * (R() % 4 ? 1 : 1e-3);
            box[j][a] = j < m ? (float)x : 0.0f;
            box[j][3 + a] = j < m ? (float)y : 0.0f;
        }
    return m;
}

static long double plane(const NodeQ &q, int a, uint32_t w, int j)
{
    return (long double)q.org[a] + (long double)((w >> (8 * j)) & 255u) * (long double)q.scale[a];
}

// every plane at least as far outside its box as the walk rounds depths by
// (3 u of the grid's length), and no more than a grid step and two margins
static void planes()
{
    long n = 0, inside = 0, wide = 0;
    for (double size : {1e-3, 1e-2, 1e-1, 1.0, 30.0})
        for (double at : {0.0, 8.0, -60.0, 300.0, -1000.0, 1e5})
            for (int it = 0; it < 4000; ++it) {
                float box[4][6];
                const int m = draw_boxes(box, size, at);
                const NodeQ q = quantize_node(box, kRef, m);
                for (int a = 0; a < 3; ++a) {
                    float lo = box[0][a], hi = box[0][3 + a];
                    for (int j = 1; j < m; ++j) {
                        lo = std::fmin(lo, box[j][a]);
                        hi = std::fmax(hi, box[j][3 + a]);
                    }
                    const long double ext = (long double)hi - lo, slack = 3 * kU * 255 * q.scale[a];
                    const long double step = 1.01L * q.scale[a] + 32 * kU * ext;
                    for (int j = 0; j < m; ++j) {
                        const long double below = box[j][a] - plane(q, a, q.lo[a], j);
                        const long double above = plane(q, a, q.hi[a], j) - box[j][3 + a];
                        ++n;
                        inside += below < slack || above < slack;
                        wide += below > step || above > step;
                    }
                }
            }
    // an infinite or NaN corner: every child stays in reach of every ray
    for (float bad : {INFINITY, -INFINITY, NAN})
        for (int it = 0; it < 2000; ++it) {
            float box[4][6];
            const int m = draw_boxes(box, 1.0, 0.0);
            const int a = (int)(R() % 3);
            const float x0 = box[0][a], y0 = box[0][3 + a];
            if (bad > 0) box[0][3 + a] = bad;
            else if (bad < 0) box[0][a] = bad;
            else box[0][a] = box[0][3 + a] = bad;
            const NodeQ q = quantize_node(box, kRef, m);
            for (int j = bad == bad ? 0 : 1; j < m; ++j) {
                const float l = j ? box[j][a] : x0, h = j ? box[j][3 + a] : y0;
                const float o = (float)U(-3, 3), d = U(-1, 1) < 0 ? -0.7f : 0.7f, inv = fast_inv(d);
                const float start = (q.org[a] - o) * inv, step = q.scale[a] * inv;
                const float near = fmaf((float)(((d < 0 ? q.hi[a] : q.lo[a]) >> (8 * j)) & 255u), step, start);
                const float far = fmaf((float)(((d < 0 ? q.lo[a] : q.hi[a]) >> (8 * j)) & 255u), step, start);
                ++n;
                const float tn = ((d < 0 ? h : l) - o) / d, tf = ((d < 0 ? l : h) - o) / d;
                inside += near > tn + 8 * 0x1p-24f * std::fabs(tn) || far < tf - 8 * 0x1p-24f * std::fabs(tf);  // (NaN: no bound)
            }
        }
    printf("planes %ld inside %ld wide %ld\n", n, inside, wide);
}

// A direction component whose reciprocal, within 1 ulp of the exact one, is
// nearly that much above (side > 0) or below it.
static float off_component(int side, float &inv)
{
    for (;;) {
        const float d = (float)(0.5 * (1.0 - U(0, 0.004))), r = (float)(1.0 / (double)d);
        inv = std::nextafterf(r, side > 0 ? 9.0f : 0.0f);
        const double ulp = (double)std::nextafterf(r, 9.0f) - r, err = std::fabs((double)inv - 1.0 / (double)d) / ulp;
        if (err <= 1.0 && err > 0.997) return d;
    }
}

struct Plane {
    long double depth;  // exact, of the single-precision ray
    float o, org, scale;
    int q;
};

// Near planes of x whose computed depth is nearly all the roundings together
// too far, far planes of y as much too near, paired where the exact depths
// meet within half a unit in the last place: the ray enters the box.
static void slack()
{
    long n = 0, lost = 0, kept = 0;
    for (int trial = 0; trial < 3; ++trial) {
        float inv[2];
        const float d[2] = {off_component(1, inv[0]), off_component(-1, inv[1])};
        const double m = 1.08;  // depths just above a power of two
        std::vector<Plane> v[2];
        for (int a = 0; a < 2; ++a) {
            for (long i = 0; i < 10000000; ++i) {
                Plane c;
                c.org = (float)U(-1e-4, 1e-4);
                c.scale = (float)U(0.5e-6, 1e-6);
                c.q = 1 + (int)(R() % 254);
                c.o = (float)-(512 * m * (1 + U(0, 2e-4)) * d[a]);
                const float t = fmaf((float)c.q, c.scale * inv[a], (c.org - c.o) * inv[a]);
                c.depth = ((long double)c.org + (long double)c.q * c.scale - c.o) / d[a];
                const long double err = (t - c.depth) / c.depth, lim = 0.972L * (2 + 3 / m) * kU;
                if (a == 0 ? err > lim : err < -lim) v[a].push_back(c);
            }
            std::sort(v[a].begin(), v[a].end(), [](const Plane &x, const Plane &y) { return x.depth < y.depth; });
        }
        for (const Plane &x : v[0])
            for (const Plane &y : v[1]) {
                const long double gap = (y.depth - x.depth) / x.depth;
                if (gap < 0) continue;
                if (gap > 0.5L * kU) break;
                const float3 step = {x.scale * inv[0], y.scale * inv[1], 0.0f};
                float3 start = {(x.org - x.o) * inv[0], (y.org - y.o) * inv[1], NAN};  // no plane of z
                float tn;
                ++n;
                lost += !slab_q<0>((uint32_t)x.q, 0u, 0u, 255u, (uint32_t)y.q, 0u, step, {start.x, start.y, start.z}, 0.0f, tn);
                start.y *= 1.0f - 4e-6f;  // a far plane clearly before the near one
                kept += slab_q<0>((uint32_t)x.q, 0u, 0u, 255u, (uint32_t)y.q, 0u, step, start, 0.0f, tn);
            }
    }
    printf("pairs %ld lost %ld kept %ld\n", n, lost, kept);
}

int main(int argc, char **argv)
{
    if (argc > 1 && !strcmp(argv[1], "planes")) planes();
    if (argc > 1 && !strcmp(argv[1], "slack")) slack();
    return 0;
}
