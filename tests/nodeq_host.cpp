// The quantized node on the CPU: quantize_node and slab_q compiled for the
// host, checked in extended precision.  argv[1] names the check.  Prints the
// number of cases and of failures.
#include <cmath>
#include <cstdint>
#include <cstdio>
#include <cstdlib>
#include <cstring>
#include <random>

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

int main(int argc, char **argv)
{
    if (argc > 1 && !strcmp(argv[1], "planes")) planes();
    return 0;
}
