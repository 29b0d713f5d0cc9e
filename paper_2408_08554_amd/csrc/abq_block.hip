// Host side of the block kernels: the choice of shape and the launch.
#include "abq_block_g128_kernels.h"

namespace abq {

struct BkShapeInfo { int bm, bn, occ; };   // rows of A, channels, workgroups a compute unit (as in block_launch)
constexpr int kBlockShapes = 5;
static const BkShapeInfo kShapes[kBlockShapes] = {{256, 256, 1}, {128, 192, 1}, {128, 128, 1}, {128, 128, 2}, {64, 128, 2}};
static int shape_bn(int p, int shape) { return shape == 0 && p == 7 ? 192 : kShapes[shape].bn; }

// What a launch costs (us): `base`, `round` for every round of resident workgroups (first loads, epilogue, and the gap to the next workgroup),
// and per step of 128 k what a unit with 1, 2 or 3 of the shape's workgroups takes.  Non-negative least squares of the relative error over
// 2400 sizes that the K-split kernel leaves (M = 48..2048, N = 256..13824, K = 512..13824), mean error 7 to 13 %.
struct Cost { float base, round, step[3]; };
struct WidthCosts { Cost block[kBlockShapes], tiled[3]; };   // tiled: 64 x 64, 64 x 128, 64 x 256
static const WidthCosts kCosts[6] = {
    {{{0, 9.436f, {1.027f, 0, 0}}, {0.125f, 6.141f, {0.471f, 0, 0}}, {1.062f, 4.048f, {0.349f, 0, 0}}, {2.211f, 3.673f, {0.353f, 0.7f, 0}}, {2.843f, 1.716f, {0.226f, 0.374f, 0}}},   // p = 1, 2
     {{4.838f, 0, {0.139f, 0.269f, 0.4f}}, {4.947f, 1.356f, {0.065f, 0.452f, 0.614f}}, {8.31f, 2.498f, {0.339f, 0.701f, 0}}}},
    {{{0, 10.526f, {1.165f, 0, 0}}, {0.719f, 6.203f, {0.62f, 0, 0}}, {1.303f, 4.349f, {0.438f, 0, 0}}, {2.376f, 3.92f, {0.457f, 0.878f, 0}}, {3.074f, 1.855f, {0.286f, 0.465f, 0}}},   // p = 3
     {{5.21f, 0, {0.131f, 0.31f, 0.464f}}, {3.924f, 2.746f, {0.324f, 0.551f, 0.798f}}, {}}},
    {{{0, 9.576f, {1.01f, 0, 0}}, {0, 6.327f, {0.455f, 0, 0}}, {0.661f, 4.709f, {0.346f, 0, 0}}, {0.766f, 3.528f, {0.467f, 0.762f, 0}}, {1.904f, 2.828f, {0.21f, 0.418f, 0}}},   // p = 4
     {{4.788f, 0, {0.15f, 0.281f, 0.468f}}, {2.312f, 4.769f, {0, 0.44f, 0.662f}}, {}}},
    {{{0, 9.587f, {1.182f, 0, 0}}, {0, 6.626f, {0.636f, 0, 0}}, {0.552f, 4.801f, {0.462f, 0, 0}}, {2.267f, 2.933f, {0.516f, 0.977f, 0}}, {1.979f, 2.725f, {0.293f, 0.533f, 0}}},   // p = 5, 6
     {{4.728f, 0, {0.187f, 0.305f, 0.569f}}, {4.94f, 1.929f, {0.377f, 0.588f, 0.853f}}, {}}},
    {{{0, 9.063f, {1.151f, 0, 0}}, {0, 7.177f, {0.86f, 0, 0}}, {0.709f, 5.01f, {0.614f, 0, 0}}, {0.842f, 5.436f, {0.634f, 1.187f, 0}}, {2.537f, 2.546f, {0.389f, 0.686f, 0}}},   // p = 7
     {{4.918f, 0, {0.235f, 0.424f, 0.702f}}, {0.179f, 6.379f, {0.148f, 0.793f, 1.114f}}, {}}},
    {{{0, 9.726f, {1.011f, 0, 0}}, {0, 6.513f, {0.535f, 0, 0}}, {0, 5.063f, {0.368f, 0, 0}}, {0, 4.122f, {0.537f, 0.888f, 0}}, {1.416f, 3.033f, {0.27f, 0.559f, 0}}},   // p = 8
     {{4.527f, 0, {0.21f, 0.335f, 0.602f}}, {3.166f, 3.019f, {0.15f, 0.554f, 0.939f}}, {}}},
};

static double cost_of(const Cost& c, int M, int N, int K, int bm, int bn, int occ)
{
    const long wgs = (long)((M + bm - 1) / bm) * ((N + bn - 1) / bn), cus = num_cus();
    const long load = (wgs + cus - 1) / cus, full = load / occ, part = load % occ;
    const double steps = 4.0 * ((K + kSuperK - 1) / kSuperK);
    return c.base + c.round * (double)(full + (part > 0)) + steps * ((double)full * c.step[occ - 1] + (part ? c.step[part - 1] : 0.f));
}

// The cheapest shape by the costs above, unless the tiled kernel's is 6 % below it (its 64 x 64 tiles, three workgroups a unit, where K is
// short or the output leaves the larger tiles' last round nearly empty).  Over those sizes the choice is 1.6 % from the best of all
// of them and takes 0.92 times the tiled kernel's time (M = 256..2048 0.91), 3 % of the sizes lose 3 % or more.
// A plan-table entry with a knob of the tiled kernel asks for that; so does a call for the int32 accumulator, which only that kernel writes.
bool block_plan(const GemmArgs& g, const WeightLayout& W, int* shape)
{
    if (W.g128 || g.acc) return false;
    PlanOverride ov;
    if (lookup_plan(g.p, g.q, g.M, g.N, g.K, &ov) && (ov.tiled_mt > 0 || ov.tiled_ntw > 0 || ov.tiled_wd > 0 || ov.tiled_band > 0)) return false;
    const int env = tuning_env("ABQ_BLOCK");   // tuning builds: -1 off, 1..5 a shape
    if (env) { *shape = env - 1; return env > 0 && env <= kBlockShapes; }
    const WidthCosts& w = kCosts[g.p <= 2 ? 0 : (g.p <= 4 ? g.p - 2 : (g.p <= 6 ? 3 : g.p - 3))];
    double best = 0;
    for (int i = 0; i < kBlockShapes; ++i) {
        const double c = cost_of(w.block[i], g.M, g.N, g.K, kShapes[i].bm, shape_bn(g.p, i), kShapes[i].occ);
        if (i == 0 || c < best) { best = c; *shape = i; }
    }
    int mt, ntw;
    tiled_shape_by_rule(g.p, g.M, g.N, g.K, &mt, &ntw);
    if (mt == 8 || (g.p >= 3 && ntw == 4)) return true;   // (one of its large tiles: those lose at every such size)
    return cost_of(w.tiled[ntw / 2], g.M, g.N, g.K, 16 * mt, 64 * ntw, ntw == 4 ? 2 : 3) * 0.94 >= best;
}

hipError_t launch_gemm_block(const GemmArgs& g, const ActLayout& A, const WeightLayout& W, int shape, hipStream_t s)
{
    const int bm = kShapes[shape].bm, bn = shape_bn(g.p, shape);
    BlockParams prm;
    for (int i = 0; i < 3; ++i) prm.fields[i] = g.w_blob + W.off_fields[i];
    prm.a = g.act_blob + A.off_codes;
    prm.aparams = (const RowParams*)(g.act_blob + A.off_params);
    prm.wparams = (const RowParams*)(g.w_blob + W.off_params);
    prm.y = g.y; prm.rq = g.rq;
    prm.M = g.M; prm.N = g.N; prm.K = g.K;
    prm.lda = A.Kp;
    prm.nsuper = A.Kp / kSuperK;
    prm.ntiles = W.NT;
    prm.oa = g.q == 8 ? 128 : 0;
    prm.ow = g.p == 8 ? 128 : 0;
    prm.narrow_sums = ((long)g.K * ((1 << g.p) - 1) < (1L << 23) && (long)g.K * ((1 << g.q) - 1) < (1L << 23)) ? 1 : 0;
    prm.tiles_m = (g.M + bm - 1) / bm;
    prm.tiles_n = (g.N + bn - 1) / bn;
    // bands of equal height, as in the tiled kernel
    const int cap = 1024 / bm, bands = (prm.tiles_m + cap - 1) / cap;
    prm.band_m = (prm.tiles_m + bands - 1) / bands;
    switch (g.p) {
        case 1: return block_launch_p1(prm, shape, s);
        case 2: return block_launch_p2(prm, shape, s);
        case 3: return block_launch_p3(prm, shape, s);
        case 4: return block_launch_p4(prm, shape, s);
        case 5: return block_launch_p5(prm, shape, s);
        case 6: return block_launch_p6(prm, shape, s);
        case 7: return block_launch_p7(prm, shape, s);
        default: return block_launch_p8(prm, shape, s);
    }
}

// ---- per-group weights
static const BkShapeInfo kG128Shapes[2] = {{256, 128, 1}, {128, 128, 2}};   // (as in block_g128_launch)

// Costs as above, from 1500 sizes of M = 48..2048 that the K-split kernel leaves; the tiled per-group kernel's by its tiles (64 x 64, 64 x 128).
static const struct { Cost block[2], tiled[2]; } kG128Costs[2] = {
    {{{0, 7.012f, {1.282f, 0, 0}}, {3.391f, 2.608f, {0.741f, 1.423f, 0}}},         // p = 1, 2, 4 (64 x 64: three workgroups a unit)
     {{0, 4.617f, {0, 0.466f, 0.705f}}, {3.42f, 2.239f, {0.417f, 0.89f, 0}}}},
    {{{0.394f, 6.649f, {1.388f, 0, 0}}, {3.63f, 2.345f, {0.816f, 1.542f, 0}}},     // p = 3, 5, 6
     {{3.511f, 0.924f, {0.233f, 0.548f, 0}}, {3.28f, 2.088f, {0.471f, 1.026f, 0}}}},
};

// The cheaper shape where it is 6 % below the tiled per-group kernel, on more than twelve groups of K (up to there the rounds' own
// cost decides, and this kernel takes 1.10 times the other's time on average).  It takes a fifth of those sizes, at 0.88 times the time (W4A8 M=1024
// 5120->13824 157 / 130 us), and none at 1.03 times or more but one in a thousand.  7- and 8-bit weights have no room for z in the byte.
bool block_g128_plan(const GemmArgs& g, int* shape)
{
    if (g.p > 6 || g.K <= 1536) return false;
    const int env = tuning_env("ABQ_BLOCK");   // tuning builds: -1 off, 1 or 2 a shape
    if (env) { *shape = env - 1; return env > 0 && env <= 2; }
    const bool merged = g.p == 3 || g.p >= 5;
    const auto& w = kG128Costs[merged ? 1 : 0];
    double c[2];
    for (int i = 0; i < 2; ++i) c[i] = cost_of(w.block[i], g.M, g.N, g.K, kG128Shapes[i].bm, kG128Shapes[i].bn, kG128Shapes[i].occ);
    *shape = c[1] < c[0] ? 1 : 0;
    const int ntw = tiled_g128_ntw(g.M, g.N);
    return cost_of(w.tiled[ntw - 1], g.M, g.N, g.K, 64, 64 * ntw, ntw == 1 && !merged ? 3 : 2) * 0.94 >= c[*shape];
}

hipError_t launch_gemm_block_g128(const GemmArgs& g, const ActLayout& A, const WeightLayout& W, int shape, hipStream_t s)
{
    const int bm = kG128Shapes[shape].bm, bn = kG128Shapes[shape].bn;
    BlockG128Params prm;
    for (int i = 0; i < 3; ++i) prm.fields[i] = g.w_blob + W.off_fields[i];
    prm.gparams = g.w_blob + W.off_gparams;
    prm.a = g.act_blob + A.off_codes;
    prm.aparams = (const RowParams*)(g.act_blob + A.off_params);
    prm.y = g.y;
    prm.M = g.M; prm.N = g.N;
    prm.lda = A.Kp;
    prm.nsuper = A.Kp / kSuperK;
    prm.ntiles = W.NT;
    prm.oa = g.q == 8 ? 128 : 0;
    prm.tiles_m = (g.M + bm - 1) / bm;
    prm.tiles_n = (g.N + bn - 1) / bn;
    const int cap = 1024 / bm, bands = (prm.tiles_m + cap - 1) / cap;
    prm.band_m = (prm.tiles_m + bands - 1) / bands;
    switch (g.p) {
        case 1: return block_g128_launch_p1(prm, shape, s);
        case 2: return block_g128_launch_p2(prm, shape, s);
        case 3: return block_g128_launch_p3(prm, shape, s);
        case 4: return block_g128_launch_p4(prm, shape, s);
        case 5: return block_g128_launch_p5(prm, shape, s);
        case 6: return block_g128_launch_p6(prm, shape, s);
        default: return hipErrorInvalidValue;
    }
}

}  // namespace abq
