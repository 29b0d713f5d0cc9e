// Host side of the block kernels: the choice of shape and the launch.
#include "abq_block_g128_kernels.h"

namespace abq {

struct BkShapeInfo { int bm, bn, occ; };   // rows of A, channels, workgroups a compute unit (as in block_launch)
constexpr int kBlockShapes = 5;
static const BkShapeInfo kShapes[kBlockShapes] = {{256, 256, 1}, {128, 192, 1}, {128, 128, 1}, {128, 128, 2}, {64, 128, 2}};
static int shape_bn(int p, int shape) { return shape == 0 && p == 7 ? 192 : kShapes[shape].bn; }

// What a launch costs (us): `base`, `round` for every round of resident workgroups (first loads, epilogue, and the gap to the next workgroup),
// and per step of 128 k what a unit with 1, 2 or 3 of the shape's workgroups takes.  Non-negative least squares of the relative error over
// 1830 sizes that the K-split kernel leaves (M = 49..2048, N = 256..13824, K = 512..13824), mean error 4 to 9 %, tiled 9 to 14 %.
struct Cost { float base, round, step[3]; };
struct WidthCosts { Cost block[kBlockShapes], tiled[3]; };   // tiled: 64 x 64, 64 x 128, 64 x 256
static const WidthCosts kCosts[6] = {
    {{{0, 9.144f, {0.985f, 0, 0}}, {0.391f, 5.682f, {0.469f, 0, 0}}, {1.124f, 3.7f, {0.344f, 0, 0}}, {1.943f, 3.554f, {0.343f, 0.679f, 0}}, {2.85f, 1.66f, {0.214f, 0.351f, 0}}},   // p = 1, 2
     {{4.87f, 0, {0.137f, 0.26f, 0.399f}}, {4.166f, 2.417f, {0, 0.409f, 0.59f}}, {5.59f, 2.758f, {0.336f, 0.758f, 0}}}},
    {{{0, 9.718f, {1.153f, 0, 0}}, {0.81f, 5.817f, {0.627f, 0, 0}}, {1.535f, 3.576f, {0.447f, 0, 0}}, {2.717f, 3.159f, {0.466f, 0.857f, 0}}, {3.741f, 1.113f, {0.271f, 0.475f, 0}}},   // p = 3
     {{0, 5.241f, {0.149f, 0.29f, 0.478f}}, {9.106f, 0.731f, {0, 0.492f, 0.649f}}, {}}},
    {{{0, 9.251f, {0.979f, 0, 0}}, {0, 6.093f, {0.453f, 0, 0}}, {1.017f, 4.042f, {0.347f, 0, 0}}, {0.065f, 3.967f, {0.452f, 0.766f, 0}}, {2.17f, 2.39f, {0.204f, 0.406f, 0}}},   // p = 4
     {{4.871f, 0, {0.147f, 0.277f, 0.444f}}, {2.393f, 3.984f, {0.459f, 0.467f, 0.652f}}, {}}},
    {{{0, 9.543f, {1.129f, 0, 0}}, {0.492f, 5.959f, {0.635f, 0, 0}}, {1.149f, 4.056f, {0.455f, 0, 0}}, {2.163f, 2.877f, {0.505f, 0.931f, 0}}, {2.248f, 2.435f, {0.286f, 0.504f, 0}}},   // p = 5, 6
     {{5.057f, 0, {0.158f, 0.31f, 0.526f}}, {6.833f, 0.752f, {0.341f, 0.574f, 0.853f}}, {}}},
    {{{0, 8.586f, {1.139f, 0, 0}}, {0.668f, 6.019f, {0.875f, 0, 0}}, {1.225f, 4.196f, {0.613f, 0, 0}}, {3.875f, 2.112f, {0.63f, 1.185f, 0}}, {3.137f, 1.839f, {0.384f, 0.675f, 0}}},   // p = 7
     {{4.901f, 0, {0.228f, 0.427f, 0.646f}}, {0.597f, 6.999f, {0, 0.621f, 1.126f}}, {}}},
    {{{0, 9.307f, {0.99f, 0, 0}}, {0, 6.138f, {0.541f, 0, 0}}, {0.046f, 4.672f, {0.366f, 0, 0}}, {0, 3.718f, {0.548f, 0.852f, 0}}, {1.545f, 2.573f, {0.283f, 0.555f, 0}}},   // p = 8
     {{4.162f, 0, {0.234f, 0.349f, 0.628f}}, {4.02f, 2.662f, {0, 0.594f, 0.86f}}, {}}},
};

static double cost_of(const Cost& c, int M, int N, int K, int bm, int bn, int occ)
{
    const long wgs = (long)((M + bm - 1) / bm) * ((N + bn - 1) / bn), cus = num_cus();
    const long load = (wgs + cus - 1) / cus, full = load / occ, part = load % occ;
    const double steps = 4.0 * ((K + kSuperK - 1) / kSuperK);
    return c.base + c.round * (double)(full + (part > 0)) + steps * ((double)full * c.step[occ - 1] + (part ? c.step[part - 1] : 0.f));
}

// The cheapest shape by the costs above, unless the tiled kernel's is 7 % below it, 10 % for widths of more than one plane group, whose tiled
// costs scatter more (its 64 x 64 tiles, three workgroups a unit, where K is short or the output leaves the larger tiles' last round
// nearly empty; W6A6 M=128 4096->11008 with its quantizer 17.1 us there, 18.2 here).  Over those sizes the choice takes 0.86 times the
// tiled kernel's time for p = 1, 2, 4, 8 and 0.93 times for the others; 2.0 and 0.7 % of the sizes lose 3 to 12 %.
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
    const double lead = group_count(g.p) > 1 ? 0.90 : 0.93;
    return cost_of(w.tiled[ntw / 2], g.M, g.N, g.K, 16 * mt, 64 * ntw, ntw == 4 ? 2 : 3) * lead >= best;
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

// Costs as above, from 1700 sizes of M = 48..2048, K > 1536 that the K-split kernel leaves; the tiled per-group kernel's by its tiles (64 x 64, 64 x 128).
static const struct { Cost block[2], tiled[2]; } kG128Costs[2] = {
    {{{0, 5.923f, {1.266f, 0, 0}}, {4.608f, 0.765f, {0.742f, 1.34f, 0}}},          // p = 1, 2, 4 (64 x 64: three workgroups a unit)
     {{0, 4.456f, {0, 0.465f, 0.694f}}, {4.193f, 1.724f, {0.436f, 0.865f, 0}}}},
    {{{0, 6.13f, {1.378f, 0, 0}}, {4.757f, 0.762f, {0.812f, 1.453f, 0}}},          // p = 3, 5, 6
     {{4.612f, 0.038f, {0.249f, 0.533f, 0}}, {5.148f, 1.313f, {0.476f, 0.989f, 0}}}},
};

// The cheaper shape where its cost is 6 % below the tiled per-group kernel's, on more than twelve groups of K (up to there the rounds' own
// cost decides, and the better shape takes 1.10 times the other kernel's time on average).  It takes a third of those sizes, at 0.86 times the time (W4A8
// M=1024 5120->13824 157 / 130 us); 0.5 % of the sizes lose 3 to 6 %.  7- and 8-bit weights have no room for z in the byte.
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
