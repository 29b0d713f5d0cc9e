// Host side of the block kernels: the choice of shape and the launch.
#include "abq_block_g128_kernels.h"

namespace abq {

struct BkShapeInfo { int bm, bn, occ; };   // rows of A, channels, workgroups a compute unit (as in block_launch)
constexpr int kBlockShapes = 5;
static const BkShapeInfo kShapes[kBlockShapes] = {{256, 256, 1}, {128, 192, 1}, {128, 128, 1}, {128, 128, 2}, {64, 128, 2}};
static int shape_bn(int p, int shape) { return shape == 0 && p == 7 ? 192 : kShapes[shape].bn; }

// What a launch costs (us): `base`, `round` for every round of resident workgroups (first loads, epilogue, and the gap to the next workgroup),
// per step of 128 k what a unit with 1, 2 or 3 of the shape's workgroups takes, and `ragged` for every workgroup a unit gets where rows of Y
// start off 16-byte boundaries (N % 8 != 0; the tiled kernels then store one half at a time, a quarter to a third of such a launch).  Least squares of
// the relative error with step costs that do not fall with the number of workgroups and rise no faster than it, over 5200 sizes that the K-split kernel leaves
// (M = 49..2048, N = 256..13824, K = 512..13824), each timed on operands in cache and on weights from memory; mean error of an entry 2 to 7 %.
struct Cost { float base, round, step[3], ragged; };
struct WidthCosts { Cost block[kBlockShapes], tiled[4]; };   // tiled: 64 x 64, 64 x 128, the width's large tile (64 x 256 for p = 1, 2, 4, else 128 x 128), 128 x 64
static const WidthCosts kCosts[8] = {
    {{{0, 9.054f, {0.94f, 0, 0}, 2.41f}, {1.365f, 4.576f, {0.456f, 0, 0}, 2.177f}, {},
      {2.58f, 2.874f, {0.356f, 0.637f, 0}, 0.714f}, {3.569f, 0.936f, {0.233f, 0.337f, 0}, 0.396f}},   // p = 1
     {{0, 4.617f, {0.139f, 0.262f, 0.372f}, 2.103f}, {4.879f, 1.175f, {0.207f, 0.396f, 0.54f}, 3.21f},
      {7.364f, 1.638f, {0.313f, 0.625f, 0}, 4.286f}}},
    {{{0, 9.12f, {0.959f, 0, 0}, 2.182f}, {1.209f, 4.577f, {0.493f, 0, 0}, 1.943f}, {},
      {1.932f, 3.411f, {0.385f, 0.666f, 0}, 0.572f}, {3.595f, 0.969f, {0.267f, 0.367f, 0}, 0.284f}},   // p = 2
     {{0, 4.577f, {0.16f, 0.279f, 0.377f}, 2.038f}, {4.328f, 1.945f, {0.197f, 0.394f, 0.546f}, 3.166f},
      {7.038f, 1.667f, {0.327f, 0.653f, 0}, 4.287f}}},
    {{{0, 9.445f, {1.145f, 0, 0}, 2.878f}, {1.09f, 5.101f, {0.64f, 0, 0}, 2.343f}, {},
      {3.441f, 2.419f, {0.489f, 0.856f, 0}, 0.777f}, {4.301f, 0.598f, {0.324f, 0.464f, 0}, 0.541f}},   // p = 3
     {{0, 4.676f, {0.162f, 0.323f, 0.475f}, 2.066f}, {4.375f, 2.142f, {0.26f, 0.519f, 0.7f}, 3.084f},
      {5.128f, 3.109f, {0.439f, 0.833f, 0}, 6.206f}}},
    {{{0, 8.805f, {1.02f, 0, 0}, 2.389f}, {0.418f, 5.744f, {0.438f, 0, 0}, 2.173f}, {1.55f, 3.841f, {0.34f, 0, 0}, 0.785f},
      {0.224f, 4.041f, {0.555f, 0.76f, 0}, 0.872f}, {2.241f, 2.414f, {0.222f, 0.408f, 0}, 0.428f}},   // p = 4
     {{0, 4.603f, {0.162f, 0.305f, 0.457f}, 2.078f}, {3.524f, 2.735f, {0.228f, 0.43f, 0.625f}, 3.196f},
      {5.184f, 3.201f, {0.46f, 0.768f, 0}, 4.556f}}},
    {{{0, 9.345f, {1.117f, 0, 0}, 2.007f}, {0.704f, 5.726f, {0.601f, 0, 0}, 2.034f}, {1.804f, 3.655f, {0.452f, 0, 0}, 0.64f},
      {1.787f, 3.265f, {0.596f, 0.9f, 0}, 0.588f}, {2.693f, 2.083f, {0.301f, 0.504f, 0}, 0.393f}},   // p = 5
     {{0, 4.698f, {0.197f, 0.348f, 0.522f}, 1.93f}, {4.768f, 1.975f, {0.289f, 0.541f, 0.782f}, 3.157f},
      {4.885f, 3.359f, {0.476f, 0.874f, 0}, 6.386f}}},
    {{{0, 9.588f, {1.147f, 0, 0}, 2.184f}, {0.786f, 5.669f, {0.637f, 0, 0}, 2.121f}, {1.685f, 3.777f, {0.481f, 0, 0}, 0.859f},
      {1.354f, 3.646f, {0.619f, 0.924f, 0}, 0.871f}, {2.481f, 2.224f, {0.353f, 0.537f, 0}, 0.549f}},   // p = 6
     {{0, 4.565f, {0.202f, 0.354f, 0.531f}, 2.136f}, {4.878f, 1.738f, {0.416f, 0.545f, 0.798f}, 3.207f},
      {4.945f, 3.576f, {0.497f, 0.859f, 0}, 6.374f}}},
    {{{0, 8.642f, {1.151f, 0, 0}, 3.241f}, {1.369f, 5.472f, {0.866f, 0, 0}, 1.997f}, {2.091f, 3.84f, {0.61f, 0, 0}, 0.632f},
      {3.73f, 2.26f, {0.715f, 1.174f, 0}, 0.653f}, {3.774f, 1.503f, {0.435f, 0.676f, 0}, 0.391f}},   // p = 7
     {{0, 5.02f, {0.277f, 0.428f, 0.642f}, 1.938f}, {6.044f, 1.491f, {0.362f, 0.703f, 0.986f}, 3.046f},
      {5.694f, 3.337f, {0.544f, 1.029f, 0}, 6.215f}, {0, 6.886f, {0.506f, 0.625f, 0}, 4.222f}}},
    {{{0, 8.824f, {1.103f, 0, 0}, 2.807f}, {0.755f, 5.422f, {0.572f, 0, 0}, 2.353f}, {1.63f, 3.505f, {0.41f, 0, 0}, 0.702f},
      {0, 4.244f, {0.659f, 0.856f, 0}, 0.882f}, {2.627f, 1.853f, {0.331f, 0.593f, 0}, 0.442f}},   // p = 8
     {{0, 4.608f, {0.194f, 0.378f, 0.567f}, 2.012f}, {4.693f, 1.574f, {0.369f, 0.592f, 0.871f}, 3.188f},
      {3.778f, 4.781f, {0.592f, 0.807f, 0}, 6.251f}}},
};

static double cost_of(const Cost& c, int M, int N, int K, int bm, int bn, int occ)
{
    const long wgs = (long)((M + bm - 1) / bm) * ((N + bn - 1) / bn), cus = num_cus();
    const long load = (wgs + cus - 1) / cus, full = load / occ, part = load % occ;
    const double steps = 4.0 * ((K + kSuperK - 1) / kSuperK);
    return c.base + c.round * (double)(full + (part > 0)) + steps * ((double)full * c.step[occ - 1] + (part ? c.step[part - 1] : 0.f)) + (N % 8 ? c.ragged * (double)load : 0.0);
}

// The cheapest shape by the costs above, unless the tiled kernel's is 5 % below it (its 64 x 64 tiles, three workgroups a unit, where K is short or the
// output leaves the larger tiles' last round nearly empty; W6A6 M=128 4096->11008 with its quantizer 17.1 us there, 18.2 on 64 x 128 here).  Over those sizes
// the choice takes 0.86 times the tiled kernel's time in cache and 0.85 times from memory, 0.84 for p = 1, 2, 4, 8 and 0.88 for the others; 0.3 % of the sizes lose
// 3 to 8 % in cache, 1.5 % lose 3 to 19 % from memory.  (Costs that were the same for all N, with steps that cost nothing at some loads, from times in cache alone: 2.3 %
// of the sizes slower than the tiled kernel by more than 3 %, 7.9 % from memory, W2A8 M=68 8958->8480 32 us against 27.)
// A plan-table entry with a knob of the tiled kernel asks for that; so does a call for the int32 accumulator, which only that kernel writes.
bool block_plan(const GemmArgs& g, const WeightLayout& W, int* shape)
{
    if (W.g128 || g.acc) return false;
    PlanOverride ov;
    if (lookup_plan(g.p, g.q, g.M, g.N, g.K, &ov) && (ov.tiled_mt > 0 || ov.tiled_ntw > 0 || ov.tiled_wd > 0 || ov.tiled_band > 0)) return false;
    const int env = tuning_env("ABQ_BLOCK");   // tuning builds: -1 off, 1..5 a shape
    if (env) { *shape = env - 1; return env > 0 && env <= kBlockShapes; }
    const WidthCosts& w = kCosts[g.p - 1];
    double best = 0;
    for (int i = 0; i < kBlockShapes; ++i) {
        if (w.block[i].step[0] == 0) continue;   // (not built)
        const double c = cost_of(w.block[i], g.M, g.N, g.K, kShapes[i].bm, shape_bn(g.p, i), kShapes[i].occ);
        if (i == 0 || c < best) { best = c; *shape = i; }
    }
    int mt, ntw;
    tiled_shape_by_rule(g.p, g.M, g.N, g.K, &mt, &ntw);
    const bool large = mt == 8 || ntw == 4;
    return cost_of(w.tiled[large ? (mt == 8 && ntw == 1 ? 3 : 2) : ntw - 1], g.M, g.N, g.K, 16 * mt, 64 * ntw, large ? 2 : 3) * 0.95 >= best;
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

// Costs as above, from 2300 sizes of M = 49..2048, K > 1536 that the K-split kernel leaves; the tiled per-group kernel's by its tiles (64 x 64, 64 x 128).
static const struct { Cost block[2], tiled[2]; } kG128Costs[2] = {
    {{{0, 5.76f, {1.266f, 0, 0}, 1.472f}, {5.255f, 0, {0.756f, 1.326f, 0}, 0.867f}},   // p = 1, 2, 4 (64 x 64: three workgroups a unit)
     {{0, 4.09f, {0.288f, 0.482f, 0.683f}, 1.972f}, {5.702f, 0.444f, {0.406f, 0.803f, 0}, 3.047f}}},
    {{{0, 6.019f, {1.374f, 0, 0}, 1.413f}, {5.457f, 0, {0.827f, 1.446f, 0}, 0.773f}},   // p = 3, 5, 6
     {{4.838f, 0, {0.266f, 0.532f, 0}, 1.948f}, {6.4f, 0.346f, {0.469f, 0.93f, 0}, 2.917f}}},
};

// The cheaper shape where its cost is 3 % below the tiled per-group kernel's, on more than twelve groups of K (up to there the rounds' own
// cost decides, and the better shape takes 1.10 times the other kernel's time on average).  It takes a third of those sizes,
// at 0.87 times the time (W4A4 M=2048 5120->13824 226 / 202 us in cache); 0.1 % of the sizes lose 3 to 8 % in cache, 0.4 % from memory.
// 7- and 8-bit weights have no room for z in the byte.
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
    return cost_of(w.tiled[ntw - 1], g.M, g.N, g.K, 64, 64 * ntw, ntw == 1 && !merged ? 3 : 2) * 0.97 >= c[*shape];
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
