// Host side of the K-split prefill kernel: the choice of shape and the launch.
#include "abq_ksplit_kernels.h"

namespace abq {

struct KsShapeInfo { int rt, ct; };
static const KsShapeInfo kShapes[4] = {{2, 1}, {2, 2}, {4, 2}, {4, 4}};   // (as in ks_launch_p)

// Unpacked rows on 64 x 64 tiles: the rows of A up to which they are packed first.  Masks, row sums and pieces of rows off 128-byte lines cost
// every tile a share of its own time, the pack launch some 2 us and the bytes of A once, and the more rows, the fewer tiles read each.
// This kernel alone / the pack launch and this kernel on packed rows, 1370 sizes of K >= 3072:
//   rows              17..64  65..128  ..192  ..256  ..384  ..512  ..1000
//   whole lines, p < 7  1.03    1.05    1.03   1.01   0.97   0.93   0.89;   p = 7, 8  0.98  0.97  0.99  0.95  0.96  0.90  0.85
//   dwords, p < 7       1.10    1.08    1.06   1.04   1.01   0.97   0.92;   p = 7, 8  1.05  1.05  1.04  1.02  0.99  0.96  0.92
//   others, p < 7       1.20    1.17    1.15   1.10   1.05   1.00   0.96;   p = 7, 8  1.13  1.10  1.08  1.10  0.94  -     0.95
static int packed_up_to(int p, int K)
{
    if (K % 128 == 0) return p >= 7 ? 0 : 256;
    return (K % 4 == 0 ? 384 : 512) - (p >= 7 ? 128 : 0);
}

// Shape: the smallest workgroup tile of which no compute unit gets more than one.  A workgroup's time goes with the operand bytes it
// pulls (about 30 bytes a clock per compute unit), and a second round of workgroups costs what the first did.  Against the other
// kernels (tiled, streaming; 957 sizes of M = 17..2048, N = 256..13824, K = 512..13824, all widths, packed and unpacked rows, per-channel
// and per-group weights, timed in replays) the choice below is 1.41 times as fast on average, 2.4 % from the best of all kernels and
// shapes at each size, and at most 7 % behind the others but for the per-group sizes named below.  Where the lines lie (this kernel / the others, us):
//   64 x 64, per-channel: the tiled kernel has overtaken while K is short (packed rows K < 1600 1.11 times, K = 3072..6144 0.92), up to
//     64 rows of p = 8 until K = 4608 (12880 ch x 3296, M = 38, with the pack launch in front of both: 16.9 / 15.9);
//   64 x 64, unpacked rows: see packed_up_to;
//   per-group: one answer for packed and unpacked rows, because the order of the binary32 sums goes with the kernel and a call on codes
//     returns the bits of packing and multiplying.  On 64 x 64 the tiled per-group kernel wins at p <= 6 (packed rows 0.75 to 0.94 times;
//     unpacked, behind a pack launch, 1.07 to 1.15) and below K = 2048 at p = 7, 8 (above 1.2 and more); on 64 x 32 it is even below
//     K = 1024 for packed rows (0.94 to 1.08; unpacked 1.5);
//   up to 48 rows, per-channel, K >= 3072: the streaming kernel splits K as well, over tiles of 16 rows (1536 ch x 10400, M = 25: 11.2 /
//     9.3; 512 ch x 5712, M = 44: 8.2 / 7.5).  With unpacked rows of a K that is no multiple of 16 it needs a pack launch and loses, and
//     above 8128 channels the prefill kernel would run in its place (8192 ch x 8192, M = 32: W5A8 12.9 / 21.4, W8A8 15.6 / 21.1).
static int shape_by_rule(const GemmArgs& g, const WeightLayout& W)
{
    int shape = 0;
    for (;; ++shape) {
        if (shape == 4) return -1;
        if ((long)((g.M + 16 * kShapes[shape].rt - 1) / (16 * kShapes[shape].rt)) * ((W.NT + kShapes[shape].ct - 1) / kShapes[shape].ct) <= (long)num_cus()) break;
    }
    const bool raw = g.a_raw != nullptr;
    if (W.g128) return shape == 3 && (g.p <= 6 || g.K < 2048) ? -1 : shape;
    if (shape == 3 && g.K < (g.p == 8 && g.M <= 64 ? 4608 : 3072)) return -1;
    if (shape == 3 && raw && g.M <= packed_up_to(g.p, g.K)) return -1;   // (packed first, and asked again)
    if (shape <= 1 && g.M <= 48 && g.K >= 3072 && (shape == 0 || g.p >= 5) && !(raw && g.K % 16 != 0) && streaming_shape(g.M, g.N)) return -1;
    return shape;
}

// False: another kernel takes the problem.
bool ksplit_plan(const GemmArgs& g, const ActLayout& A, const WeightLayout& W, int* shape)
{
    if (!W.has_fields || g.M <= 16) return false;
    // (unpacked rows: any length of at least one 16-byte load; per-group weights, of whole ones)
    if (g.a_raw ? g.K < 16 || (W.g128 && g.K % 16 != 0) : !A.has_fields) return false;
    if (W.g128 && (g.acc || g.rq.codes)) return false;
    // A plan-table entry is followed where it asks for a shape of the kernel that runs instead (per-channel only: the key does not tell
    // the kinds of blobs apart, and the per-group kernels above 16 rows have no knobs).
    PlanOverride ov;
    if (!W.g128 && lookup_plan(g.p, g.q, g.M, g.N, g.K, &ov) && (streaming_shape(g.M, g.N) ? skinny_entry_fits(g, A, W, ov) : ov.tiled_mt > 0 || ov.tiled_ntw > 0)) return false;
    const int env = tuning_env("ABQ_KS");   // tuning builds: -1 off, 1..4 a shape
    *shape = env < 0 ? -1 : (env >= 1 && env <= 4 && (!W.g128 || ks_has_gq(g.p, kShapes[env - 1].rt * kShapes[env - 1].ct)) ? env - 1 : shape_by_rule(g, W));
    return *shape >= 0;
}

hipError_t launch_gemm_ksplit(const GemmArgs& g, const ActLayout& A, const WeightLayout& W, int shape, hipStream_t s)
{
    const KsShapeInfo& sh = kShapes[shape];
    KsplitParams prm;
    for (int i = 0; i < 3; ++i) prm.fields[i] = (const u4v*)(g.w_blob + W.off_fields[i]);
    const bool raw = g.a_raw != nullptr;
    prm.a = raw ? g.a_raw : g.act_blob + A.off_codes;
    prm.aparams = raw ? nullptr : (const RowParams*)(g.act_blob + A.off_params);
    prm.a_scale = g.a_scale;
    prm.a_zero = g.a_zero;
    prm.wparams = (const RowParams*)(g.w_blob + W.off_params);
    prm.gparams = W.g128 ? (const u4v*)(g.w_blob + W.off_gparams) : nullptr;
    prm.y = g.y; prm.acc = g.acc; prm.rq = g.rq;
    prm.M = g.M; prm.N = g.N; prm.K = g.K;
    prm.lda = raw ? g.K : A.Kp;
    prm.nsuper = A.Kp / kSuperK;
    prm.ntiles = W.NT;
    prm.oa = g.q == 8 ? 128 : 0;
    prm.ow = g.p == 8 ? 128 : 0;
    prm.a_mask = ((1u << g.q) - 1u) * 0x01010101u;
    prm.tiles_m = (g.M + 16 * sh.rt - 1) / (16 * sh.rt);
    prm.tiles_n = (W.NT + sh.ct - 1) / sh.ct;
    // bands of equal height, as in the tiled kernel
    const int cap = (g.p <= 4 ? 512 : 1024) / (16 * sh.rt);
    const int bands = (prm.tiles_m + cap - 1) / cap;
    prm.band_m = (prm.tiles_m + bands - 1) / bands;
    switch (g.p) {
        case 1: return ksplit_launch_p1(prm, shape, raw, W.g128, s);
        case 2: return ksplit_launch_p2(prm, shape, raw, W.g128, s);
        case 3: return ksplit_launch_p3(prm, shape, raw, W.g128, s);
        case 4: return ksplit_launch_p4(prm, shape, raw, W.g128, s);
        case 5: return ksplit_launch_p5(prm, shape, raw, W.g128, s);
        case 6: return ksplit_launch_p6(prm, shape, raw, W.g128, s);
        case 7: return ksplit_launch_p7(prm, shape, raw, W.g128, s);
        default: return ksplit_launch_p8(prm, shape, raw, W.g128, s);
    }
}

}  // namespace abq
