// Device code of the K-split prefill kernel and the templates that launch its variants.  Included by the host translation
// unit (abq_ksplit.hip) and by the translation units that hold the instantiations.
//
// Matmul for 17 rows of A and more where the output has few tiles per compute unit (batches of decoding requests, short
// prompts, narrow layers).  There the time is load latency, not arithmetic: a kernel whose waves share operands through LDS
// advances one load latency and one barrier per step of K, and few workgroups keep few bytes in flight.  Here the waves of a
// workgroup split K instead of the tile: every wave multiplies the whole workgroup tile (16 RT rows of A x 16 CT rows of W)
// over its own phases of 256 k (wave, wave + S, ...), both operands loaded into its own registers one phase (or half of one) ahead.
// Weights are multiplied from there; rows of A pass through a block of LDS that only their wave uses, to change lanes.  There is no
// barrier before the partial tiles meet in LDS at the end, so the waves never wait for each other; the operand bytes a compute unit
// pulls are the same (each wave its own k).  The price is RT x CT accumulator tiles in every wave.
// RAW: rows of A are unpacked codes (one byte each): masked to q bits and made signed in registers, their sums taken on the way,
// so a call needs no pack launch.  GQ: per-group weight parameters (groups of 128 along K); the groups of a wave's phases are
// flushed into binary32 partial tiles.
#pragma once
#include "abq_internal.h"

#include <type_traits>

namespace abq {

typedef int v4i __attribute__((ext_vector_type(4)));
typedef float v4f __attribute__((ext_vector_type(4)));
typedef unsigned int u4v __attribute__((ext_vector_type(4)));
typedef int v4i_byte __attribute__((ext_vector_type(4), aligned(1)));

struct KsplitParams {
    const u4v* fields[3];
    const uint8_t* a;            // packed rows (int8, stride lda) or unpacked codes
    const RowParams* aparams;    // packed rows
    const float* a_scale;        // unpacked codes
    const int32_t* a_zero;
    const RowParams* wparams;
    const u4v* gparams;          // GQ: [ntiles][nsuper][16 channels] records
    uint16_t* y;                 // may be null when rq.codes is given
    int32_t* acc;
    Requant rq;
    int M, N, K, lda, nsuper, ntiles;
    int oa, ow;
    uint32_t a_mask;             // (2^q - 1) in every byte
    int tiles_m, tiles_n, band_m;
    int phase_q, phase_r;        // phases of a wave: phase_q, one more in the first phase_r waves
};

// Registers of one phase (256 k) of one 16-row tile of W: a b-bit group takes max(b/2, 1) of its 1 KiB chunks (a 1-bit chunk spans
// both phases of a super-chunk and is fetched for each).
__host__ __device__ constexpr int ks_chunks(int b) { return b >= 2 ? b / 2 : 1; }
__host__ __device__ constexpr int ks_base(int p, int g)
{
    return g == 0 ? 0 : (g == 1 ? ks_chunks(group_width(p, 0)) : ks_chunks(group_width(p, 0)) + ks_chunks(group_width(p, 1)));
}
__host__ __device__ constexpr int ks_regs(int p) { return ks_base(p, group_count(p) - 1) + ks_chunks(group_width(p, group_count(p) - 1)); }

// One dword of a slice's operand (slice SL = 0..3 of the phase), all plane groups merged into one byte per weight.  1-bit groups
// have been shifted right by four times the phase's parity ahead of this.
template <int P, int SL, int G0 = 0>
__device__ __forceinline__ uint32_t ks_dword(const u4v* w, int j)
{
    constexpr int b = group_width(P, G0), shift = group_shift(P, G0), T = 8 / b;
    constexpr int local = b == 1 ? 0 : SL / T, t = b == 1 ? SL : SL % T;
    const uint32_t x = w[ks_base(P, G0) + local][j];
    uint32_t v;
    if constexpr (b == 8) {
        v = x;
    } else {
        constexpr int sh = b * t - shift;
        constexpr uint32_t mask = (((1u << b) - 1u) * 0x01010101u) << shift;
        if constexpr (sh > 0) v = (x >> sh) & mask;
        else if constexpr (sh < 0) v = (x << (-sh)) & mask;
        else v = x & mask;
    }
    if constexpr (G0 + 1 < group_count(P)) v |= ks_dword<P, SL, G0 + 1>(w, j);
    return v;
}
template <int P, int SL>
__device__ __forceinline__ v4i ks_operand(const u4v* w)
{
    v4i r;
#pragma unroll
    for (int j = 0; j < 4; ++j) r[j] = (int)ks_dword<P, SL>(w, j);
    return r;
}

// Per-group weights on 64 x 64 tiles exist for p = 7, 8 only: below, the tiled per-group kernel is ahead of them (see shape_by_rule).
__host__ __device__ constexpr bool ks_has_gq(int p, int tiles) { return p >= 7 || tiles < 16; }

// Workgroup shapes: index -> rows / 16, channels / 16, waves, halves of a phase that the rows of A are fetched in, waves per SIMD
// that the registers are held to.
template <int RT_, int CT_, int S_, int AH_, int OCC_>
struct KsShape {
    static constexpr int RT = RT_, CT = CT_, S = S_, AH = AH_, OCC = OCC_;
};

template <int P, class SH, bool RAW, bool GQ>
__global__ __launch_bounds__(64 * SH::S, SH::OCC) void ksplit_kernel(KsplitParams prm)
{
    constexpr int RT = SH::RT, CT = SH::CT, S = SH::S, AH = SH::AH, NSL = 4 / AH, PR = ks_regs(P);
    constexpr int kBM = 16 * RT, kBN = 16 * CT;
    // per wave: the rows of A on their way to the operand's order, later the partial tiles
    constexpr int kWaveLds = 1024 * (RT * CT > RT * NSL ? RT * CT : RT * NSL);
    __shared__ __align__(16) v4i lds[S * kWaveLds / 16];
    __shared__ RowParams par_a[kBM], par_w[kBN];
    __shared__ int32_t row_part[RAW && !GQ ? S : 1][kBM];
    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6), waves = blockDim.x >> 6;
    const int r = lane & 15, G = lane >> 4;
    // tile order: a contiguous run of the banded order per XCD (workgroup b runs on XCD b % 8), M fastest inside a band, so that
    // the workgroups of one XCD share rows of A and tiles of W through its L2
    const int nwg = prm.tiles_m * prm.tiles_n;
    const int xcd = blockIdx.x & 7, slot = blockIdx.x >> 3;
    const int per = nwg >> 3, rem = nwg & 7;
    const int vid = xcd * per + min(xcd, rem) + slot;
    const int band = vid / (prm.band_m * prm.tiles_n), in_band = vid - band * prm.band_m * prm.tiles_n;
    const int band_rows = min(prm.band_m, prm.tiles_m - band * prm.band_m);
    const int m_blk = band * prm.band_m + in_band % band_rows, n_blk = in_band / band_rows;
    const int m0 = m_blk * kBM, n0 = n_blk * kBN, tile0 = n_blk * CT;

    // the epilogue's parameters are requested first (their wait leaves the operand loads in flight), every load unconditional
    v4i pa{0, 0, 0, 0}, pw{0, 0, 0, 0};
    {
        const int m = min(m0 + min(tid, kBM - 1), prm.M - 1);
        if constexpr (RAW) { pa.y = __float_as_int(prm.a_scale[m]); pa.z = prm.a_zero[m]; }
        else pa = reinterpret_cast<const v4i*>(prm.aparams)[m];
        if constexpr (!GQ) pw = reinterpret_cast<const v4i*>(prm.wparams)[min(n0 + min(tid, kBN - 1), prm.N - 1)];
    }

    // Rows of A are requested in lane order: a load covers 8 rows x 128 k, lane l the 16 bytes at 16 (l % 8) of row l / 8, and a pair of
    // loads 16 rows.  In the MFMA operand's own order (16 rows x 64 k, neighbouring lanes in different rows) the same bytes keep
    // the address path busy several times as long: W8A8 M=512 11008->4096 55 us against 36.  The operand's order is restored through
    // a block of LDS that only this wave uses (no barrier): the 16 bytes of slice t, k block G, row r at 1024 t + 256 G +
    // 16 (r ^ (4 t + G)), so that neither the writes (one row, eight pieces) nor the reads (16 rows, one piece) meet on a bank.
    unsigned a_off[RT][2];
#pragma unroll
    for (int rt = 0; rt < RT; ++rt)
#pragma unroll
        for (int i = 0; i < 2; ++i)
            a_off[rt][i] = (unsigned)(min(m0 + 16 * rt + 8 * i + (lane >> 3), prm.M - 1) - m0) * (unsigned)prm.lda + (RAW ? 0u : 16u * (lane & 7));
    const uint8_t* const a_tile = prm.a + (size_t)m0 * prm.lda;

    // Loads of phase j: all unconditional.  Rows past M and tiles past the last re-read valid ones (never stored); unpacked rows are
    // clamped to their last 16 bytes and put right before use.
    typedef __attribute__((address_space(1))) uint8_t a_byte;
    typedef __attribute__((address_space(1))) typename std::conditional<RAW, v4i_byte, v4i>::type a_vec;   // (unpacked rows of any length start on any byte)
    auto load_a = [&](int j, int h, v4i (*a)[RT]) {
#pragma unroll
        for (int s = 0; s < NSL; s += 2) {
            const int k = 256 * j + 64 * (h * NSL + s);
            const unsigned kk = RAW ? (unsigned)min(k + 16 * (lane & 7), prm.K - 16) : 0u;
            const a_byte* base = (const a_byte*)(RAW ? a_tile : a_tile + k);
            // Scalar base + 32-bit lane offset where registers are short (left alone, the step goes into 64-bit lane addresses, 16
            // registers more, and 64 x 32 tiles at p = 7 are 2-5 % slower or go to scratch)
            if constexpr (!RAW && P == 7 && !GQ) asm("" : "+s"(base));
#pragma unroll
            for (int rt = 0; rt < RT; ++rt)
#pragma unroll
                for (int i = 0; i < 2; ++i) a[s + i][rt] = *reinterpret_cast<const a_vec*>(base + (a_off[rt][i] + kk));
        }
    };
    uint8_t* const a_lds = reinterpret_cast<uint8_t*>(&lds[wave * (kWaveLds / 16)]);
    const int w_pos = 256 * (lane & 7) + 16 * ((lane >> 3) ^ (lane & 7)), r_pos = 256 * G + 16 * (r ^ G);
    auto read_a = [&](int s, v4i* aop) {   // (4 t + G) ^ r = r ^ G ^ 4 for the second slice of a pair
        const uint8_t* const p = a_lds + 2048 * RT * (s >> 1) + 1024 * (s & 1) + (r_pos ^ (64 * (s & 1)));
#pragma unroll
        for (int rt = 0; rt < RT; ++rt) aop[rt] = *reinterpret_cast<const v4i*>(p + 2048 * rt);
    };
    auto load_w = [&](int j, u4v (*w)[PR], u4v* gq) {
        const int sc = j >> 1, ph = j & 1;
#pragma unroll
        for (int ct = 0; ct < CT; ++ct) {
            const int tile = min(tile0 + ct, prm.ntiles - 1);
            if constexpr (GQ) gq[ct] = prm.gparams[((size_t)tile * prm.nsuper + sc) * 16 + r];
#pragma unroll
            for (int g = 0; g < group_count(P); ++g) {
                const int b = group_width(P, g), cpp = ks_chunks(b);
                const u4v* const base = prm.fields[g] + (((size_t)tile * prm.nsuper + sc) * b + (b == 1 ? 0 : cpp * ph)) * 64;
#pragma unroll
                for (int i = 0; i < cpp; ++i) w[ct][ks_base(P, g) + i] = base[i * 64 + lane];
            }
        }
    };

    typedef typename std::conditional<GQ, v4f, v4i>::type acc_t;
    acc_t acc[RT][CT];
#pragma unroll
    for (int rt = 0; rt < RT; ++rt)
#pragma unroll
        for (int ct = 0; ct < CT; ++ct) acc[rt][ct] = acc_t{0, 0, 0, 0};
    int code_sum[RT][2];   // of the operand bytes: the codes less oa
#pragma unroll
    for (int rt = 0; rt < RT; ++rt) code_sum[rt][0] = code_sum[rt][1] = 0;
    int nzc[GQ ? RT : 1][4];   // GQ: the token's zero-points of the accumulator rows, less oa, negated

    const uint32_t flip = prm.oa ? 0x80808080u : 0u;
    // loaded rows -> LDS; RAW: codes -> signed operand bytes (bits above q dropped, as the packers drop them), zero past K, and their sums
    auto stage_part = [&](auto TC, int klive, v4i (*a)[RT]) {
        constexpr bool TAIL = decltype(TC)::value;
#pragma unroll
        for (int s = 0; s < NSL; s += 2) {
            // TAIL: the loads began `sh` bytes early, and `live` bytes of a lane's vectors lie inside their rows.  Masks once for all rows: a wave
            // that ends in a tail is the last of its workgroup, and the compiler merges masks written per vector only by chance (per vector / once,
            // unpacked rows, 70 sizes: 32 x 16 tiles 0.957, 32 x 32 0.980, 64 x 32 0.926 times; W3A5 77x1003x4091 7.67 -> 7.53 us a pass).
            const int live = klive - 64 * s - 16 * (lane & 7), sh = max(16 - live, 0);
            uint32_t keep[4], fl[4];
#pragma unroll
            for (int d = 0; d < 4; ++d) {
                const uint32_t inside = TAIL ? (uint32_t)((1ull << (8 * min(max(live - 4 * d, 0), 4))) - 1) : ~0u;
                keep[d] = prm.a_mask & inside;
                fl[d] = flip & inside;
            }
#pragma unroll
            for (int rt = 0; rt < RT; ++rt)
#pragma unroll
                for (int i = 0; i < 2; ++i) {
                    v4i v = a[s + i][rt];
                    if constexpr (RAW) {
                        if constexpr (TAIL) {
                            if (sh > 0) {
                                if (sh & 8) v = v4i{v.z, v.w, 0, 0};
                                if (sh & 4) v = v4i{v.y, v.z, v.w, 0};
                                const uint32_t bits = 8 * (sh & 3);
                                v = v4i{(int)__builtin_amdgcn_alignbit((uint32_t)v.y, (uint32_t)v.x, bits), (int)__builtin_amdgcn_alignbit((uint32_t)v.z, (uint32_t)v.y, bits),
                                        (int)__builtin_amdgcn_alignbit((uint32_t)v.w, (uint32_t)v.z, bits), (int)((uint32_t)v.w >> bits)};
                            }
                        }
#pragma unroll
                        for (int d = 0; d < 4; ++d) {
                            v[d] = (int)(((uint32_t)v[d] & keep[d]) ^ fl[d]);
                            if constexpr (!GQ) code_sum[rt][i] = __builtin_amdgcn_sdot4(v[d], 0x01010101, code_sum[rt][i], false);
                        }
                    }
                    *reinterpret_cast<v4i*>(a_lds + 1024 * RT * s + 2048 * rt + (w_pos ^ (128 * i))) = v;
                }
        }
    };
    auto stage_a = [&](int j, int h, v4i (*a)[RT]) {
        const int klive = prm.K - (256 * j + 64 * h * NSL);
        // (the same for every lane; per-group weights hold their zero-point past K, so whatever stands there adds nothing)
        if (RAW && !GQ && klive < 64 * NSL) stage_part(std::true_type{}, klive, a);
        else stage_part(std::false_type{}, klive, a);
    };
    // 1-bit groups: the phase's four fields to the low half of the byte
    auto prepare_w = [&](int j, u4v (*w)[PR]) {
#pragma unroll
        for (int g = 0; g < group_count(P); ++g)
            if (group_width(P, g) == 1) {
                const int sh = 4 * (j & 1);
#pragma unroll
                for (int ct = 0; ct < CT; ++ct) w[ct][ks_base(P, g)] = w[ct][ks_base(P, g)] >> (unsigned)sh;
            }
    };
    // slices SL0 .. of the phase against the operands a[0..NSL-1]
    auto multiply = [&](auto HC, const u4v (*w)[PR]) {
        constexpr int H = decltype(HC)::value;
        auto slice = [&](auto SC) {
            constexpr int s = decltype(SC)::value, SL = H * NSL + s;
            v4i a[RT];
            read_a(s, a);
#pragma unroll
            for (int ct = 0; ct < CT; ++ct) {
                const v4i b = ks_operand<P, SL>(w[ct]);
#pragma unroll
                for (int rt = 0; rt < RT; ++rt) acc[rt][ct] = __builtin_amdgcn_mfma_i32_16x16x64_i8(b, a[rt], acc[rt][ct], 0, 0, 0);
            }
            __builtin_amdgcn_sched_barrier(0);   // (left alone, all slices' operands are expanded ahead and the registers run out)
        };
        slice(std::integral_constant<int, 0>{});
        slice(std::integral_constant<int, 1>{});
        if constexpr (NSL == 4) {
            slice(std::integral_constant<int, 2>{});
            slice(std::integral_constant<int, 3>{});
        }
    };
    // The same for per-group parameters: two slices are one group.  The A operand comes first here, so a lane's accumulators are four
    // rows of one channel, whose scale and zero-point are the lane's own record.  p <= 6: the operand byte is w - z (two's
    // complement: 128 + w - z never borrows from its neighbour, for zero-points of 0..2^p-1), what is left is the token's
    // zero-point; p = 7, 8: both corrections from operand sums, as in tiled_g128_kernel.
    auto multiply_g128 = [&](auto HC, int j, const u4v (*w)[PR], const u4v* gq) {
        constexpr int H = decltype(HC)::value;
        const v4i ones{0x01010101, 0x01010101, 0x01010101, 0x01010101}, zero4{0, 0, 0, 0};
        auto group = [&](auto JC) {
            constexpr int s0 = 2 * decltype(JC)::value, SL = H * NSL + s0;
            const int gj = 2 * (j & 1) + SL / 2;     // group of the super-chunk
            v4i a0[RT], a1[RT], asum[P > 6 ? RT : 1];
            read_a(s0, a0);
            read_a(s0 + 1, a1);
            if constexpr (P > 6) {
#pragma unroll
                for (int rt = 0; rt < RT; ++rt) {
                    asum[rt] = __builtin_amdgcn_mfma_i32_16x16x64_i8(a0[rt], ones, zero4, 0, 0, 0);
                    asum[rt] = __builtin_amdgcn_mfma_i32_16x16x64_i8(a1[rt], ones, asum[rt], 0, 0, 0);
                }
            }
#pragma unroll
            for (int ct = 0; ct < CT; ++ct) {
                const int z = ((int)(gq[ct].z << (24 - 8 * gj))) >> 24;
                const uint32_t sbits = ((j & 1) ? gq[ct].y : gq[ct].x) >> (16 * (SL / 2));
                const float sc = __half2float(__ushort_as_half((unsigned short)(sbits & 0xFFFFu)));
                v4i b0 = ks_operand<P, SL>(w[ct]), b1 = ks_operand<P, SL + 1>(w[ct]);
                if constexpr (P <= 6) {
                    const uint32_t off = __builtin_amdgcn_perm(0u, (uint32_t)(128 - z), 0u);   // its low byte in all four
#pragma unroll
                    for (int d = 0; d < 4; ++d) {
                        b0[d] = (int)(((uint32_t)b0[d] + off) ^ 0x80808080u);
                        b1[d] = (int)(((uint32_t)b1[d] + off) ^ 0x80808080u);
                    }
                }
                v4i wsum = __builtin_amdgcn_mfma_i32_16x16x64_i8(ones, b0, zero4, 0, 0, 0);
                wsum = __builtin_amdgcn_mfma_i32_16x16x64_i8(ones, b1, wsum, 0, 0, 0);   // every row: the column's sum
                const int wz = P <= 6 ? wsum.x : wsum.x - 128 * z;
#pragma unroll
                for (int rt = 0; rt < RT; ++rt) {
                    v4i c = __builtin_amdgcn_mfma_i32_16x16x64_i8(a0[rt], b0, zero4, 0, 0, 0);
                    c = __builtin_amdgcn_mfma_i32_16x16x64_i8(a1[rt], b1, c, 0, 0, 0);
#pragma unroll
                    for (int reg = 0; reg < 4; ++reg) {
                        int t = __mul24(nzc[rt][reg], wz) + c[reg];
                        if constexpr (P > 6) t += __mul24(-z, asum[rt][reg]);
                        acc[rt][ct][reg] = fmaf((float)t, sc, acc[rt][ct][reg]);
                    }
                }
            }
            __builtin_amdgcn_sched_barrier(0);
        };
        group(std::integral_constant<int, 0>{});
        if constexpr (NSL == 4) group(std::integral_constant<int, 1>{});
    };
    auto compute = [&](auto HC, int j, v4i (*a)[RT], const u4v (*w)[PR], const u4v* gq) {
        __builtin_amdgcn_sched_barrier(0);
        stage_a(j, decltype(HC)::value, a);
        if constexpr (GQ) multiply_g128(HC, j, w, gq);
        else multiply(HC, w);
    };
    typedef std::integral_constant<int, 0> H0;
    typedef std::integral_constant<int, 1> H1;

    v4i a0[NSL][RT], a1[NSL][RT];
    u4v w0[CT][PR], w1[CT][PR], g0[CT], g1[CT];
    int j = wave, n = prm.phase_q + (wave < prm.phase_r ? 1 : 0);
    constexpr bool kSwapA = AH == 1;   // (with halves the buffers of A are back in place after a phase)
    // An even number of phases starts in the other buffers, so that every wave ends in the same ones (64-row tiles short of registers; see below)
    constexpr bool kOneEnd = RT == 4 && (CT == 2 ? GQ || RAW || P == 7 : !GQ || (P == 7 && !RAW));
    const bool even = kOneEnd && (n & 1) == 0;
    if (even) {
        load_w(j, w1, g1);
        load_a(j, 0, kSwapA ? a1 : a0);
    } else {
        load_w(j, w0, g0);
        load_a(j, 0, a0);
    }
    if (tid < kBM) *reinterpret_cast<v4i*>(&par_a[tid]) = pa;
    if (!GQ && tid < kBN) *reinterpret_cast<v4i*>(&par_w[tid]) = pw;
    if constexpr (GQ) {
        __syncthreads();
#pragma unroll
        for (int rt = 0; rt < RT; ++rt)
#pragma unroll
            for (int reg = 0; reg < 4; ++reg) nzc[rt][reg] = prm.oa - par_a[16 * rt + 4 * G + reg].zero;
    }
    // One phase with the next one's loads under it, and the wave's last phase, which stands outside the loop, so that no load is issued
    // for a phase that does not exist and every wait counts exactly the loads behind it.
    auto phase = [&](u4v (*w)[PR], u4v* gq, u4v (*wn)[PR], u4v* gqn, v4i (*a)[RT], v4i (*an)[RT]) {
        const int jn = j + waves;
        if constexpr (AH == 1) {
            load_w(jn, wn, gqn);
            load_a(jn, 0, an);
            prepare_w(j, w);
            compute(H0{}, j, a, w, gq);
        } else {
            load_a(j, 1, an);
            prepare_w(j, w);
            compute(H0{}, j, a, w, gq);
            load_w(jn, wn, gqn);
            load_a(jn, 0, a);
            compute(H1{}, j, an, w, gq);
        }
        j = jn;
    };
    auto last_phase = [&](u4v (*w)[PR], u4v* gq, v4i (*a)[RT], v4i (*an)[RT]) {
        if constexpr (AH == 2) load_a(j, 1, an);
        prepare_w(j, w);
        compute(H0{}, j, a, w, gq);
        if constexpr (AH == 2) compute(H1{}, j, an, w, gq);
    };
    if constexpr (kOneEnd) {
        // One last phase for both parities.  With one for each, as below, the buffers of one end stay alive across the other, and
        // 64-row tiles went to scratch (M=256 1920 ch, K=2048, packed rows: per-group p = 3, 5, 7, 8 8.4, 10.0, 14.8, 8.7 us, now
        // 6.9, 7.0, 7.9, 7.5; per-channel p = 7 8.2, now 6.6).  32-row tiles have the registers, and a short K is 2-4 % faster without a
        // choice of buffers ahead of its first loads; so have the other per-group 64 x 64 tiles (M=512 2000 ch, K=8192 34.5 / 35.6), and 64 x 32
        // tiles of packed rows but for p = 7: there one end is 1 % faster where every wave has an odd count, and 1-2 % slower, up to 3, elsewhere
        // (125 sizes).
        if (even) phase(w1, g1, w0, g0, kSwapA ? a1 : a0, kSwapA ? a0 : a1);
        for (; n > 2; n -= 2) {
            phase(w0, g0, w1, g1, a0, a1);
            phase(w1, g1, w0, g0, kSwapA ? a1 : a0, kSwapA ? a0 : a1);
        }
        last_phase(w0, g0, a0, a1);
    } else {
        for (; n > 2; n -= 2) {
            phase(w0, g0, w1, g1, a0, a1);
            phase(w1, g1, w0, g0, kSwapA ? a1 : a0, kSwapA ? a0 : a1);
        }
        if (n == 2) {
            phase(w0, g0, w1, g1, a0, a1);
            last_phase(w1, g1, kSwapA ? a1 : a0, kSwapA ? a0 : a1);
        } else {
            asm volatile("; one phase" ::: "memory");
            last_phase(w0, g0, a0, a1);
        }
    }

    // the waves' partial tiles meet in LDS
#pragma unroll
    for (int rt = 0; rt < RT; ++rt)
#pragma unroll
        for (int ct = 0; ct < CT; ++ct) *reinterpret_cast<acc_t*>(a_lds + (rt * CT + ct) * 1024 + lane * 16) = acc[rt][ct];
    if constexpr (RAW && !GQ) {
#pragma unroll
        for (int rt = 0; rt < RT; ++rt) {
#pragma unroll
            for (int i = 0; i < 2; ++i) {
                int v = code_sum[rt][i];
                v += __shfl_xor(v, 1, 64);
                v += __shfl_xor(v, 2, 64);
                v += __shfl_xor(v, 4, 64);
                if ((lane & 7) == 0) row_part[wave][16 * rt + 8 * i + (lane >> 3)] = v;
            }
        }
    }
    __syncthreads();
    for (int v = wave; v < RT * CT; v += waves) {
        const int rt = v / CT, ct = v % CT;
        acc_t t = *reinterpret_cast<const acc_t*>(&lds[v * 64 + lane]);
        for (int s = 1; s < waves; ++s) t += *reinterpret_cast<const acc_t*>(&lds[s * (kWaveLds / 16) + v * 64 + lane]);
        if constexpr (GQ) {
            const int n = n0 + 16 * ct + r;
#pragma unroll
            for (int reg = 0; reg < 4; ++reg) {
                const int ml = 16 * rt + 4 * G + reg, m = m0 + ml;
                const float val = par_a[ml].scale * t[reg];
                uint32_t h;
                asm("v_cvt_f16_f32 %0, %1" : "=v"(h) : "v"(val));
                if (m < prm.M && n < prm.N) prm.y[(size_t)m * prm.N + n] = (uint16_t)h;
            }
        } else {
            const int ml = 16 * rt + r, m = m0 + ml, nl = 16 * ct + 4 * G, n = n0 + nl;
            RowParams ap = par_a[ml];
            if constexpr (RAW) {
                ap.sum = prm.oa * prm.K;
                for (int s = 0; s < waves; ++s) ap.sum += row_part[s][ml];
            }
            if (m < prm.M) {
                const size_t idx = (size_t)m * prm.N + n;
                if (prm.acc == nullptr && prm.rq.codes == nullptr && (prm.N & 3) == 0) {
                    if (n < prm.N) {   // (whole groups of four channels)
                        uint32_t hv[4];
                        int32_t raw;
#pragma unroll
                        for (int reg = 0; reg < 4; ++reg) hv[reg] = epilogue_value(t[reg], prm.oa, prm.ow, prm.K, ap, par_w[nl + reg], &raw);
                        uint2 h4;
                        h4.x = hv[0] | (hv[1] << 16);
                        h4.y = hv[2] | (hv[3] << 16);
                        *reinterpret_cast<uint2*>(prm.y + idx) = h4;
                    }
                } else {
#pragma unroll
                    for (int reg = 0; reg < 4; ++reg)
                        if (n + reg < prm.N) epilogue_store(t[reg], prm.oa, prm.ow, prm.K, ap, par_w[nl + reg], idx + reg, prm.y, prm.acc, prm.rq, m);
                }
            }
        }
    }
}

typedef KsShape<2, 1, 8, 1, 2> Ks21;
typedef KsShape<2, 2, 8, 1, 2> Ks22;
typedef KsShape<4, 2, 8, 2, 2> Ks42;
typedef KsShape<4, 4, 4, 2, 1> Ks44;

template <int P, class SH, bool RAW, bool GQ>
static hipError_t ks_launch_one(KsplitParams prm, hipStream_t s)
{
    const int nphase = 2 * prm.nsuper, waves = nphase < SH::S ? nphase : SH::S;
    prm.phase_q = nphase / waves;
    prm.phase_r = nphase % waves;
    ksplit_kernel<P, SH, RAW, GQ><<<dim3((unsigned)(prm.tiles_m * prm.tiles_n)), 64 * waves, 0, s>>>(prm);
    return hipGetLastError();
}
template <int P, class SH>
static hipError_t ks_launch_shape(const KsplitParams& prm, bool raw, bool gq, hipStream_t s)
{
    if (gq) {
        if constexpr (ks_has_gq(P, SH::RT * SH::CT)) return raw ? ks_launch_one<P, SH, true, true>(prm, s) : ks_launch_one<P, SH, false, true>(prm, s);
        else return hipErrorInvalidValue;
    }
    return raw ? ks_launch_one<P, SH, true, false>(prm, s) : ks_launch_one<P, SH, false, false>(prm, s);
}
template <int P>
static hipError_t ks_launch_p(const KsplitParams& prm, int shape, bool raw, bool gq, hipStream_t s)
{
    switch (shape) {
        case 0: return ks_launch_shape<P, Ks21>(prm, raw, gq, s);
        case 1: return ks_launch_shape<P, Ks22>(prm, raw, gq, s);
        case 2: return ks_launch_shape<P, Ks42>(prm, raw, gq, s);
        default: return ks_launch_shape<P, Ks44>(prm, raw, gq, s);
    }
}
hipError_t ksplit_launch_p1(const KsplitParams& prm, int shape, bool raw, bool gq, hipStream_t s);
hipError_t ksplit_launch_p2(const KsplitParams& prm, int shape, bool raw, bool gq, hipStream_t s);
hipError_t ksplit_launch_p3(const KsplitParams& prm, int shape, bool raw, bool gq, hipStream_t s);
hipError_t ksplit_launch_p4(const KsplitParams& prm, int shape, bool raw, bool gq, hipStream_t s);
hipError_t ksplit_launch_p5(const KsplitParams& prm, int shape, bool raw, bool gq, hipStream_t s);
hipError_t ksplit_launch_p6(const KsplitParams& prm, int shape, bool raw, bool gq, hipStream_t s);
hipError_t ksplit_launch_p7(const KsplitParams& prm, int shape, bool raw, bool gq, hipStream_t s);
hipError_t ksplit_launch_p8(const KsplitParams& prm, int shape, bool raw, bool gq, hipStream_t s);

}  // namespace abq
