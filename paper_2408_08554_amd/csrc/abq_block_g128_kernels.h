// Device code of the block kernel for per-group weights (a scale and a zero-point per 128 k, p <= 6) and the templates that launch
// its variants.  Loads, LDS ring and tile order are the block kernel's (abq_block_kernels.h); a step of 128 k is one group.
//
// A group's sums are integers: t = sum_k (a' - zc)(w' - z) = c - zc sum_k (w' - z), with c the product of the stored rows with the operand
// bytes w' - z (one add and one flip a dword of four: 128 + w' - z stays inside its byte), zc the token's zero-point less oa, and
// sum_k (w' - z) from an MFMA against ones.  They are flushed through the group's scale into binary32 tiles, group after group:
// the same integers in the same order as in the tiled kernel, so the results are the same bits.
//
// What bounds it is the vector ALU: a multiply-add, a conversion and a fused multiply-add per element and group (48 clocks a tile of 16 x 16, against 32 of
// its two MFMAs), and the operands' expansion.  Waves of 128 x 32 make that expansion serve eight tiles (the tiled kernel's 64 x 32: four), which leaves
// 73 clocks of vector issue a tile, and a row's flush runs under the next row's MFMAs.  Measured at 256 x 128: 2950-3030 clocks a step, of them 2340 of vector
// issue (586 instructions a SIMD, 78 %) and 1150 of MFMAs.  W4A8 M=1024 5120->13824 on the tiled kernel / 256 x 128 / 128 x 128, two a unit, replays in cache 122 / 115 /
// 114 us, from memory 127 / 120 / 119; W4A4 M=2048 226 / 225 / 202 and 231 / 231 / 205.  Three waves a SIMD (64 x 32 each) spill, two such are no faster.
#pragma once
#include "abq_block_kernels.h"

namespace abq {

typedef float v4f __attribute__((ext_vector_type(4)));

struct BlockG128Params {
    const uint8_t* fields[3];
    const uint8_t* gparams;      // records of 16 bytes: [ntiles][nsuper][16 channels] (four binary16 scales, four zero-points as bytes)
    const uint8_t* a;            // packed rows (int8, stride lda)
    const RowParams* aparams;
    uint16_t* y;
    int M, N, lda, nsuper, ntiles, oa;
    int tiles_m, tiles_n, band_m;
};

// A wave multiplies 16 MT rows by 16 NT channels; two places in the ring.
template <int P, int RW, int CW, int MT, int NT, int OCC>
__global__ __launch_bounds__(64 * RW * CW, OCC) void block_g128_kernel(BlockG128Params prm)
{
    constexpr int kWaves = RW * CW, kBM = 16 * MT * RW, kTW = NT * CW;
    constexpr int kABytes = kBM * kBkStep, kBuf = kABytes + kTW * bk_fast_chunks(P) * 1024;
    constexpr int kSlow = kTW * bk_slow_groups(P) * 1024;
    constexpr int kRecA = (kBM + 63) / 64, kRecG = (kTW + 3) / 4;       // wave loads of 64 records
    static_assert(P <= 6, "128 + w' - z has to stay inside a byte");
    __shared__ __align__(1024) uint8_t ring[2 * kBuf];
    __shared__ __align__(1024) uint8_t lds_slow[kSlow > 0 ? kSlow : 16];
    __shared__ __align__(16) uint8_t grec[kRecG * 1024];         // the super-chunk's group records, 256 bytes a tile
    __shared__ __align__(16) RowParams par_a[64 * kRecA];
    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int rw = wave / CW, cw = wave % CW;
    const int r = lane & 15, G = lane >> 4;
    const int nwg = prm.tiles_m * prm.tiles_n;
    const int xcd = blockIdx.x & 7, slot = blockIdx.x >> 3;
    const int per = nwg >> 3, rem = nwg & 7;
    const int vid = xcd * per + min(xcd, rem) + slot;
    const int band = vid / (prm.band_m * prm.tiles_n), in_band = vid - band * prm.band_m * prm.tiles_n;
    const int band_rows = min(prm.band_m, prm.tiles_m - band * prm.band_m);
    const int m_blk = band * prm.band_m + in_band % band_rows, n_blk = in_band / band_rows;
    const int m0 = m_blk * kBM, n0 = n_blk * 16 * kTW, tile0 = n_blk * kTW;
    const int nsteps = prm.nsuper * 4;

    // ---- loads (see block_kernel)
    auto lds_addr = [](const void* p) { return (unsigned)(uintptr_t)(const __attribute__((address_space(3))) uint8_t*)p; };
    auto lds_load = [](const void* base, unsigned off, unsigned dst) {
        asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %1, %2" : : "s"(dst), "v"(off), "s"(base) : "memory", "m0");
    };
    constexpr int kALoads = kBM / 8 / kWaves;
    unsigned a_goff[kALoads];
#pragma unroll
    for (int u = 0; u < kALoads; ++u) {
        const int row = 8 * (wave * kALoads + u) + (lane >> 3);
        a_goff[u] = (unsigned)(min(m0 + row, prm.M - 1) - m0) * (unsigned)prm.lda + ((lane & 7) ^ ((row >> 1) & 7)) * 16;
    }
    const uint8_t* a_tile = prm.a + (size_t)m0 * prm.lda;
    constexpr int kWLoads = (kTW + kWaves - 1) / kWaves, kChunks = bk_fast_chunks(P), kB0 = group_width(P, 0);
    int w_place[kWLoads], w_row[kWLoads];
    const uint8_t* w_tile[kWLoads];
#pragma unroll
    for (int u = 0; u < kWLoads; ++u) {
        w_place[u] = min(u * kWaves + wave, kTW - 1);
        w_row[u] = min(tile0 + w_place[u], prm.ntiles - 1);
        w_tile[u] = prm.fields[0] + (size_t)w_row[u] * (prm.nsuper * kB0) * 1024;
    }
    constexpr int kLoads = kALoads + kWLoads * kChunks;
    auto load_piece = [&](int i, int step, const uint8_t* buf) {
        if (i < kALoads) lds_load(a_tile + (size_t)step * kBkStep, a_goff[i], lds_addr(buf) + (wave * kALoads + i) * 1024);
        else if constexpr (kChunks > 0) {
            const int u = i - kALoads;
            lds_load(w_tile[u], lane * 16 + step * 1024, lds_addr(buf) + kABytes + w_place[u] * 1024);
        }
    };
    const uint8_t* rec_base = prm.gparams + (size_t)tile0 * prm.nsuper * 256;
    const unsigned rec_off = (unsigned)(min(tile0 + (wave % kRecG) * 4 + G, prm.ntiles - 1) - tile0) * (unsigned)prm.nsuper * 256u + r * 16;   // (waves past the records load some again)
    auto load_slow = [&](auto TC, int step) {                     // the narrow groups' chunks and the group records that `step` = T modulo 4 begins
        constexpr int T = decltype(TC)::value;
        auto group = [&](auto GC) {
            constexpr int g = decltype(GC)::value;
            if constexpr (bk_slow_begins(P, g, T)) {
                constexpr int b = group_width(P, g);
#pragma unroll
                for (int u = 0; u < kWLoads; ++u)
                    lds_load(prm.fields[g] + (size_t)w_row[u] * (prm.nsuper * b) * 1024, lane * 16 + (b == 2 ? step >> 1 : step >> 2) * 1024,
                             lds_addr(lds_slow) + (bk_slow_index(P, g) * kTW + w_place[u]) * 1024);
            }
        };
        group(std::integral_constant<int, 0>{});
        group(std::integral_constant<int, 1>{});
        group(std::integral_constant<int, 2>{});
        if constexpr (T == 0) lds_load(rec_base, rec_off + (unsigned)(step >> 2) * 256u, lds_addr(grec) + (wave % kRecG) * 1024);
    };
    auto sync = [&](auto LC) {
        constexpr int left = decltype(LC)::value;
        __builtin_amdgcn_sched_barrier(0);
        __builtin_amdgcn_s_waitcnt(0x0070 | (left & 15) | ((left >> 4) << 14));   // vmcnt(left) lgkmcnt(0)
        __builtin_amdgcn_s_barrier();
        asm volatile("" ::: "memory");
        __builtin_amdgcn_sched_barrier(0);
    };
    for (int i = wave; i < kRecA; i += kWaves) lds_load(prm.aparams, (unsigned)min(m0 + i * 64 + lane, prm.M - 1) * 16u, lds_addr(par_a + i * 64));
    load_slow(std::integral_constant<int, 0>{}, 0);
#pragma unroll
    for (int s = 0; s < 2; ++s)
#pragma unroll
        for (int i = 0; i < kLoads; ++i) load_piece(i, min(s, nsteps - 1), ring + s * kBuf);

    // ---- a wave's registers
    const int a_off = (rw * MT * 16 + r) * kBkStep, swz = (r >> 1) & 7;
    const int a_o0 = a_off + ((G ^ swz) << 4), a_o1 = a_off + (((4 + G) ^ swz) << 4);
    const v4i ones{0x01010101, 0x01010101, 0x01010101, 0x01010101}, zero4{0, 0, 0, 0};
    v4f facc[MT][NT];
#pragma unroll
    for (int mt = 0; mt < MT; ++mt)
#pragma unroll
        for (int nt = 0; nt < NT; ++nt) facc[mt][nt] = v4f{0.f, 0.f, 0.f, 0.f};
    v4i a[4][2], w[2][2][NT], raw[NT][3], c[2][NT], wz[2][NT];   // rows of A (four on their way), operands of two steps, products of two rows
    v4f sc[2][NT];
    uint2 scales[NT][4];                                          // of this lane's four channels: the super-chunk's four groups
    uint32_t zeros[NT];                                           // of the channel whose operand bytes this lane holds
    int32_t nzc[MT];                                              // minus the zero-point (less oa) of row r of every tile
    auto read_a = [&](int mt, const uint8_t* buf) {
        a[mt & 3][0] = *reinterpret_cast<const v4i*>(buf + a_o0 + mt * 16 * kBkStep);
        a[mt & 3][1] = *reinterpret_cast<const v4i*>(buf + a_o1 + mt * 16 * kBkStep);
    };
    auto read_raw = [&](auto TC, int nt, const uint8_t* buf) {   // what a step = T modulo 4 begins
        constexpr int T = decltype(TC)::value;
        auto group = [&](auto GC) {
            constexpr int g = decltype(GC)::value;
            if constexpr (g < group_count(P)) {
                if constexpr (group_width(P, g) == 4) raw[nt][g] = *reinterpret_cast<const v4i*>(buf + kABytes + (cw * NT + nt) * 1024 + lane * 16);
                else if constexpr (bk_slow_begins(P, g, T))
                    raw[nt][g] = *reinterpret_cast<const v4i*>(lds_slow + (bk_slow_index(P, g) * kTW + cw * NT + nt) * 1024 + lane * 16);
            }
        };
        group(std::integral_constant<int, 0>{});
        group(std::integral_constant<int, 1>{});
        group(std::integral_constant<int, 2>{});
        if constexpr (T == 0) {
            const uint8_t* rec = grec + (cw * NT + nt) * 256;
            zeros[nt] = *reinterpret_cast<const uint32_t*>(rec + r * 16 + 8);
#pragma unroll
            for (int reg = 0; reg < 4; ++reg) scales[nt][reg] = *reinterpret_cast<const uint2*>(rec + (4 * G + reg) * 16);
        }
    };
    // operand dword: four bytes w' - z
    auto expand = [&](auto TC, int set, int nt, int slice, int j) {
        constexpr int T = decltype(TC)::value;
        const uint32_t z = ((int)(zeros[nt] << (24 - 8 * T))) >> 24;
        const uint32_t off = __builtin_amdgcn_perm(0u, 128u - z, 0u);   // its low byte in all four
        const uint32_t x = slice ? bk_dword<P, 2 * T + 1>(raw[nt], j) : bk_dword<P, 2 * T>(raw[nt], j);
        w[set][slice][nt][j] = (int)((x + off) ^ 0x80808080u);
    };
    auto group_scales = [&](auto TC, int set) {
        constexpr int T = decltype(TC)::value;
#pragma unroll
        for (int nt = 0; nt < NT; ++nt)
#pragma unroll
            for (int reg = 0; reg < 4; ++reg) {
                const uint32_t bits = (T < 2 ? scales[nt][reg].x : scales[nt][reg].y) >> (16 * (T & 1));
                sc[set][nt][reg] = __half2float(__ushort_as_half((unsigned short)(bits & 0xFFFFu)));
            }
    };
    // A row of tiles is flushed two elements at a time, in three stages a slot apart, so that no instruction waits for the one before it.
    int ft[2] = {0, 0};
    float fv[2] = {0.f, 0.f};
    constexpr int kPairs = 2 * NT;                                // of a row
    auto flush = [&](int mt, int set, int u) {                    // slot u: the multiply-adds of pair u, the conversions of u - 1, the sums of u - 2
        if (u >= 2 && u < kPairs + 2) {
            const int e = 2 * (u - 2);
#pragma unroll
            for (int h = 0; h < 2; ++h) facc[mt][(e + h) / 4][(e + h) % 4] = fmaf(fv[h], sc[set][(e + h) / 4][(e + h) % 4], facc[mt][(e + h) / 4][(e + h) % 4]);
        }
        if (u >= 1 && u < kPairs + 1) { fv[0] = (float)ft[0]; fv[1] = (float)ft[1]; }
        if (u < kPairs) {
            const int e = 2 * u;
#pragma unroll
            for (int h = 0; h < 2; ++h) ft[h] = __mul24(nzc[mt], wz[set][(e + h) / 4][(e + h) % 4]) + c[mt & 1][(e + h) / 4][(e + h) % 4];
        }
    };

    sync(std::integral_constant<int, kLoads>{});
#pragma unroll
    for (int mt = 0; mt < MT; ++mt) nzc[mt] = prm.oa - par_a[(rw * MT + mt) * 16 + r].zero;
#pragma unroll
    for (int mt = 0; mt < 4; ++mt) read_a(mt, ring);
#pragma unroll
    for (int nt = 0; nt < NT; ++nt) {
        read_raw(std::integral_constant<int, 0>{}, nt, ring);
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            expand(std::integral_constant<int, 0>{}, 0, nt, 0, j);
            expand(std::integral_constant<int, 0>{}, 0, nt, 1, j);
        }
    }
#pragma unroll
    for (int nt = 0; nt < NT; ++nt) { c[0][nt] = c[1][nt] = zero4; wz[1][nt] = zero4; sc[1][nt] = v4f{0.f, 0.f, 0.f, 0.f}; }   // (nothing to flush before the first row)

    // ---- one step = one group.  Row after row of tiles; under a row's MFMAs the row before is flushed.  The barrier stands behind row MT - 4,
    // when the last rows of the step have been read: past it the step's place in the ring is loaded again, the next step's operands are read and made.
    auto step_body = [&](auto TC, int step, const uint8_t* cur, const uint8_t* nxt) {
        constexpr int T = decltype(TC)::value, TN = (T + 1) & 3, set = T & 1;
        constexpr int kSlots = 2 * NT, kMake = 8 * NT;           // MFMAs of a row, dwords of the next step's operands
        group_scales(TC, set);
#pragma unroll
        for (int nt = 0; nt < NT; ++nt) wz[set][nt] = __builtin_amdgcn_mfma_i32_16x16x64_i8(w[set][0][nt], ones, zero4, 0, 0, 0);
#pragma unroll
        for (int nt = 0; nt < NT; ++nt) wz[set][nt] = __builtin_amdgcn_mfma_i32_16x16x64_i8(w[set][1][nt], ones, wz[set][nt], 0, 0, 0);
        const int ahead = min(step + 2, nsteps - 1);
#pragma unroll
        for (int mt = 0; mt < MT; ++mt) {
            // the row that is flushed, and the one before it, whose last two stages stand in the first two slots
            const int fm = (mt + MT - 1) % MT, fset = mt == 0 ? set ^ 1 : set, fm2 = (mt + MT - 2) % MT, fset2 = mt < 2 ? set ^ 1 : set;
#pragma unroll
            for (int i = 0; i < kSlots; ++i) {
                const int nt = i % NT, slice = i / NT;
                c[mt & 1][nt] = __builtin_amdgcn_mfma_i32_16x16x64_i8(w[set][slice][nt], a[mt & 3][slice], slice ? c[mt & 1][nt] : zero4, 0, 0, 0);
                if (i < 2) flush(fm2, fset2, kPairs + i);
                flush(fm, fset, i);
                if (mt > MT - 4) {
                    const int k = (mt - (MT - 3)) * kSlots + i;          // of 3 kSlots
                    if (mt == MT - 3 && i < NT) read_raw(std::integral_constant<int, TN>{}, i, nxt);
#pragma unroll
                    for (int u = 0; u < kLoads; ++u)
                        if (u * 3 * kSlots / kLoads == k) load_piece(u, ahead, cur);
#pragma unroll
                    for (int u = 0; u < kMake; ++u)
                        if (mt > MT - 3 && u * 2 * kSlots / kMake == k - kSlots) expand(std::integral_constant<int, TN>{}, set ^ 1, u / 8, (u / 4) & 1, u & 3);
                }
                __builtin_amdgcn_sched_barrier(0);
            }
            if (mt == MT - 4) {
                sync(std::integral_constant<int, 0>{});
                load_slow(std::integral_constant<int, (T + 2) & 3>{}, min(step + 2, nsteps - 4 + ((T + 2) & 3)));
            }
            if (mt < MT - 4) read_a(mt + 4, cur);
            else read_a(mt + 4 - MT, nxt);
        }
    };
    for (int s = 0; s < prm.nsuper; ++s) {
        step_body(std::integral_constant<int, 0>{}, 4 * s, ring, ring + kBuf);
        step_body(std::integral_constant<int, 1>{}, 4 * s + 1, ring + kBuf, ring);
        step_body(std::integral_constant<int, 2>{}, 4 * s + 2, ring, ring + kBuf);
        step_body(std::integral_constant<int, 3>{}, 4 * s + 3, ring + kBuf, ring);
    }
#pragma unroll
    for (int u = 0; u < kPairs + 2; ++u) {
        if (u < 2) flush(MT - 2, 1, kPairs + u);
        flush(MT - 1, 1, u);
    }
    __builtin_amdgcn_s_waitcnt(0x0070);                           // (the last loads, for nobody, land before LDS is given back)

    // ---- epilogue: Y = half(a_scale * sum over groups); lanes exchange as in block_kernel
    static_assert(NT == 2, "tiles in pairs");
    const int n = n0 + (cw * NT + (G & 1)) * 16 + (G >> 1) * 8;
#pragma unroll
    for (int mt = 0; mt < MT; ++mt) {
        const int row = (rw * MT + mt) * 16 + r, m = m0 + row;
        const float sa = par_a[row].scale;
        uint32_t d[2][2];
#pragma unroll
        for (int h = 0; h < 2; ++h) {
            uint32_t hv[4];
#pragma unroll
            for (int reg = 0; reg < 4; ++reg) {
                const float v = sa * facc[mt][h][reg];
                asm("v_cvt_f16_f32 %0, %1" : "=v"(hv[reg]) : "v"(v));
            }
            d[h][0] = __builtin_amdgcn_perm(hv[1], hv[0], 0x05040100u);
            d[h][1] = __builtin_amdgcn_perm(hv[3], hv[2], 0x05040100u);
        }
        const auto lo = __builtin_amdgcn_permlane16_swap(d[0][0], d[1][0], false, false);
        const auto hi = __builtin_amdgcn_permlane16_swap(d[0][1], d[1][1], false, false);
        if (m < prm.M && n < prm.N) store_row_part8(prm.y + (size_t)m * prm.N + n, n, prm.N, lo[0], hi[0], lo[1], hi[1]);
    }
}

// Workgroup shapes (sizes: kG128Shapes in abq_block.hip)
template <int P>
static hipError_t block_g128_launch(const BlockG128Params& prm, int shape, hipStream_t s)
{
    const unsigned grid = (unsigned)(prm.tiles_m * prm.tiles_n);
    if (shape == 0) block_g128_kernel<P, 2, 4, 8, 2, 2><<<grid, 512, 0, s>>>(prm);   // 256 x 128, one a unit
    else if (shape == 1) block_g128_kernel<P, 1, 4, 8, 2, 2><<<grid, 256, 0, s>>>(prm);              // 128 x 128, two
    else return hipErrorInvalidValue;
    return hipGetLastError();
}

#define ABQ_BLOCK_G128_LAUNCH(P) hipError_t block_g128_launch_p##P(const BlockG128Params& prm, int shape, hipStream_t s)
ABQ_BLOCK_G128_LAUNCH(1);
ABQ_BLOCK_G128_LAUNCH(2);
ABQ_BLOCK_G128_LAUNCH(3);
ABQ_BLOCK_G128_LAUNCH(4);
ABQ_BLOCK_G128_LAUNCH(5);
ABQ_BLOCK_G128_LAUNCH(6);

}  // namespace abq
