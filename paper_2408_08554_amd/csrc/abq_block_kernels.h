// Device code of the block kernel and the templates that launch its variants.  Included by the host translation unit
// (abq_block.hip) and by the translation units that hold the instantiations.
//
// Matmul for prompts (and large batches) whose output has enough tiles to give every compute unit one of 64 x 128 or more.  A
// workgroup of RW x CW waves multiplies 16 MT RW rows of A by 16 NT CW rows of W, wave (rw, cw) its MT x NT accumulator tiles
// of 16 x 16 on the int8 MFMA.  Both operands go from global memory straight into LDS, S steps of 128 k in a ring: packed weights as
// they are stored (p/8 byte a weight; every wave expands the fields of its own tiles in registers, one dword at a time under the
// MFMAs), rows of A as whole 128-byte lines, XOR-swizzled so that the operand reads have no bank conflicts.  (Unpacked rows, masked and
// made signed in registers, take 1.3 to 2 times as long: every wave of a row of waves converts them again.  They are packed first.)
//
// What bounds it is the matrix pipe and, past that, power: at 256 x 256 tiles the K loop keeps the pipe 90-93 % busy on operands in cache (2200-2280
// clocks a step of 2048 clocks of MFMAs), 82-85 % with weights from memory, while the chip holds 1.65 (W8A8) to 2.1 GHz (W4A4).  How it gets there: eight waves
// of 128 x 64 take the fewest LDS bytes per MFMA that 256 registers allow; the one barrier of a step stands inside its second slice, where
// every operand of the MFMAs around it is in registers already; reads, loads and expansions stand one by one between MFMAs, because behind the
// barrier all waves run in step, and what stands in a row of its own there is time of the matrix pipe.
// Before / now (tiled kernel / this one, rows packed, replays): W4A4 M=2048 5120->13824 135 / 111 us, W8A8 147 / 119, M=1024 70 / 51 and
// 79 / 60, W8A8 M=512 4096->11008 32.5 / 26.5, 11008->4096 42 / 29.
#pragma once
#include "abq_rows.h"

#include <type_traits>

namespace abq {

typedef int v4i __attribute__((ext_vector_type(4)));

struct BlockParams {
    const uint8_t* fields[3];
    const uint8_t* a;            // packed rows (int8, stride lda)
    const RowParams* aparams;
    const RowParams* wparams;
    uint16_t* y;                 // may be null when rq.codes is given
    Requant rq;
    int M, N, K, lda, nsuper, ntiles;
    int oa, ow;
    int tiles_m, tiles_n;        // workgroup tiles along M and N (1-D grid of tiles_m * tiles_n workgroups)
    int band_m;                  // row blocks per band of the tile order
    int narrow_sums;             // 1: every row sum of codes is below 2^23 (the epilogue then multiplies at the 24-bit rate)
};

constexpr int kBkStep = 128;     // k per step: one chunk of a 4-bit group, two 64-k slices

// Chunks of a tile that change with every step (8- and 4-bit groups), and those that serve two or four (2- and 1-bit groups, one place each).
__host__ __device__ constexpr int bk_fast_chunks(int p) { return p == 8 ? 2 : (p >= 4 ? 1 : 0); }
__host__ __device__ constexpr int bk_slow_groups(int p) { return group_count(p) - (p >= 4 ? 1 : 0); }
__host__ __device__ constexpr int bk_slow_index(int p, int g) { return p >= 4 ? g - 1 : g; }
// whether group g has a chunk that begins with a step = T modulo 4 of the super-chunk, and is not loaded with every step
__host__ __device__ constexpr bool bk_slow_begins(int p, int g, int T)
{
    return g < group_count(p) && ((group_width(p, g) == 2 && T % 2 == 0) || (group_width(p, g) == 1 && T == 0));
}

// Operand dword j of slice SL (0..7 inside a super-chunk): all plane groups merged into one byte per weight.  raw: the tile's chunks.
template <int P, int SL, int G0 = 0>
__device__ __forceinline__ uint32_t bk_dword(const v4i* raw, int j)
{
    constexpr int b = group_width(P, G0), shift = group_shift(P, G0), t = SL % (8 / b), sh = b * t - shift;
    const uint32_t x = (uint32_t)raw[G0][j];
    constexpr uint32_t mask = (((1u << b) - 1u) * 0x01010101u) << shift;
    uint32_t v;
    if constexpr (sh > 0) v = (x >> sh) & mask;
    else if constexpr (sh < 0) v = (x << (-sh)) & mask;
    else v = x & mask;
    if constexpr (G0 + 1 < group_count(P)) v |= bk_dword<P, SL, G0 + 1>(raw, j);
    return v;
}

// a * b + c, low 32 bits, factors of 24 bits (written as the instruction: the compiler otherwise splits it)
__device__ __forceinline__ int32_t bk_mad24(int32_t a, int32_t b, int32_t c)
{
    int32_t d;
    asm("v_mad_i32_i24 %0, %1, %2, %3" : "=v"(d) : "v"(a), "v"(b), "v"(c));
    return d;
}

// What the epilogue needs of a channel: the sum over the codes less their zero-points is acc + raw0 + wz sumA - az cw.
struct alignas(16) ColParams { int32_t raw0, cw, wz; float scale; };

// OCC: waves per SIMD that the registers are held to.
template <int P, int RW, int CW, int MT, int NT, int S, int OCC>
__global__ __launch_bounds__(64 * RW * CW, OCC) void block_kernel(BlockParams prm)
{
    constexpr int kWaves = RW * CW, kBM = 16 * MT * RW, kTW = NT * CW, kBN = 16 * kTW;
    constexpr int kABytes = kBM * kBkStep, kBuf = kABytes + kTW * bk_fast_chunks(P) * 1024;
    constexpr int kSlow = kTW * bk_slow_groups(P) * 1024;
    constexpr int kRecA = (kBM + 63) / 64, kRecW = (kBN + 63) / 64;   // wave loads of 64 records
    __shared__ __align__(1024) uint8_t ring[S * kBuf];
    __shared__ __align__(1024) uint8_t lds_slow[kSlow > 0 ? kSlow : 16];
    __shared__ __align__(16) RowParams par_a[64 * kRecA], par_w[64 * kRecW];
    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int rw = wave / CW, cw = wave % CW;
    const int r = lane & 15, G = lane >> 4;
    // tile order: as in tiled_kernel (a contiguous run of the banded order per XCD)
    const int nwg = prm.tiles_m * prm.tiles_n;
    const int xcd = blockIdx.x & 7, slot = blockIdx.x >> 3;
    const int per = nwg >> 3, rem = nwg & 7;
    const int vid = xcd * per + min(xcd, rem) + slot;
    const int band = vid / (prm.band_m * prm.tiles_n), in_band = vid - band * prm.band_m * prm.tiles_n;
    const int band_rows = min(prm.band_m, prm.tiles_m - band * prm.band_m);
    const int m_blk = band * prm.band_m + in_band % band_rows, n_blk = in_band / band_rows;
    const int m0 = m_blk * kBM, n0 = n_blk * kBN, tile0 = n_blk * kTW;
    const int nsteps = prm.nsuper * 4;

    // ---- loads.  1 KiB a wave and instruction: 16 bytes per lane from base + off (all but off wave-uniform) to LDS address dst + 16 lane.
    // Written as the instruction: the compiler takes the builtin for an LDS access of unknown order and waits for every outstanding
    // LDS read behind it.  It has no result register; sync() below waits for these loads.
    auto lds_addr = [](const void* p) { return (unsigned)(uintptr_t)(const __attribute__((address_space(3))) uint8_t*)p; };
    auto lds_load = [](const void* base, unsigned off, unsigned dst) {
        asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %1, %2" : : "s"(dst), "v"(off), "s"(base) : "memory", "m0");
    };
    // Rows of A: load u of a wave fills rows 8 (wave kALoads + u) .. + 7, lane L row L / 8, position L % 8, which holds the row's
    // 16-byte piece (L % 8) ^ ((row / 2) % 8) (an operand read's sixteen rows then lie on different banks).  Rows past M re-read row M - 1, their outputs
    // are never stored.
    constexpr int kALoads = kBM / 8 / kWaves;
    static_assert(kBM % (8 * kWaves) == 0, "whole loads");
    unsigned a_goff[kALoads];
#pragma unroll
    for (int u = 0; u < kALoads; ++u) {
        const int row = 8 * (wave * kALoads + u) + (lane >> 3);
        const unsigned piece = ((lane & 7) ^ ((row >> 1) & 7)) * 16;
        a_goff[u] = (unsigned)(min(m0 + row, prm.M - 1) - m0) * (unsigned)prm.lda + piece;
    }
    const uint8_t* a_tile = prm.a + (size_t)m0 * prm.lda;
    // Chunks of W: as many loads from every wave, so that one count of outstanding loads holds for all (the last tile may be loaded twice).
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
    auto load_piece = [&](int i, int step, const uint8_t* buf) {   // i-th load of a step
        if (i < kALoads) {
            lds_load(a_tile + (size_t)step * kBkStep, a_goff[i], lds_addr(buf) + (wave * kALoads + i) * 1024);
        } else if constexpr (kChunks > 0) {
            const int u = (i - kALoads) / kChunks, c = (i - kALoads) % kChunks;
            lds_load(w_tile[u], lane * 16 + (step * kChunks + c) * 1024, lds_addr(buf) + kABytes + (w_place[u] * kChunks + c) * 1024);
        }
    };
    auto load_slow = [&](auto TC, int step) {                      // the narrow groups' chunks that `step` = T modulo 4 begins
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
    };
    // At most `left` loads of this wave are outstanding past it, none of its LDS reads, and every other wave is there too.  (The bare
    // barrier: a workgroup fence would wait for every load.)
    auto sync = [&](auto LC) {
        constexpr int left = decltype(LC)::value < 63 ? decltype(LC)::value : 63;
        __builtin_amdgcn_sched_barrier(0);
        __builtin_amdgcn_s_waitcnt(0x0070 | (left & 15) | ((left >> 4) << 14));   // vmcnt(left) lgkmcnt(0)
        __builtin_amdgcn_s_barrier();
        asm volatile("" ::: "memory");
        __builtin_amdgcn_sched_barrier(0);
    };

    v4i acc[MT][NT];
#pragma unroll
    for (int mt = 0; mt < MT; ++mt)
#pragma unroll
        for (int nt = 0; nt < NT; ++nt) acc[mt][nt] = v4i{0, 0, 0, 0};

    // the epilogue's records first: whatever waits for a later load waits for them
    for (int i = wave; i < kRecA + kRecW; i += kWaves) {
        if (i >= kRecA) lds_load(prm.wparams, (unsigned)min(n0 + (i - kRecA) * 64 + lane, prm.N - 1) * 16u, lds_addr(par_w + (i - kRecA) * 64));
        else lds_load(prm.aparams, (unsigned)min(m0 + i * 64 + lane, prm.M - 1) * 16u, lds_addr(par_a + i * 64));
    }
    load_slow(std::integral_constant<int, 0>{}, 0);
#pragma unroll
    for (int s = 0; s < S; ++s)
#pragma unroll
        for (int i = 0; i < kLoads; ++i) load_piece(i, min(s, nsteps - 1), ring + s * kBuf);

    // ---- operands of a wave: the current slice's rows of A (replaced by the next slice's one by one), the expanded weights of both slices
    // of a step, the chunks that they are made from
    const int a_off = (rw * MT * 16 + r) * kBkStep, swz = (r >> 1) & 7;
    const int a_o0 = a_off + ((G ^ swz) << 4), a_o1 = a_off + (((4 + G) ^ swz) << 4);
    v4i a[MT], w0[NT], w1[NT], raw[NT][3];
    auto read_a = [&](int mt, int o, const uint8_t* buf) { a[mt] = *reinterpret_cast<const v4i*>(buf + o + mt * 16 * kBkStep); };
    auto read_w8 = [&](int nt, int slice, const uint8_t* buf) {
        return *reinterpret_cast<const v4i*>(buf + kABytes + ((cw * NT + nt) * 2 + slice) * 1024 + lane * 16);
    };
    auto read_raw = [&](auto TC, int nt, const uint8_t* buf) {   // the groups whose chunk begins with a step = T modulo 4
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
    };
    sync(std::integral_constant<int, (S - 1) * kLoads>{});
#pragma unroll
    for (int nt = 0; nt < NT; ++nt) {
        if constexpr (P == 8) w0[nt] = read_w8(nt, 0, ring);
        else {
            read_raw(std::integral_constant<int, 0>{}, nt, ring);
#pragma unroll
            for (int j = 0; j < 4; ++j) w0[nt][j] = (int)bk_dword<P, 0>(raw[nt], j);
        }
    }
#pragma unroll
    for (int mt = 0; mt < MT; ++mt) read_a(mt, a_o0, ring);

    // ---- one step: two slices of 64 k, MT x NT MFMAs each
    constexpr int kHold = MT >= 8 ? 2 : 1;                       // rows of the second slice multiplied ahead of the barrier
    constexpr int kSlots = MT * NT, kPast = kSlots - kHold * NT; // MFMAs of a slice; of those, past the barrier
    auto step_body = [&](auto TC, int step, const uint8_t* cur, const uint8_t* nxt) {
        constexpr int T = decltype(TC)::value, TN = (T + 1) & 3;
        // first slice; its rows of A are replaced by the second's as they are used up
#pragma unroll
        for (int i = 0; i < kSlots; ++i) {
            const int mt = i / NT, nt = i % NT;
            acc[mt][nt] = __builtin_amdgcn_mfma_i32_16x16x64_i8(w0[nt], a[mt], acc[mt][nt], 0, 0, 0);
            if (nt == NT - 1) read_a(mt, a_o1, cur);
            if constexpr (P == 8) { if (i % 2 == 0 && i / 2 < NT) w1[i / 2] = read_w8(i / 2, 1, cur); }
            else {
#pragma unroll
                for (int u = 0; u < 4 * NT; ++u)
                    if (u * kSlots / (4 * NT) == i) w1[u / 4][u % 4] = (int)bk_dword<P, 2 * T + 1>(raw[u / 4], u % 4);
            }
            __builtin_amdgcn_sched_barrier(0);
        }
        // second slice: past the barrier this step's place in the ring is free, and the next step has landed
        const int ahead = min(step + S, nsteps - 1);             // (past the end the last step is loaded again, for nobody)
#pragma unroll
        for (int i = 0; i < kSlots; ++i) {
            const int mt = i / NT, nt = i % NT, j = i - kHold * NT;   // the j-th MFMA past the barrier
            acc[mt][nt] = __builtin_amdgcn_mfma_i32_16x16x64_i8(w1[nt], a[mt], acc[mt][nt], 0, 0, 0);
            if (j >= 0) {
                if (j % 2 == 0 && j / 2 < NT) {
                    if constexpr (P == 8) w0[j / 2] = read_w8(j / 2, 0, nxt);
                    else read_raw(std::integral_constant<int, TN>{}, j / 2, nxt);
                }
                if (j % 2 == 1 && j / 2 < kHold) read_a(j / 2, a_o0, nxt);
                if (nt == NT - 1) read_a(mt, a_o0, nxt);
#pragma unroll
                for (int u = 0; u < kLoads; ++u)
                    if (1 + u * (kPast - 1) / kLoads == j) load_piece(u, ahead, cur);
                if constexpr (P < 8) {
#pragma unroll
                    for (int u = 0; u < 4 * NT; ++u)
                        if (kPast / 2 + u * (kPast - kPast / 2) / (4 * NT) == j) w0[u / 4][u % 4] = (int)bk_dword<P, 2 * TN>(raw[u / 4], u % 4);
                }
            }
            __builtin_amdgcn_sched_barrier(0);
            if (j == -1) {
                // The narrow groups' chunks of step + 1 were asked for a step ago, ahead of that step's kLoads.
                constexpr bool slow = bk_slow_begins(P, 0, TN) || bk_slow_begins(P, 1, TN) || bk_slow_begins(P, 2, TN);
                sync(std::integral_constant<int, S == 2 ? 0 : (slow ? kLoads : (S - 2) * kLoads)>{});
                load_slow(std::integral_constant<int, (T + 2) & 3>{}, min(step + 2, nsteps - 4 + ((T + 2) & 3)));
            }
        }
    };
    if constexpr (S == 2) {
        for (int sc = 0; sc < prm.nsuper; ++sc) {
            step_body(std::integral_constant<int, 0>{}, 4 * sc, ring, ring + kBuf);
            step_body(std::integral_constant<int, 1>{}, 4 * sc + 1, ring + kBuf, ring);
            step_body(std::integral_constant<int, 2>{}, 4 * sc + 2, ring, ring + kBuf);
            step_body(std::integral_constant<int, 3>{}, 4 * sc + 3, ring + kBuf, ring);
        }
    } else {
        unsigned place = 0;
        auto go = [&](auto TC, int step) {
            const unsigned nxt = place + kBuf == S * kBuf ? 0u : place + kBuf;
            step_body(TC, step, ring + place, ring + nxt);
            place = nxt;
        };
        for (int sc = 0; sc < prm.nsuper; ++sc) {
            go(std::integral_constant<int, 0>{}, 4 * sc);
            go(std::integral_constant<int, 1>{}, 4 * sc + 1);
            go(std::integral_constant<int, 2>{}, 4 * sc + 2);
            go(std::integral_constant<int, 3>{}, 4 * sc + 3);
        }
    }

    // ---- epilogue.  Lane (G, r) holds channels 4 G .. 4 G + 3 of row r of every tile; two neighbouring tiles exchange quarters of
    // a wave, after which a lane has eight adjacent channels: one 16-byte store.  (The outputs leave faster than the vector ALU makes
    // them, 4 us a 256 x 256 tile; staged through LDS they take the same time.)
    // Output codes are made from the same eight values and leave as one 8-byte store, with a row's parameters loaded once: nothing runs beside a
    // workgroup's epilogue here.  (With 32-bit multiplies, parameters loaded and a byte stored per element, calls with codes took 1.02 to 1.06 times the
    // tiled kernel's time, up to 1.39, over 100 sizes that the rule takes; now 0.70 with the values and 0.73 without, pack launch
    // included: W8A8 M=512 4096->11008 55.8 us tiled, 53.5 so, 40.5 now.)
    __builtin_amdgcn_s_waitcnt(0x0070);                          // (the last loads, for nobody, land before LDS is given back)
    for (int i = tid; i < kBN; i += 64 * kWaves) {               // a channel's record becomes what the epilogue needs of it
        const RowParams pw = par_w[i];
        ColParams c;
        c.raw0 = (int32_t)((uint32_t)prm.oa * (uint32_t)pw.sum - (uint32_t)prm.K * (uint32_t)prm.oa * (uint32_t)prm.ow);
        c.cw = (int32_t)((uint32_t)pw.sum - (uint32_t)prm.K * (uint32_t)pw.zero);
        c.wz = (int32_t)((uint32_t)prm.ow - (uint32_t)pw.zero);
        c.scale = pw.scale;
        reinterpret_cast<ColParams*>(par_w)[i] = c;
    }
    __syncthreads();
    const int wm0 = m0 + rw * MT * 16, wn0 = n0 + cw * NT * 16;
    const bool vec_ok = (prm.N & 3) == 0;                        // (of an odd tile: rows of Y 8-byte aligned)
    auto dequant = [&](auto narrow, auto coded) {                // coded: the next layer's codes as well as (or instead of) the values
        float rq_scale[MT];
        int rq_zero[MT];
        if constexpr (decltype(coded)::value) {
#pragma unroll
            for (int mt = 0; mt < MT; ++mt) {
                const int m = min(wm0 + mt * 16 + r, prm.M - 1);
                rq_scale[mt] = prm.rq.scale[m];
                rq_zero[mt] = prm.rq.zero[m];
            }
        }
#pragma unroll
        for (int np = 0; np < NT; np += 2) {
            const int two = np + 1 < NT ? 2 : 1;                 // (an odd tile is left on its own: 8-byte stores)
            ColParams pw[2][4];
#pragma unroll
            for (int h = 0; h < 2; ++h)
#pragma unroll
                for (int reg = 0; reg < 4; ++reg)
                    if (h < two) pw[h][reg] = reinterpret_cast<const ColParams*>(par_w)[(cw * NT + np + h) * 16 + 4 * G + reg];
#pragma unroll
            for (int mt = 0; mt < MT; ++mt) {
                const RowParams pa = par_a[(rw * MT + mt) * 16 + r];
                const int m = wm0 + mt * 16 + r;
                const int32_t naz = (int32_t)(0u - (uint32_t)pa.zero);
                uint32_t d[2][2] = {{0u, 0u}, {0u, 0u}};
#pragma unroll
                for (int h = 0; h < 2; ++h) {
                    if (h >= two) break;
                    uint32_t hv[4];
#pragma unroll
                    for (int reg = 0; reg < 4; ++reg) {
                        const ColParams& c = pw[h][reg];
                        const int32_t s = (int32_t)((uint32_t)acc[mt][np + h < NT ? np + h : 0][reg] + (uint32_t)c.raw0);
                        int32_t centered;
                        if constexpr (decltype(narrow)::value)
                            centered = bk_mad24(naz, c.cw, bk_mad24(c.wz, pa.sum, s));
                        else
                            centered = (int32_t)((uint32_t)s + (uint32_t)c.wz * (uint32_t)pa.sum + (uint32_t)naz * (uint32_t)c.cw);
                        const float v = ((float)centered * pa.scale) * c.scale;
                        asm("v_cvt_f16_f32 %0, %1" : "=v"(hv[reg]) : "v"(v));   // (the instruction itself: see epilogue_value)
                    }
                    d[h][0] = __builtin_amdgcn_perm(hv[1], hv[0], 0x05040100u);   // the low halves of both
                    d[h][1] = __builtin_amdgcn_perm(hv[3], hv[2], 0x05040100u);
                }
                int n = wn0 + np * 16 + 4 * G;
                uint32_t w4[4] = {d[0][0], d[0][1], 0u, 0u};
                if (two == 2) {
                    const auto lo = __builtin_amdgcn_permlane16_swap(d[0][0], d[1][0], false, false);
                    const auto hi = __builtin_amdgcn_permlane16_swap(d[0][1], d[1][1], false, false);
                    n = wn0 + (np + (G & 1)) * 16 + (G >> 1) * 8;
                    w4[0] = lo[0]; w4[1] = hi[0]; w4[2] = lo[1]; w4[3] = hi[1];
                }
                if (m >= prm.M || n >= prm.N) continue;
                if constexpr (decltype(coded)::value) {
                    uint32_t c8[2] = {0u, 0u};
#pragma unroll
                    for (int e = 0; e < 8; ++e)
                        if (e < 4 * two) c8[e >> 2] |= (uint32_t)requant_code((uint16_t)(w4[e >> 1] >> (16 * (e & 1))), rq_scale[mt], rq_zero[mt], prm.rq.qmax) << (8 * (e & 3));
                    uint8_t* dst = prm.rq.codes + (size_t)m * prm.N + n;
                    if (two == 2 && n + 8 <= prm.N) *reinterpret_cast<u32x2_byte*>(dst) = u32x2_byte{c8[0], c8[1]};
                    else {
#pragma unroll
                        for (int e = 0; e < 8; ++e)
                            if (e < 4 * two && n + e < prm.N) dst[e] = (uint8_t)(c8[e >> 2] >> (8 * (e & 3)));
                    }
                }
                if (!decltype(coded)::value || prm.y) {
                    uint16_t* dst = prm.y + (size_t)m * prm.N + n;
                    if (two == 2) store_row_part8(dst, n, prm.N, w4[0], w4[1], w4[2], w4[3]);
                    else if (vec_ok) *reinterpret_cast<uint2*>(dst) = uint2{w4[0], w4[1]};
                    else {
#pragma unroll
                        for (int e = 0; e < 4; ++e)
                            if (n + e < prm.N) dst[e] = (uint16_t)(w4[e >> 1] >> (16 * (e & 1)));
                    }
                }
            }
        }
    };
    if (prm.rq.codes == nullptr) {                               // (the same for every thread, as is narrow_sums)
        if (prm.narrow_sums) dequant(std::true_type{}, std::false_type{});
        else dequant(std::false_type{}, std::false_type{});
    } else {
        if (prm.narrow_sums) dequant(std::true_type{}, std::true_type{});
        else dequant(std::false_type{}, std::true_type{});
    }
}

template <int P, int RW, int CW, int MT, int NT, int S, int OCC>
static hipError_t block_go(const BlockParams& prm, hipStream_t s)
{
    block_kernel<P, RW, CW, MT, NT, S, OCC><<<(unsigned)(prm.tiles_m * prm.tiles_n), 64 * RW * CW, 0, s>>>(prm);
    return hipGetLastError();
}

// Workgroup shapes (sizes: kShapes in abq_block.hip).  Places in the ring: as many as fit beside what the shape's occupancy leaves of
// 160 KiB, at most six; at 256 x 256 a step lasts longer than a load, and two are as fast as three.
template <int P>
static hipError_t block_launch(const BlockParams& prm, int shape, hipStream_t s)
{
    constexpr bool few = P < 4;   // (narrow groups only: no weights in the ring)
    switch (shape) {
        case 0: return block_go<P, 2, 4, 8, P == 7 ? 3 : 4, 2, 2>(prm, s);                      // 256 x 256 (p = 7: 192, or it spills), one a unit
        case 1: return block_go<P, 2, 4, 4, 3, P == 8 ? 3 : (few ? 6 : 4), 2>(prm, s);          // 128 x 192, one
        case 2:                                                                                  // 128 x 128, one (for p < 4 the costs pick it nowhere: 1.2 times the best other shape's time)
            if constexpr (!few) return block_go<P, 2, 4, 4, 2, P == 8 ? 4 : 5, 2>(prm, s);
            else return hipErrorInvalidValue;
        case 3: return block_go<P, 2, 2, 4, 4, P >= 4 ? 2 : 3, 2>(prm, s);                      // 128 x 128 by four waves, two
        case 4: return block_go<P, 1, 4, 4, 2, P >= 7 ? 3 : 4, 2>(prm, s);                      // 64 x 128 by four waves, two
        default: return hipErrorInvalidValue;
    }
}

#define ABQ_BLOCK_LAUNCH(P) hipError_t block_launch_p##P(const BlockParams& prm, int shape, hipStream_t s)
ABQ_BLOCK_LAUNCH(1);
ABQ_BLOCK_LAUNCH(2);
ABQ_BLOCK_LAUNCH(3);
ABQ_BLOCK_LAUNCH(4);
ABQ_BLOCK_LAUNCH(5);
ABQ_BLOCK_LAUNCH(6);
ABQ_BLOCK_LAUNCH(7);
ABQ_BLOCK_LAUNCH(8);

}  // namespace abq
