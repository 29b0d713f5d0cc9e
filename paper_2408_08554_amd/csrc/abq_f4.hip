// The very-low-bit matmul on gfx950's 4-bit floating-point MFMA: operands of one or two bits (weights AND activations).
//
// Appendix B decomposes a p x q-bit matmul into p*q binary ones because the tensor cores it targets multiply 1-bit
// planes; the point of Sec. 3.4 / Table 4 is that narrower operands should run faster.  The int8 MFMA path of this
// library carries a whole byte per operand whatever p and q are.  gfx950 has a 16x16x128 MFMA on 4-bit E2M1 operands at
// twice the int8 rate, and the codes 0..3 are E2M1 values (0, 1, 2, 3 = 0b0000, 0b0010, 0b0100, 0b0101): their products
// (<= 9) and the sums of them are exact in the instruction's binary32 accumulator as long as K * 9 < 2^24, far beyond
// any K the library accepts, so the accumulator converts to the same int32 the other kernels produce, and the fused
// dequant epilogue (Fig. 3b) is theirs.  Block scales of the instruction are 2^0.
//
// Both operands use ONE packed layout (so one packer serves weights and activations): after the header and the row
// parameters, [row tiles of 16][K blocks of 128][64 lanes][16 bytes] — 1 KiB per (16 rows x 128 k), lane L holding row
// L % 16, k = 128 block + 32 (L / 16) .. + 31 as 32 nibbles, which is the MFMA operand of that block as it stands.
// Rows past the end and k past K hold code 0.
//
// Kernel: both operands through an LDS ring, workgroup tiles of 32 x 64 to 256 x 256 (see f4_gemm_kernel).
#include "abq_rows.h"
#include "../../include/abq.h"

#include <type_traits>

namespace abq {

typedef int v4i_f4 __attribute__((ext_vector_type(4)));
typedef int v8i_f4 __attribute__((ext_vector_type(8)));
typedef float v4f_f4 __attribute__((ext_vector_type(4)));

constexpr int kF4BlockK = 128;                 // k per operand block

static inline int f4_row_tiles(int rows) { return (rows + 15) / 16; }
static inline int f4_k_blocks(int K) { return (K + kF4BlockK - 1) / kF4BlockK; }

size_t f4_packed_bytes(int rows, int K)
{
    return kHeaderBytes + align_up((size_t)rows * sizeof(RowParams), 256) + (size_t)f4_row_tiles(rows) * f4_k_blocks(K) * 1024;
}
static inline size_t f4_off_params() { return kHeaderBytes; }
static inline size_t f4_off_blocks(int rows) { return kHeaderBytes + align_up((size_t)rows * sizeof(RowParams), 256); }

// ---- packer ---------------------------------------------------------------------------------------------------------
// Four codes in the bytes of a dword (already masked to 0..3) -> their four E2M1 nibbles in the low 16 bits: a code c
// becomes c << 1, except 3, which becomes 5 (0, 1, 2, 3 = 0b0000, 0b0010, 0b0100, 0b0101).
__device__ __forceinline__ uint32_t f4_nibbles(uint32_t x)
{
    const uint32_t three = x & (x >> 1) & 0x01010101u;             // 1 in the bytes that hold 3
    const uint32_t nib = (x << 1) ^ (three * 3u);                  // one E2M1 value per byte
    const uint32_t pairs = (nib | (nib >> 4)) & 0x00FF00FFu;       // bytes 0, 2: nibble pairs (0,1), (2,3)
    return (pairs | (pairs >> 8)) & 0xFFFFu;
}

// The whole blob in one launch (a pack of the activations sits in front of every matmul: three dependent launches
// cost more than the work).  One workgroup of sixteen waves per tile of 16 rows; wave w packs the K blocks w, w + 16, ...:
// lane L takes 32 codes of row L % 16 at k = 128 kb + 32 (L / 16) -> 32 E2M1 nibbles (16 bytes, the operand layout), and
// keeps the sum of its codes; the sums meet across the lanes of a row, then across the waves through LDS, and become the
// rows' parameter records {sum of codes, scale, zero}.  vec: K is a multiple of 16 and the rows are 16-byte aligned, so
// the 32 codes are two 128-bit loads.  Workgroup 0 also writes the header.
constexpr int kF4PackWaves = 16;
__global__ __launch_bounds__(64 * kF4PackWaves) void f4_pack_kernel(const uint8_t* codes, int rows, int K, int kblocks, uint32_t mask, int vec,
                                                                    const float* scale, const int32_t* zero, int bits, uint32_t* hdr,
                                                                    RowParams* params, v4i_f4* out, int ksplit)
{
    __shared__ uint32_t part[kF4PackWaves][16];
    const int tid = (int)threadIdx.x, lane = tid & 63, wave = tid >> 6;
    // ksplit = 2: two workgroups per row tile, one per half of the K blocks (a pack of 2048 rows is otherwise 128
    // workgroups: half the chip); the second writes its sums of codes into the record's spare word
    const int rt = (int)blockIdx.x / ksplit, half = (int)blockIdx.x % ksplit;
    const int kb_per = (kblocks + ksplit - 1) / ksplit, kb_lo = half * kb_per, kb_hi = min(kblocks, kb_lo + kb_per);
    const int row = rt * 16 + (lane & 15);
    const uint8_t* src = codes + (size_t)min(row, rows - 1) * K;   // (rows past the end: a valid row is read, zeros are stored)
    const uint32_t m4 = mask * 0x01010101u;
    uint32_t sum = 0;
    // up to four K blocks of the wave at a time: their loads are all requested before the first is packed
    constexpr int NB = 4;
    for (int kb0 = kb_lo + wave; kb0 < kb_hi; kb0 += kF4PackWaves * NB) {
        v4i_f4 lo[NB], hi[NB];
        bool fast[NB];
#pragma unroll
        for (int u = 0; u < NB; ++u) {
            const int kb = kb0 + kF4PackWaves * u, k0 = kb * kF4BlockK + (lane >> 4) * 32;
            fast[u] = vec && kb < kb_hi && k0 + 32 <= K;
            lo[u] = hi[u] = v4i_f4{0, 0, 0, 0};
            if (fast[u]) {
                lo[u] = *reinterpret_cast<const v4i_f4*>(src + k0);
                hi[u] = *reinterpret_cast<const v4i_f4*>(src + k0 + 16);
            }
        }
#pragma unroll
        for (int u = 0; u < NB; ++u) {
            const int kb = kb0 + kF4PackWaves * u, k0 = kb * kF4BlockK + (lane >> 4) * 32;
            if (kb >= kb_hi) break;   // (the same for the whole wave)
            uint32_t w[4] = {0, 0, 0, 0};
            if (fast[u]) {
                const uint32_t c[8] = {(uint32_t)lo[u].x & m4, (uint32_t)lo[u].y & m4, (uint32_t)lo[u].z & m4, (uint32_t)lo[u].w & m4,
                                       (uint32_t)hi[u].x & m4, (uint32_t)hi[u].y & m4, (uint32_t)hi[u].z & m4, (uint32_t)hi[u].w & m4};
#pragma unroll
                for (int e = 0; e < 8; ++e) sum = __builtin_amdgcn_sad_u8(c[e], 0u, sum);
#pragma unroll
                for (int e = 0; e < 4; ++e) w[e] = f4_nibbles(c[2 * e]) | (f4_nibbles(c[2 * e + 1]) << 16);
            } else {
                for (int e = 0; e < 32; ++e) {
                    const int k = k0 + e;
                    const uint32_t c = k < K ? (src[k] & mask) : 0u;
                    sum += c;
                    const uint32_t nib = c == 3 ? 5u : (c << 1);
                    w[e >> 3] |= nib << (4 * (e & 7));
                }
            }
            if (row >= rows) w[0] = w[1] = w[2] = w[3] = 0;
            out[((size_t)rt * kblocks + kb) * 64 + lane] = v4i_f4{(int)w[0], (int)w[1], (int)w[2], (int)w[3]};
        }
    }
    sum += (uint32_t)__shfl_xor((int)sum, 16);
    sum += (uint32_t)__shfl_xor((int)sum, 32);
    if (lane < 16) part[wave][lane] = sum;
    __syncthreads();
    if (tid < 16 && row < rows) {
        uint32_t total = 0;
#pragma unroll
        for (int w = 0; w < kF4PackWaves; ++w) total += part[w][tid];
        if (half == 0) {
            params[row].sum = (int32_t)total;
            params[row].scale = scale[row];
            params[row].zero = zero[row];
            if (ksplit == 1) params[row].pad = 0;
        } else {
            params[row].pad = (int32_t)total;   // (the matmul adds the two)
        }
    }
    if (blockIdx.x == 0 && tid >= 64 && tid < 128) {
        const int t = tid - 64;
        hdr[t] = t == 0 ? 0x34514241u /* "ABQ4" */ : (t == 1 ? 0x34460001u : (t == 2 ? (uint32_t)bits : (t == 3 ? (uint32_t)rows : (t == 4 ? (uint32_t)K : 0u))));
    }
}

hipError_t launch_f4_pack(int bits, int rows, int K, const uint8_t* codes, const float* scale, const int32_t* zero, uint8_t* blob, hipStream_t s)
{
    const uint32_t mask = (1u << bits) - 1u;
    const int vec = (K % 16 == 0) ? 1 : 0;   // (the entry point checks that `codes` is 16-byte aligned)
    const int ksplit = (f4_k_blocks(K) >= 32 && 2L * f4_row_tiles(rows) <= (long)num_cus()) ? 2 : 1;
    f4_pack_kernel<<<(unsigned)(f4_row_tiles(rows) * ksplit), 64 * kF4PackWaves, 0, s>>>(codes, rows, K, f4_k_blocks(K), mask, vec, scale, zero, bits, (uint32_t*)blob,
                                                                                         (RowParams*)(blob + f4_off_params()), (v4i_f4*)(blob + f4_off_blocks(rows)), ksplit);
    return hipGetLastError();
}

// ---- matmul ---------------------------------------------------------------------------------------------------------
struct F4Params {
    const v4i_f4* a_blocks;    // [row tiles][kblocks][64]
    const v4i_f4* w_blocks;
    const RowParams* aparams;
    const RowParams* wparams;
    uint16_t* y;
    int32_t* acc;              // may be null
    int M, N, K, kblocks;
    int a_tiles, w_tiles;      // 16-row tiles of the two operands
    int tiles_m, tiles_n;      // workgroup tiles
    int band_m;                // row tiles per band of the tile order
};

// Y = dequant(A W^T) on the 4-bit floating-point MFMA.  RW x CW waves, each MT x NT accumulator tiles of 16 x 16; S places in the LDS
// ring; OCC: waves per SIMD that the registers are held to.  The loop is the int8 block kernel's (abq_block_kernels.h, which says why it is
// built so): both operands go global -> LDS, where an operand block lands as the operand layout, a step is one block of 128 k, its barrier stands
// behind its first rows of MFMAs, and reads and loads stand one by one between the others.  (Two blocks a step: 1 to 6 % slower.)
// The kernel before this one read its rows into registers by hand-written loads, waited for by hand, and took the eight W blocks of a step through LDS
// in four waves of 64 x 128.  The gain is at few and middling rows: 400 sizes of M = 1..2048 take 0.69 times its time in cache, 0.61 with weights from memory (17..63
// rows 0.60 and 0.52, from 1024 on 0.83 and 0.80; 5 and 4 of them are 3 to 10 % slower).  W2A2 M=2048 5120->13824 traced 72.2 us, 65.6, but a pass
// with its pack, 68-74 us by process, is hardly faster than it was (72-75).
template <int RW, int CW, int MT, int NT, int S, int OCC>
__global__ __launch_bounds__(64 * RW * CW, OCC) void f4_gemm_kernel(F4Params prm)
{
    constexpr int kWaves = RW * CW, kTA = MT * RW, kTW = NT * CW, kBuf = (kTA + kTW) * 1024;   // a step: one block of every tile
    constexpr int kRecA = (kTA + 3) / 4, kRecW = (kTW + 3) / 4;                                // wave loads of 64 records
    __shared__ __align__(1024) uint8_t ring[S * kBuf];
    __shared__ __align__(16) RowParams par_a[64 * kRecA], par_w[64 * kRecW];
    const int tid = (int)threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int rw = wave / CW, cw = wave % CW;
    const int r = lane & 15, G = lane >> 4;
    // Workgroup b runs on XCD b % 8 and each XCD has its own L2: give every XCD a contiguous run of the tile order, row tiles in bands, so that the
    // workgroups resident on an XCD at one time cover about as many row tiles as column tiles, which is the least operand traffic into its L2.
    const int nwg = prm.tiles_m * prm.tiles_n;
    const int xcd = (int)blockIdx.x & 7, slot = (int)blockIdx.x >> 3;
    const int per = nwg >> 3, rem = nwg & 7;
    const int vid = xcd * per + min(xcd, rem) + slot;
    const int band_wgs = prm.band_m * prm.tiles_n, band = vid / band_wgs, in_band = vid - band * band_wgs;
    const int band_rows = min(prm.band_m, prm.tiles_m - prm.band_m * band);
    const int m_blk = prm.band_m * band + in_band % band_rows, n_blk = in_band / band_rows;
    const int m0 = m_blk * 16 * kTA, n0 = n_blk * 16 * kTW;
    const int nsteps = prm.kblocks;

    // ---- loads: 1 KiB a wave and instruction, lane L 16 bytes at base + off to LDS address dst + 16 L (see the block kernel)
    auto lds_addr = [](const void* p) { return (unsigned)(uintptr_t)(const __attribute__((address_space(3))) uint8_t*)p; };
    auto lds_load = [](const void* base, unsigned off, unsigned dst) {
        asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %1, %2" : : "s"(dst), "v"(off), "s"(base) : "memory", "m0");
    };
    constexpr int kTiles = kTA + kTW, kTileLoads = (kTiles + kWaves - 1) / kWaves, kLoads = kTileLoads;
    const uint8_t* src[kTileLoads];      // tile u * kWaves + wave: rows of A first, then channels of W (the last may be loaded twice)
    int place_of[kTileLoads];
#pragma unroll
    for (int u = 0; u < kTileLoads; ++u) {
        const int t = min(u * kWaves + wave, kTiles - 1);
        place_of[u] = t;
        src[u] = t < kTA ? (const uint8_t*)(prm.a_blocks + (size_t)min(m0 / 16 + t, prm.a_tiles - 1) * prm.kblocks * 64)
                         : (const uint8_t*)(prm.w_blocks + (size_t)min(n0 / 16 + t - kTA, prm.w_tiles - 1) * prm.kblocks * 64);
    }
    auto load_piece = [&](int i, int step, const uint8_t* buf) {   // i-th load of a step
        lds_load(src[i], lane * 16 + step * 1024, lds_addr(buf) + place_of[i] * 1024);
    };
    // At most `left` loads of this wave are outstanding past it, none of its LDS reads, and every other wave is there too.
    auto sync = [&](auto LC) {
        constexpr int left = decltype(LC)::value;
        __builtin_amdgcn_sched_barrier(0);
        __builtin_amdgcn_s_waitcnt(0x0070 | (left & 15) | ((left >> 4) << 14));   // vmcnt(left) lgkmcnt(0)
        __builtin_amdgcn_s_barrier();
        asm volatile("" ::: "memory");
        __builtin_amdgcn_sched_barrier(0);
    };
    for (int i = wave; i < kRecA + kRecW; i += kWaves) {
        if (i < kRecA) lds_load(prm.aparams, (unsigned)min(m0 + i * 64 + lane, prm.M - 1) * 16u, lds_addr(par_a + i * 64));
        else lds_load(prm.wparams, (unsigned)min(n0 + (i - kRecA) * 64 + lane, prm.N - 1) * 16u, lds_addr(par_w + (i - kRecA) * 64));
    }
#pragma unroll
    for (int s = 0; s < S; ++s)
#pragma unroll
        for (int i = 0; i < kLoads; ++i) load_piece(i, min(s, nsteps - 1), ring + s * kBuf);

    v4f_f4 acc[MT][NT];
#pragma unroll
    for (int mt = 0; mt < MT; ++mt)
#pragma unroll
        for (int nt = 0; nt < NT; ++nt) acc[mt][nt] = v4f_f4{0.f, 0.f, 0.f, 0.f};
    const int one = 0x7F7F7F7F;   // block scales of 2^0
    const int a_off = rw * MT * 1024 + lane * 16, w_off = (kTA + cw * NT) * 1024 + lane * 16;
    v4i_f4 a[MT], w[2][NT];
    auto read_a = [&](int mt, const uint8_t* buf) { a[mt] = *reinterpret_cast<const v4i_f4*>(buf + a_off + mt * 1024); };
    auto read_w = [&](int nt, int set, const uint8_t* buf) { w[set][nt] = *reinterpret_cast<const v4i_f4*>(buf + w_off + nt * 1024); };
    auto mfma = [&](int set, int mt, int nt) {   // (weights first: a lane's four results are four channels of a row)
        const v4i_f4 b = w[set][nt];
        acc[mt][nt] = __builtin_amdgcn_mfma_scale_f32_16x16x128_f8f6f4(v8i_f4{b.x, b.y, b.z, b.w, 0, 0, 0, 0}, v8i_f4{a[mt].x, a[mt].y, a[mt].z, a[mt].w, 0, 0, 0, 0},
                                                                       acc[mt][nt], 4, 4, 0, one, 0, one);
    };
    sync(std::integral_constant<int, (S - 1) * kLoads>{});
#pragma unroll
    for (int nt = 0; nt < NT; ++nt) read_w(nt, 0, ring);
#pragma unroll
    for (int mt = 0; mt < MT; ++mt) read_a(mt, ring);

    constexpr int kHold = MT >= 8 ? 2 : 1, kSlots = MT * NT, kPast = kSlots - kHold * NT;
    unsigned place = 0;
    auto step_body = [&](auto SC, int step) {
        constexpr int set = decltype(SC)::value;
        const uint8_t* const cur = ring + place;
        place = place + kBuf == S * kBuf ? 0u : place + kBuf;
        const uint8_t* const nxt = ring + place;
        const int ahead = min(step + S, nsteps - 1);              // (past the end the last block is loaded again, for nobody)
#pragma unroll
        for (int i = 0; i < kSlots; ++i) {
            const int mt = i / NT, nt = i % NT, j = i - kHold * NT;
            mfma(set, mt, nt);
            if (j >= 0) {
#pragma unroll
                for (int u = 0; u < NT; ++u)
                    if (u * (kPast / 2) / NT == j) read_w(u, set ^ 1, nxt);
#pragma unroll
                for (int u = 0; u < kHold; ++u)
                    if (u * (kPast / 2) / kHold == j) read_a(u, nxt);
                if (nt == NT - 1) read_a(mt, nxt);
#pragma unroll
                for (int u = 0; u < kLoads; ++u)
                    if (1 + u * (kPast - 1) / kLoads == j) load_piece(u, ahead, cur);
            }
            __builtin_amdgcn_sched_barrier(0);
            if (j == -1) sync(std::integral_constant<int, (S - 2) * kLoads>{});
        }
    };
    int step = 0;
    for (; step + 2 <= nsteps; step += 2) {
        step_body(std::integral_constant<int, 0>{}, step);
        step_body(std::integral_constant<int, 1>{}, step + 1);
    }
    if (step < nsteps) step_body(std::integral_constant<int, 0>{}, step);
    __builtin_amdgcn_s_waitcnt(0x0070);                           // (the last loads, for nobody, land before LDS is given back)

    // ---- epilogue: the fused dequant of the other kernels (Fig. 3b), with the terms that depend on the column only taken out of the inner loop:
    // centered = S - wz asum - az (wsum - K wz).  A record's sum of codes may come in two parts, the second in its spare word (see f4_pack_kernel).
    const int wm0 = m0 + rw * MT * 16, wn0 = n0 + cw * NT * 16;
    if (prm.acc == nullptr) {
        // Every term here is an integer below 2^24 in magnitude (K * 9 < 2^24: the entry point checks it), and so is every
        // partial sum, so binary32 fused multiply-adds give the int32 arithmetic's value exactly, at four times the rate
        // of 32-bit integer multiplies; the accumulator needs no conversion either.  Stores as in the block kernel.
        static_assert(NT % 2 == 0, "tiles in pairs");
#pragma unroll
        for (int np = 0; np < NT; np += 2) {
            float wz[2][4], cwz[2][4], sw[2][4];
#pragma unroll
            for (int h = 0; h < 2; ++h)
#pragma unroll
                for (int reg = 0; reg < 4; ++reg) {
                    const RowParams pw = par_w[(cw * NT + np + h) * 16 + 4 * G + reg];
                    wz[h][reg] = -(float)pw.zero;
                    cwz[h][reg] = (float)(pw.sum + pw.pad - prm.K * pw.zero);
                    sw[h][reg] = pw.scale;
                }
#pragma unroll
            for (int mt = 0; mt < MT; ++mt) {
                const RowParams pa = par_a[(rw * MT + mt) * 16 + r];
                const float asum = (float)(pa.sum + pa.pad), az = -(float)pa.zero;
                uint32_t d[2][2];
#pragma unroll
                for (int h = 0; h < 2; ++h) {
                    uint32_t hv[4];
#pragma unroll
                    for (int reg = 0; reg < 4; ++reg) {
                        const float centered = __builtin_fmaf(az, cwz[h][reg], __builtin_fmaf(wz[h][reg], asum, acc[mt][np + h][reg]));
                        const float v = (centered * pa.scale) * sw[h][reg];
                        asm("v_cvt_f16_f32 %0, %1" : "=v"(hv[reg]) : "v"(v));   // (the instruction itself: see epilogue_value)
                    }
                    d[h][0] = __builtin_amdgcn_perm(hv[1], hv[0], 0x05040100u);
                    d[h][1] = __builtin_amdgcn_perm(hv[3], hv[2], 0x05040100u);
                }
                const auto lo = __builtin_amdgcn_permlane16_swap(d[0][0], d[1][0], false, false);
                const auto hi = __builtin_amdgcn_permlane16_swap(d[0][1], d[1][1], false, false);
                const int m = wm0 + mt * 16 + r, n = wn0 + (np + (G & 1)) * 16 + (G >> 1) * 8;
                if (m < prm.M && n < prm.N) store_row_part8(prm.y + (size_t)m * prm.N + n, n, prm.N, lo[0], hi[0], lo[1], hi[1]);
            }
        }
        return;
    }
#pragma unroll
    for (int mt = 0; mt < MT; ++mt) {
        RowParams pa = par_a[(rw * MT + mt) * 16 + r];
        pa.sum += pa.pad;
        const int m = wm0 + mt * 16 + r;
#pragma unroll
        for (int nt = 0; nt < NT; ++nt)
#pragma unroll
            for (int reg = 0; reg < 4; ++reg) {
                RowParams pw = par_w[(cw * NT + nt) * 16 + 4 * G + reg];
                pw.sum += pw.pad;
                const int n = wn0 + nt * 16 + 4 * G + reg;
                if (m < prm.M && n < prm.N) epilogue_store((int32_t)acc[mt][nt][reg], 0, 0, prm.K, pa, pw, (size_t)m * prm.N + n, prm.y, prm.acc);
            }
    }
}

// Workgroup shapes (rows of A, channels, workgroups a compute unit) and what a launch of each costs (us): `base`, `round` for every round of resident
// workgroups, and per block of 128 k what a unit with one or two of them takes.  Non-negative least squares of the relative error over 400 sizes
// (M = 17..2048, N = 256..13824, K = 512..13824) in cache, mean error 5 to 8 %; two shapes more (256 x 128, 128 x 256 by four waves) gained nothing there.
struct F4ShapeInfo { int bm, bn, occ; float base, round, step[2]; };
constexpr int kF4Shapes = 5;
static const F4ShapeInfo kF4ShapeInfo[kF4Shapes] = {{256, 256, 1, 0, 7.391f, {0.495f, 0}}, {128, 128, 1, 0, 4.353f, {0.18f, 0}}, {128, 128, 2, 0, 5.002f, {0.179f, 0.434f}},
                                                    {64, 128, 2, 0.651f, 3.477f, {0.119f, 0.29f}}, {32, 64, 2, 2.437f, 1.186f, {0.074f, 0.127f}}};

template <int RW, int CW, int MT, int NT, int S, int OCC>
static hipError_t f4_launch(const F4Params& prm, hipStream_t s)
{
    f4_gemm_kernel<RW, CW, MT, NT, S, OCC><<<(unsigned)(prm.tiles_m * prm.tiles_n), 64 * RW * CW, 0, s>>>(prm);
    return hipGetLastError();
}

hipError_t launch_f4_gemm(int M, int N, int K, const uint8_t* act_blob, const uint8_t* w_blob, uint16_t* y, int32_t* acc, hipStream_t s)
{
    F4Params prm;
    prm.a_blocks = (const v4i_f4*)(act_blob + f4_off_blocks(M));
    prm.w_blocks = (const v4i_f4*)(w_blob + f4_off_blocks(N));
    prm.aparams = (const RowParams*)(act_blob + f4_off_params());
    prm.wparams = (const RowParams*)(w_blob + f4_off_params());
    prm.y = y; prm.acc = acc;
    prm.M = M; prm.N = N; prm.K = K; prm.kblocks = f4_k_blocks(K);
    prm.a_tiles = f4_row_tiles(M); prm.w_tiles = f4_row_tiles(N);
    int shape = 0;
    double best = 0;
    for (int i = 0; i < kF4Shapes; ++i) {
        const F4ShapeInfo& f = kF4ShapeInfo[i];
        const long wgs = (long)((M + f.bm - 1) / f.bm) * ((N + f.bn - 1) / f.bn), cus = num_cus();
        const long load = (wgs + cus - 1) / cus, full = load / f.occ, part = load % f.occ;
        const double cost = f.base + f.round * (double)(full + part) + prm.kblocks * ((double)full * f.step[f.occ - 1] + (part ? f.step[0] : 0.f));
        if (i == 0 || cost < best) { best = cost; shape = i; }
    }
    const int bm = kF4ShapeInfo[shape].bm, bn = kF4ShapeInfo[shape].bn;
    prm.tiles_m = (M + bm - 1) / bm;
    prm.tiles_n = (N + bn - 1) / bn;
    const int cap = 2048 / bm, bands = (prm.tiles_m + cap - 1) / cap;   // (bands of equal height)
    prm.band_m = (prm.tiles_m + bands - 1) / bands;
    switch (shape) {
        case 0: return f4_launch<2, 4, 8, 4, 3, 2>(prm, s);
        case 1: return f4_launch<2, 4, 4, 2, 6, 2>(prm, s);
        case 2: return f4_launch<2, 2, 4, 4, 4, 2>(prm, s);
        case 3: return f4_launch<1, 4, 4, 2, 6, 2>(prm, s);
        default: return f4_launch<1, 2, 2, 2, 8, 2>(prm, s);
    }
}

}  // namespace abq
