// Rows of activations as the row kernels (one workgroup per token) read, quantize and write them: 16-byte vectors of
// rows that may start at any element, the per-token quantizer, and the choice of workgroup for a row length.
#pragma once
#include "abq_internal.h"

#include <type_traits>

namespace abq {

// Global memory takes vector accesses at element alignment; a row of K elements that is no whole number of vectors
// therefore goes by vectors too, all but its last K % 8 elements.
typedef uint32_t u32x4_half __attribute__((ext_vector_type(4), aligned(2)));
typedef uint32_t u32x4_byte __attribute__((ext_vector_type(4), aligned(1)));
typedef uint32_t u32x2_byte __attribute__((ext_vector_type(2), aligned(1)));

// Vector v (eight halves) of a row of K; elements past the row are zero.  The load is unconditional (clamped), the
// row's tail is gathered by the one lane that holds it.
template <bool RAGGED>
__device__ __forceinline__ void load_half8(const uint16_t* row, int v, int K, uint32_t* out)
{
    const int nfull = K >> 3;
    if (!RAGGED || nfull > 0) {
        const int vc = v < nfull ? v : nfull - 1;
        if constexpr (RAGGED) {
            const u32x4_half a = *reinterpret_cast<const u32x4_half*>(row + 8 * vc);
            out[0] = a.x; out[1] = a.y; out[2] = a.z; out[3] = a.w;
        } else {
            const uint4 a = *reinterpret_cast<const uint4*>(row + 8 * vc);
            out[0] = a.x; out[1] = a.y; out[2] = a.z; out[3] = a.w;
        }
    }
    if (v >= nfull) {
#pragma unroll
        for (int j = 0; j < 4; ++j) out[j] = 0u;
        if (RAGGED && v == nfull) {
#pragma unroll
            for (int e = 0; e < 7; ++e)
                if (8 * v + e < K) out[e >> 1] |= (uint32_t)row[8 * v + e] << (16 * (e & 1));
        }
    }
}

// Eight halves of an output row from channel n on (four dwords), up to the row's end.  A row that starts off a 16-byte boundary takes the
// same vector store (one store per half instead: W1A8 2048 x 6463 x 6832 96 us, 85 so).
__device__ __forceinline__ void store_row_part8(uint16_t* dst, int n, int N, uint32_t w0, uint32_t w1, uint32_t w2, uint32_t w3)
{
    if (n + 8 <= N) {
        *reinterpret_cast<u32x4_half*>(dst) = u32x4_half{w0, w1, w2, w3};
    } else {
        const uint32_t w[4] = {w0, w1, w2, w3};
#pragma unroll
        for (int e = 0; e < 7; ++e)
            if (n + e < N) dst[e] = (uint16_t)(w[e >> 1] >> (16 * (e & 1)));
    }
}

template <bool RAGGED>
__device__ __forceinline__ void store_half8(uint16_t* row, int v, int K, const uint32_t* in)
{
    const int nfull = K >> 3;
    if (v < nfull) {
        if constexpr (RAGGED) *reinterpret_cast<u32x4_half*>(row + 8 * v) = u32x4_half{in[0], in[1], in[2], in[3]};
        else *reinterpret_cast<uint4*>(row + 8 * v) = uint4{in[0], in[1], in[2], in[3]};
    } else if (RAGGED && v == nfull) {
#pragma unroll
        for (int e = 0; e < 7; ++e)
            if (8 * v + e < K) row[8 * v + e] = (uint16_t)(in[e >> 1] >> (16 * (e & 1)));
    }
}

template <bool RAGGED>
__device__ __forceinline__ void store_bytes8(uint8_t* row, int v, int K, const uint32_t* in)
{
    const int nfull = K >> 3;
    if (v < nfull) {
        if constexpr (RAGGED) *reinterpret_cast<u32x2_byte*>(row + 8 * v) = u32x2_byte{in[0], in[1]};
        else *reinterpret_cast<uint2*>(row + 8 * v) = uint2{in[0], in[1]};
    } else if (RAGGED && v == nfull) {
#pragma unroll
        for (int e = 0; e < 7; ++e)
            if (8 * v + e < K) row[8 * v + e] = (uint8_t)(in[e >> 2] >> (8 * (e & 3)));
    }
}

// The per-token quantizer: lo <= 0 <= hi the row's range, Delta = (hi - lo) / (2^q - 1) (1 if the range is empty),
// z = clamp(rint(-lo / Delta)), code = clamp(rint(x / Delta) + z); every float step one correctly rounded binary32
// operation, since they decide integer codes.
struct TokenQuantizer {
    typedef short s2v __attribute__((ext_vector_type(2)));
    float delta, inv;
    int z;
    s2v z2, top2;   // z and 2^q - 1, both halves
    __device__ __forceinline__ TokenQuantizer(float lo, float hi, int qmax)
    {
        delta = 1.0f;
        z = 0;
        if (hi != lo) {
            delta = __fdiv_rn(__fsub_rn(hi, lo), (float)qmax);
            const float r = rintf(__fdiv_rn(-lo, delta));
            z = r < 0.0f ? 0 : (r > (float)qmax ? qmax : (int)r);
        }
        inv = __fdiv_rn(1.0f, delta);
        z2 = s2v{(short)z, (short)z};
        top2 = s2v{(short)qmax, (short)qmax};
    }
    // The correctly rounded x / Delta from inv, the correctly rounded 1 / Delta: two residual corrections of x * inv, the
    // first brings it within one unit in the last place, the second rounds it correctly (P. Markstein, IBM J. Res. Dev.
    // 34, 1990, theorem on division from a correctly rounded reciprocal).  No step over- or underflows: |x| is zero or
    // 2^-24 .. 2^16 and Delta is 2^-32 .. 2^17.  Five operations; a general division is some fourteen, and one per
    // element was what bounded these kernels.
    __device__ __forceinline__ float quotient(float x) const
    {
        float t = __fmul_rn(x, inv);
        t = __fmaf_rn(__fmaf_rn(-t, delta, x), inv, t);
        return __fmaf_rn(__fmaf_rn(-t, delta, x), inv, t);
    }
    // Two halves -> their codes as 16-bit integers.  The conversion to integers takes a NaN to 0, which gives it the code of zero (as in
    // rows with planes); sums and clamps then go two at a time.  2048 x 5120 halves 8.3 us (clamped as floats, where a NaN became
    // code 0, 8.4; one integer at a time 8.9).
    __device__ __forceinline__ s2v codes2(uint32_t pair) const
    {
        const float r0 = rintf(quotient(__half2float(__ushort_as_half((unsigned short)(pair & 0xFFFFu)))));
        const float r1 = rintf(quotient(__half2float(__ushort_as_half((unsigned short)(pair >> 16)))));
        const s2v c = __builtin_bit_cast(s2v, __builtin_amdgcn_cvt_pk_i16((int)r0, (int)r1)) + z2;
        return __builtin_elementwise_min(__builtin_elementwise_max(c, s2v{0, 0}), top2);
    }
    // one half (as a float) -> its code
    __device__ __forceinline__ int code(float x) const
    {
        const int c = (int)rintf(quotient(x)) + z;
        return c < 0 ? 0 : (c > top2.x ? top2.x : c);
    }
    // four halves -> four code bytes
    __device__ __forceinline__ uint32_t codes4(uint32_t pair0, uint32_t pair1) const
    {
        return __builtin_amdgcn_perm(__builtin_bit_cast(uint32_t, codes2(pair1)), __builtin_bit_cast(uint32_t, codes2(pair0)), 0x06040200u);
    }
    // eight halves -> eight code bytes
    __device__ __forceinline__ void codes8(const uint32_t* half8, uint32_t* out) const
    {
        out[0] = codes4(half8[0], half8[1]);
        out[1] = codes4(half8[2], half8[3]);
    }
};

// Workgroup of a row kernel: BLOCK threads of VPT vectors of eight elements each, BLOCK * VPT >= nvec.  Few rows leave
// the chip idle and a row's latency is the time: as many threads as the row has vectors.  Many rows fill it: fewer,
// busier threads, whose reductions cost less per element.  `launch` is called with both as compile-time constants; false:
// the row is too long (more than 32768 elements) for a workgroup's registers.
template <class F>
static inline bool for_row_shape(int nvec, int M, F&& launch)
{
    auto go = [&](auto block, auto vpt) { launch(block, vpt); return true; };
    using std::integral_constant;
    if (nvec <= 64) return go(integral_constant<int, 64>{}, integral_constant<int, 1>{});
    if (nvec <= 128) return go(integral_constant<int, 128>{}, integral_constant<int, 1>{});
    if (nvec <= 256) return go(integral_constant<int, 256>{}, integral_constant<int, 1>{});
    if (M <= 256) {
        if (nvec <= 512) return go(integral_constant<int, 512>{}, integral_constant<int, 1>{});
        if (nvec <= 1024) return go(integral_constant<int, 1024>{}, integral_constant<int, 1>{});
        if (nvec <= 2048) return go(integral_constant<int, 1024>{}, integral_constant<int, 2>{});
    }
    if (nvec <= 512) return go(integral_constant<int, 256>{}, integral_constant<int, 2>{});
    if (nvec <= 768) return go(integral_constant<int, 256>{}, integral_constant<int, 3>{});
    if (nvec <= 1024) return go(integral_constant<int, 512>{}, integral_constant<int, 2>{});
    if (nvec <= 1536) return go(integral_constant<int, 512>{}, integral_constant<int, 3>{});
    if (nvec <= 2048) return go(integral_constant<int, 512>{}, integral_constant<int, 4>{});
    if (nvec <= 4096) return go(integral_constant<int, 1024>{}, integral_constant<int, 4>{});
    return false;
}

}  // namespace abq
