// Arithmetic of the per-token int8 activation quantizer (paper Eq. 1-2 with n = 8), shared by the
// stand-alone quantization kernel and the decode GEMM that quantizes its few tokens in its prologue.
// Every step is a single correctly rounded fp32 operation:
//   amax = max_k |x|            sx = amax / 127          inv = 127 / amax
//   code = clamp(rne(x * inv), -127, 127)                (all-zero token: sx = 1, codes 0)
#ifndef QL_QUANT_MATH_H
#define QL_QUANT_MATH_H

#include <hip/hip_fp16.h>
#include <hip/hip_runtime.h>

namespace ql {

constexpr int CHUNK = 16;               // elements per lane per step: 32 B in, 16 B out

struct alignas(16) Half16 {
    uint4 lo, hi;                       // 16 fp16 values
};

__device__ inline unsigned abs_max_bits(const Half16 &v, unsigned m)
{
    // |h| as an integer is monotonic in |value| for finite fp16, so the maximum can be taken on bits, two at a time
    typedef unsigned short us2 __attribute__((ext_vector_type(2)));
    const unsigned w[8] = {v.lo.x, v.lo.y, v.lo.z, v.lo.w, v.hi.x, v.hi.y, v.hi.z, v.hi.w};
    us2 p = __builtin_bit_cast(us2, w[0] & 0x7fff7fffu);
#pragma unroll
    for (int i = 1; i < 8; ++i) p = __builtin_elementwise_max(p, __builtin_bit_cast(us2, w[i] & 0x7fff7fffu));
    return max(m, max((unsigned)p[0], (unsigned)p[1]));
}

__device__ inline float half_bits_to_float(unsigned bits)
{
    return __half2float(__ushort_as_half((unsigned short)bits));
}

// Codes of four values t = x * inv (one fp32 multiply each, already within +-127): adding 1.5 * 2^23 rounds to the nearest
// integer, ties to even, and leaves the code's two's complement in the low byte -- an addition and 3/4 of a byte
// permute per code instead of a round, a clamp, a conversion and the masks and shifts that assemble the word.
__device__ inline unsigned code_word(float t0, float t1, float t2, float t3)
{
    const float magic = 12582912.0f;
    const unsigned u0 = __float_as_uint(t0 + magic), u1 = __float_as_uint(t1 + magic);
    const unsigned u2 = __float_as_uint(t2 + magic), u3 = __float_as_uint(t3 + magic);
    const unsigned lo = __builtin_amdgcn_perm(u1, u0, 0x0c0c0400u), hi = __builtin_amdgcn_perm(u3, u2, 0x0c0c0400u);
    return __builtin_amdgcn_perm(hi, lo, 0x05040100u);
}

__device__ inline float clamped(float x, float inv) { return fminf(fmaxf(x * inv, -127.0f), 127.0f); }

__device__ inline unsigned clamped_word(unsigned w0, unsigned w1, float inv)
{
    return code_word(clamped(half_bits_to_float(w0 & 0xffffu), inv), clamped(half_bits_to_float(w0 >> 16), inv),
                     clamped(half_bits_to_float(w1 & 0xffffu), inv), clamped(half_bits_to_float(w1 >> 16), inv));
}

__device__ inline unsigned quant_word(unsigned w0, unsigned w1, float inv)   // 4 halves -> 4 codes
{
    // |x| <= amax and inv = 127 / amax rounded: |x * inv| <= 127 + one ulp, which rounds to 127 -- no clamp.  The widening
    // and the multiply are one instruction (fma with 0: the sum with +0 changes nothing but the sign of a zero).
    return code_word(__builtin_fmaf(half_bits_to_float(w0 & 0xffffu), inv, 0.0f), __builtin_fmaf(half_bits_to_float(w0 >> 16), inv, 0.0f),
                     __builtin_fmaf(half_bits_to_float(w1 & 0xffffu), inv, 0.0f), __builtin_fmaf(half_bits_to_float(w1 >> 16), inv, 0.0f));
}

// The fast codes hold for finite tokens.  One with an infinity (inv = 0) or a NaN (inv = NaN) takes the products through the
// clamp, where a NaN becomes -127: its codes say nothing, but they are the same in every kernel and mode.  The clamp
// changes no code of a finite token, so all lanes of a wavefront go the same way: a scalar branch, decided on the maximum
// (`finite`), which is known before the division that gives inv.
__device__ inline bool no_lane(bool c) { return __builtin_amdgcn_ballot_w64(c) == 0; }

__device__ inline bool finite_tokens(unsigned amax_bits) { return no_lane(amax_bits >= 0x7c00u); }

__device__ inline uint4 quant_chunk(const Half16 &v, float inv, bool finite)
{
    uint4 q;
    if (finite) [[likely]] {
        q.x = quant_word(v.lo.x, v.lo.y, inv);
        q.y = quant_word(v.lo.z, v.lo.w, inv);
        q.z = quant_word(v.hi.x, v.hi.y, inv);
        q.w = quant_word(v.hi.z, v.hi.w, inv);
    } else {
        asm volatile("");               // or the compiler computes both sides for every token and selects
        q.x = clamped_word(v.lo.x, v.lo.y, inv);
        q.y = clamped_word(v.lo.z, v.lo.w, inv);
        q.z = clamped_word(v.hi.x, v.hi.y, inv);
        q.w = clamped_word(v.hi.z, v.hi.w, inv);
    }
    return q;
}

// the same code decision for fp32 values (operands after one of the paper's transforms, Eq. 3-4).  Here inv also overflows,
// when amax is below 127 / FLT_MAX: such tokens take the clamp too (which commutes with the rounding, its bounds are
// integers).
__device__ inline uint4 quant_chunk_f32(const float (&v)[16], float inv)
{
    unsigned q[4];
    if (no_lane(!(inv > 0.0f && inv <= 3.402823466e38f))) [[likely]] {
#pragma unroll
        for (int i = 0; i < 4; ++i) q[i] = code_word(v[4 * i] * inv, v[4 * i + 1] * inv, v[4 * i + 2] * inv, v[4 * i + 3] * inv);
    } else {
        asm volatile("");
#pragma unroll
        for (int i = 0; i < 4; ++i)
            q[i] = code_word(clamped(v[4 * i], inv), clamped(v[4 * i + 1], inv), clamped(v[4 * i + 2], inv), clamped(v[4 * i + 3], inv));
    }
    return make_uint4(q[0], q[1], q[2], q[3]);
}

__device__ inline void token_scales_f32(float amax, float &scale, float &inv)
{
    const bool zero = (amax == 0.0f);
    scale = zero ? 1.0f : amax / 127.0f;    // IEEE fp32 division
    inv = zero ? 0.0f : 127.0f / amax;      // IEEE fp32 division
}

// SwiGLU of the gated MLP in front of the quantizer (textbook definition: h = silu(gate) * up, silu(g) = g / (1 +
// exp(-g)); the paper names no activation function).  The result is that of correctly rounded fp32 operations one by one, the
// exponential included -- clamp, range reduction by n = rint(t log2 e) with a two-constant ln 2, degree-7 Horner
// polynomial in 1/k! (multiply, then add), exact scaling by 2^n -- so that the codes are a function of the inputs alone.
// Here the sequence is shorter by six: the multiply and add of n and of the first five Horner steps are one fused operation
// each, with the first three coefficients a few ulps from 1/7!, 1/6! and 1/5!, chosen so that silu(g) has the same bits for every
// one of the 63488 finite fp16 gates -- there are no other arguments (with 1/k! three gates differ; of the last two steps fused no
// coefficients were found, nor of n times the second constant of ln 2).  These operations, not memory, take most of the
// quantizer's time (4096 x 11008: 225 MB in 56 us).  us, before and after: 4096 x 11008 56.8 / 50.4, 1900 x 6144 19.7 / 17.8,
// 512 x 11008 11.7 / 10.7.
__device__ inline float exp_steps(float t)      // t = -g in [-80, 80], g an fp16 value
{
    // n = rint(t log2 e): adding 1.5 * 2^23 rounds to the nearest integer, ties to even, and leaves n in the low bits
    const float magic = 12582912.0f;
    const float z = __builtin_fmaf(t, 1.4426950408889634f, magic);
    const float n = z - magic;
    float r = __builtin_fmaf(-n, 0.693359375f, t);      // n * (355 / 512) is exact: the same as multiply, then subtract
    r = r - n * -2.12194440e-4f;
    float p = 0x1.a03c88p-13f;                           // 1/5040 + 6.4e-8
    p = __builtin_fmaf(p, r, 0x1.6c142ap-10f);           // 1/720 - 3.9e-8
    p = __builtin_fmaf(p, r, 0x1.11116cp-7f);            // 1/120 + 4.2e-8
    p = __builtin_fmaf(p, r, (float)(1.0 / 24));
    p = __builtin_fmaf(p, r, (float)(1.0 / 6));
    p = __builtin_fmaf(p, r, 0.5f);
    p = p * r + 1.0f;
    p = p * r + 1.0f;
    // times 2^n by adding n to the exponent, exact: |n| <= 116 and 0.7 < p < 1.42 (the shift leaves n of z's bits only)
    return __uint_as_float((__float_as_uint(z) << 23) + __float_as_uint(p));
}

// 1 / d correctly rounded for the d = 1 + exp(t) that an fp16 gate can give (1 <= d < 2^116: no operand or result near the
// ends of the exponent range, where the general division spends most of its instructions): the hardware's
// approximation and one Newton step in fused operations.  Checked for every fp16 gate against the IEEE division.
__device__ inline float reciprocal_of_sum(float d)
{
    const float y = __builtin_amdgcn_rcpf(d);
    return __builtin_fmaf(__builtin_fmaf(-d, y, 1.0f), y, y);
}

__device__ inline float swiglu_f32(float g, float u)
{
    const float t = fminf(fmaxf(-g, -80.0f), 80.0f);
    const float d = 1.0f + exp_steps(t);
    // u's widening and the multiply in one (as in quant_word): 4096 x 11008 49 / 47.8 us, 1900 x 6144 16.7 / 16.3, 512 x 11008 9.9 / 9.5
    return __builtin_fmaf(g * reciprocal_of_sum(d), u, 0.0f);
}

// {a, b} = {v of this lane, v of lane ^ OFF}, in either order, without the hundred cycles of a shuffle through LDS: for operations
// that commute, in the pairs of a butterfly.  us, shuffles / these steps: SmoothQuant + Hadamard quantizer and W4A8 GEMM of 3001 x
// 4096 x 4096 70.5 / 67.5; decoder layer with the quantizer in the decode GEMMs, 1 token W8A8 52.4 / 51.5, 8 tokens W4A8 48.0 / 46.7;
// RMSNorm of 2048 x 14336 31.6 / 30.8.
template <int OFF>
__device__ inline void lane_pair(unsigned v, unsigned &a, unsigned &b)
{
    static_assert(OFF == 32 || OFF == 16 || OFF == 8 || OFF == 4 || OFF == 2 || OFF == 1, "a power of two below 64");
    a = v;
    if constexpr (OFF == 32) {
        const auto s = __builtin_amdgcn_permlane32_swap(v, v, false, false);     // lower halves, upper halves
        a = s[0], b = s[1];
    } else if constexpr (OFF == 16) {
        const auto s = __builtin_amdgcn_permlane16_swap(v, v, false, false);     // even rows, odd rows
        a = s[0], b = s[1];
    } else if constexpr (OFF == 8) {
        b = (unsigned)__builtin_amdgcn_mov_dpp((int)v, 0x128, 0xf, 0xf, true);   // row_ror:8
    } else if constexpr (OFF == 4) {
        const int up = __builtin_amdgcn_update_dpp(0, (int)v, 0x104, 0xf, 0x5, false);   // row_shl:4 into banks 0 and 2
        b = (unsigned)__builtin_amdgcn_update_dpp(up, (int)v, 0x114, 0xf, 0xa, false);   // row_shr:4 into banks 1 and 3
    } else {
        b = (unsigned)__builtin_amdgcn_mov_dpp((int)v, OFF == 2 ? 0x4E : 0xB1, 0xf, 0xf, true);   // quad_perm
    }
}

template <int OFF>
__device__ inline unsigned max_pair(unsigned v)
{
    unsigned a, b;
    lane_pair<OFF>(v, a, b);
    return max(a, b);
}

template <int OFF>
__device__ inline double sum_pair(double v)
{
    const uint64_t u = __builtin_bit_cast(uint64_t, v);
    unsigned a0, a1, b0, b1;
    lane_pair<OFF>((unsigned)u, a0, b0);
    lane_pair<OFF>((unsigned)(u >> 32), a1, b1);
    return __builtin_bit_cast(double, (uint64_t)a1 << 32 | a0) + __builtin_bit_cast(double, (uint64_t)b1 << 32 | b0);
}

// Maximum over the wavefront, or over its first 16 lanes, in steps inside the registers: a shuffle through LDS takes about a
// hundred cycles, every token waited for six of them in turn and then read the wavefronts' maxima one by one.  us, before / after
// (the first figure also has the branch in front of the loads): SwiGLU 512 x 11008 10.7 / 9.9, 1900 x 6144 17.8 / 16.7,
// 4096 x 11008 50.4 / 48.9; plain 300 x 4096 3.7 / 3.2, 512 x 11008 6.9 / 6.3, 2048 x 14336 24.4 / 21.0; RMSNorm 1900 x 1536
// 5.1 / 4.9, 2048 x 14336 33.2 / 30.7.
template <bool WHOLE>
__device__ inline unsigned max_over_lanes(unsigned v)
{
    v = max(v, (unsigned)__builtin_amdgcn_update_dpp(0, (int)v, 0x111, 0xf, 0xf, true));        // row_shr:1, 2, 4, 8
    v = max(v, (unsigned)__builtin_amdgcn_update_dpp(0, (int)v, 0x112, 0xf, 0xf, true));
    v = max(v, (unsigned)__builtin_amdgcn_update_dpp(0, (int)v, 0x114, 0xf, 0xf, true));
    v = max(v, (unsigned)__builtin_amdgcn_update_dpp(0, (int)v, 0x118, 0xf, 0xf, true));
    if constexpr (!WHOLE) return (unsigned)__builtin_amdgcn_readlane((int)v, 15);
    v = max(v, (unsigned)__builtin_amdgcn_update_dpp(0, (int)v, 0x142, 0xa, 0xf, false));       // row_bcast:15 into rows 1 and 3
    v = max(v, (unsigned)__builtin_amdgcn_update_dpp(0, (int)v, 0x143, 0xc, 0xf, false));       // row_bcast:31 into rows 2 and 3
    return (unsigned)__builtin_amdgcn_readlane((int)v, 63);
}

// token scale and its reciprocal from the bit pattern of the largest |x|
__device__ inline void token_scales(unsigned amax_bits, float &scale, float &inv)
{
    const float amax = half_bits_to_float(amax_bits);
    const bool zero = (amax_bits == 0);
    scale = zero ? 1.0f : amax / 127.0f;    // IEEE fp32 division
    inv = zero ? 0.0f : 127.0f / amax;      // IEEE fp32 division
}

}  // namespace ql
#endif
