// The operand transforms of the paper's two enhanced W4A8 configurations, for gfx950:
//   SmoothQuant (Eq. 3):  Y = (X S^-1)(S W),  s_j = max|X_j|^alpha / max|W_j|^(1-alpha)
//   Hadamard   (Eq. 4):  Y = (X H)(H^T W),   H a normalized Hadamard matrix
// Online: the activation side (per-channel multiply by 1/s_j, or a fast Walsh-Hadamard transform of every
// token) is fused in front of the per-token int8 quantizer (Eq. 1-2), one workgroup per token, fp32 throughout.
// Offline: calibration statistics, the scale vector, and the transformed fp32 weights handed to the weight
// quantizer.
//
// H is the natural-order (Sylvester) matrix, block diagonal with blocks of B = the largest power of two that
// divides K (at most 4096) so that any K % 64 == 0 works.  It is applied as the in-place butterfly in fp32,
// stages h = 1, 2, ..., B/2 in that order, every output one addition or subtraction, then one multiply by
// fp32(1/sqrt(B)): a fixed sequence of single fp32 operations per element, whatever lane does them.
// A wavefront holds whole blocks: one chunk of 16 consecutive elements per lane covers 1024 elements, larger blocks take two
// or four chunks per lane.  So no stage leaves the wavefront: stages h <= 8 and h >= 1024 are in registers, the four in
// between inside a row of 16 lanes are one lane-permuting multiply-add each, the two across the rows swap registers.
#include "common.h"
#include "quant_math.h"
#include <algorithm>
#include <cmath>
#include <type_traits>

namespace ql {
namespace {

// ---- Hadamard transform of blocks of 2^LB elements held by one wavefront.  NIT = chunks per lane; element
//   k = (it * 64 + l) * 16 + i   of the wavefront's piece sits in v[it][i] of the lane whose logical number is l.
// Logical lane l of physical lane p: l = p ^ (p & 4 ? 3 : 0), so that a step of one bit in l is a step in p that a
// lane-permuting operand modifier can make: l^1 and l^2 are p^1, p^2 (quad permutes), l^4 is p^7 (half-row mirror), l^8
// is p^8 (row rotation).
constexpr int hadamard_chunks(int lb) { return lb > 10 ? 1 << (lb - 10) : 1; }

__device__ inline int logical_lane(int p) { return p ^ ((p & 4) ? 3 : 0); }

// One stage between logical lanes that differ in one bit.  The lower lane needs a + b and the upper a - b; both compute
// (own value) + s * (partner's), s = +1 below and -1 above, a single rounding each: the upper lane is left with the negative
// of its result.  Every value of a lane then carries the same sign, -1 to the number of such stages in which the lane was
// the upper one; partners agree in it (they differ in the stage's own bit only), and the final multiply takes it out.
// Written as one block of multiply-adds whose first operand is permuted (the compiler keeps the permutation a move of its
// own, with wait states in front of each).  gfx950 needs two wait states between a vector write of a register and its
// permuted read or lane-register swap: the leading s_nop covers them for the first multiply-add, the last one for whatever
// follows -- the compiler counts them for its own instructions but does not see writes inside the block.  Every lane of
// the wavefront is active here and every source lane exists.
#define QL_FMAC_DPP(i, ctrl) "v_fmac_f32_dpp %" #i ", %" #i ", %16 " ctrl " row_mask:0xf bank_mask:0xf\n\t"
#define QL_LANE_STAGE(name, ctrl)                                                                                                     \
    __device__ inline void name(float (&v)[16], float s)                                                                              \
    {                                                                                                                                 \
        asm("s_nop 1\n\t" QL_FMAC_DPP(0, ctrl) QL_FMAC_DPP(1, ctrl) QL_FMAC_DPP(2, ctrl) QL_FMAC_DPP(3, ctrl) QL_FMAC_DPP(4, ctrl)      \
                QL_FMAC_DPP(5, ctrl) QL_FMAC_DPP(6, ctrl) QL_FMAC_DPP(7, ctrl) QL_FMAC_DPP(8, ctrl) QL_FMAC_DPP(9, ctrl)               \
                    QL_FMAC_DPP(10, ctrl) QL_FMAC_DPP(11, ctrl) QL_FMAC_DPP(12, ctrl) QL_FMAC_DPP(13, ctrl) QL_FMAC_DPP(14, ctrl)       \
                        QL_FMAC_DPP(15, ctrl) "s_nop 1"                                                                               \
            : "+v"(v[0]), "+v"(v[1]), "+v"(v[2]), "+v"(v[3]), "+v"(v[4]), "+v"(v[5]), "+v"(v[6]), "+v"(v[7]), "+v"(v[8]), "+v"(v[9]),  \
              "+v"(v[10]), "+v"(v[11]), "+v"(v[12]), "+v"(v[13]), "+v"(v[14]), "+v"(v[15])                                            \
            : "v"(s));                                                                                                                \
    }
QL_LANE_STAGE(stage_lane1, "quad_perm:[1,0,3,2]")
QL_LANE_STAGE(stage_lane2, "quad_perm:[2,3,0,1]")
QL_LANE_STAGE(stage_lane4, "row_half_mirror")
QL_LANE_STAGE(stage_lane8, "row_ror:8")
#undef QL_LANE_STAGE
#undef QL_FMAC_DPP

// Swap between two registers and lanes 16 (32) apart: afterwards `a` holds, in lanes with that bit clear, what it held
// there, and in lanes with it set, what `b` held in the lane 16 (32) below; `b` the rest.  Its own inverse.
template <int DIST>
__device__ inline void lane_register_swap(unsigned &a, unsigned &b)
{
    const auto r = DIST == 16 ? __builtin_amdgcn_permlane16_swap(a, b, false, false) : __builtin_amdgcn_permlane32_swap(a, b, false, false);
    a = r[0], b = r[1];
}

template <int DIST>
__device__ inline void lane_register_swap(float &a, float &b)
{
    unsigned x = __float_as_uint(a), y = __float_as_uint(b);
    lane_register_swap<DIST>(x, y);
    a = __uint_as_float(x), b = __uint_as_float(y);
}

// The transform, multiplied by `norm`.  Where LB >= 9 (10) lane bit 4 (5) and register bit 2 (3) have changed places on
// return: v[it][8 * c5 + 4 * c4 + j] is then element 8 * (lane bit 5) + 4 * (lane bit 4) + j of the chunk of logical lane
// (l & 15) + 16 * c4 + 32 * c5 (LB = 9: bit 4 only).  unswap_words / unswap_values put things back.
template <int LB, int NIT>
__device__ inline void hadamard_wave(float (&v)[NIT][16], int l, float norm)
{
    static_assert(LB == 0 || LB >= 4, "no transform, or whole chunks");
    if (LB > 0) {
#pragma unroll
        for (int it = 0; it < NIT; ++it)
#pragma unroll
            for (int h = 1; h < 16; h <<= 1)
#pragma unroll
                for (int i = 0; i < 16; ++i)
                    if ((i & h) == 0) {
                        const float a = v[it][i], b = v[it][i | h];
                        v[it][i] = a + b;
                        v[it][i | h] = a - b;
                    }
    }
#pragma unroll
    for (int it = 0; it < NIT; ++it) {
        if (LB > 4) stage_lane1(v[it], (l & 1) ? -1.0f : 1.0f);
        if (LB > 5) stage_lane2(v[it], (l & 2) ? -1.0f : 1.0f);
        if (LB > 6) stage_lane4(v[it], (l & 4) ? -1.0f : 1.0f);
        if (LB > 7) stage_lane8(v[it], (l & 8) ? -1.0f : 1.0f);
    }
    // across the rows: after the swap both operands of a pair sit in one lane
    if (LB > 8) {
#pragma unroll
        for (int it = 0; it < NIT; ++it)
#pragma unroll
            for (int i = 0; i < 16; ++i)
                if ((i & 4) == 0) {
                    lane_register_swap<16>(v[it][i], v[it][i | 4]);
                    const float a = v[it][i], b = v[it][i | 4];
                    v[it][i] = a + b;
                    v[it][i | 4] = a - b;
                }
    }
    if (LB > 9) {
#pragma unroll
        for (int it = 0; it < NIT; ++it)
#pragma unroll
            for (int i = 0; i < 16; ++i)
                if ((i & 8) == 0) {
                    lane_register_swap<32>(v[it][i], v[it][i | 8]);
                    const float a = v[it][i], b = v[it][i | 8];
                    v[it][i] = a + b;
                    v[it][i | 8] = a - b;
                }
    }
#pragma unroll
    for (int bit = 1; bit < NIT; bit <<= 1)
#pragma unroll
        for (int it = 0; it < NIT; ++it)
            if ((it & bit) == 0) {
#pragma unroll
                for (int i = 0; i < 16; ++i) {
                    const float a = v[it][i], b = v[it | bit][i];
                    v[it][i] = a + b;
                    v[it | bit][i] = a - b;
                }
            }
    if (LB > 0) {
        const int dpp_bits = LB >= 8 ? 15 : LB == 7 ? 7 : LB == 6 ? 3 : LB == 5 ? 1 : 0;
        const float scale = (__popc(l & dpp_bits) & 1) ? -norm : norm;
#pragma unroll
        for (int it = 0; it < NIT; ++it)
#pragma unroll
            for (int i = 0; i < 16; ++i) v[it][i] *= scale;
    }
}

template <int LB>
__device__ inline void unswap_words(unsigned (&w)[4])   // one 32-bit word per four registers of a chunk
{
    if (LB > 9) lane_register_swap<32>(w[0], w[2]), lane_register_swap<32>(w[1], w[3]);
    if (LB > 8) lane_register_swap<16>(w[0], w[1]), lane_register_swap<16>(w[2], w[3]);
}

template <int LB>
__device__ inline void unswap_values(float (&v)[16])
{
    if (LB > 9) {
#pragma unroll
        for (int i = 0; i < 8; ++i) lane_register_swap<32>(v[i], v[i | 8]);
    }
    if (LB > 8) {
#pragma unroll
        for (int i = 0; i < 16; ++i)
            if ((i & 4) == 0) lane_register_swap<16>(v[i], v[i | 4]);
    }
}

__device__ inline __amdgpu_buffer_rsrc_t buffer_of(const void *p, size_t bytes)
{
    return __builtin_amdgcn_make_buffer_rsrc(const_cast<void *>(p), 0, (int)(unsigned)bytes, 0x00020000);
}

// the wavefront's chunks of one row as fp32, times the optional per-channel factors (one fp32 multiply each)
template <int NIT>
__device__ inline void load_row(const __half *row, bool present, int K, const float *factor, int c0, float (&v)[NIT][16])
{
    typedef unsigned v4u __attribute__((ext_vector_type(4)));
    const __amdgpu_buffer_rsrc_t rs = buffer_of(row, present ? (size_t)K * sizeof(__half) : 0);
    const __amdgpu_buffer_rsrc_t rf = buffer_of(factor, factor ? (size_t)K * sizeof(float) : 0);
    v4u raw[NIT][2];
#pragma unroll
    for (int it = 0; it < NIT; ++it)
#pragma unroll
        for (int q = 0; q < 2; ++q)
            raw[it][q] = __builtin_bit_cast(v4u, __builtin_amdgcn_raw_buffer_load_b128(rs, (unsigned)(c0 + it * 64) * 32u + q * 16u, 0, 0));
#pragma unroll
    for (int it = 0; it < NIT; ++it) {
#pragma unroll
        for (int i = 0; i < 8; ++i) {
            v[it][2 * i] = half_bits_to_float(raw[it][i / 4][i % 4] & 0xffffu);
            v[it][2 * i + 1] = half_bits_to_float(raw[it][i / 4][i % 4] >> 16);
        }
        if (factor) {
#pragma unroll
            for (int q = 0; q < 4; ++q) {
                const v4u f = __builtin_bit_cast(v4u, __builtin_amdgcn_raw_buffer_load_b128(rf, (unsigned)(c0 + it * 64) * 64u + q * 16u, 0, 0));
#pragma unroll
                for (int e = 0; e < 4; ++e) v[it][4 * q + e] *= __uint_as_float(f[e]);
            }
        }
    }
}

// Row of this workgroup: workgroup ids go to the 8 XCDs in turn, every XCD takes one contiguous range of whole groups of
// `unit` rows (rows that share 128-byte lines of the tile order), so that the lines are completed in one L2.
__device__ inline int row_of_workgroup(int rows, int unit)
{
    const int groups = (rows + unit - 1) / unit, xcd = blockIdx.x % 8, in_xcd = blockIdx.x / 8;
    const int mine = groups / 8 + (xcd < groups % 8 ? 1 : 0);
    if (in_xcd >= unit * mine) return rows;
    return unit * (xcd * (groups / 8) + (xcd < groups % 8 ? xcd : groups % 8)) + in_xcd;
}

inline int workgroups_for(int rows, int unit) { return 8 * unit * ceil_div(ceil_div(rows, unit), 8); }

constexpr int MAX_WAVES = 16;

// Activations: one workgroup per token, one chunk per lane whatever the block.  The stages of blocks of 2048 and 4096 that
// lie above a wavefront's 1024 elements are taken behind one exchange through LDS in which each of the W = 2 or 4
// wavefronts of a block gets its 16 / W values of every lane from all of them; the codes go back the same way, a quarter
// of the bytes.  (Bound by the 3 bytes per element and, where all tokens are resident at once, by the time the last of them
// takes from its last byte on: with W chunks per lane in one wavefront 1 x 4096 took 5.4 us instead of 3.8 and
// 4096 x 4096 20.2 instead of 18.2; with 256 lanes per token, two operations per element and lane stage, a
// bpermute for the stages across rows and two exchanges of all values, 22.2.)
template <int LB>
__global__ __launch_bounds__(MAX_WAVES * 64) void act_quant_hadamard_kernel(const __half *__restrict__ x, int64_t ldx, int M, int K,
                                                                             const float *__restrict__ inv_smooth, float norm,
                                                                             int8_t *__restrict__ xq_rm, int8_t *__restrict__ xq_kl,
                                                                             float *__restrict__ sx)
{
    constexpr int W = hadamard_chunks(LB);          // wavefronts per block
    constexpr int LANE_LB = LB > 10 ? 10 : LB;
    __shared__ float red[MAX_WAVES];
    extern __shared__ __attribute__((aligned(16))) float4 exch[];   // W > 1: [wavefront][4 planes of 4 registers][64 lanes]
    const int m = row_of_workgroup(M, 8);
    if (m >= M) return;
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6, nwaves = blockDim.x >> 6;
    const int l = logical_lane(lane), c = wave * 64 + l;            // chunk of this lane
    float v[1][16];
    load_row<1>(x + (size_t)m * ldx, true, K, inv_smooth, c, v);
    hadamard_wave<LANE_LB>(v, l, W > 1 ? 1.0f : norm);
    const int first = wave / W * W, part = wave % W;                // wavefronts of the block; this one's share of the registers
    constexpr int P = 4 / W;                                        // planes per share
    if constexpr (W > 1) {
#pragma unroll
        for (int p = 0; p < 4; ++p) exch[(wave * 4 + p) * 64 + lane] = make_float4(v[0][4 * p], v[0][4 * p + 1], v[0][4 * p + 2], v[0][4 * p + 3]);
        __syncthreads();
#pragma unroll
        for (int src = 0; src < W; ++src)
#pragma unroll
            for (int p = 0; p < P; ++p) {
                const float4 f = exch[((first + src) * 4 + part * P + p) * 64 + lane];
                const int at = 4 * (src * P + p);
                v[0][at] = f.x, v[0][at + 1] = f.y, v[0][at + 2] = f.z, v[0][at + 3] = f.w;
            }
#pragma unroll
        for (int bit = 1; bit < W; bit <<= 1)
#pragma unroll
            for (int src = 0; src < W; ++src)
                if ((src & bit) == 0) {
#pragma unroll
                    for (int e = 0; e < 4 * P; ++e) {
                        const float f = v[0][4 * src * P + e], g = v[0][4 * (src | bit) * P + e];
                        v[0][4 * src * P + e] = f + g;
                        v[0][4 * (src | bit) * P + e] = f - g;
                    }
                }
#pragma unroll
        for (int i = 0; i < 16; ++i) v[0][i] *= norm;
    }
    float amax = 0.0f;
#pragma unroll
    for (int i = 0; i < 16; ++i) amax = __builtin_elementwise_maximum(amax, fabsf(v[0][i]));   // passes a NaN on
    amax = __uint_as_float(max_over_lanes<true>(__float_as_uint(amax)));   // not negative, a NaN above all: ordered like their bits
    if (nwaves > 1) {
        if (lane == 0) red[wave] = amax;
        __syncthreads();
        static_assert(MAX_WAVES <= 16, "one row of lanes takes the wavefronts' maxima");
        amax = __uint_as_float(max_over_lanes<false>(lane < nwaves ? __float_as_uint(red[lane]) : 0u));
    }
    float scale, inv;
    token_scales_f32(amax, scale, inv);
    if (threadIdx.x == 0) sx[m] = scale;
    const uint4 s = quant_chunk_f32(v[0], inv);
    unsigned w[4] = {s.x, s.y, s.z, s.w};
    if constexpr (W > 1) {   // word (src, p) of this share is word part * P + p of the chunk that wavefront `src` started from
        unsigned *words = reinterpret_cast<unsigned *>(exch);
#pragma unroll
        for (int src = 0; src < W; ++src)
#pragma unroll
            for (int p = 0; p < P; ++p) words[((first + src) * 64 + lane) * 4 + part * P + p] = w[src * P + p];
        __syncthreads();
        const uint4 q = *reinterpret_cast<const uint4 *>(words + (wave * 64 + lane) * 4);
        w[0] = q.x, w[1] = q.y, w[2] = q.z, w[3] = q.w;
    }
    unswap_words<LANE_LB>(w);
    if (c < K / 16) {
        const uint4 q = make_uint4(w[0], w[1], w[2], w[3]);
        if (xq_rm) *reinterpret_cast<uint4 *>(xq_rm + (size_t)m * K + (size_t)c * 16) = q;
        if (xq_kl) *reinterpret_cast<uint4 *>(xq_kl + tile_offset_i8(m, c * 16, K)) = q;
    }
}

// A wavefront's 64 chunks of 16 fp32 values (first chunk `c_first`, this lane's is `l`) to row[0, K): through its 4 KB of LDS, so
// that a store instruction covers 1024 contiguous bytes.  Straight from the registers it takes 16 bytes out of every lane's
// 64: four instructions touch each 128-byte line, and 180 MB of them held the kernel at 3.6 TB/s (4096 x 11008, int4: 98 us
// against 62).  Within a chunk the four pieces are rotated by the chunk's number, or the 64-byte stride would meet the same banks.
// Non-temporal: nothing here reads the values again, and the fp16 weights that the next calls read stay cached
// (calibration, scales and this kernel 98.5 against 86 us; non-temporal stores straight from the registers: 161 us here).
__device__ inline void store_chunks(float *row, int K, float4 *stage, int c_first, int l, int lane, const float (&v)[16])
{
    typedef float f4 __attribute__((ext_vector_type(4)));
#pragma unroll
    for (int q = 0; q < 4; ++q) stage[l * 4 + (q ^ ((l >> 1) & 3))] = make_float4(v[4 * q], v[4 * q + 1], v[4 * q + 2], v[4 * q + 3]);
    asm volatile("" ::: "memory");   // (same wavefront, LDS operations complete in order: only the compiler must keep them so)
    __builtin_amdgcn_wave_barrier();
#pragma unroll
    for (int r = 0; r < 4; ++r) {
        const int chunk = r * 16 + lane / 4, q = lane % 4;
        const float4 f = stage[chunk * 4 + (q ^ ((chunk >> 1) & 3))];
        if (c_first + chunk < K / 16)
            __builtin_nontemporal_store(f4{f.x, f.y, f.z, f.w}, reinterpret_cast<f4 *>(row + (size_t)(c_first + chunk) * 16 + q * 4));
    }
    asm volatile("" ::: "memory");
    __builtin_amdgcn_wave_barrier();
}

// Codes of a chunk, a byte each: clamp(rint(w / s)) with the IEEE fp32 division by the stored scale, ties to even, that the
// quantizer of weight_quant.hip makes -- but by one reciprocal for the chunk and a multiplication per weight wherever that cannot
// matter: w * (1 / s) lies within 1.5 * 2^-23 of the divided value (relative; 1.3e-6 at the largest int4 code, 2.3e-5 at the largest
// int8 code), so both round to the same integer unless the product comes closer than the margin below to the middle between
// two.  A wavefront with such a weight (in fp32 normal data about 1 % of them with int4, 10 % with int8), or with a scale whose
// reciprocal or own rounding is not that accurate (fp32 below 2^-125 or above 2^125, fp16 subnormal, non-finite; there the clamp
// counts as well), divides.  4096 x 11008 with the transform: int4 62.4 to 61.5 us alone, calibration, scales and this together 85.9 to 77.9.
template <int LIMIT>
__device__ inline void weight_codes(const float (&v)[16], float s, unsigned (&q)[4])
{
    constexpr float MAGIC = 12582912.0f, MIDDLE = LIMIT == 7 ? 0.499995f : 0.49995f;
    constexpr float SMALLEST = LIMIT == 7 ? 6.103515625e-5f : 2.35098870e-38f, LARGEST = 4.25352959e37f;   // 2^-14, 2^-125; 2^125
    const float inv = 1.0f / s;
    float worst = 0.0f;
#pragma unroll
    for (int i = 0; i < 16; ++i) {
        const float t = v[i] * inv;
        worst = __builtin_elementwise_maximum(worst, fabsf(t - ((t + MAGIC) - MAGIC)));   // passes a NaN on
    }
    if (no_lane(!(worst <= MIDDLE && s >= SMALLEST && s <= LARGEST))) [[likely]] {
#pragma unroll
        for (int i = 0; i < 4; ++i) q[i] = code_word(v[4 * i] * inv, v[4 * i + 1] * inv, v[4 * i + 2] * inv, v[4 * i + 3] * inv);
    } else {
        asm volatile("");               // or the compiler computes both sides for every chunk and selects
#pragma unroll
        for (int i = 0; i < 4; ++i) q[i] = 0;
#pragma unroll
        for (int i = 0; i < 16; ++i) q[i / 4] |= (unsigned)((int)fminf(fmaxf(rintf(v[i] / s), (float)-LIMIT), (float)LIMIT) & 0xff) << (8 * (i % 4));
    }
}

// Offline: S W and / or H^T W of one weight row (output channel) per workgroup, its fp32 values stored (w32) and quantized
// from the registers in the same pass (bound by HBM: 2 bytes in, 4 + 2 x codes out per weight; as two kernels the
// fp32 values were read back: 145 us for 4096 x 11008, int4, against 62 in one).  Rows N .. 32-row padding: zero codes.
// STORED: quantizes what an earlier launch left in w32 (only where the results take the place of the inputs).
template <int LB, int BITS, bool STORED = false>
__global__ __launch_bounds__(MAX_WAVES * 64) void weight_transform_quant_kernel(const __half *__restrict__ w, int N, int Npad, int K,
                                                                                 const float *__restrict__ smooth, float norm,
                                                                                 float *__restrict__ w32, uint8_t *__restrict__ canon,
                                                                                 void *__restrict__ scales, uint8_t *__restrict__ kl,
                                                                                 __half *__restrict__ kl_scales, __half *__restrict__ kl_scales_dec)
{
    constexpr int NIT = hadamard_chunks(LB);
    __shared__ float red[MAX_WAVES];
    extern __shared__ __attribute__((aligned(16))) float4 stage[];   // 4 KB per wavefront (none if STORED)
    const int n = row_of_workgroup(Npad, 32);
    if (n >= Npad) return;
    const bool real = n < N;
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6, nwaves = blockDim.x >> 6;
    const int l = logical_lane(lane), c0 = wave * NIT * 64 + l, G = K / 128;
    float v[NIT][16];
    if constexpr (STORED) {
        static_assert(LB == 0, "already transformed");
#pragma unroll
        for (int it = 0; it < NIT; ++it) {
            const int c = c0 + it * 64;
            const bool there = real && c < K / 16;
#pragma unroll
            for (int i = 0; i < 16; ++i) v[it][i] = there ? w32[(size_t)n * K + (size_t)c * 16 + i] : 0.0f;
        }
    } else {
        load_row<NIT>(w + (size_t)(real ? n : 0) * K, real, K, smooth, c0, v);
        hadamard_wave<LB>(v, l, norm);
#pragma unroll
        for (int it = 0; it < NIT; ++it) unswap_values<LB>(v[it]);
    }
    float amax[NIT];
#pragma unroll
    for (int it = 0; it < NIT; ++it) {
        amax[it] = 0.0f;
#pragma unroll
        for (int i = 0; i < 16; ++i) amax[it] = fmaxf(amax[it], fabsf(v[it][i]));
        if constexpr (!STORED) store_chunks(w32 + (size_t)n * K, real ? K : 0, stage + wave * 256, c0 - l + it * 64, l, lane, v[it]);
    }
    if constexpr (BITS == 8) {
        float mx = amax[0];
#pragma unroll
        for (int it = 1; it < NIT; ++it) mx = fmaxf(mx, amax[it]);
        mx = __uint_as_float(max_over_lanes<true>(__float_as_uint(mx)));
        if (lane == 0) red[wave] = mx;
        __syncthreads();
        mx = __uint_as_float(max_over_lanes<false>(lane < nwaves ? __float_as_uint(red[lane]) : 0u));
        float s = mx / 127.0f;
        if (s == 0.0f) s = 1.0f;
        if (real && scales && threadIdx.x == 0) static_cast<float *>(scales)[n] = s;
#pragma unroll
        for (int it = 0; it < NIT; ++it) {
            const int c = c0 + it * 64;
            unsigned q[4];
            weight_codes<127>(v[it], s, q);
            const uint4 o = make_uint4(q[0], q[1], q[2], q[3]);
            if (c < K / 16) {
                if (real && canon) *reinterpret_cast<uint4 *>(canon + (size_t)n * K + (size_t)c * 16) = o;
                if (kl) *reinterpret_cast<uint4 *>(kl + tile_offset_i8(n, c * 16, K)) = o;
            }
        }
    } else {
#pragma unroll
        for (int it = 0; it < NIT; ++it) {
            const int c = c0 + it * 64;
            float mx = amax[it];   // a group of 128 is the eight chunks of lanes 8i .. 8i + 7
            mx = __uint_as_float(max_pair<4>(max_pair<2>(max_pair<1>(__float_as_uint(mx)))));
            __half s16 = __float2half_rn(mx / 7.0f);
            if (__half2float(s16) == 0.0f) s16 = __float2half_rn(1.0f);
            const float s = __half2float(s16);
            unsigned q[4];
            weight_codes<7>(v[it], s, q);
            if (c >= K / 16) continue;
            const int g = c / 8;
            if (c % 8 == 0) {
                if (real && scales) static_cast<__half *>(scales)[(size_t)n * G + g] = s16;
                if (kl) {
                    kl_scales[(size_t)g * Npad + n] = s16;
                    kl_scales_dec[((size_t)(n / 16) * G + g) * 16 + n % 16] = s16;
                }
            }
            if (real && canon) {   // even k in the low nibbles, odd k in the high ones
                unsigned even, odd, lo, hi;
                even = __builtin_amdgcn_perm(q[1], q[0], 0x06040200u), odd = __builtin_amdgcn_perm(q[1], q[0], 0x07050301u);
                lo = (even & 0x0f0f0f0fu) | ((odd << 4) & 0xf0f0f0f0u);
                even = __builtin_amdgcn_perm(q[3], q[2], 0x06040200u), odd = __builtin_amdgcn_perm(q[3], q[2], 0x07050301u);
                hi = (even & 0x0f0f0f0fu) | ((odd << 4) & 0xf0f0f0f0u);
                *reinterpret_cast<uint2 *>(canon + (size_t)n * (K / 2) + (size_t)c * 8) = make_uint2(lo, hi);
            }
            if (kl) {   // the first four k of a word in its low nibbles, the other four in the high ones (w4_nibble_pos)
                const unsigned w0 = (q[0] & 0x0f0f0f0fu) | ((q[1] << 4) & 0xf0f0f0f0u), w1 = (q[2] & 0x0f0f0f0fu) | ((q[3] << 4) & 0xf0f0f0f0u);
                *reinterpret_cast<uint2 *>(kl + tile_offset_w4_word(n, c * 16, K)) = make_uint2(w0, w1);
            }
        }
    }
}

// Calibration: running max|X_j| per input channel (non-negative floats order like their bit patterns).  A workgroup takes
// 256 channels x 64 tokens: 8 channels (16 bytes) per lane, 8 tokens side by side, one atomic per channel at the end.
__global__ __launch_bounds__(256) void channel_absmax_kernel(const __half *__restrict__ x, int64_t ldx, int M, int K,
                                                             unsigned *__restrict__ xmax_bits)
{
    __shared__ float red[8][256 + 8];
    const int col = threadIdx.x & 31, r = threadIdx.x >> 5;
    const int k0 = blockIdx.x * 256 + col * 8, m0 = blockIdx.y * 64;
    float mx[8] = {0, 0, 0, 0, 0, 0, 0, 0};
    if (k0 < K) {
#pragma unroll
        for (int i = 0; i < 8; ++i) {
            const int m = m0 + r + 8 * i;
            if (m < M) {
                const uint4 h = *reinterpret_cast<const uint4 *>(x + (size_t)m * ldx + k0);
                const unsigned w[4] = {h.x, h.y, h.z, h.w};
#pragma unroll
                for (int e = 0; e < 4; ++e) {
                    mx[2 * e] = fmaxf(mx[2 * e], fabsf(half_bits_to_float(w[e] & 0xffffu)));
                    mx[2 * e + 1] = fmaxf(mx[2 * e + 1], fabsf(half_bits_to_float(w[e] >> 16)));
                }
            }
        }
    }
#pragma unroll
    for (int e = 0; e < 8; ++e) red[r][col * 8 + e] = mx[e];
    __syncthreads();
    const int k = blockIdx.x * 256 + threadIdx.x;
    if (k >= K) return;
    float a = 0.0f;
#pragma unroll
    for (int i = 0; i < 8; ++i) a = fmaxf(a, red[i][threadIdx.x]);
    atomicMax(xmax_bits + k, __float_as_uint(a));
}

// s_j = xmax_j^alpha / wmax_j^(1-alpha), 1 where either maximum is 0; inv_j = 1 / s_j (IEEE fp32 division)
__device__ inline void smooth_scale(float xm, float wmax, float alpha, float *s, float *inv_s)
{
    float sj = 1.0f;
    if (xm > 0.0f && wmax > 0.0f) sj = (float)(pow((double)xm, (double)alpha) / pow((double)wmax, 1.0 - (double)alpha));
    *s = sj;
    *inv_s = 1.0f / sj;
}

// A workgroup finds the column maxima of 64 channels over N rows (8 channels per lane, 64 rows side by side, 8 loads of each
// lane in flight: a strip of 128 bytes per row streams at the rate one CU can pull, about 30 GB/s) -- one lane per channel
// walking down the rows took 1570 us for 4096 x 11008.  PART: of `rows` rows per blockIdx.y, into the larger of what inv_s holds (as
// bits; zeroed before) and of what the other workgroups of the strip find; smooth_scales_finish_kernel does the rest.
template <bool PART>
__global__ __launch_bounds__(512) void smooth_scales_kernel(const float *__restrict__ xmax, const __half *__restrict__ w, int N, int K, int rows,
                                                            float alpha, float *__restrict__ s, float *__restrict__ inv_s)
{
    __shared__ float red[8][64];
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6, col = lane & 7;
    const __half *base = w + (size_t)blockIdx.x * 64 + col * 8;
    float mx[8] = {0, 0, 0, 0, 0, 0, 0, 0};
    const int end = PART ? min(N, (int)(blockIdx.y + 1) * rows) : N;
    for (int n0 = PART ? blockIdx.y * rows : 0; n0 < end; n0 += 512) {
        uint4 h[8];
#pragma unroll
        for (int i = 0; i < 8; ++i) {   // (a row behind the last one: the last one again)
            const int n = n0 + i * 64 + wave * 8 + (lane >> 3);
            h[i] = *reinterpret_cast<const uint4 *>(base + (size_t)(n < end ? n : end - 1) * K);
        }
#pragma unroll
        for (int i = 0; i < 8; ++i) {
            const unsigned q[4] = {h[i].x, h[i].y, h[i].z, h[i].w};
#pragma unroll
            for (int e = 0; e < 4; ++e) {
                mx[2 * e] = fmaxf(mx[2 * e], fabsf(half_bits_to_float(q[e] & 0xffffu)));
                mx[2 * e + 1] = fmaxf(mx[2 * e + 1], fabsf(half_bits_to_float(q[e] >> 16)));
            }
        }
    }
#pragma unroll
    for (int e = 0; e < 8; ++e) {
#pragma unroll
        for (int off = 8; off < 64; off <<= 1) mx[e] = fmaxf(mx[e], __shfl_xor(mx[e], off, 64));
        if (lane < 8) red[wave][col * 8 + e] = mx[e];
    }
    __syncthreads();
    if (threadIdx.x >= 64) return;
    float wmax = 0.0f;
#pragma unroll
    for (int i = 0; i < 8; ++i) wmax = fmaxf(wmax, red[i][threadIdx.x]);
    const int k = blockIdx.x * 64 + threadIdx.x;
    if constexpr (PART) atomicMax(reinterpret_cast<unsigned *>(inv_s) + k, __float_as_uint(wmax));   // (non-negative: ordered like their bits)
    else smooth_scale(xmax[k], wmax, alpha, s + k, inv_s + k);
}

__global__ __launch_bounds__(256) void smooth_scales_clear_kernel(int K, float *__restrict__ inv_s)
{
    const int k = blockIdx.x * 256 + threadIdx.x;
    if (k < K) inv_s[k] = 0.0f;
}

__global__ __launch_bounds__(256) void smooth_scales_finish_kernel(const float *__restrict__ xmax, int K, float alpha, float *__restrict__ s,
                                                                   float *__restrict__ inv_s)
{
    const int k = blockIdx.x * 256 + threadIdx.x;
    if (k < K) smooth_scale(xmax[k], inv_s[k], alpha, s + k, inv_s + k);
}

float block_norm(int hblock) { return (float)(1.0 / std::sqrt((double)hblock)); }

}  // namespace

int hadamard_block_of(int K)
{
    const int b = K & -K;
    return b < 4096 ? b : 4096;
}

// calls f(integral constant LB) for the block's exponent (0: no transform)
template <typename F>
static int by_block(int hblock, F f)
{
    int lb = 0;
    while (hblock > 1 && (1 << lb) < hblock) ++lb;
    switch (lb) {
    case 0: return f(std::integral_constant<int, 0>{});
    case 4: return f(std::integral_constant<int, 4>{});
    case 5: return f(std::integral_constant<int, 5>{});
    case 6: return f(std::integral_constant<int, 6>{});
    case 7: return f(std::integral_constant<int, 7>{});
    case 8: return f(std::integral_constant<int, 8>{});
    case 9: return f(std::integral_constant<int, 9>{});
    case 10: return f(std::integral_constant<int, 10>{});
    case 11: return f(std::integral_constant<int, 11>{});
    case 12: return f(std::integral_constant<int, 12>{});
    default: return fail(QL_ERR_UNSUPPORTED, "hadamard_block=%d", hblock);
    }
}

int launch_act_quant_transform(const __half *x, int64_t ldx, int M, int K, const float *inv_smooth, int hblock,
                               int8_t *xq_rm, int8_t *xq_kl, float *sx, hipStream_t st)
{
    if (M == 0) return QL_OK;
    const float norm = block_norm(hblock > 1 ? hblock : 1);
    return by_block(hblock, [&](auto lb) {
        constexpr int LB = decltype(lb)::value;
        const int waves = ceil_div(K / 16, 64);   // (a block of W > 1 wavefronts divides K: every block is complete)
        const unsigned lds = LB > 10 ? waves * 4096u : 0u;
        hipLaunchKernelGGL((act_quant_hadamard_kernel<LB>), dim3(workgroups_for(M, 8)), dim3(waves * 64), lds, st, x, ldx, M, K, inv_smooth,
                           norm, xq_rm, xq_kl, sx);
        return check_hip(hipGetLastError(), "act_quant_hadamard launch");
    });
}

int launch_weight_transform_quant(const __half *w, int N, int K, int bits, int group, const float *smooth, int hblock, float *w32,
                                  void *canon, void *scales, void *kl, hipStream_t st)
{
    const float norm = block_norm(hblock > 1 ? hblock : 1);
    const int Npad = round_up(N, TILE_ROWS), rows = kl ? Npad : N;   // padding rows exist in the kernel layout only
    uint8_t *blob = static_cast<uint8_t *>(kl);
    __half *kls = (kl && bits == 4) ? reinterpret_cast<__half *>(blob + w4_scales_offset(N, K)) : nullptr;
    __half *klsd = (kl && bits == 4) ? reinterpret_cast<__half *>(blob + w4_scales_dec_offset(N, K, group)) : nullptr;
    return by_block(hblock, [&](auto lb) {
        constexpr int LB = decltype(lb)::value;
        const dim3 grid(workgroups_for(rows, 32)), block(ceil_div(K / 16, 64 * hadamard_chunks(LB)) * 64);
        if (bits == 8)
            hipLaunchKernelGGL((weight_transform_quant_kernel<LB, 8>), grid, block, block.x * 64, st, w, N, rows, K, smooth, norm, w32,
                               static_cast<uint8_t *>(canon), scales, blob, kls, klsd);
        else
            hipLaunchKernelGGL((weight_transform_quant_kernel<LB, 4>), grid, block, block.x * 64, st, w, N, rows, K, smooth, norm, w32,
                               static_cast<uint8_t *>(canon), scales, blob, kls, klsd);
        return check_hip(hipGetLastError(), "weight_transform_quant launch");
    });
}

int launch_weight_transform_then_quant(const __half *w, int N, int K, int bits, int group, const float *smooth, int hblock, float *w32,
                                       void *canon, void *scales, void *kl, hipStream_t st)
{
    QL_TRY(launch_weight_transform_quant(w, N, K, 8, 0, smooth, hblock, w32, nullptr, nullptr, nullptr, st));   // fills w32
    const int Npad = round_up(N, TILE_ROWS), rows = kl ? Npad : N;
    uint8_t *blob = static_cast<uint8_t *>(kl);
    __half *kls = (kl && bits == 4) ? reinterpret_cast<__half *>(blob + w4_scales_offset(N, K)) : nullptr;
    __half *klsd = (kl && bits == 4) ? reinterpret_cast<__half *>(blob + w4_scales_dec_offset(N, K, group)) : nullptr;
    const dim3 grid(workgroups_for(rows, 32)), block(ceil_div(K / 16, 64 * hadamard_chunks(0)) * 64);
    auto kern = bits == 8 ? weight_transform_quant_kernel<0, 8, true> : weight_transform_quant_kernel<0, 4, true>;
    hipLaunchKernelGGL(kern, grid, block, 0, st, nullptr, N, rows, K, nullptr, 1.0f, w32, static_cast<uint8_t *>(canon), scales, blob,
                       kls, klsd);
    return check_hip(hipGetLastError(), "weight_transform_quant launch (stored)");
}

int launch_channel_absmax(const __half *x, int64_t ldx, int M, int K, float *xmax, hipStream_t st)
{
    if (M == 0) return QL_OK;
    hipLaunchKernelGGL(channel_absmax_kernel, dim3(ceil_div(K, 256), ceil_div(M, 64)), dim3(256), 0, st, x, ldx, M, K,
                       reinterpret_cast<unsigned *>(xmax));
    return check_hip(hipGetLastError(), "channel_absmax launch");
}

int launch_smooth_scales(const float *xmax, const __half *w, int N, int K, float alpha, float *s, float *inv_s,
                         hipStream_t st)
{
    // One workgroup per 64 channels pulls its N x 128 bytes in 2 + N / 235 us, however few of them there are.  Several per strip and two
    // small launches around them take 7 us + the bytes at 4 TB/s: taken where that is a tenth less, unless a result lies over an
    // input that a later launch reads.  N x K, us, one against several, weights from HBM: 4608 x 1536 21.2 / 10.4, 6144 x 2048 26.7 / 13.0,
    // 12288 x 4096 52.0 / 30.1, 4096 x 4096 20.4 / 15.8, 2048 x 2048 11.4 / 9.3; the other way 1536 x 6144 10.9 / 12.5, 3000 x 8192 16.6 /
    // 18.0.  Not below 2048 rows: there one workgroup takes anything from 5.8 to 10.7 us by the row's length (fewest where it is no multiple
    // of 1 KB) and several 8.0 to 9.9 (1484 x 512 6.3 / 8.1, 2007 x 512 7.4 / 8.2, 1992 x 1920 9.4 / 9.9; 1902 x 1024 10.7 / 9.7).
    // Weights that are still in a cache have one the faster up to 3800 rows: 2048 x 2048 6.0 / 7.5, 3072 x 1024 7.0 / 7.7, 4096 x 1024 8.0 / 7.8.
    const int strips = K / 64, parts = std::min(ceil_div(384, strips), N / 512);
    const bool several = N >= 2048 && parts > 1 && 7.0 + 0.5e-6 * N * K < 0.9 * (2.0 + N / 235.0);
    auto over_inputs = [&](const float *p) {
        return bytes_overlap(p, (size_t)K * 4, xmax, (size_t)K * 4) || bytes_overlap(p, (size_t)K * 4, w, (size_t)N * K * 2);
    };
    if (several && !over_inputs(s) && !over_inputs(inv_s)) {
        const int rows = round_up(ceil_div(N, parts), 64);
        hipLaunchKernelGGL(smooth_scales_clear_kernel, dim3(ceil_div(K, 256)), dim3(256), 0, st, K, inv_s);
        hipLaunchKernelGGL(smooth_scales_kernel<true>, dim3(strips, ceil_div(N, rows)), dim3(512), 0, st, xmax, w, N, K, rows, alpha, s, inv_s);
        hipLaunchKernelGGL(smooth_scales_finish_kernel, dim3(ceil_div(K, 256)), dim3(256), 0, st, xmax, K, alpha, s, inv_s);
        return check_hip(hipGetLastError(), "smooth_scales launch");
    }
    hipLaunchKernelGGL(smooth_scales_kernel<false>, dim3(strips), dim3(512), 0, st, xmax, w, N, K, N, alpha, s, inv_s);
    return check_hip(hipGetLastError(), "smooth_scales launch");
}

}  // namespace ql
