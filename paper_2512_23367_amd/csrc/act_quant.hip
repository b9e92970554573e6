// Per-token dynamic int8 activation quantization (paper Eq. 1-2 with n = 8; one scale per token
// over its whole feature dimension, Preliminary section) for gfx950.
//
// The rows are read once and stay in registers between their maximum and their codes, which leave row-major and/or in
// the GEMM's tile order.
//
// Arithmetic (every step a single correctly rounded fp32 operation):
//   amax = max_k |x|            sx = amax / 127          inv = 127 / amax
//   code = clamp(rne(x * inv), -127, 127)                (all-zero token: sx = 1, codes 0)
#include "common.h"
#include "quant_math.h"

namespace ql {
namespace {

typedef unsigned v4u __attribute__((ext_vector_type(4)));

// MODE 0: the quantizer alone.
// MODE 1: the SmoothQuant variant (paper Eq. 3): every element is first multiplied by inv_smooth[k] = 1 / s_k (one
// fp32 multiply), the row maximum is taken on those fp32 products.
// MODE 2: RMSNorm in front of the quantizer (textbook definition; the normalisation a decoder layer applies to the
// input of its QKV and gate/up projections):  h_k = x_k / sqrt(mean(x^2) + eps) * gamma_k, then Eq. 1-2 on h.
//   ss = fp32(sum x^2): the squares are exact, they are added in fp64 (per lane in k order, a butterfly
//        across the lanes, the wavefronts in order) and rounded to fp32 once -- the fp64 sum is within ~1e-13 of the
//        exact one, so this is the correctly rounded exact sum except within that distance of a rounding boundary;
//   mean = ss / K,  r = 1 / sqrt(mean + eps),  h = (x * r) * gamma: one correctly rounded fp32 operation each.
// MODE 3: SwiGLU in front of the quantizer: x is the fused gate+up projection output [M, 2K] (gate = columns 0..K-1,
// up = columns K..2K-1), the quantized value is h_k = silu(gate_k) * up_k in fp32 (swiglu_f32: a fixed sequence of
// single fp32 operations).
//
// What bounds it: HBM (3 B per element, SwiGLU 5) for many tokens, one memory round trip for few.  One workgroup per
// token, NC chunks of 16 consecutive elements per lane (1 up to K = 16384: K / 1024 wavefronts, rounded up, share the token):
// few registers, so a CU holds many tokens whose loads and arithmetic cover each other.  Range-checked buffer loads: a lane
// behind the row's end reads zeros, without a branch.  With the row spread over at most 8 wavefronts of several chunks, loaded
// under conditions, SwiGLU of 4096 x 11008 took 84 us (2.7 TB/s) against 64 us (3.5 TB/s), of 32 x 11008 7.6 against 5.5 us.
// (Workgroups that stay and keep several tokens in flight in an LDS ring were slower: 69 us.)
// Longer rows (the down projections of 70B-class layers: 28672) keep 2, 4 or 8 chunks per lane in as many wavefronts as they
// need.  The fp32 values stay in registers between maximum and codes (SwiGLU: its ~45 operations per element are done once);
// with 8 chunks there is room for the fp16 values only, and RMSNorm forms its products again.  K = 28672, plain / RMSNorm /
// SwiGLU, against rows read twice (three times) by 8 wavefronts: 32 tokens 4.6 / 6.7 / 11.3 us, before 5.3 / 7.6 / 15.3;
// 4096 tokens 75 / 105 / 145, before 161 / 181 / 229.
constexpr int MAX_WAVES = 16;
constexpr int ROW_CHUNKS = MAX_WAVES * 64;                      // chunks of a row held one per lane
constexpr int ROW4_MAX_K = 4 * ROW_CHUNKS * CHUNK;              // 65536: longer SmoothQuant and SwiGLU rows are read twice

__device__ inline void widen(const Half16 &h, float (&f)[16])
{
    const unsigned w[8] = {h.lo.x, h.lo.y, h.lo.z, h.lo.w, h.hi.x, h.hi.y, h.hi.z, h.hi.w};
#pragma unroll
    for (int i = 0; i < 8; ++i) {
        f[2 * i] = half_bits_to_float(w[i] & 0xffffu);
        f[2 * i + 1] = half_bits_to_float(w[i] >> 16);
    }
}

__device__ inline __amdgpu_buffer_rsrc_t buffer_of(const void *p, size_t bytes)
{
    return __builtin_amdgcn_make_buffer_rsrc(const_cast<void *>(p), 0, (int)(unsigned)bytes, 0x00020000);
}

constexpr unsigned ABSENT = 0xFFFFFFE0u;   // behind any buffer: such loads read zeros, such stores are dropped

__device__ inline Half16 chunk_of(v4u lo, v4u hi) { return Half16{uint4{lo[0], lo[1], lo[2], lo[3]}, uint4{hi[0], hi[1], hi[2], hi[3]}}; }

__device__ inline Half16 load_chunk(__amdgpu_buffer_rsrc_t rs, unsigned off)
{
    const v4u lo = __builtin_bit_cast(v4u, __builtin_amdgcn_raw_buffer_load_b128(rs, off, 0, 0));
    const v4u hi = __builtin_bit_cast(v4u, __builtin_amdgcn_raw_buffer_load_b128(rs, off + 16u, 0, 0));
    return chunk_of(lo, hi);
}

// Workgroup ids go to the 8 XCDs in turn.  Every XCD takes one contiguous range of tokens (whole groups of 8: the tokens that
// share 128-byte lines of the tile order), so that what it writes at a time is a window of a few dozen tokens that its L2
// holds until the lines are whole.  M: nothing to do.
__device__ inline int token_of_workgroup(int M)
{
    const int groups = (M + 7) / 8, xcd = blockIdx.x % 8, in_xcd = blockIdx.x / 8;
    if (in_xcd >= 8 * (groups / 8 + (xcd < groups % 8 ? 1 : 0))) return M;
    return 8 * (xcd * (groups / 8) + (xcd < groups % 8 ? xcd : groups % 8)) + in_xcd;
}

template <int MODE, int NC>
__global__ __launch_bounds__(MAX_WAVES * 64) void act_quant_kernel(const __half *__restrict__ x, int64_t ldx, int M, int K,
                                                                    const float *__restrict__ inv_smooth,
                                                                    const __half *__restrict__ gamma, float eps,
                                                                    int8_t *__restrict__ xq_rm, int8_t *__restrict__ xq_kl,
                                                                    float *__restrict__ sx)
{
    static_assert(NC <= 4 || MODE == 0 || MODE == 2, "SmoothQuant, SwiGLU: the fp32 values of a row stay in registers");
    constexpr bool KEEP = MODE != 0 && NC <= 4;      // the values to quantize stay in registers as fp32
    __shared__ unsigned red[MAX_WAVES];
    __shared__ double red_ss[MODE == 2 ? MAX_WAVES : 1];
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6, nwaves = blockDim.x >> 6;
    const int m = token_of_workgroup(M);
    // no branch in front of the loads (those of an absent token read zeros); with RMSNorm it measured no gain
    const bool absent = (MODE == 0 || MODE == 3) && m >= M;
    if (MODE != 0 && MODE != 3 && m >= M) return;

    // this lane's chunks of the row: threadIdx.x, threadIdx.x + blockDim.x, ...
    auto chunk = [&](int it) { return (int)threadIdx.x + it * (int)blockDim.x; };
    auto have = [&](int it) { return chunk(it) < K / CHUNK; };
    auto at = [&](int it, unsigned bytes) { return have(it) ? (unsigned)chunk(it) * bytes : ABSENT; };
    const __amdgpu_buffer_rsrc_t rs = buffer_of(x + (absent ? (size_t)0 : (size_t)m * ldx), absent ? 0u : (MODE == 3 ? 4u : 2u) * (unsigned)K);
    const __amdgpu_buffer_rsrc_t rv = MODE == 1 ? buffer_of(inv_smooth, (size_t)K * sizeof(float))
                                                : buffer_of(gamma, MODE == 2 ? (size_t)K * sizeof(__half) : 0);
    Half16 v[NC];
#pragma unroll
    for (int it = 0; it < NC; ++it) v[it] = load_chunk(rs, at(it, 32u));
    Half16 u[MODE == 3 ? NC : 1], gm[MODE == 2 && KEEP ? NC : 1];
    if constexpr (MODE == 3) {
#pragma unroll
        for (int it = 0; it < NC; ++it) u[it] = load_chunk(rs, have(it) ? (unsigned)chunk(it) * 32u + 2u * (unsigned)K : ABSENT);
    }
    if constexpr (MODE == 2 && KEEP) {
#pragma unroll
        for (int it = 0; it < NC; ++it) gm[it] = load_chunk(rv, at(it, 32u));
    }
    // RMSNorm, 8 chunks: the widened values of one pass must not stay for the next (the registers do not hold them)
    auto fp16_only = [&]() {
        if constexpr (MODE == 2 && !KEEP) {
#pragma unroll
            for (int it = 0; it < NC; ++it)
                asm volatile("" : "+v"(v[it].lo.x), "+v"(v[it].lo.y), "+v"(v[it].lo.z), "+v"(v[it].lo.w), "+v"(v[it].hi.x), "+v"(v[it].hi.y),
                             "+v"(v[it].hi.z), "+v"(v[it].hi.w)::"memory");
        }
    };
    float rnorm = 0.0f;
    if constexpr (MODE == 2) {
        // sum of squares first (the maximum needs the normalised values); squares of fp16 values are exact, absent chunks zeros
        double ss = 0.0;
#pragma unroll
        for (int it = 0; it < NC; ++it) {
            float f[16];
            widen(v[it], f);
#pragma unroll
            for (int e = 0; e < 16; ++e) ss = __builtin_fma((double)f[e], (double)f[e], ss);
        }
        ss = sum_pair<1>(sum_pair<2>(sum_pair<4>(sum_pair<8>(sum_pair<16>(sum_pair<32>(ss))))));
        if (lane == 0) red_ss[wave] = ss;
        __syncthreads();
        double tot = 0.0;
        for (int w = 0; w < nwaves; ++w) tot += red_ss[w];
        const float mean = (float)tot / (float)K;
        rnorm = 1.0f / sqrtf(mean + eps);
        fp16_only();
    }
    // the values to quantize: fp16 bits as loaded, or fp32 after the mode's arithmetic (absent chunks are zeros, which
    // change no maximum)
    auto values = [&](int it, float (&f)[16]) {
        widen(v[it], f);
        if constexpr (MODE == 1) {
            v4u sm[4];
#pragma unroll
            for (int q = 0; q < 4; ++q)
                sm[q] = __builtin_bit_cast(v4u, __builtin_amdgcn_raw_buffer_load_b128(rv, have(it) ? (unsigned)chunk(it) * 64u + q * 16u : ABSENT, 0, 0));
#pragma unroll
            for (int e = 0; e < 16; ++e) f[e] *= __uint_as_float(sm[e / 4][e % 4]);
        }
        if constexpr (MODE == 2) {
            float g[16];
            widen(KEEP ? gm[KEEP ? it : 0] : load_chunk(rv, at(it, 32u)), g);
#pragma unroll
            for (int e = 0; e < 16; ++e) f[e] = __builtin_fmaf(__builtin_fmaf(f[e], rnorm, 0.0f), g[e], 0.0f);   // widened in the multiply
        }
        if constexpr (MODE == 3) {
            float up[16];
            widen(u[it], up);
#pragma unroll
            for (int e = 0; e < 16; ++e) f[e] = swiglu_f32(f[e], up[e]);
        }
    };
    float kept[KEEP ? NC : 1][16];
    unsigned mx = 0;
    if constexpr (MODE == 0) {
#pragma unroll
        for (int it = 0; it < NC; ++it) mx = abs_max_bits(v[it], mx);
    } else {
        float mf = 0.0f;
#pragma unroll
        for (int it = 0; it < NC; ++it) {
            float (&f)[16] = kept[KEEP ? it : 0];
            values(it, f);
#pragma unroll
            for (int e = 0; e < 16; ++e) mf = __builtin_elementwise_maximum(mf, fabsf(f[e]));   // passes a NaN on
            if (!KEEP) __builtin_amdgcn_sched_barrier(0);   // (nor do the vectors of all chunks at once)
        }
        mx = __float_as_uint(mf);   // non-negative floats order like their bit patterns
    }
    mx = max_over_lanes<true>(mx);
    if (lane == 0) red[wave] = mx;
    __syncthreads();
    static_assert(MAX_WAVES == 16, "one row of lanes takes the wavefronts' maxima");
    mx = max_over_lanes<false>(lane < nwaves ? red[lane] : 0u);
    const bool finite = MODE == 0 && finite_tokens(mx);
    float scale, inv;
    if (MODE != 0) token_scales_f32(__uint_as_float(mx), scale, inv);
    else token_scales(mx, scale, inv);
    if (absent) return;
    if (threadIdx.x == 0) sx[m] = scale;
    fp16_only();
#pragma unroll
    for (int it = 0; it < NC; ++it) {
        const int c = chunk(it);
        if (!have(it)) break;                        // (the chunks of a lane ascend)
        uint4 q;
        if constexpr (MODE == 0) {
            q = quant_chunk(v[it], inv, finite);
        } else if constexpr (KEEP) {
            q = quant_chunk_f32(kept[it], inv);
        } else {
            float f[16];
            values(it, f);
            q = quant_chunk_f32(f, inv);
            __builtin_amdgcn_sched_barrier(0);
        }
        if (xq_rm) *reinterpret_cast<uint4 *>(xq_rm + (size_t)m * K + (size_t)c * CHUNK) = q;
        if (xq_kl) *reinterpret_cast<uint4 *>(xq_kl + tile_offset_i8(m, c * CHUNK, K)) = q;
    }
}

// Many tokens, plain and SmoothQuant (MODE 0, 1): one workgroup per 8 tokens.  A wavefront covers 8 tokens x 8 chunks per
// step (lane = token % 8 + 8 * chunk), so that in the tile order the 8 lanes of one chunk write one whole 128-byte line
// (8 token slots x 16 bytes) and in the row-major copy each token gets 128 contiguous bytes per step; up to 8 wavefronts
// split K.  Whole lines are worth more than small workgroups once the writes come from HBM's side: 4096 x 4096
// 10.9 us against 12.9 with a workgroup per token, 16384 x 1536 16.2 against 20.0; at 3001 x 4096 (10.2 / 10.1),
// 1024 x 4096 (6.5 / 5.4) and below it is the other way round.
// NIT: steps per wavefront kept in registers (up to K = 12288).
// RPB: 8 tokens per workgroup, or 1 (SmoothQuant rows of 65536 < K <= 98304: the fp16 values fit 8 wavefronts of 12 chunks).
constexpr int ROWS8_WAVES = 8, ROWS8_MIN_M = 3072, ROWS8_MAX_K = 12288, ROW12_MAX_K = 12 * 64 * ROWS8_WAVES * CHUNK;

template <int NIT, int MODE, int RPB = 8>
__global__ __launch_bounds__(ROWS8_WAVES * 64) void act_quant_rows8_kernel(const __half *__restrict__ x, int64_t ldx, int M, int K,
                                                                            int per_wave, const float *__restrict__ inv_smooth,
                                                                            int8_t *__restrict__ xq_rm, int8_t *__restrict__ xq_kl,
                                                                            float *__restrict__ sx)
{
    __shared__ unsigned red[RPB][ROWS8_WAVES];
    constexpr int CPS = 64 / RPB;                     // chunks per wavefront per step
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6, nwaves = blockDim.x >> 6;
    const int r = lane % RPB, cl = lane / RPB;
    const int m = blockIdx.x * RPB + r;
    const bool valid = m < M;
    const int nchunks = K / CHUNK;
    const int s0 = wave * per_wave;
    // (the product is formed again for the codes: cheaper than keeping fp32 copies in registers)
    auto smoothed = [&](const Half16 &h, int c, float (&f)[16]) {
        widen(h, f);
#pragma unroll
        for (int i = 0; i < 16; i += 4) {
            const float4 s4 = *reinterpret_cast<const float4 *>(inv_smooth + (size_t)c * CHUNK + i);
            f[i] *= s4.x, f[i + 1] *= s4.y, f[i + 2] *= s4.z, f[i + 3] *= s4.w;
        }
    };
    Half16 v[NIT];
    unsigned mx = 0;
    if constexpr (MODE == 0) {
        // All NIT chunks of a lane are requested at once, through range-checked buffer loads with no branch around them (a
        // chunk beyond the row, the wavefront's share or the last token reads zeros): with a conditional load per step the
        // compiler waits for each step's data before it issues the next step's loads.  The buffer is the workgroup's
        // 8 rows, so the 32-bit offsets hold for any M.
        const int rows = M - (int)blockIdx.x * RPB < RPB ? M - (int)blockIdx.x * RPB : RPB;
        const __amdgpu_buffer_rsrc_t rs = buffer_of(x + (size_t)blockIdx.x * RPB * ldx, ((size_t)(rows - 1) * ldx + K) * sizeof(__half));
#pragma unroll
        for (int i = 0; i < NIT; ++i) {
            const int c = (s0 + i) * CPS + cl;
            const bool ok = i < per_wave && c < nchunks && valid;
            v[i] = load_chunk(rs, ok ? (unsigned)r * (unsigned)ldx * 2u + (unsigned)c * 32u : ABSENT);
        }
#pragma unroll
        for (int i = 0; i < NIT; ++i) mx = abs_max_bits(v[i], mx);
    } else {
        // (a step's scale vector is requested together with its chunk; with the chunks requested ahead of all the scale
        // vectors the kernel measured 18 % slower at K = 11008)
        const Half16 *row = reinterpret_cast<const Half16 *>(x + (size_t)(valid ? m : 0) * ldx);
#pragma unroll
        for (int i = 0; i < NIT; ++i) {
            const int c = (s0 + i) * CPS + cl;
            if (i < per_wave && c < nchunks && valid) {
                v[i] = row[c];
                float f[16];
                smoothed(v[i], c, f);
#pragma unroll
                for (int e = 0; e < 16; ++e) mx = max(mx, __float_as_uint(fabsf(f[e])));
            }
        }
    }
#pragma unroll
    for (int off = 32; off >= RPB; off >>= 1) mx = max(mx, (unsigned)__shfl_xor((int)mx, off, 64));
    if (cl == 0) red[r][wave] = mx;
    __syncthreads();
    mx = 0;
    for (int w = 0; w < nwaves; ++w) mx = max(mx, red[r][w]);
    const bool finite = MODE == 0 && finite_tokens(mx);
    float scale, inv;
    if (MODE != 0) token_scales_f32(__uint_as_float(mx), scale, inv);
    else token_scales(mx, scale, inv);
    if (wave == 0 && cl == 0 && valid) sx[m] = scale;
#pragma unroll
    for (int i = 0; i < NIT; ++i) {
        const int c = (s0 + i) * CPS + cl;
        if (i < per_wave && c < nchunks && valid) {
            uint4 q;
            if constexpr (MODE == 0) {
                q = quant_chunk(v[i], inv, finite);
            } else {
                float f[16];
                smoothed(v[i], c, f);
                q = quant_chunk_f32(f, inv);
            }
            if (xq_rm) *reinterpret_cast<uint4 *>(xq_rm + (size_t)m * K + (size_t)c * CHUNK) = q;
            if (xq_kl) *reinterpret_cast<uint4 *>(xq_kl + tile_offset_i8(m, c * CHUNK, K)) = q;
        }
    }
}

// SwiGLU rows too long for registers (K > 65536): the row is read twice and the arithmetic done twice.
constexpr int LONG_WAVES = 8;

__global__ __launch_bounds__(LONG_WAVES * 64) void act_quant_swiglu_long_kernel(const __half *__restrict__ x, int64_t ldx, int M, int K,
                                                                                int8_t *__restrict__ xq_rm, int8_t *__restrict__ xq_kl,
                                                                                float *__restrict__ sx)
{
    __shared__ unsigned red[LONG_WAVES];
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    // (up to 64 tokens: no XCD holds more than 8 of them either way, and 8 XCDs read faster than one: 8 x 98304 45 us against 49)
    const int m = M <= 64 ? (int)blockIdx.x : token_of_workgroup(M), nchunks = K / CHUNK;
    if (m >= M) return;
    const Half16 *row = reinterpret_cast<const Half16 *>(x + (size_t)m * ldx);
    const Half16 *row_up = reinterpret_cast<const Half16 *>(x + (size_t)m * ldx + K);
    auto values = [&](int c, float (&f)[16]) {
        float g[16];
        widen(row[c], f);
        widen(row_up[c], g);
#pragma unroll
        for (int e = 0; e < 16; ++e) f[e] = swiglu_f32(f[e], g[e]);
    };
    unsigned mx = 0;
    for (int c = threadIdx.x; c < nchunks; c += LONG_WAVES * 64) {
        float f[16];
        values(c, f);
#pragma unroll
        for (int e = 0; e < 16; ++e) mx = max(mx, __float_as_uint(fabsf(f[e])));
    }
#pragma unroll
    for (int off = 32; off > 0; off >>= 1) mx = max(mx, (unsigned)__shfl_xor((int)mx, off, 64));
    if (lane == 0) red[wave] = mx;
    __syncthreads();
    mx = 0;
    for (int w = 0; w < LONG_WAVES; ++w) mx = max(mx, red[w]);
    float scale, inv;
    token_scales_f32(__uint_as_float(mx), scale, inv);
    if (threadIdx.x == 0) sx[m] = scale;
    for (int c = threadIdx.x; c < nchunks; c += LONG_WAVES * 64) {
        float f[16];
        values(c, f);
        const uint4 q = quant_chunk_f32(f, inv);
        if (xq_rm) *reinterpret_cast<uint4 *>(xq_rm + (size_t)m * K + (size_t)c * CHUNK) = q;
        if (xq_kl) *reinterpret_cast<uint4 *>(xq_kl + tile_offset_i8(m, c * CHUNK, K)) = q;
    }
}

// SmoothQuant, long rows of many tokens (the factors, 4 bytes per element from L2, are shared by RPB = 8 tokens; lane = token %
// 8 + 8 * chunk as above) and rows beyond the registers: read twice, the wavefronts take contiguous ranges of K.
// 2048 x 40960 83 us against 95 with a workgroup per token, 4096 x 16448 67 against 72 (below 2048 tokens it is the
// other way round: 1024 x 28672 45 against 32).  RPB = 1: at most 512 tokens of K > 98304.
template <int RPB>
__global__ __launch_bounds__(LONG_WAVES * 64) void act_quant_smooth_long_kernel(const __half *__restrict__ x, int64_t ldx, int M, int K,
                                                                                const float *__restrict__ inv_smooth,
                                                                                int8_t *__restrict__ xq_rm, int8_t *__restrict__ xq_kl,
                                                                                float *__restrict__ sx)
{
    __shared__ unsigned red[RPB][LONG_WAVES];
    constexpr int CPS = 64 / RPB;                        // chunks per wavefront per step
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6, r = lane % RPB, cl = lane / RPB;
    const int m = blockIdx.x * RPB + r, nchunks = K / CHUNK;
    const bool valid = m < M;
    const int steps = (nchunks + CPS - 1) / CPS, per_wave = (steps + LONG_WAVES - 1) / LONG_WAVES, s0 = wave * per_wave;
    const Half16 *row = reinterpret_cast<const Half16 *>(x + (size_t)(valid ? m : 0) * ldx);
    auto products = [&](int c, float (&f)[16]) {
        widen(row[c], f);
#pragma unroll
        for (int i = 0; i < 16; i += 4) {
            const float4 s4 = *reinterpret_cast<const float4 *>(inv_smooth + (size_t)c * CHUNK + i);
            f[i] *= s4.x, f[i + 1] *= s4.y, f[i + 2] *= s4.z, f[i + 3] *= s4.w;
        }
    };
    unsigned mx = 0;
    for (int i = 0; i < per_wave; ++i) {
        const int c = (s0 + i) * CPS + cl;
        if (c < nchunks && valid) {
            float f[16];
            products(c, f);
#pragma unroll
            for (int e = 0; e < 16; ++e) mx = max(mx, __float_as_uint(fabsf(f[e])));
        }
    }
#pragma unroll
    for (int off = 32; off >= RPB; off >>= 1) mx = max(mx, (unsigned)__shfl_xor((int)mx, off, 64));
    if (cl == 0) red[r][wave] = mx;
    __syncthreads();
    mx = 0;
    for (int w = 0; w < LONG_WAVES; ++w) mx = max(mx, red[r][w]);
    float scale, inv;
    token_scales_f32(__uint_as_float(mx), scale, inv);
    if (wave == 0 && cl == 0 && valid) sx[m] = scale;
    for (int i = 0; i < per_wave; ++i) {
        const int c = (s0 + i) * CPS + cl;
        if (c < nchunks && valid) {
            float f[16];
            products(c, f);
            const uint4 q = quant_chunk_f32(f, inv);
            if (xq_rm) *reinterpret_cast<uint4 *>(xq_rm + (size_t)m * K + (size_t)c * CHUNK) = q;
            if (xq_kl) *reinterpret_cast<uint4 *>(xq_kl + tile_offset_i8(m, c * CHUNK, K)) = q;
        }
    }
}

constexpr int SMOOTH_LONG_MIN_M = 2048;

// The other quantizer forms of the Preliminary section (not the hot path; one workgroup per token, the row is
// read twice).  Eq. 1 as printed: code = rne(x / s) with the stored fp32 scale s (IEEE division), then Eq. 2's
// clamp.  range 1 = Eq. 2 as printed (s = 2 amax / 255, codes in [-128, 127]); scope: the token's own maximum,
// the whole tensor's (tensor_amax: its bit pattern, found by a kernel before this one) or a calibrated scale
// supplied by the caller (static_scale).  sx still gets one entry per token, so the GEMM epilogue is unchanged.
__device__ inline float act_scale_of(float amax, int range)
{
    return range == QL_RANGE_EQ2 ? (2.0f * amax) / 255.0f : amax / 127.0f;   // one IEEE fp32 division
}

__global__ __launch_bounds__(256) void act_quant_opt_kernel(const __half *__restrict__ x, int64_t ldx, int M, int K,
                                                            int range, const unsigned *__restrict__ tensor_amax,
                                                            const float *__restrict__ static_scale,
                                                            int8_t *__restrict__ xq_rm, int8_t *__restrict__ xq_kl,
                                                            float *__restrict__ sx)
{
    __shared__ unsigned red[4];
    const int m = blockIdx.x;
    const int nchunks = K / CHUNK;
    const Half16 *row = reinterpret_cast<const Half16 *>(x + (size_t)m * ldx);
    float s;
    if (static_scale) {
        s = *static_scale;
    } else if (tensor_amax) {
        s = act_scale_of(__uint_as_float(*tensor_amax), range);
    } else {
        unsigned mx = 0;
        for (int c = threadIdx.x; c < nchunks; c += 256) mx = abs_max_bits(row[c], mx);
#pragma unroll
        for (int off = 32; off > 0; off >>= 1) mx = max(mx, (unsigned)__shfl_xor((int)mx, off, 64));
        if ((threadIdx.x & 63) == 0) red[threadIdx.x >> 6] = mx;
        __syncthreads();
        mx = max(max(red[0], red[1]), max(red[2], red[3]));
        s = act_scale_of(half_bits_to_float(mx), range);
    }
    if (s == 0.0f) s = 1.0f;
    if (threadIdx.x == 0) sx[m] = s;
    const float lo = range == QL_RANGE_EQ2 ? -128.0f : -127.0f;
    for (int c = threadIdx.x; c < nchunks; c += 256) {
        const Half16 h = row[c];
        const unsigned w[8] = {h.lo.x, h.lo.y, h.lo.z, h.lo.w, h.hi.x, h.hi.y, h.hi.z, h.hi.w};
        unsigned q[4] = {0, 0, 0, 0};
#pragma unroll
        for (int i = 0; i < 16; ++i) {
            const float v = half_bits_to_float((w[i / 2] >> (16 * (i % 2))) & 0xffffu);
            const float r = fminf(fmaxf(rintf(v / s), lo), 127.0f);   // IEEE fp32 division, ties to even, clamp
            q[i / 4] |= (unsigned)((int)r & 0xff) << (8 * (i % 4));
        }
        const uint4 o = make_uint4(q[0], q[1], q[2], q[3]);
        if (xq_rm) *reinterpret_cast<uint4 *>(xq_rm + (size_t)m * K + (size_t)c * CHUNK) = o;
        if (xq_kl) *reinterpret_cast<uint4 *>(xq_kl + tile_offset_i8(m, c * CHUNK, K)) = o;
    }
}

// max |x| over all tokens, as a bit pattern (accumulates into *out) or, with `as_scale`, as Eq. 2's scale for
// the given range (the scale is a non-decreasing function of the maximum, so the largest scale any workgroup
// derives is the scale of the largest value): a calibrated scale is the running maximum over batches
__global__ __launch_bounds__(256) void act_absmax_kernel(const __half *__restrict__ x, int64_t ldx, int M, int K,
                                                         int range, bool as_scale, unsigned *__restrict__ out)
{
    __shared__ unsigned red[4];
    const int nchunks = K / CHUNK;
    unsigned mx = 0;
    for (int m = blockIdx.x; m < M; m += gridDim.x) {
        const Half16 *row = reinterpret_cast<const Half16 *>(x + (size_t)m * ldx);
        for (int c = threadIdx.x; c < nchunks; c += 256) mx = abs_max_bits(row[c], mx);
    }
#pragma unroll
    for (int off = 32; off > 0; off >>= 1) mx = max(mx, (unsigned)__shfl_xor((int)mx, off, 64));
    if ((threadIdx.x & 63) == 0) red[threadIdx.x >> 6] = mx;
    __syncthreads();
    if (threadIdx.x == 0) {
        mx = max(max(red[0], red[1]), max(red[2], red[3]));
        const float amax = half_bits_to_float(mx);
        const float v = as_scale ? act_scale_of(amax, range) : amax;
        if (v > 0.0f) atomicMax(out, __float_as_uint(v));
    }
}

__global__ void fill_word_kernel(unsigned *p, unsigned v) { *p = v; }

__global__ void act_repack_kernel(const int8_t *__restrict__ xq_rm, int M, int K,
                                  int8_t *__restrict__ xq_kl)
{
    const int nchunks = K / CHUNK;
    const size_t total = (size_t)M * nchunks;
    for (size_t i = blockIdx.x * (size_t)blockDim.x + threadIdx.x; i < total;
         i += (size_t)gridDim.x * blockDim.x) {
        const int m = (int)(i / nchunks), c = (int)(i % nchunks);
        const uint4 q = *reinterpret_cast<const uint4 *>(xq_rm + (size_t)m * K + (size_t)c * CHUNK);
        *reinterpret_cast<uint4 *>(xq_kl + tile_offset_i8(m, c * CHUNK, K)) = q;
    }
}

}  // namespace

// (the documented limit of the row stride)
static int check_row_stride(int64_t ldx)
{
    if (ldx > MAX_ROW_STRIDE) return fail(QL_ERR_SHAPE, "row stride %lld beyond 2^27 elements", (long long)ldx);
    return QL_OK;
}

template <int MODE>
static void launch_rows8(const __half *x, int64_t ldx, int M, int K, const float *inv_smooth, int8_t *xq_rm, int8_t *xq_kl, float *sx,
                         hipStream_t st)
{
    const int steps = ceil_div(K / CHUNK, 64 / 8);
    const int nw = steps < ROWS8_WAVES ? steps : ROWS8_WAVES, per_wave = ceil_div(steps, nw);
    const dim3 grid(ceil_div(M, 8)), block(nw * 64);
#define QL_LAUNCH_ROWS8(NIT) \
    hipLaunchKernelGGL((act_quant_rows8_kernel<NIT, MODE>), grid, block, 0, st, x, ldx, M, K, per_wave, inv_smooth, xq_rm, xq_kl, sx)
    if (per_wave <= 1) QL_LAUNCH_ROWS8(1);
    else if (per_wave <= 2) QL_LAUNCH_ROWS8(2);
    else if (per_wave <= 4) QL_LAUNCH_ROWS8(4);
    else if (per_wave <= 8) QL_LAUNCH_ROWS8(8);
    else QL_LAUNCH_ROWS8(12);
#undef QL_LAUNCH_ROWS8
}

template <int MODE>
static int launch_aq(const __half *x, int64_t ldx, int M, int K, const float *inv_smooth, const __half *gamma, float eps,
                     int8_t *xq_rm, int8_t *xq_kl, float *sx, hipStream_t st)
{
    if constexpr (MODE <= 1) {
        if (M > ROWS8_MIN_M && K <= ROWS8_MAX_K) {
            launch_rows8<MODE>(x, ldx, M, K, inv_smooth, xq_rm, xq_kl, sx, st);
            return check_hip(hipGetLastError(), "act_quant (8 tokens per workgroup) launch");
        }
    }
    const dim3 grid(64 * ceil_div(M, 64));   // 8 equal ranges of whole groups of 8 tokens; what a range has too few ends at once
    const int chunks = K / CHUNK;
    if constexpr (MODE == 1) {
        if (K > ROW4_MAX_K && K <= ROW12_MAX_K && M < SMOOTH_LONG_MIN_M) {
            hipLaunchKernelGGL((act_quant_rows8_kernel<12, 1, 1>), dim3(M), dim3(ROWS8_WAVES * 64), 0, st, x, ldx, M, K,
                               ceil_div(ceil_div(chunks, 64), ROWS8_WAVES), inv_smooth, xq_rm, xq_kl, sx);
            return check_hip(hipGetLastError(), "act_quant (long rows) launch");
        }
        if (K > ROW12_MAX_K && M <= 512) {
            hipLaunchKernelGGL(act_quant_smooth_long_kernel<1>, dim3(M), dim3(LONG_WAVES * 64), 0, st, x, ldx, M, K, inv_smooth, xq_rm, xq_kl, sx);
            return check_hip(hipGetLastError(), "act_quant (long rows) launch");
        }
        if (K > ROW4_MAX_K || (chunks > ROW_CHUNKS && M >= SMOOTH_LONG_MIN_M)) {
            hipLaunchKernelGGL(act_quant_smooth_long_kernel<8>, dim3(ceil_div(M, 8)), dim3(LONG_WAVES * 64), 0, st, x, ldx, M, K, inv_smooth,
                               xq_rm, xq_kl, sx);
            return check_hip(hipGetLastError(), "act_quant (long rows) launch");
        }
    }
    if constexpr (MODE == 3) {
        if (K > ROW4_MAX_K) {
            hipLaunchKernelGGL(act_quant_swiglu_long_kernel, grid, dim3(LONG_WAVES * 64), 0, st, x, ldx, M, K, xq_rm, xq_kl, sx);
            return check_hip(hipGetLastError(), "act_quant (long rows) launch");
        }
    }
#define QL_LAUNCH_ROW(NC)                                                                                                       \
    hipLaunchKernelGGL((act_quant_kernel<MODE, NC>), grid, dim3(ceil_div(ceil_div(chunks, NC), 64) * 64), 0, st, x, ldx, M, K, inv_smooth, \
                       gamma, eps, xq_rm, xq_kl, sx)
    if (chunks <= ROW_CHUNKS) QL_LAUNCH_ROW(1);
    else if (chunks <= 2 * ROW_CHUNKS) QL_LAUNCH_ROW(2);
    else if (chunks <= 4 * ROW_CHUNKS) QL_LAUNCH_ROW(4);
    else if constexpr (MODE == 0 || MODE == 2) QL_LAUNCH_ROW(8);   // the last: K <= 131072
#undef QL_LAUNCH_ROW
    return check_hip(hipGetLastError(), "act_quant launch");
}

int launch_act_quant(const __half *x, int64_t ldx, int M, int K, int8_t *xq_rm, int8_t *xq_kl,
                     float *sx, hipStream_t st)
{
    if (M == 0) return QL_OK;
    QL_TRY(check_row_stride(ldx));
    return launch_aq<0>(x, ldx, M, K, nullptr, nullptr, 0.0f, xq_rm, xq_kl, sx, st);
}

int launch_act_quant_smooth(const __half *x, int64_t ldx, int M, int K, const float *inv_smooth, int8_t *xq_rm,
                            int8_t *xq_kl, float *sx, hipStream_t st)
{
    if (M == 0) return QL_OK;
    QL_TRY(check_row_stride(ldx));
    return launch_aq<1>(x, ldx, M, K, inv_smooth, nullptr, 0.0f, xq_rm, xq_kl, sx, st);
}

int launch_act_quant_opt(const __half *x, int64_t ldx, int M, int K, int range, int scope,
                         const float *static_scale, unsigned *amax_scratch, int8_t *xq_rm, int8_t *xq_kl, float *sx,
                         hipStream_t st)
{
    if (M == 0) return QL_OK;
    const unsigned *ta = nullptr;
    if (scope == QL_SCOPE_TENSOR) {
        hipLaunchKernelGGL(fill_word_kernel, dim3(1), dim3(1), 0, st, amax_scratch, 0u);
        hipLaunchKernelGGL(act_absmax_kernel, dim3(M < 1024 ? M : 1024), dim3(256), 0, st, x, ldx, M, K, range, false,
                           amax_scratch);
        QL_TRY(check_hip(hipGetLastError(), "act_absmax launch"));
        ta = amax_scratch;
    }
    hipLaunchKernelGGL(act_quant_opt_kernel, dim3(M), dim3(256), 0, st, x, ldx, M, K, range, ta,
                       scope == QL_SCOPE_STATIC ? static_scale : nullptr, xq_rm, xq_kl, sx);
    return check_hip(hipGetLastError(), "act_quant (options) launch");
}

int launch_act_calibrate(const __half *x, int64_t ldx, int M, int K, int range, float *scale, hipStream_t st)
{
    if (M == 0) return QL_OK;
    hipLaunchKernelGGL(act_absmax_kernel, dim3(M < 1024 ? M : 1024), dim3(256), 0, st, x, ldx, M, K, range, true,
                       reinterpret_cast<unsigned *>(scale));
    return check_hip(hipGetLastError(), "act_calibrate launch");
}

int launch_act_quant_rmsnorm(const __half *x, int64_t ldx, int M, int K, const __half *gamma, float eps, int8_t *xq_rm,
                             int8_t *xq_kl, float *sx, hipStream_t st)
{
    if (M == 0) return QL_OK;
    QL_TRY(check_row_stride(ldx));
    return launch_aq<2>(x, ldx, M, K, nullptr, gamma, eps, xq_rm, xq_kl, sx, st);
}

int launch_act_quant_swiglu(const __half *gate_up, int64_t ld, int M, int K, int8_t *xq_rm, int8_t *xq_kl, float *sx,
                            hipStream_t st)
{
    if (M == 0) return QL_OK;
    return launch_aq<3>(gate_up, ld, M, K, nullptr, nullptr, 0.0f, xq_rm, xq_kl, sx, st);
}

int launch_act_repack(const int8_t *xq_rm, int M, int K, int8_t *xq_kl, hipStream_t st)
{
    if (M == 0) return QL_OK;
    const size_t total = (size_t)M * (K / CHUNK);
    int blocks = (int)((total + 255) / 256);
    if (blocks > 4096) blocks = 4096;
    hipLaunchKernelGGL(act_repack_kernel, dim3(blocks), dim3(256), 0, st, xq_rm, M, K, xq_kl);
    return check_hip(hipGetLastError(), "act_repack launch");
}

}  // namespace ql
