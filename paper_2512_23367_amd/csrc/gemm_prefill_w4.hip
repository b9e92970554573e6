// Prefill GEMM + dequantization epilogue of the W4A8 linear layer for gfx950 (integer accumulation per group of 128 k, one
// fp16 scale per channel and group; Y = XW).
//
// Operands arrive as in the int8 kernel: activations in 32-row x 32-k int8 tiles, weights as nibbles in 1024-byte tile
// pairs (32 rows x 64 k), both fetched by `buffer_load_dwordx4 ... lds`.  A stage is one scale group (128 k).  The matrix
// instruction is 16x16x64: lane (row r = lane % 16, chunk ch = lane / 16) takes 16 bytes of weights that hold its 16 k of
// k-blocks 2 (ch / 2) and 2 (ch / 2) + 1, unpacked by shift and mask into 16 * code per byte, so two instructions cover the
// group for a 16 x 16 block; their int32 sums are folded into the fp32 accumulators right behind them (accf += float(sum) *
// scale).  Because a group is only two instructions deep, the integer sums are transient (16 registers) instead of a
// second copy of the accumulators, and a wavefront holds 128 tokens x 64 channels: half the unpacking per product of a
// 64 x 64 wavefront tile, and one pass over a 256 x 256 tile's output instead of two.
//
// What bounds it: the vector port.  Measured on gfx950, matrix and vector instructions of a SIMD add up (16 cycles per
// 16x16x64, 2 to 4 per vector operation whichever of the two wavefronts issues it), and the fold takes two operations per
// accumulator element and group: in registers alone 4.2 POP/s of products become 2.9 with the fold and 2.5 with the unpack.
// The loop below runs at 2.1 (2.02 us per stage of a 256 x 256 tile per CU, + ~7 us per tile: whole kernels at 1.9).  The
// 32x32x32 kernel further down (64 x 64 wavefront tiles in two ping-pong groups, 128 x 256 tiles) takes 2 x 1.07 us and 2 x 9
// us for the same: 4096 x 4096 x 12288 237 against 217 us, 3001 x 4096 x 4096 74 against 58 (192 x 256), 4096 x 11008 x
// 4096 205 against 184 -- it is the better one where 128 x 256 tiles fit one pass.
// Per wavefront the 8 multiplies of a token block and its 32 fold operations stay in clusters: interleaving them,
// folding a block late, fp32 scales instead of mixed-precision multiply-adds and wave priorities all measured the
// same or slower.
#include "gemm_tiles.h"
#include <type_traits>

namespace ql {
namespace {

struct W4Params {
    const int8_t *xq;
    const void *wq;
    const float *sx;
    const __half *wscales;   // [K/128][Npad] fp16
    const __half *bias;
    __half *y;
    int64_t ldy;
    int32_t *acc;
    int64_t ldacc;
    int32_t *partials;
    int row0, nrows;
    int M, N, K, Npad;
    int tiles_m, tiles_n, group_m;   // group_m: token tiles per strip of the tile order (see tile_coords)
    int tail_tiles_m, tail_tiles_n, tail_group_m;   // 128 x 256 tiles of the channels behind the first tiles_n tiles
    unsigned x_bytes, w_bytes, s_bytes;
    void *part;              // split-K: partial sums [split][workgroup][wavefront][channel block][token block][64 lanes x 16 B]
    int stages_per_split;    // split-K: blockIdx.y takes stages [y * stages_per_split, ...); otherwise all of them
};

// Writes a wavefront's staged block of 32 tokens to y, 16 bytes per lane (LPR lanes per row).
template <int LPR>
__device__ __forceinline__ void store_rows(const W4Params &p, const char *stg, int row_bytes, int m0, int n0, int lane)
{
    constexpr int RPI = 64 / LPR;
    static_assert(64 % LPR == 0 && 32 % RPI == 0, "whole rows per read-back instruction");
    asm volatile("" ::: "memory");   // (same wavefront, LDS operations complete in order: only the compiler must keep them so)
    __builtin_amdgcn_wave_barrier();
#pragma unroll
    for (int t = 0; t < 32 / RPI; ++t) {
        const int row = t * RPI + lane / LPR, c = lane % LPR;
        const uint4 v = *reinterpret_cast<const uint4 *>(stg + row * row_bytes + c * 16);
        const int mm = m0 + row, nn = n0 + c * 8;
        if (mm < p.M && nn < p.N) {
            __half *dst = p.y + (size_t)mm * p.ldy + nn;
            if (nn + 7 < p.N) {
                *reinterpret_cast<uint4 *>(dst) = v;
            } else {
                const unsigned w[4] = {v.x, v.y, v.z, v.w};
                for (int e = 0; e < 8 && nn + e < p.N; ++e)
                    dst[e] = __ushort_as_half((unsigned short)(w[e / 2] >> (16 * (e % 2))));
            }
        }
    }
    asm volatile("" ::: "memory");
    __builtin_amdgcn_wave_barrier();
}

// One workgroup tile: WAVES_M x WAVES_N wavefronts of 16 TB tokens x 16 CB channels; (tm, tn): the tile's position in
// units of its own size.
template <int WAVES_M, int WAVES_N, int TB, int CB, int STAGES, int EPI>
__device__ __forceinline__ void w4_tile(const W4Params &p, int tm, int tn, char *smem)
{
    constexpr int NW = WAVES_M * WAVES_N;
    constexpr int TM = WAVES_M * TB * 16, TN = WAVES_N * CB * 16;
    static_assert(TB % 2 == 0 && CB % 2 == 0, "wavefront tiles are whole 32-row blocks");
    constexpr int XFR = TM / 32 * 4, WFR = TN / 32 * 2;      // 1024-byte fragments per stage (128 k)
    constexpr int WOFF = XFR * 1024;
    constexpr int STAGE_BYTES = (XFR + WFR) * 1024;
    constexpr int FR = XFR + WFR;
    constexpr int LPW_HI = (FR + NW - 1) / NW + 1, LPW_LO = FR / NW + 1, NHI = FR % NW;

    constexpr int SXI = (TM + NW * 64 - 1) / (NW * 64), SBI = (TN + NW * 64 - 1) / (NW * 64);
    float *side_sx = reinterpret_cast<float *>(smem + STAGES * STAGE_BYTES);
    float *side_b = side_sx + SXI * NW * 64;
    char *scale_slots = reinterpret_cast<char *>(side_b + SBI * NW * 64);

    const int lane = threadIdx.x & 63;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int wm = wave % WAVES_M, wn = wave / WAVES_M;

    // epilogue operands: requested in front of the first stages, parked in registers, stored to LDS behind them (loads
    // return in order; range-checked, so no branch).  Each array is padded to whole entries per thread.
    int r_sx[SXI];
    short r_b[SBI];
    if (EPI == EPI_F16) {
        const __amdgpu_buffer_rsrc_t rx = make_rsrc(p.sx, (unsigned)p.M * 4u);
        const __amdgpu_buffer_rsrc_t rb = make_rsrc(p.bias, p.bias ? (unsigned)p.N * 2u : 0u);
#pragma unroll
        for (int it = 0; it < SXI; ++it)
            r_sx[it] = __builtin_amdgcn_raw_buffer_load_b32(rx, (unsigned)(tm * TM + threadIdx.x + it * NW * 64) * 4u, 0, 0);
#pragma unroll
        for (int it = 0; it < SBI; ++it)
            r_b[it] = __builtin_amdgcn_raw_buffer_load_b16(rb, (unsigned)(tn * TN + threadIdx.x + it * NW * 64) * 2u, 0, 0);
    }

    const int stage0 = blockIdx.y * p.stages_per_split;
    const int nstages = min(p.stages_per_split, p.K / 128 - stage0);
    const unsigned lane16 = lane * 16;
    const unsigned KB = p.K / 32;
    // Range checking: the whole byte offset travels in the per-lane offset; row-blocks beyond ceil32(M) / ceil32(N) return
    // nothing, dead stages behind the last one use buffers of zero length.  Fragment f of a stage is loaded by wavefront f % NW.
    // The group scales of the wavefront's channels (4 bytes per lane, the first CB * 8 lanes carry them) are loaded by every
    // wavefront of a channel column, the same bytes into the same slot: equal counts for all.
    auto issue_stage = [&](int s) {
        const bool live = s < nstages;
        const __amdgpu_buffer_rsrc_t xr = make_rsrc(p.xq, live ? p.x_bytes : 0u);
        const __amdgpu_buffer_rsrc_t wr = make_rsrc(p.wq, live ? p.w_bytes : 0u);
        char *buf = smem + (s % STAGES) * STAGE_BYTES;
        auto load_fragment = [&](int i) {
            const int f = i * NW + wave;
            const bool is_x = (XFR % NW == 0) ? (i < XFR / NW) : (f < XFR);
            if (is_x) {
                const unsigned off = ((unsigned)(tm * (TM / 32) + f / 4) * KB + (stage0 + s) * 4 + f % 4) * 1024u;
                __builtin_amdgcn_raw_ptr_buffer_load_lds(xr, LDS_PTR(buf + f * 1024), 16, lane16 + off, 0, 0, 0);
            } else {
                const int g = f - XFR;
                const unsigned off = ((unsigned)(tn * (TN / 32) + g / 2) * (KB / 2) + (stage0 + s) * 2 + g % 2) * 1024u;
                __builtin_amdgcn_raw_ptr_buffer_load_lds(wr, LDS_PTR(buf + f * 1024), 16, lane16 + off, 0, 0, 0);
            }
        };
#pragma unroll
        for (int i = 0; i < FR / NW; ++i) load_fragment(i);
        if (NHI != 0 && wave < NHI) load_fragment(FR / NW);
        const __amdgpu_buffer_rsrc_t sr = make_rsrc(p.wscales, live ? p.s_bytes : 0u);
        const unsigned off = ((unsigned)(stage0 + s) * p.Npad + tn * TN + wn * CB * 16) * 2u;
        __builtin_amdgcn_raw_ptr_buffer_load_lds(sr, LDS_PTR(scale_slots + ((s % STAGES) * WAVES_N + wn) * 256), 4, lane * 4 + off, 0, 0, 0);
    };
    // all but this wavefront's loads of the newest `newer` stages have landed
    auto wait_stages = [&](auto newer) {
        constexpr int n = decltype(newer)::value;
        if (NHI == 0 || wave < NHI) wait_vmcnt<n * LPW_HI>();
        else wait_vmcnt<n * LPW_LO>();
    };

    float accf[CB][TB][4];
    int tot[EPI == EPI_ACC ? CB : 1][EPI == EPI_ACC ? TB : 1][4];
#pragma unroll
    for (int i = 0; i < CB; ++i)
#pragma unroll
        for (int j = 0; j < TB; ++j)
#pragma unroll
            for (int e = 0; e < 4; ++e) {
                accf[i][j][e] = 0.0f;
                if (EPI == EPI_ACC) tot[i][j][e] = 0;
            }

#pragma unroll
    for (int s = 0; s < STAGES; ++s) issue_stage(s);
    if (EPI == EPI_F16) {
#pragma unroll
        for (int it = 0; it < SXI; ++it) side_sx[threadIdx.x + it * NW * 64] = __int_as_float(r_sx[it]);
#pragma unroll
        for (int it = 0; it < SBI; ++it)
            side_b[threadIdx.x + it * NW * 64] = __half2float(__ushort_as_half((unsigned short)r_b[it]));
    }

    const int ch = lane >> 4, r = lane & 15;
    const int xlane = (wm * TB / 2) * 4096 + (ch / 2) * 2048 + (r + 32 * (ch % 2)) * 16;
    const int wlane = WOFF + (wn * CB / 2) * 2048 + (ch / 2) * 1024 + (r + 32 * (ch % 2)) * 16;
    v4i wp[CB];              // packed weights of the stage, 128 k of 16 channels each
    v4i xf[2][2];
    h4 sg[CB], sn[CB];       // group scales of the stage being multiplied; of the one whose weights were read last
    auto read_weights = [&](int s) {
        const char *buf = smem + (s % STAGES) * STAGE_BYTES + wlane;
#pragma unroll
        for (int i = 0; i < CB; ++i) wp[i] = *reinterpret_cast<const v4i *>(buf + (i / 2) * 2048 + (i % 2) * 256);
        const char *slot = scale_slots + ((s % STAGES) * WAVES_N + wn) * 256 + ch * 8;
#pragma unroll
        for (int i = 0; i < CB; ++i) sn[i] = *reinterpret_cast<const h4 *>(slot + i * 32);
    };
    auto read_tokens = [&](int s, int j) {
        const char *buf = smem + (s % STAGES) * STAGE_BYTES + xlane;
#pragma unroll
        for (int t = 0; t < 2; ++t)
            xf[j & 1][t] = *reinterpret_cast<const v4i *>(buf + (j / 2) * 4096 + (j % 2) * 256 + t * 1024);
    };

    auto fold = [&](int g, int i, int j, const v4i &q) {   // group g's sums of channel block i, token block j
#pragma unroll
        for (int e = 0; e < 4; ++e) {
            if (EPI != EPI_ACC) {
                accf[i][j][e] = __builtin_fmaf((float)q[e], (float)sg[i][e], accf[i][j][e]);
            } else {
                tot[i][j][e] += q[e];
                if (p.partials) {
                    const int m = tm * TM + (wm * TB + j) * 16 + r, n = tn * TN + (wn * CB + i) * 16 + 4 * ch + e;
                    if (m >= p.row0 && m < p.row0 + p.nrows && m < p.M && n < p.N)
                        p.partials[((size_t)(m - p.row0) * (p.K / 128) + stage0 + g) * p.N + n] = q[e] >> 4;
                }
            }
        }
    };

    // Main loop, one barrier per stage.  Token fragments are read one block ahead; in front of the last block's products
    // the wavefront hands its stage over (own reads done, own loads of the next stage landed, barrier: then everyone's
    // have), refills the freed buffer and reads the next stage's weights and first tokens, whose latency the last
    // block's products and fold cover.
    wait_stages(std::integral_constant<int, STAGES - 1>{});
    __builtin_amdgcn_s_barrier();
    read_weights(0);
    read_tokens(0, 0);
    for (int it = 0; it < nstages; ++it) {
        v4i wf[CB][2];
#pragma unroll
        for (int i = 0; i < CB; ++i)
#pragma unroll
            for (int t = 0; t < 2; ++t) {
                const unsigned w0 = (unsigned)wp[i][2 * t], w1 = (unsigned)wp[i][2 * t + 1];
                wf[i][t][0] = (int)((w0 << 4) & 0xF0F0F0F0u);
                wf[i][t][1] = (int)(w0 & 0xF0F0F0F0u);
                wf[i][t][2] = (int)((w1 << 4) & 0xF0F0F0F0u);
                wf[i][t][3] = (int)(w1 & 0xF0F0F0F0u);
            }
#pragma unroll
        for (int i = 0; i < CB; ++i) sg[i] = sn[i];
        __builtin_amdgcn_sched_barrier(0);
#pragma unroll
        for (int j = 0; j < TB; ++j) {
            if (j + 1 < TB) {
                read_tokens(it, j + 1);
            } else {
                __builtin_amdgcn_s_waitcnt(0xC07F);   // lgkmcnt(0)
                wait_stages(std::integral_constant<int, STAGES - 2>{});
                __builtin_amdgcn_s_barrier();
                issue_stage(it + STAGES);
                read_weights(it + 1);
                read_tokens(it + 1, 0);
            }
            __builtin_amdgcn_sched_barrier(0);
            v4i q[CB];
#pragma unroll
            for (int i = 0; i < CB; ++i) q[i] = __builtin_amdgcn_mfma_i32_16x16x64_i8(wf[i][0], xf[j & 1][0], v4i{0, 0, 0, 0}, 0, 0, 0);
#pragma unroll
            for (int i = 0; i < CB; ++i) q[i] = __builtin_amdgcn_mfma_i32_16x16x64_i8(wf[i][1], xf[j & 1][1], q[i], 0, 0, 0);
            __builtin_amdgcn_sched_barrier(0);
#pragma unroll
            for (int i = 0; i < CB; ++i) fold(it, i, j, q[i]);
            __builtin_amdgcn_sched_barrier(0);
        }
    }
    wait_vmcnt<0>();   // drain the dead tail loads before the LDS is released

    if constexpr (EPI == EPI_PART) {
        char *dst = static_cast<char *>(p.part) + (((size_t)blockIdx.y * gridDim.x + blockIdx.x) * NW + wave) * (size_t)(CB * TB * 1024);
#pragma unroll
        for (int i = 0; i < CB; ++i)
#pragma unroll
            for (int j = 0; j < TB; ++j)
                *reinterpret_cast<float4 *>(dst + (i * TB + j) * 1024 + lane * 16) =
                    float4{accf[i][j][0], accf[i][j][1], accf[i][j][2], accf[i][j][3]};
        return;
    }
    if constexpr (EPI == EPI_ACC) {
#pragma unroll
        for (int j = 0; j < TB; ++j)
#pragma unroll
            for (int i = 0; i < CB; ++i)
#pragma unroll
                for (int e = 0; e < 4; ++e) {
                    const int m = tm * TM + (wm * TB + j) * 16 + r, n = tn * TN + (wn * CB + i) * 16 + 4 * ch + e;
                    if (m < p.M && n < p.N) p.acc[(size_t)m * p.ldacc + n] = tot[i][j][e] >> 4;
                }
        return;
    }

    constexpr int ROW_BYTES = CB * 16 * 2 + 16;
    static_assert(NW * 32 * ROW_BYTES <= STAGES * STAGE_BYTES, "staging patch fits the pipeline buffers");
    __syncthreads();
    char *stg = smem + wave * (32 * ROW_BYTES);
    const int n_wave0 = tn * TN + wn * CB * 16, m_wave0 = tm * TM + wm * TB * 16;
    float sx_r[TB];
    float4 b_r[CB];
#pragma unroll
    for (int j = 0; j < TB; ++j) sx_r[j] = side_sx[(wm * TB + j) * 16 + r] * 0.0625f;
#pragma unroll
    for (int i = 0; i < CB; ++i) b_r[i] = *reinterpret_cast<const float4 *>(side_b + (wn * CB + i) * 16 + 4 * ch);
#pragma unroll
    for (int jb = 0; jb < TB / 2; ++jb) {
#pragma unroll
        for (int jj = 0; jj < 2; ++jj) {
            const int j = 2 * jb + jj;
#pragma unroll
            for (int i = 0; i < CB; ++i) {
                const float b4[4] = {b_r[i].x, b_r[i].y, b_r[i].z, b_r[i].w};
                h4 o;
#pragma unroll
                for (int e = 0; e < 4; ++e) {
                    float v = __builtin_fmaf(accf[i][j][e], sx_r[j], b4[e]);
                    asm("" : "+v"(v));   // rounded to fp32, then to fp16, in every kernel variant
                    o[e] = (_Float16)v;
                }
                *reinterpret_cast<h4 *>(stg + (jj * 16 + r) * ROW_BYTES + (i * 16 + 4 * ch) * 2) = o;
            }
        }
        store_rows<CB * 2>(p, stg, ROW_BYTES, m_wave0 + jb * 32, n_wave0, lane);
    }
}

template <int WAVES_M, int WAVES_N, int TB, int CB, int STAGES>
struct W4Tile {
    static constexpr int NW = WAVES_M * WAVES_N, TM = WAVES_M * TB * 16, TN = WAVES_N * CB * 16, THREADS = NW * 64;
    static constexpr int LDS = (TM / 32 * 4 + TN / 32 * 2) * 1024 * STAGES +
                               ((TM + THREADS - 1) / THREADS + (TN + THREADS - 1) / THREADS) * THREADS * 4 + STAGES * WAVES_N * 256;
};

template <int WAVES_M, int WAVES_N, int TB, int CB, int STAGES, int EPI, int OCC>
__global__ __launch_bounds__(WAVES_M *WAVES_N * 64, OCC) void gemm_w4_kernel(W4Params p)
{
    extern __shared__ __attribute__((aligned(1024))) char smem[];
    int tm, tn;
    tile_coords(blockIdx.x, p.tiles_m, p.tiles_n, p.group_m, tm, tn);
    w4_tile<WAVES_M, WAVES_N, TB, CB, STAGES, EPI>(p, tm, tn, smem);
}

// 256 x 256 tiles for the first tiles_n channel tiles (whole passes over the CUs), 128 x 256 for the rest: the last pass
// is half as long instead of a whole one that most CUs sit out (22016 channels, 4096 tokens: 5.4 passes).
__global__ __launch_bounds__(512, 1) void gemm_w4_tail_kernel(W4Params p)
{
    extern __shared__ __attribute__((aligned(1024))) char smem[];
    int tm, tn;
    const int first = p.tiles_m * p.tiles_n;
    if ((int)blockIdx.x < first) {
        tile_coords(blockIdx.x, p.tiles_m, p.tiles_n, p.group_m, tm, tn);
        w4_tile<2, 4, 8, 4, 3, EPI_F16>(p, tm, tn, smem);
    } else {
        tile_coords(blockIdx.x - first, p.tail_tiles_m, p.tail_tiles_n, p.tail_group_m, tm, tn);
        w4_tile<2, 4, 4, 4, 4, EPI_F16>(p, tm, p.tiles_n + tn, smem);
    }
}

// 128 x 256 tiles on the 32x32x32 instruction: 8 wavefronts of 64 x 64 in two ping-pong groups (w and w + 4, one of each per
// SIMD) one phase apart -- while one reads a stage's fragments, folds the previous group's int32 sums (accf += float(sum) *
// scale) and waits for its loads, the other unpacks and multiplies; every phase ends with the workgroup barrier.  A 64 x 64
// wavefront tile has nothing to gain from transient sums (its unpacking is per 64 tokens either way), and the two
// phases cover each other's LDS and barrier latency, which counts where a launch is one pass over part of the CUs: against the
// 16x16x64 loop on the same tile 512 x 4096 x 12288 43.3 -> 37.6 us, 1536 x 11008 x 4096 104 -> 89, 3001 x 6144 x 1536
// 58.8 -> 50.2, with all 256 CUs busy (2048 x 4096 x 4096) 45.6 -> 42.2.
constexpr int PP_STAGES = 4, PP_TM = 128, PP_TN = 256, PP_THREADS = 512;
constexpr int PP_STAGE_BYTES = (PP_TM / 32 * 4 + PP_TN / 32 * 2) * 1024;
constexpr int PP_SLOTS = 8;                               // ring of scale slots: a group's scales are read one stage later than its fragments
constexpr int PP_LDS = PP_STAGES * PP_STAGE_BYTES + 2 * PP_THREADS * 4 + PP_SLOTS * 8 * 256;

template <bool SPLIT>   // split-K: raw partial sums [split][workgroup][wavefront][channel block][token block][quad][64 lanes x 16 B]
__global__ __launch_bounds__(PP_THREADS, 1) void gemm_w4_pp_kernel(W4Params p)
{
    typedef int v16i __attribute__((ext_vector_type(16)));
    constexpr int NW = 8, WB = 2;                            // 32-row blocks of a wavefront tile, either way
    constexpr int XFR = PP_TM / 32 * 4, WOFF = XFR * 1024, FR = PP_STAGE_BYTES / 1024, LPW = FR / NW + 1;
    static_assert(FR % NW == 0 && XFR % NW == 0 && PP_TM <= PP_THREADS && PP_TN <= PP_THREADS, "equal shares");
    extern __shared__ __attribute__((aligned(1024))) char smem[];
    float *side_sx = reinterpret_cast<float *>(smem + PP_STAGES * PP_STAGE_BYTES);
    float *side_b = side_sx + PP_THREADS;
    char *scale_slots = reinterpret_cast<char *>(side_b + PP_THREADS);    // [slot][wavefront] 256 bytes

    const int lane = threadIdx.x & 63;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int wm = wave % 2, wn = wave / 2;
    int tm, tn;
    tile_coords(blockIdx.x, p.tiles_m, p.tiles_n, p.group_m, tm, tn);

    // epilogue operands: requested in front of the first stages, stored to LDS behind them
    int r_sx = 0;
    short r_b = 0;
    if (!SPLIT) {
        r_sx = __builtin_amdgcn_raw_buffer_load_b32(make_rsrc(p.sx, (unsigned)p.M * 4u), (unsigned)(tm * PP_TM + threadIdx.x) * 4u, 0, 0);
        r_b = __builtin_amdgcn_raw_buffer_load_b16(make_rsrc(p.bias, p.bias ? (unsigned)p.N * 2u : 0u), (unsigned)(tn * PP_TN + threadIdx.x) * 2u, 0, 0);
    }
    const int stage0 = SPLIT ? blockIdx.y * p.stages_per_split : 0;
    const int nstages = SPLIT ? min(p.stages_per_split, p.K / 128 - stage0) : p.K / 128;
    const unsigned lane16 = lane * 16, KB = p.K / 32;
    auto issue_stage = [&](int s) {                          // as in w4_tile; the scales of a wavefront's 64 channels into a slot of its own
        const bool live = s < nstages;
        const __amdgpu_buffer_rsrc_t xr = make_rsrc(p.xq, live ? p.x_bytes : 0u);
        const __amdgpu_buffer_rsrc_t wr = make_rsrc(p.wq, live ? p.w_bytes : 0u);
        char *buf = smem + (s % PP_STAGES) * PP_STAGE_BYTES;
#pragma unroll
        for (int i = 0; i < FR / NW; ++i) {
            const int f = i * NW + wave;
            if (i < XFR / NW) {
                const unsigned off = ((unsigned)(tm * (PP_TM / 32) + f / 4) * KB + (stage0 + s) * 4 + f % 4) * 1024u;
                __builtin_amdgcn_raw_ptr_buffer_load_lds(xr, LDS_PTR(buf + f * 1024), 16, lane16 + off, 0, 0, 0);
            } else {
                const int g = f - XFR;
                const unsigned off = ((unsigned)(tn * (PP_TN / 32) + g / 2) * (KB / 2) + (stage0 + s) * 2 + g % 2) * 1024u;
                __builtin_amdgcn_raw_ptr_buffer_load_lds(wr, LDS_PTR(buf + f * 1024), 16, lane16 + off, 0, 0, 0);
            }
        }
        const __amdgpu_buffer_rsrc_t sr = make_rsrc(p.wscales, live ? p.s_bytes : 0u);
        const unsigned off = ((unsigned)(stage0 + s) * p.Npad + tn * PP_TN + wn * 64) * 2u;
        __builtin_amdgcn_raw_ptr_buffer_load_lds(sr, LDS_PTR(scale_slots + ((s % PP_SLOTS) * NW + wave) * 256), 4, lane * 4 + off, 0, 0, 0);
    };

    // element 4 q + e of a 32x32 block (i, j): channel 8 q + 4 (lane / 32) + e, token lane % 32
    v16i acc[WB][WB];
    float accf[WB][WB][16];
    h4 sg[WB][4];                                            // scales of the group whose sums sit in acc
#pragma unroll
    for (int i = 0; i < WB; ++i) {
#pragma unroll
        for (int q = 0; q < 4; ++q) sg[i][q] = h4{0, 0, 0, 0};
#pragma unroll
        for (int j = 0; j < WB; ++j)
#pragma unroll
            for (int r = 0; r < 16; ++r) acc[i][j][r] = 0, accf[i][j][r] = 0.0f;
    }
    const v16i zero16 = acc[0][0];
    auto read_scales = [&](int g) {
        const char *slot = scale_slots + ((g % PP_SLOTS) * NW + wave) * 256;
#pragma unroll
        for (int i = 0; i < WB; ++i)
#pragma unroll
            for (int q = 0; q < 4; ++q) sg[i][q] = *reinterpret_cast<const h4 *>(slot + (i * 32 + 8 * q + 4 * (lane >> 5)) * 2);
    };
    auto fold = [&]() {
#pragma unroll
        for (int i = 0; i < WB; ++i)
#pragma unroll
            for (int j = 0; j < WB; ++j)
#pragma unroll
                for (int r = 0; r < 16; ++r) accf[i][j][r] = __builtin_fmaf((float)acc[i][j][r], (float)sg[i][r / 4][r % 4], accf[i][j][r]);
    };

#pragma unroll
    for (int s = 0; s < PP_STAGES - 1; ++s) issue_stage(s);
    if (!SPLIT) {                                            // (entries beyond the tile are not used)
        side_sx[threadIdx.x] = __int_as_float(r_sx);
        side_b[threadIdx.x] = __half2float(__ushort_as_half((unsigned short)r_b));
    }

    const bool late = wave >= NW / 2;
    v4i wp[2][WB], xf[4][WB];
    wait_vmcnt<(PP_STAGES - 2) * LPW>();                     // stage 0 has landed (this wavefront's part)
    __builtin_amdgcn_s_barrier();                            // ... everyone's
    if (late) __builtin_amdgcn_s_barrier();                  // phase shift
    for (int it = 0; it < nstages; ++it) {
        // ---- memory phase
        const char *buf = smem + (it % PP_STAGES) * PP_STAGE_BYTES;
        if (it > 0) read_scales(it - 1);
#pragma unroll
        for (int kp = 0; kp < 2; ++kp)
#pragma unroll
            for (int i = 0; i < WB; ++i) wp[kp][i] = *reinterpret_cast<const v4i *>(buf + WOFF + ((wn * WB + i) * 2 + kp) * 1024 + lane16);
#pragma unroll
        for (int kb = 0; kb < 4; ++kb)
#pragma unroll
            for (int j = 0; j < WB; ++j) xf[kb][j] = *reinterpret_cast<const v4i *>(buf + ((wm * WB + j) * 4 + kb) * 1024 + lane16);
        issue_stage(it + PP_STAGES - 1);                     // into the buffer of stage it - 1: both groups have read it
        fold();                                              // group it - 1 (the first time: zeros)
        __builtin_amdgcn_sched_barrier(0);                   // the fold stays in front of the wait: it covers the loads' latency
        wait_vmcnt<(PP_STAGES - 2) * LPW>();                 // own loads of stage it + 1 have landed
        __builtin_amdgcn_s_waitcnt(0xC07F);                  // lgkmcnt(0): fragments are in registers, the buffer may be refilled
        __builtin_amdgcn_s_barrier();
        // ---- compute phase
        __builtin_amdgcn_sched_barrier(0);
#pragma unroll
        for (int kb = 0; kb < 4; ++kb)
#pragma unroll
            for (int i = 0; i < WB; ++i) {
                const unsigned w0 = (unsigned)wp[kb / 2][i][2 * (kb % 2)], w1 = (unsigned)wp[kb / 2][i][2 * (kb % 2) + 1];
                v4i wf;
                wf[0] = (int)((w0 << 4) & 0xF0F0F0F0u);
                wf[1] = (int)(w0 & 0xF0F0F0F0u);
                wf[2] = (int)((w1 << 4) & 0xF0F0F0F0u);
                wf[3] = (int)(w1 & 0xF0F0F0F0u);
#pragma unroll
                for (int j = 0; j < WB; ++j)
                    acc[i][j] = __builtin_amdgcn_mfma_i32_32x32x32_i8(wf, xf[kb][j], kb == 0 ? zero16 : acc[i][j], 0, 0, 0);
            }
        __builtin_amdgcn_sched_barrier(0);
        __builtin_amdgcn_s_barrier();
    }
    if (!late) __builtin_amdgcn_s_barrier();
    read_scales(nstages - 1);
    fold();
    wait_vmcnt<0>();                                         // drain the dead tail loads before the LDS is reused

    if constexpr (SPLIT) {
        char *dst = static_cast<char *>(p.part) + (((size_t)blockIdx.y * gridDim.x + blockIdx.x) * NW + wave) * (size_t)(WB * WB * 4096);
#pragma unroll
        for (int i = 0; i < WB; ++i)
#pragma unroll
            for (int j = 0; j < WB; ++j)
#pragma unroll
                for (int q = 0; q < 4; ++q)
                    *reinterpret_cast<float4 *>(dst + ((i * WB + j) * 4 + q) * 1024 + lane16) =
                        float4{accf[i][j][4 * q], accf[i][j][4 * q + 1], accf[i][j][4 * q + 2], accf[i][j][4 * q + 3]};
        return;
    }
    constexpr int ROW_BYTES = WB * 64 + 16;
    static_assert(NW * 32 * ROW_BYTES <= PP_STAGES * PP_STAGE_BYTES, "staging patch fits the pipeline buffers");
    __syncthreads();
    char *stg = smem + wave * (32 * ROW_BYTES);
    const int n_wave0 = tn * PP_TN + wn * 64, m_wave0 = tm * PP_TM + wm * 64;
#pragma unroll
    for (int j = 0; j < WB; ++j) {
        const float sxm = side_sx[(wm * WB + j) * 32 + (lane & 31)] * 0.0625f;
#pragma unroll
        for (int i = 0; i < WB; ++i)
#pragma unroll
            for (int q = 0; q < 4; ++q) {
                const float4 b = *reinterpret_cast<const float4 *>(side_b + (wn * WB + i) * 32 + 8 * q + 4 * (lane >> 5));
                const float b4[4] = {b.x, b.y, b.z, b.w};
                h4 o;
#pragma unroll
                for (int e = 0; e < 4; ++e) {
                    float v = __builtin_fmaf(accf[i][j][4 * q + e], sxm, b4[e]);
                    asm("" : "+v"(v));   // rounded to fp32, then to fp16, in every kernel variant
                    o[e] = (_Float16)v;
                }
                *reinterpret_cast<h4 *>(stg + (lane & 31) * ROW_BYTES + (i * 32 + 8 * q + 4 * (lane >> 5)) * 2) = o;
            }
        store_rows<WB * 4>(p, stg, ROW_BYTES, m_wave0 + j * 32, n_wave0, lane);
    }
}

// Split-K, second kernel: adds the splits' fp32 partial sums, split 0 first, then the dequantization of the fused
// epilogue.  A workgroup per wavefront of the first kernel, a quarter of its 16 x 16 blocks per wavefront; all loads of a
// split are issued before the first is used.
struct W4FinishParams {
    const float *part;
    const float *sx;
    const __half *bias;
    __half *y;
    int64_t ldy;
    int M, N, tiles_m, tiles_n, group_m, splits;
};

// SQUARE32: the blocks of 1024 bytes are quads of 32x32 blocks (gemm_w4_pp_kernel) instead of 16x16 blocks; TB, CB as there.
template <int WAVES_M, int WAVES_N, int TB, int CB, bool SQUARE32 = false>
__global__ __launch_bounds__(256) void w4_finish_kernel(W4FinishParams f)
{
    constexpr int NW = WAVES_M * WAVES_N, BLOCKS = CB * TB, PER = BLOCKS / 4;
    const int lane = threadIdx.x & 63, part = threadIdx.x >> 6;
    const int tile = blockIdx.x / NW, wave = blockIdx.x % NW;
    int tm, tn;
    tile_coords(tile, f.tiles_m, f.tiles_n, f.group_m, tm, tn);
    const int wm = wave % WAVES_M, wn = wave / WAVES_M;
    const size_t stride = (size_t)f.tiles_m * f.tiles_n * NW * BLOCKS * 256;     // floats per split
    const float *src = f.part + (size_t)blockIdx.x * BLOCKS * 256 + (size_t)part * PER * 256 + lane * 4;
    float4 v[PER];
#pragma unroll
    for (int b = 0; b < PER; ++b) v[b] = *reinterpret_cast<const float4 *>(src + b * 256);
    for (int s = 1; s < f.splits; ++s) {
        float4 u[PER];
#pragma unroll
        for (int b = 0; b < PER; ++b) u[b] = *reinterpret_cast<const float4 *>(src + s * stride + b * 256);
#pragma unroll
        for (int b = 0; b < PER; ++b) v[b].x += u[b].x, v[b].y += u[b].y, v[b].z += u[b].z, v[b].w += u[b].w;
    }
#pragma unroll
    for (int b = 0; b < PER; ++b) {
        const int at = part * PER + b;
        int m, n0;
        if (SQUARE32) {
            const int i = at / (2 * TB), j = at / 4 % (TB / 2), q = at % 4;
            m = ((tm * WAVES_M + wm) * (TB / 2) + j) * 32 + (lane & 31), n0 = ((tn * WAVES_N + wn) * (CB / 2) + i) * 32 + 8 * q + 4 * (lane >> 5);
        } else {
            const int i = at / TB, j = at % TB;
            m = ((tm * WAVES_M + wm) * TB + j) * 16 + (lane & 15), n0 = ((tn * WAVES_N + wn) * CB + i) * 16 + 4 * (lane >> 4);
        }
        if (m >= f.M || n0 >= f.N) continue;
        const float sxm = f.sx[m] * 0.0625f;
        const float a[4] = {v[b].x, v[b].y, v[b].z, v[b].w};
        h4 o;
#pragma unroll
        for (int e = 0; e < 4; ++e) {
            float t = __builtin_fmaf(a[e], sxm, f.bias && n0 + e < f.N ? __half2float(f.bias[n0 + e]) : 0.0f);
            asm("" : "+v"(t));   // rounded to fp32, then to fp16, as in the fused epilogue
            o[e] = (_Float16)t;
        }
        __half *dst = f.y + (size_t)m * f.ldy + n0;
        if (n0 + 3 < f.N) {
            *reinterpret_cast<h4 *>(dst) = o;         // 8 bytes: row starts are 16-byte aligned, n0 % 4 == 0
        } else {
            for (int e = 0; e < 4 && n0 + e < f.N; ++e) reinterpret_cast<_Float16 *>(dst)[e] = o[e];
        }
    }
}

inline W4Params w4_params(const GemmArgs &a)
{
    W4Params p = {};
    p.xq = a.xq;
    p.wq = a.wq;
    p.sx = a.sx;
    p.bias = a.bias;
    p.y = a.y;
    p.ldy = a.ldy;
    p.acc = a.acc;
    p.ldacc = a.ldacc ? a.ldacc : a.N;
    p.partials = a.partials;
    p.row0 = a.row0;
    p.nrows = a.nrows;
    p.M = a.M;
    p.N = a.N;
    p.K = a.K;
    p.Npad = round_up(a.N, TILE_ROWS);
    p.x_bytes = (unsigned)act_kernel_bytes(a.M, a.K);
    p.w_bytes = (unsigned)w4_codes_bytes(a.N, a.K);
    p.wscales = reinterpret_cast<const __half *>(static_cast<const char *>(a.wq) + w4_scales_offset(a.N, a.K));
    p.s_bytes = (unsigned)(a.K / 128) * p.Npad * 2u;
    p.stages_per_split = a.K / 128;
    return p;
}

// once per kernel and process
template <typename F>
int set_lds(F kern, int bytes)
{
    return check_hip(hipFuncSetAttribute(reinterpret_cast<const void *>(kern), hipFuncAttributeMaxDynamicSharedMemorySize, bytes),
                     "hipFuncSetAttribute(max dynamic LDS)");
}

template <int WAVES_M, int WAVES_N, int TB, int CB, int STAGES, int EPI, int OCC>
int launch_w4(const GemmArgs &a, hipStream_t st, int splits = 1)
{
    using T = W4Tile<WAVES_M, WAVES_N, TB, CB, STAGES>;
    static_assert(T::LDS * OCC <= 160 * 1024, "LDS budget");
    auto kern = gemm_w4_kernel<WAVES_M, WAVES_N, TB, CB, STAGES, EPI, OCC>;
    static const int attr_status = set_lds(kern, T::LDS);   // the initialisation of a function-local static is thread-safe
    if (attr_status != QL_OK) return attr_status;
    W4Params p = w4_params(a);
    p.tiles_m = ceil_div(a.M, T::TM);
    p.tiles_n = ceil_div(a.N, T::TN);
    // (an activation row costs twice the bytes of a weight row)
    p.group_m = strip_height(p.tiles_m, p.tiles_n, T::TM * 2, T::TN, OCC);
    const int nstages = a.K / 128;
    p.stages_per_split = ceil_div(nstages, splits);
    splits = ceil_div(nstages, p.stages_per_split);   // no empty split
    if (EPI == EPI_PART) {
        const size_t need = (size_t)splits * p.tiles_m * p.tiles_n * T::TM * T::TN * 4;
        if (!a.ws || need > a.ws_bytes) return fail(QL_ERR_WORKSPACE, "split-K needs %zu bytes of workspace", need);
    }
    p.part = a.ws;
    hipLaunchKernelGGL(kern, dim3(p.tiles_m * p.tiles_n, splits), dim3(T::THREADS), T::LDS, st, p);
    QL_TRY(check_hip(hipGetLastError(), "gemm_w4 launch"));
    if (EPI != EPI_PART) return QL_OK;
    W4FinishParams f = {static_cast<const float *>(a.ws), a.sx, a.bias, a.y, a.ldy, a.M, a.N, p.tiles_m, p.tiles_n, p.group_m, splits};
    hipLaunchKernelGGL((w4_finish_kernel<WAVES_M, WAVES_N, TB, CB>), dim3(p.tiles_m * p.tiles_n * T::NW), dim3(256), 0, st, f);
    return check_hip(hipGetLastError(), "w4_finish launch");
}

inline size_t pp_split_bytes(const GemmArgs &a, int splits) { return (size_t)splits * ceil_div(a.M, PP_TM) * ceil_div(a.N, PP_TN) * PP_TM * PP_TN * 4; }

template <bool SPLIT>
int launch_w4_pp(const GemmArgs &a, hipStream_t st, int splits = 1)
{
    static_assert(PP_LDS <= 160 * 1024, "LDS budget");
    static const int attr_status = set_lds(gemm_w4_pp_kernel<SPLIT>, PP_LDS);
    if (attr_status != QL_OK) return attr_status;
    W4Params p = w4_params(a);
    p.tiles_m = ceil_div(a.M, PP_TM);
    p.tiles_n = ceil_div(a.N, PP_TN);
    p.group_m = strip_height(p.tiles_m, p.tiles_n, PP_TM * 2, PP_TN, 1);
    p.stages_per_split = ceil_div(a.K / 128, splits);
    splits = ceil_div(a.K / 128, p.stages_per_split);   // no empty split
    if (SPLIT && (!a.ws || pp_split_bytes(a, splits) > a.ws_bytes))
        return fail(QL_ERR_WORKSPACE, "split-K needs %zu bytes of workspace", pp_split_bytes(a, splits));
    p.part = a.ws;
    hipLaunchKernelGGL(gemm_w4_pp_kernel<SPLIT>, dim3(p.tiles_m * p.tiles_n, splits), dim3(PP_THREADS), PP_LDS, st, p);
    QL_TRY(check_hip(hipGetLastError(), "gemm_w4_pp launch"));
    if (!SPLIT) return QL_OK;
    W4FinishParams f = {static_cast<const float *>(a.ws), a.sx, a.bias, a.y, a.ldy, a.M, a.N, p.tiles_m, p.tiles_n, p.group_m, splits};
    hipLaunchKernelGGL((w4_finish_kernel<2, 4, 4, 4, true>), dim3(p.tiles_m * p.tiles_n * 8), dim3(256), 0, st, f);
    return check_hip(hipGetLastError(), "w4_finish launch");
}

// the first `first_tiles` channel tiles in 256 x 256 tiles, the rest in 128 x 256 (0 < first_tiles < all of them)
int launch_w4_tail(const GemmArgs &a, int first_tiles, hipStream_t st)
{
    using Big = W4Tile<2, 4, 8, 4, 3>;
    using Small = W4Tile<2, 4, 4, 4, 4>;
    constexpr int LDS = Big::LDS > Small::LDS ? Big::LDS : Small::LDS;
    static_assert(LDS <= 160 * 1024 && Big::TN == Small::TN && Big::THREADS == Small::THREADS, "one launch");
    static const int attr_status = set_lds(gemm_w4_tail_kernel, LDS);
    if (attr_status != QL_OK) return attr_status;
    W4Params p = w4_params(a);
    p.tiles_m = ceil_div(a.M, Big::TM);
    p.tiles_n = first_tiles;
    p.group_m = strip_height(p.tiles_m, p.tiles_n, Big::TM * 2, Big::TN, 1);
    p.tail_tiles_m = ceil_div(a.M, Small::TM);
    p.tail_tiles_n = ceil_div(a.N, Small::TN) - first_tiles;
    p.tail_group_m = strip_height(p.tail_tiles_m, p.tail_tiles_n, Small::TM * 2, Small::TN, 1);
    hipLaunchKernelGGL(gemm_w4_tail_kernel, dim3(p.tiles_m * p.tiles_n + p.tail_tiles_m * p.tail_tiles_n), dim3(Big::THREADS), LDS, st, p);
    return check_hip(hipGetLastError(), "gemm_w4_tail launch");
}

// The automatic choice.  Estimated time of a tile shape: 3 us + passes over the 256 CUs x (o + stages x c), fitted to 25
// shapes (64..8192 tokens, N 1536..22016, K 1536..16384; weights from HBM, every CU busy):
//   256 x 256  o 7  c 2.02;   192 x 256  5  1.60;   128 x 256 (ping-pong)  3  1.12, a last pass of at most 224 tiles 2.5  1.00
//   128 x 128  0.5  0.78 alone on its CU, 4  1.12 for two per CU; a last pass of at most 256 tiles runs alone
// (operations per us of a full pass at K = 4096: 119, 113, 106, 106 GOP -- the largest tile wins where it fills its passes; a
// launch that leaves CUs idle runs at a higher clock).  Over 165 shapes (96..4096 tokens, N 1536..22016, K 1024..11008) the
// pick is within 0.3 % of the fastest form on average, 5 % at worst.
// Combined form: p whole passes of 256 x 256, the remaining channels in 128 x 256 tiles (c 1.10, o 5: the 16x16x64 loop).
// Split-K (few tiles, long K), taken when 10 % ahead: on 128 x 128 tiles + 8 us and 0.16 us per MB of partial sums for the second
// kernel; on 128 x 256 tiles, one pass, 8.8 us + stages x 0.87 + 0.43 us per MB, both kernels (144 splits, within 5 % on
// average; 1536 x 6144 x 1536 32 us, 128 x 128 unsplit 39; 512 x 11008 x 4096 42, split on 128 x 128 44).
enum W4Shape { W4_256 = 26, W4_192 = 35, W4_128X256 = 37, W4_128 = 13, W4_TAIL = 43, W4_SPLIT = 200, W4_SPLIT256 = 300 };   // ql_set_kernel_variant values

struct W4Choice {
    int shape, splits, first_tiles;
    double us;
};

inline double w4_passes(long tiles, double o, double c, int stages) { return (double)((tiles + 255) / 256) * (o + c * stages); }

inline double w4_128_us(long tiles, int stages)
{
    const long rest = tiles % 512;
    return (double)(tiles / 512 + (rest > 256)) * (4.0 + 1.12 * stages) + (rest > 0 && rest <= 256 ? 0.5 + 0.78 * stages : 0.0);
}

inline double w4_pp_us(long tiles, int stages)
{
    const long rest = tiles % 256, full = tiles / 256 + (rest > 224);
    return (double)full * (3.0 + 1.12 * stages) + (rest > 0 && rest <= 224 ? 2.5 + 1.0 * stages : 0.0);
}

inline W4Choice choose_w4(const GemmArgs &a, size_t scratch, bool dump_partials)
{
    const int stages = a.K / 128;
    auto tiles = [&](int tm, int tn) { return (long)ceil_div(a.M, tm) * ceil_div(a.N, tn); };
    W4Choice best = {W4_256, 1, 0, 3.0 + w4_passes(tiles(256, 256), 7.0, 2.02, stages)};
    auto offer = [&](int shape, int first, double us, double ahead) {
        if (us < best.us * ahead) best = {shape, 1, first, us};
    };
    offer(W4_192, 0, 3.0 + w4_passes(tiles(192, 256), 5.0, 1.60, stages), 0.99);
    offer(W4_128X256, 0, 3.0 + w4_pp_us(tiles(128, 256), stages), 0.99);
    offer(W4_128, 0, 3.0 + w4_128_us(tiles(128, 128), stages), 0.99);
    const int tm = ceil_div(a.M, 256), tn = ceil_div(a.N, 256);
    for (int p = 1; p * 256 / tm < tn && p * 256 >= tm; ++p) {   // (fewer than 256 token tiles: whole columns fit a pass)
        const int first = p * 256 / tm;
        offer(W4_TAIL, first, 3.0 + w4_passes((long)tm * first, 7.0, 2.02, stages) +
                                     w4_passes((long)ceil_div(a.M, 128) * (tn - first), 5.0, 1.10, stages), 0.98);
    }
    if (scratch && !dump_partials) {
        W4Choice split = {W4_SPLIT, 1, 0, 1e30};
        for (int s = 2; s <= 32 && stages / s >= 4; ++s) {
            auto consider = [&](int shape, size_t bytes, double us) {
                if (bytes <= scratch && us < split.us) split = {shape, s, 0, us};
            };
            const size_t b128 = (size_t)s * tiles(128, 128) * 128 * 128 * 4, b256 = pp_split_bytes(a, s);
            consider(W4_SPLIT, b128, 11.0 + w4_128_us(tiles(128, 128) * s, ceil_div(stages, s)) + 0.16e-6 * b128);
            if (tiles(128, 256) * s <= 256) consider(W4_SPLIT256, b256, 8.8 + 0.87 * ceil_div(stages, s) + 0.43e-6 * b256);
        }
        if (split.us < best.us * 0.9) best = split;
    }
    return best;
}

}  // namespace

double prefill_w4_estimate_us(const GemmArgs &a) { return choose_w4(a, a.ws ? a.ws_bytes : 0, a.partials != nullptr).us; }

void prefill_w4_plan(const GemmArgs &a, int *variant, int *tile_tokens, int *tile_channels, int *splits)
{
    const W4Choice c = choose_w4(a, a.ws ? a.ws_bytes : 0, a.partials != nullptr);
    *splits = c.splits;
    *variant = c.shape >= W4_SPLIT ? c.shape + c.splits : c.shape;
    *tile_tokens = c.shape == W4_256 || c.shape == W4_TAIL ? 256 : c.shape == W4_192 ? 192 : 128;
    *tile_channels = c.shape == W4_128 || c.shape == W4_SPLIT ? 128 : 256;
}

int launch_gemm_prefill_w4(const GemmArgs &a, int variant, hipStream_t st)
{
    if (a.M == 0) return QL_OK;
    if (a.acc) return launch_w4<2, 4, 4, 4, 4, EPI_ACC, 1>(a, st);   // the accumulator dump has one shape
    W4Choice c = {W4_128X256, 1, 0, 0.0};
    switch (variant) {
    case 0: case 2: c = choose_w4(a, a.ws ? a.ws_bytes : 0, false); break;
    case 6: case 26: c.shape = W4_256; break;
    case 15: case 35: c.shape = W4_192; break;
    case 4: case 11: case 13: case 19: case 20: case 39: c.shape = W4_128; break;
    case 23: case 43: c = {W4_TAIL, 1, (2 * ceil_div(a.N, 256) + 2) / 3, 0.0}; break;   // two thirds of the channel tiles in front
    default:
        if (variant >= 202 && variant <= 232) c = {W4_SPLIT, variant - 200, 0, 0.0};
        if (variant >= 302 && variant <= 332 && a.ws && pp_split_bytes(a, variant - 300) <= a.ws_bytes) c = {W4_SPLIT256, variant - 300, 0, 0.0};
    }
    if (c.shape == W4_TAIL && c.first_tiles >= ceil_div(a.N, 256)) c.shape = W4_256;
    switch (c.shape) {
    case W4_256: return launch_w4<2, 4, 8, 4, 3, EPI_F16, 1>(a, st);
    case W4_192: return launch_w4<2, 4, 6, 4, 3, EPI_F16, 1>(a, st);
    case W4_128: return launch_w4<2, 4, 4, 2, 3, EPI_F16, 2>(a, st);
    case W4_TAIL: return launch_w4_tail(a, c.first_tiles, st);
    case W4_SPLIT: return launch_w4<2, 4, 4, 2, 3, EPI_PART, 2>(a, st, c.splits);
    case W4_SPLIT256: return launch_w4_pp<true>(a, st, c.splits);
    default: return launch_w4_pp<false>(a, st);
    }
}

}  // namespace ql
