// Prefill GEMM + dequantization epilogue of the W4A8 linear layer for gfx950 (integer accumulation per group of 128 k, one
// fp16 scale per channel and group; Y = XW).
//
// Operands arrive as in the int8 kernel: activations in 32-row x 32-k int8 tiles, weights as nibbles in 1024-byte tile
// pairs (32 rows x 64 k).  A stage is one scale group (128 k).  The matrix instruction is 16x16x64 with the tokens as its first
// operand: a lane ends up with four tokens of ONE channel, so a group's scale is one register per 16 channels.  Two
// instructions cover the group for a 16 x 16 block; their int32 sums are folded into the fp32 accumulators
// (accf += float(sum) * scale) and dropped, so a wavefront holds up to 128 tokens x 64 channels.
//
// What bounds it: issue slots.  Measured on gfx950: a 16x16x64 instruction takes 16 cycles and leaves room for two vector
// operations of ANOTHER wavefront; a wavefront alone issues one vector operation per 4.7 cycles and none of its own while its
// matrix instruction runs.  The fold needs two operations per accumulator and group (four per instruction), so two or more
// wavefronts per SIMD, out of step, are what fills both pipes: workgroups of four wavefronts, two to four of them per
// CU, each with barriers of its own -- one workgroup of eight in step ran the same products at 2.02 us per 256 x 256 x 128, now
// 1.83.  That is 4000 cycles and more (2.16 GHz in a continuous run, 2.3 to 2.4 in single launches, matrix pipes busy 41 to 45 % of the
// cycles, half of that beside vector work); register-only loops with the fold take 3000 (1.50 us, held to 2.0 GHz by power): a third of the
// cycles is neither these two pipes nor power, and has not been taken apart.  Within a wavefront a block's fold is spread between
// the next block's matrix instructions: where a CU has one workgroup only, 64 multiplies + 128 folds take 1.05 instead of 1.40 us.
// Tokens go through LDS (global -> LDS loads, three stages); weights and scales, which no other wavefront of a workgroup wants,
// straight to registers, one or two stages ahead (two: 5 % at one workgroup per CU).
#include "gemm_tiles.h"
#include <algorithm>
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
    int tail_tiles_n, tail_group_m;  // 128 x 128 tiles of the channels behind the first tiles_n tiles
    unsigned x_bytes, w_bytes, s_bytes;
    void *part;              // split-K: partial sums [split][workgroup][wavefront][token block][channel block][64 lanes x 16 B]
    int stages_per_split;    // split-K: part y (blockIdx.y, or the K group of a wavefront) takes stages [y * stages_per_split, ...)
};

// A workgroup: KG groups of WAVES_M x WAVES_N wavefronts of 16 TB tokens x 16 CB channels; the groups take one part of K each.
// WPF: stages that the weights are requested ahead.
template <int WAVES_M, int WAVES_N, int TB, int CB, int WPF, int KG = 1>
struct W4Tile {
    static constexpr int NW = WAVES_M * WAVES_N, THREADS = KG * NW * 64, TM = WAVES_M * TB * 16, TN = WAVES_N * CB * 16, STAGES = 3;
    static constexpr int STAGE_BYTES = TM / 32 * 4096, GROUP_BYTES = STAGES * STAGE_BYTES;
    static constexpr int ROW_BYTES = CB * 32 + 16, PATCH_ROWS = KG == TB ? 16 : 32;
    static constexpr int SUMS = KG == 1 ? 0 : KG * NW * TB * CB * 1024;             // the groups' sums, over the stages
    static constexpr int PATCH = KG * NW * PATCH_ROWS * ROW_BYTES;                  // behind them
    static constexpr int MAIN = KG * GROUP_BYTES > SUMS + PATCH ? KG * GROUP_BYTES : SUMS + PATCH;
    static constexpr int SXI = (TM + THREADS - 1) / THREADS, SBI = (TN + THREADS - 1) / THREADS;
    static constexpr int LDS = MAIN + (SXI + SBI) * THREADS * 4;
};

template <int WAVES_M, int WAVES_N, int TB, int CB, int WPF, int EPI, int KG = 1>
__device__ __forceinline__ void w4_tile(const W4Params &p, int tm, int tn, char *smem)
{
    using T = W4Tile<WAVES_M, WAVES_N, TB, CB, WPF, KG>;
    constexpr int NW = T::NW, TM = T::TM, TN = T::TN, STAGES = T::STAGES, XL = TM / 32 * 4 / NW;   // XL: token loads per wavefront and stage
    static_assert(TB % 2 == 0 && CB % 2 == 0 && TM / 32 * 4 % NW == 0, "whole 32-row blocks, equal shares of the loads");
    static_assert(KG == 1 || ((KG == TB || 2 * KG == TB) && EPI == EPI_F16), "at the end each group takes one or two token blocks");
    float *side_sx = reinterpret_cast<float *>(smem + T::MAIN);
    float *side_b = side_sx + T::SXI * T::THREADS;

    const int lane = threadIdx.x & 63;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6) % NW, group = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6) / NW;
    const int wm = wave / WAVES_N, wn = wave % WAVES_N;

    // epilogue operands: requested in front of the first stages, parked in registers, stored to LDS behind them (loads
    // return in order; range-checked, so no branch).  Each array is padded to whole entries per thread.
    int r_sx[T::SXI];
    short r_b[T::SBI];
    if (EPI == EPI_F16) {
        const __amdgpu_buffer_rsrc_t rx = make_rsrc(p.sx, (unsigned)p.M * 4u);
        const __amdgpu_buffer_rsrc_t rb = make_rsrc(p.bias, p.bias ? (unsigned)p.N * 2u : 0u);
#pragma unroll
        for (int it = 0; it < T::SXI; ++it)
            r_sx[it] = __builtin_amdgcn_raw_buffer_load_b32(rx, (unsigned)(tm * TM + threadIdx.x + it * T::THREADS) * 4u, 0, 0);
#pragma unroll
        for (int it = 0; it < T::SBI; ++it)
            r_b[it] = __builtin_amdgcn_raw_buffer_load_b16(rb, (unsigned)(tn * TN + threadIdx.x + it * T::THREADS) * 2u, 0, 0);
    }

    // This wavefront's stages: own of them from stage0 on; every group of a workgroup makes the same number of steps.
    const int all = p.K / 128, stage0 = EPI == EPI_PART ? blockIdx.y * p.stages_per_split : KG > 1 ? group * p.stages_per_split : 0;
    const int own = min(p.stages_per_split, all - stage0), steps = KG > 1 ? p.stages_per_split : own;
    const unsigned KB = p.K / 32;
    const int ch = lane >> 4, r = lane & 15;
    char *ring = smem + group * T::GROUP_BYTES;
    // Range checking: row-blocks beyond ceil32(M) / ceil32(N) return nothing (their offset alone is behind the buffer); stages behind
    // the last one are requested as the last one again, into buffers that nobody reads.  Token fragment f of a
    // stage (row-block f / 4, k-block f % 4) is loaded by wavefront f % NW.
    unsigned xoff[XL], woff[CB / 2];
#pragma unroll
    for (int i = 0; i < XL; ++i) {
        const int f = i * NW + wave;
        xoff[i] = lane * 16 + ((unsigned)(tm * (TM / 32) + f / 4) * KB + f % 4) * 1024u;
    }
#pragma unroll
    for (int i = 0; i < CB / 2; ++i)
        woff[i] = ((unsigned)(tn * (TN / 32) + wn * (CB / 2) + i) * (KB / 2) + ch / 2) * 1024u + (r + 32 * (ch % 2)) * 16;
    const unsigned soff = (unsigned)(tn * TN + wn * CB * 16 + r) * 2u;
    auto issue_tokens = [&](int s) {
        const int k = min(stage0 + s, all - 1);
        const __amdgpu_buffer_rsrc_t xr = make_rsrc(p.xq, p.x_bytes);
        char *buf = ring + (s % STAGES) * T::STAGE_BYTES + wave * 1024;
#pragma unroll
        for (int i = 0; i < XL; ++i) {
            const unsigned off = xoff[i];
            __builtin_amdgcn_raw_ptr_buffer_load_lds(xr, LDS_PTR(buf + i * NW * 1024), 16, off, k * 4096, 0, 0);
        }
    };
    v4i wp[WPF][CB];         // packed weights, 128 k of 16 channels each, and their scales: lane (r, ch) has 16 bytes of channel r
    short sn[WPF][CB];
    auto issue_weights = [&](int s, v4i (&w)[CB], short (&sc)[CB]) {
        const int k = min(stage0 + s, all - 1);
        const __amdgpu_buffer_rsrc_t wr = make_rsrc(p.wq, p.w_bytes), sr = make_rsrc(p.wscales, p.s_bytes);
#pragma unroll
        for (int i = 0; i < CB; ++i) {
            const unsigned off = woff[i / 2] + (i % 2) * 256;
            w[i] = __builtin_bit_cast(v4i, __builtin_amdgcn_raw_buffer_load_b128(wr, off, k * 2048, 0));
        }
#pragma unroll
        for (int i = 0; i < CB; ++i) {
            const unsigned off = soff + i * 32;
            if constexpr (EPI == EPI_ACC) sc[i] = 0;
            else sc[i] = __builtin_amdgcn_raw_buffer_load_b16(sr, off, k * p.Npad * 2, 0);
        }
    };

    float accf[EPI == EPI_ACC ? 1 : CB][EPI == EPI_ACC ? 1 : TB][4];
    int tot[EPI == EPI_ACC ? CB : 1][EPI == EPI_ACC ? TB : 1][4];
#pragma unroll
    for (int i = 0; i < CB; ++i)
#pragma unroll
        for (int j = 0; j < TB; ++j)
#pragma unroll
            for (int e = 0; e < 4; ++e) {
                if constexpr (EPI == EPI_ACC) tot[i][j][e] = 0;
                else accf[i][j][e] = 0.0f;
            }

    issue_tokens(0);
    issue_tokens(1);
#pragma unroll
    for (int s = 0; s < WPF; ++s) issue_weights(s, wp[s], sn[s]);
    issue_tokens(2);
    if (EPI == EPI_F16) {
#pragma unroll
        for (int it = 0; it < T::SXI; ++it) side_sx[threadIdx.x + it * T::THREADS] = __int_as_float(r_sx[it]);
#pragma unroll
        for (int it = 0; it < T::SBI; ++it)
            side_b[threadIdx.x + it * T::THREADS] = __half2float(__ushort_as_half((unsigned short)r_b[it]));
    }

    const int xlane = wm * (TB / 2) * 4096 + (ch / 2) * 2048 + (r + 32 * (ch % 2)) * 16;
    v4i xf[2][2];
    auto read_tokens = [&](int s, int j) {
        const char *buf = ring + (s % STAGES) * T::STAGE_BYTES + xlane;
#pragma unroll
        for (int t = 0; t < 2; ++t)
            xf[j & 1][t] = *reinterpret_cast<const v4i *>(buf + (j / 2) * 4096 + (j % 2) * 256 + t * 1024);
    };
    v4i q[2][CB];            // a block's sums while the next one is multiplied
    float sg[CB], so[CB];    // scales of the stage; of the one before, to which the last block's sums belong
#pragma unroll
    for (int i = 0; i < CB; ++i) q[0][i] = q[1][i] = v4i{0, 0, 0, 0}, sg[i] = 0.0f;
    auto fold = [&](int g, int j, int from, int to) {   // values [from, to) of token block j, group g of this wavefront's
#pragma unroll
        for (int n = from; n < to; ++n) {
            const int i = n / 4, e = n % 4;
            if constexpr (EPI != EPI_ACC) {
                accf[i][j][e] = __builtin_fmaf((float)q[j & 1][i][e], j == TB - 1 ? so[i] : sg[i], accf[i][j][e]);
            } else {
                tot[i][j][e] += q[j & 1][i][e];
                if (p.partials && g >= 0) {
                    const int m = tm * TM + (wm * TB + j) * 16 + 4 * ch + e, nn = tn * TN + (wn * CB + i) * 16 + r;
                    if (m >= p.row0 && m < p.row0 + p.nrows && m < p.M && nn < p.N)
                        p.partials[((size_t)(m - p.row0) * (p.K / 128) + g) * p.N + nn] = q[j & 1][i][e] >> 4;
                }
            }
        }
    };

    // Main loop, one barrier per stage.  Token fragments are read one block ahead; in front of the last block's products the
    // wavefront hands its stage over (own reads done; its share of the next stage had landed before it unpacked this one;
    // barrier: then everyone's has) and refills the freed buffer.
    // Loads issued behind a stage's weights: the tokens of one stage, the weights and scales of WPF - 1 (the accumulator dump uses no
    // scales, and the compiler leaves their loads out: counting them let a stage be handed over before its tokens were there)
    constexpr int NEWER = XL + (WPF - 1) * (EPI == EPI_ACC ? 1 : 2) * CB;
    auto stage = [&](int it, v4i (&w)[CB], short (&sc)[CB]) {
        wait_vmcnt<NEWER>();
        v4i wf[CB][2];
#pragma unroll
        for (int i = 0; i < CB; ++i) {
#pragma unroll
            for (int t = 0; t < 2; ++t) {
                const unsigned w0 = (unsigned)w[i][2 * t], w1 = (unsigned)w[i][2 * t + 1];
                wf[i][t][0] = (int)((w0 << 4) & 0xF0F0F0F0u);
                wf[i][t][1] = (int)(w0 & 0xF0F0F0F0u);
                wf[i][t][2] = (int)((w1 << 4) & 0xF0F0F0F0u);
                wf[i][t][3] = (int)(w1 & 0xF0F0F0F0u);
            }
            so[i] = sg[i];
            sg[i] = __half2float(__ushort_as_half((unsigned short)sc[i]));
            if (KG > 1 && it >= own) sg[i] = 0.0f;      // a group that has fewer stages than the others
            asm("" : "+v"(sg[i]));                       // converted here, not in every multiply-add (those at half the rate)
        }
        __builtin_amdgcn_sched_barrier(0);
        issue_weights(it + WPF, w, sc);
        __builtin_amdgcn_sched_barrier(0);
#pragma unroll
        for (int j = 0; j < TB; ++j) {
            if (j + 1 < TB) {
                read_tokens(it, j + 1);
            } else {
                __builtin_amdgcn_s_waitcnt(0xC07F);      // lgkmcnt(0)
                __builtin_amdgcn_s_barrier();
                issue_tokens(it + STAGES);
                read_tokens(it + 1, 0);
            }
            __builtin_amdgcn_sched_barrier(0);
            const int c = j & 1, pj = (j + TB - 1) % TB, g = j == 0 ? it - 1 : it;
#pragma unroll
            for (int n = 0; n < 2 * CB; ++n) {
                const int i = n % CB, t = n / CB;
                q[c][i] = __builtin_amdgcn_mfma_i32_16x16x64_i8(xf[c][t], wf[i][t], t == 0 ? v4i{0, 0, 0, 0} : q[c][i], 0, 0, 0);
                __builtin_amdgcn_sched_barrier(0);
                fold(g, pj, n, n + 1);
                __builtin_amdgcn_sched_barrier(0);
            }
            fold(g, pj, 2 * CB, 4 * CB);
            __builtin_amdgcn_sched_barrier(0);
        }
    };
    wait_vmcnt<NEWER>();
    __builtin_amdgcn_s_barrier();
    read_tokens(0, 0);
    if constexpr (WPF == 1) {
        for (int it = 0; it < steps; ++it) stage(it, wp[0], sn[0]);
    } else {
        int it = 0;
        for (; it + 1 < steps; it += 2) {
            stage(it, wp[0], sn[0]);
            stage(it + 1, wp[1], sn[1]);
        }
        if (it < steps) stage(it, wp[0], sn[0]);
    }
#pragma unroll
    for (int i = 0; i < CB; ++i) so[i] = sg[i];
    fold(steps - 1, TB - 1, 0, 4 * CB);
    wait_vmcnt<0>();   // drain the loads behind the last stage before the LDS is released

    if constexpr (EPI == EPI_PART) {
        char *dst = static_cast<char *>(p.part) + (((size_t)blockIdx.y * gridDim.x + blockIdx.x) * NW + wave) * (size_t)(CB * TB * 1024);
#pragma unroll
        for (int j = 0; j < TB; ++j)
#pragma unroll
            for (int i = 0; i < CB; ++i)
                *reinterpret_cast<float4 *>(dst + (j * CB + i) * 1024 + lane * 16) =
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
                    const int m = tm * TM + (wm * TB + j) * 16 + 4 * ch + e, n = tn * TN + (wn * CB + i) * 16 + r;
                    if (m < p.M && n < p.N) p.acc[(size_t)m * p.ldacc + n] = tot[i][j][e] >> 4;
                }
        return;
    }

    __syncthreads();
    char *stg = smem + T::SUMS + (group * NW + wave) * (T::PATCH_ROWS * T::ROW_BYTES);
    const int n_wave0 = tn * TN + wn * CB * 16;
    const bool odd = lane & 1;
    char *at = stg + (4 * ch + (odd ? 2 : 0)) * T::ROW_BYTES + (r & ~1) * 2;
    float b_r[CB];
#pragma unroll
    for (int i = 0; i < CB; ++i) b_r[i] = side_b[(wn * CB + i) * 16 + r];
    auto to_patch = [&](char *dst, float4 s4, const float (&a)[4], float b) {
        const float sx4[4] = {s4.x * 0.0625f, s4.y * 0.0625f, s4.z * 0.0625f, s4.w * 0.0625f};
        float v[4];
#pragma unroll
        for (int e = 0; e < 4; ++e) {
            v[e] = __builtin_fmaf(a[e], sx4[e], b);
            asm("" : "+v"(v[e]));   // rounded to fp32, then to fp16, in every kernel variant
        }
        patch_quad(dst, T::ROW_BYTES, odd, v);
    };
    if constexpr (KG > 1) {         // the groups' sums meet in LDS; each group adds up its share of the token blocks, first part first
        constexpr int BLOCKS = TB / KG;
#pragma unroll
        for (int j = 0; j < TB; ++j)
#pragma unroll
            for (int i = 0; i < CB; ++i)
                *reinterpret_cast<float4 *>(smem + (((group * NW + wave) * TB + j) * CB + i) * 1024 + lane * 16) =
                    float4{accf[i][j][0], accf[i][j][1], accf[i][j][2], accf[i][j][3]};
        __syncthreads();
#pragma unroll
        for (int b = 0; b < BLOCKS; ++b) {
            const int j = group * BLOCKS + b;
            const float4 s4 = *reinterpret_cast<const float4 *>(side_sx + (wm * TB + j) * 16 + 4 * ch);
#pragma unroll
            for (int i = 0; i < CB; ++i) {
                float a[4] = {0, 0, 0, 0};
#pragma unroll
                for (int g = 0; g < KG; ++g) {
                    const float4 u = *reinterpret_cast<const float4 *>(smem + (((g * NW + wave) * TB + j) * CB + i) * 1024 + lane * 16);
                    if (g == 0) a[0] = u.x, a[1] = u.y, a[2] = u.z, a[3] = u.w;
                    else a[0] += u.x, a[1] += u.y, a[2] += u.z, a[3] += u.w;
                }
                to_patch(at + b * 16 * T::ROW_BYTES + i * 32, s4, a, b_r[i]);
            }
        }
        store_rows<CB * 2, T::PATCH_ROWS>(p.y, p.ldy, p.M, p.N, stg, T::ROW_BYTES, tm * TM + (wm * TB + group * BLOCKS) * 16, n_wave0, lane);
    } else {
#pragma unroll
        for (int jb = 0; jb < TB / 2; ++jb) {
#pragma unroll
            for (int jj = 0; jj < 2; ++jj) {
                const float4 s4 = *reinterpret_cast<const float4 *>(side_sx + (wm * TB + 2 * jb + jj) * 16 + 4 * ch);
#pragma unroll
                for (int i = 0; i < CB; ++i) to_patch(at + jj * 16 * T::ROW_BYTES + i * 32, s4, accf[i][2 * jb + jj], b_r[i]);
            }
            store_rows<CB * 2, 32>(p.y, p.ldy, p.M, p.N, stg, T::ROW_BYTES, tm * TM + (wm * TB + 2 * jb) * 16, n_wave0, lane);
        }
    }
}

// WPS: wavefronts per SIMD that the registers must leave room for
template <int WAVES_M, int WAVES_N, int TB, int CB, int WPF, int EPI, int KG, int WPS>
__global__ __launch_bounds__(WAVES_M *WAVES_N *KG * 64, WPS) void gemm_w4_kernel(W4Params p)
{
    extern __shared__ __attribute__((aligned(1024))) char smem[];
    int tm, tn;
    tile_coords(blockIdx.x, p.tiles_m, p.tiles_n, p.group_m, tm, tn);
    w4_tile<WAVES_M, WAVES_N, TB, CB, WPF, EPI, KG>(p, tm, tn, smem);
}

// 128 x 256 tiles for the first tiles_n channel tiles (whole passes over the CUs, two tiles each), 128 x 128 for the rest: the last
// pass is spread more evenly.
__global__ __launch_bounds__(256, 2) void gemm_w4_tail_kernel(W4Params p)
{
    extern __shared__ __attribute__((aligned(1024))) char smem[];
    int tm, tn;
    const int first = p.tiles_m * p.tiles_n;
    if ((int)blockIdx.x < first) {
        tile_coords(blockIdx.x, p.tiles_m, p.tiles_n, p.group_m, tm, tn);
        w4_tile<1, 4, 8, 4, 1, EPI_F16>(p, tm, tn, smem);
    } else {
        tile_coords(blockIdx.x - first, p.tiles_m, p.tail_tiles_n, p.tail_group_m, tm, tn);
        w4_tile<1, 4, 8, 2, 2, EPI_F16>(p, tm, 2 * p.tiles_n + tn, smem);
    }
}

// Split-K over workgroups, second kernel: adds the splits' fp32 partial sums, split 0 first, then the dequantization of the fused
// epilogue.  A wavefront takes 32 tokens x 16 CB channels; the loads of four splits are issued before the first is used.
template <int WAVES_M, int WAVES_N, int TB, int CB>
__global__ __launch_bounds__(256) void w4_finish_kernel(W4Params p, int splits)
{
    constexpr int NW = WAVES_M * WAVES_N, JB = TB / 2, ROW_BYTES = CB * 32 + 16, BLOCKS = 2 * CB, AHEAD = 4;
    __shared__ __attribute__((aligned(16))) char patch[4 * 32 * ROW_BYTES];
    const int lane = threadIdx.x & 63, w4 = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int unit = blockIdx.x * 4 + w4;
    const int tile = unit / (NW * JB), wave = unit / JB % NW, jb = unit % JB;
    if (tile >= p.tiles_m * p.tiles_n) return;
    int tm, tn;
    tile_coords(tile, p.tiles_m, p.tiles_n, p.group_m, tm, tn);
    const int wm = wave / WAVES_N, wn = wave % WAVES_N, ch = lane >> 4, r = lane & 15;
    const int m0 = ((tm * WAVES_M + wm) * TB + 2 * jb) * 16, n0 = (tn * WAVES_N + wn) * CB * 16;
    if (m0 >= p.M || n0 >= p.N) return;
    const size_t stride = (size_t)p.tiles_m * p.tiles_n * NW * TB * CB * 256;
    const float *src = static_cast<const float *>(p.part) + ((size_t)(tile * NW + wave) * TB + 2 * jb) * CB * 256 + lane * 4;
    float4 v[BLOCKS];
    for (int s0 = 0; s0 < splits; s0 += AHEAD) {
        float4 u[AHEAD][BLOCKS];
#pragma unroll
        for (int a = 0; a < AHEAD; ++a)
            if (s0 + a < splits)
#pragma unroll
                for (int b = 0; b < BLOCKS; ++b) u[a][b] = *reinterpret_cast<const float4 *>(src + (s0 + a) * stride + b * 256);
#pragma unroll
        for (int a = 0; a < AHEAD; ++a)
            if (s0 + a < splits)
#pragma unroll
                for (int b = 0; b < BLOCKS; ++b) {
                    if (s0 + a == 0) v[b] = u[a][b];
                    else v[b].x += u[a][b].x, v[b].y += u[a][b].y, v[b].z += u[a][b].z, v[b].w += u[a][b].w;
                }
    }
    char *stg = patch + w4 * 32 * ROW_BYTES;
    const bool odd = lane & 1;
    char *at = stg + (4 * ch + (odd ? 2 : 0)) * ROW_BYTES + (r & ~1) * 2;
#pragma unroll
    for (int b = 0; b < BLOCKS; ++b) {
        const int jj = b / CB, i = b % CB, n = n0 + i * 16 + r;
        const float bias = p.bias && n < p.N ? __half2float(p.bias[n]) : 0.0f;
        const float a4[4] = {v[b].x, v[b].y, v[b].z, v[b].w};
        float o[4];
#pragma unroll
        for (int e = 0; e < 4; ++e) {
            const int m = m0 + jj * 16 + 4 * ch + e;
            o[e] = __builtin_fmaf(a4[e], (m < p.M ? p.sx[m] : 0.0f) * 0.0625f, bias);
            asm("" : "+v"(o[e]));   // rounded to fp32, then to fp16, as in the fused epilogue
        }
        patch_quad(at + jj * 16 * ROW_BYTES + i * 32, ROW_BYTES, odd, o);
    }
    store_rows<CB * 2, 32>(p.y, p.ldy, p.M, p.N, stg, ROW_BYTES, m0, n0, lane);
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

// scratch of a K range split over workgroups, for tiles of tm x tn
inline size_t split_bytes(const GemmArgs &a, int tm, int tn, int splits)
{
    return (size_t)splits * ceil_div(a.M, tm) * ceil_div(a.N, tn) * tm * tn * 4;
}

// once per kernel and process
template <typename F>
int set_lds(F kern, int bytes)
{
    return check_hip(hipFuncSetAttribute(reinterpret_cast<const void *>(kern), hipFuncAttributeMaxDynamicSharedMemorySize, bytes),
                     "hipFuncSetAttribute(max dynamic LDS)");
}

// OCC: workgroups per CU
template <int WAVES_M, int WAVES_N, int TB, int CB, int WPF, int EPI, int OCC, int KG = 1>
int launch_w4(const GemmArgs &a, hipStream_t st, int splits = 1)
{
    using T = W4Tile<WAVES_M, WAVES_N, TB, CB, WPF, KG>;
    static_assert(T::LDS * OCC <= 160 * 1024, "LDS budget");
    auto kern = gemm_w4_kernel<WAVES_M, WAVES_N, TB, CB, WPF, EPI, KG, OCC * T::NW * KG / 4>;
    static const int attr_status = set_lds(kern, T::LDS);   // the initialisation of a function-local static is thread-safe
    if (attr_status != QL_OK) return attr_status;
    W4Params p = w4_params(a);
    p.tiles_m = ceil_div(a.M, T::TM);
    p.tiles_n = ceil_div(a.N, T::TN);
    // (an activation row costs twice the bytes of a weight row)
    p.group_m = strip_height(p.tiles_m, p.tiles_n, T::TM * 2, T::TN, OCC);
    p.stages_per_split = ceil_div(a.K / 128, KG > 1 ? KG : splits);
    splits = ceil_div(a.K / 128, p.stages_per_split);   // no empty split
    if (EPI == EPI_PART) {
        const size_t need = split_bytes(a, T::TM, T::TN, splits);
        if (!a.ws || need > a.ws_bytes) return fail(QL_ERR_WORKSPACE, "split-K needs %zu bytes of workspace", need);
    }
    p.part = a.ws;
    hipLaunchKernelGGL(kern, dim3(p.tiles_m * p.tiles_n, EPI == EPI_PART ? splits : 1), dim3(T::THREADS), T::LDS, st, p);
    QL_TRY(check_hip(hipGetLastError(), "gemm_w4 launch"));
    if constexpr (EPI == EPI_PART) {
        hipLaunchKernelGGL((w4_finish_kernel<WAVES_M, WAVES_N, TB, CB>), dim3(ceil_div(p.tiles_m * p.tiles_n * T::NW * (TB / 2), 4)), dim3(256),
                           0, st, p, splits);
        return check_hip(hipGetLastError(), "w4_finish launch");
    }
    return QL_OK;
}

// the first `first_tiles` channel tiles in 128 x 256 tiles, the rest in 128 x 128 (0 < first_tiles < all of them)
int launch_w4_tail(const GemmArgs &a, int first_tiles, hipStream_t st)
{
    using Big = W4Tile<1, 4, 8, 4, 1>;
    using Small = W4Tile<1, 4, 8, 2, 2>;
    constexpr int LDS = Big::LDS > Small::LDS ? Big::LDS : Small::LDS;
    static_assert(2 * LDS <= 160 * 1024 && Big::TN == 2 * Small::TN && Big::TM == Small::TM && Big::THREADS == Small::THREADS, "one launch");
    static const int attr_status = set_lds(gemm_w4_tail_kernel, LDS);
    if (attr_status != QL_OK) return attr_status;
    W4Params p = w4_params(a);
    p.tiles_m = ceil_div(a.M, Big::TM);
    p.tiles_n = first_tiles;
    p.group_m = strip_height(p.tiles_m, p.tiles_n, Big::TM * 2, Big::TN, 2);
    p.tail_tiles_n = ceil_div(a.N, Small::TN) - 2 * first_tiles;
    p.tail_group_m = strip_height(p.tiles_m, p.tail_tiles_n, Small::TM * 2, Small::TN, 2);
    hipLaunchKernelGGL(gemm_w4_tail_kernel, dim3(p.tiles_m * (p.tiles_n + p.tail_tiles_n)), dim3(Big::THREADS), LDS, st, p);
    return check_hip(hipGetLastError(), "gemm_w4_tail launch");
}

// The automatic choice.  Estimated time of a tile form: 3 us + the packed weights at 20 TB/s + what the busiest CU does, in rounds of as many workgroups as fit it
// together; a round of n takes o[n - 1] + stages x c[n - 1].  Fitted to 173 shapes (40..8192 tokens, N 1536..22016, K 1536..11008;
// weights from HBM), within 2.5 to 5 % on average each; the pick is within 0.3 % of the fastest form on average, 5 % at worst.
// (TOP/s of a CU full of them: 128 x 256 9.2, 96 x 256 9.1, 128 x 128 8.3, 96 x 128 7.9, 64 x 128 7.4: large tiles where there
// are many, small ones where the larger would leave CUs or a last round empty.  1024 x 4096 x 4096: 128 x 256
// 44 us, 96 x 256 35, 128 x 256 by eight wavefronts 34, 128 x 128 28, 64 x 128 25; 4096 x 4096 x 22016: 370, 404, 419, 384, 424.)
// One 128 x 256 tile per CU by eight wavefronts (1 x 8 of 128 x 32): one round only, 2048 x 4096 x 4096 39.9 us, the others 42.6..54.
// Combined form: whole passes of 128 x 256 (512 tiles), possibly half a one, the remaining channels in 128 x 128 tiles, two
// per CU: 2048 x 4096 x 22016 183.6 us, 128 x 256 alone 197, 128 x 128 alone 192; 3500 tokens 325 / 329 / 332.
// K in parts (only where the scratch offered holds the partial sums, which is how a caller allows them to be taken in parts):
//   over two or four groups of four wavefronts of one workgroup, 64 x 128 tiles, where these fit one pass: the sums meet in LDS,
//   the scratch is not touched.  512 x 11008 x 4096 32.1 us (four; two 34.9; 64 x 128 unsplit 49.5, split over
//   workgroups 41.5), 1280 x 6144 x 1536 18.7 / 19.2 / 24.7 / 28.8, 512 x 4096 x 4096 15.1 / 15.4 / 18.8 / 24.4.  Not up to 64 tokens,
//   which the weight-streaming kernels take in one block (4096 channels 6.9 us, here 13.3);
//   over workgroups, partial sums in the scratch and a second kernel, 3 us + 0.27 us per MB: few tiles that do not fit one pass
//   of 64 x 128 (1536 x 6144 x 1536, three parts: 32.3 us; 96 x 128 unsplit 32.2, 64 x 128 33.3, both groups 35).
enum W4Shape { W4_128X256 = 26, W4_96X256 = 35, W4_ONE = 37, W4_128X128 = 4, W4_64X128 = 13, W4_96X128 = 19, W4_TAIL = 43,
               W4_SPLIT = 200, W4_GROUPS2 = 202, W4_SPLIT256 = 300, W4_GROUPS4 = 304 };   // ql_set_kernel_variant values

struct W4Form {
    int shape, tm, tn, per_cu;
    double o[4], c[4];
};
constexpr W4Form W4_FORMS[] = {
    {W4_128X256, 128, 256, 2, {3.0, 7.0}, {1.17, 1.83}},
    {W4_96X256, 96, 256, 2, {2.4, 5.5}, {0.92, 1.39}},
    {W4_ONE, 128, 256, 1, {2.3}, {0.93}},
    {W4_128X128, 128, 128, 3, {1.6, 3.7, 4.6}, {0.69, 1.00, 1.52}},
    {W4_64X128, 64, 128, 4, {0.0, 1.2, 2.5, 2.9}, {0.50, 0.65, 0.89, 1.14}},
    {W4_96X128, 96, 128, 3, {1.3, 2.4, 3.0}, {0.60, 0.83, 1.19}},
};

// rounds of `tiles` workgroups of a form, at most per_cu of them together on a CU
inline double w4_rounds_us(const W4Form &f, long tiles, int stages, int per_cu)
{
    auto round = [&](int n) { return f.o[n - 1] + f.c[n - 1] * stages; };
    const long busiest = (tiles + 255) / 256;
    return (double)(busiest / per_cu) * round(per_cu) + (busiest % per_cu ? round((int)(busiest % per_cu)) : 0.0);
}

struct W4Choice {
    int shape, splits, first_tiles;
    double us;
};

// What a caller has to offer before K is taken in two or four parts: the bytes of the split over workgroups that the value stands for
// (the groups touch none of it).  One rule for the automatic choice and for the values asked for.
inline size_t groups_scratch(const GemmArgs &a, int groups) { return split_bytes(a, 128, groups == 2 ? 128 : 256, groups); }

inline W4Choice choose_w4(const GemmArgs &a, size_t scratch)
{
    const int stages = a.K / 128;
    auto tiles = [&](int tm, int tn) { return (long)ceil_div(a.M, tm) * ceil_div(a.N, tn); };
    W4Choice best = {0, 1, 0, 1e30};
    auto offer = [&](int shape, int splits, int first, double us) {
        if (us < best.us) best = {shape, splits, first, us};
    };
    const double base = 3.0 + 0.5 * a.N * a.K / 20e6;
    const W4Form &big = W4_FORMS[0], &one = W4_FORMS[2], &mid = W4_FORMS[3];
    for (const W4Form &f : W4_FORMS) {
        const long t = tiles(f.tm, f.tn);
        if (f.shape != W4_ONE || t <= 256) offer(f.shape, 1, 0, base + w4_rounds_us(f, t, stages, f.per_cu));
    }
    const int tm = ceil_div(a.M, 128), tn = ceil_div(a.N, 256);
    for (int half = 1; half * 256 / tm < tn; ++half) {   // `half` half passes (whole columns of tiles: a little less)
        const int first = half * 256 / tm;
        const long rest = (long)tm * (ceil_div(a.N, 128) - 2 * first);
        if (first == 0 || (half % 2 && rest > 256)) continue;
        double us = base + half / 2 * (big.o[1] + big.c[1] * stages);
        if (half % 2) us += 0.75 * (big.o[0] + big.c[0] * stages) + 0.25 * (big.o[1] + big.c[1] * stages);   // beside the small tiles
        else us += w4_rounds_us(mid, rest, stages, 2);
        if (us < 0.99 * best.us) offer(W4_TAIL, 1, first, us);
    }
    if (!scratch) return best;
    if (a.M > 64 && tiles(64, 128) <= 256) {
        if (scratch >= groups_scratch(a, 2)) offer(W4_GROUPS2, 2, 0, base + 0.6 + 0.66 * ceil_div(stages, 2));
        if (scratch >= groups_scratch(a, 4)) offer(W4_GROUPS4, 4, 0, base + 2.1 + 1.22 * ceil_div(stages, 4));
    }
    for (int s = 2; s <= 32 && stages / s >= 4; ++s)
        for (const W4Form *f : {&mid, &one}) {
            const long t = tiles(f->tm, f->tn) * s;
            const size_t bytes = split_bytes(a, f->tm, f->tn, s);
            if (bytes > scratch || (f == &one && t > 256) || (f == &mid && s == 2) || (f == &one && s == 4)) continue;   // (2 and 4: the groups' values)
            const double us = base + 3.0 + w4_rounds_us(*f, t, ceil_div(stages, s), f->per_cu) + 0.27e-6 * bytes;
            if (us < 0.95 * best.us) offer((f == &mid ? W4_SPLIT : W4_SPLIT256) + s, s, 0, us);
        }
    return best;
}

}  // namespace

double prefill_w4_estimate_us(const GemmArgs &a) { return choose_w4(a, a.ws ? a.ws_bytes : 0).us; }

void prefill_w4_plan(const GemmArgs &a, int *variant, int *tile_tokens, int *tile_channels, int *splits)
{
    const W4Choice c = choose_w4(a, a.ws ? a.ws_bytes : 0);
    *splits = c.splits;
    *variant = c.shape;
    const bool groups = c.shape == W4_GROUPS2 || c.shape == W4_GROUPS4;
    *tile_tokens = groups ? 64 : 128, *tile_channels = !groups && (c.shape > W4_SPLIT256 || c.shape == W4_TAIL) ? 256 : 128;
    for (const W4Form &f : W4_FORMS)
        if (f.shape == c.shape) *tile_tokens = f.tm, *tile_channels = f.tn;
}

int launch_gemm_prefill_w4(const GemmArgs &a, int variant, hipStream_t st)
{
    if (a.M == 0) return QL_OK;
    if (a.acc) return launch_w4<1, 4, 4, 2, 2, EPI_ACC, 1>(a, st);   // the accumulator dump has one shape
    const size_t scratch = a.ws ? a.ws_bytes : 0;
    W4Choice c = {W4_ONE, 1, 0, 0.0};
    switch (variant) {
    case 0: case 2: c = choose_w4(a, scratch); break;
    case 6: case 26: c.shape = W4_128X256; break;
    case 15: case 35: c.shape = W4_96X256; break;
    case 4: case 11: c.shape = W4_128X128; break;
    case 13: c.shape = W4_64X128; break;
    case 19: case 20: case 39: c.shape = W4_96X128; break;
    case 23: case 43: c = {W4_TAIL, 1, (2 * ceil_div(a.N, 256) + 2) / 3, 0.0}; break;   // two thirds of the channel tiles in front
    default:
        if (variant >= 202 && variant <= 232) c = {variant, variant - W4_SPLIT, 0, 0.0};
        if (variant >= 302 && variant <= 332 && split_bytes(a, 128, 256, variant - W4_SPLIT256) <= scratch)   // (304: groups_scratch)
            c = {variant, variant - W4_SPLIT256, 0, 0.0};
    }
    if (c.shape == W4_TAIL && c.first_tiles >= ceil_div(a.N, 256)) c.shape = W4_128X256;
    switch (c.shape) {
    case W4_128X256: return launch_w4<1, 4, 8, 4, 1, EPI_F16, 2>(a, st);
    case W4_96X256: return launch_w4<1, 4, 6, 4, 2, EPI_F16, 2>(a, st);
    case W4_ONE: return launch_w4<1, 8, 8, 2, 2, EPI_F16, 1>(a, st);
    case W4_128X128: return launch_w4<1, 4, 8, 2, 2, EPI_F16, 3>(a, st);
    case W4_64X128: return launch_w4<1, 4, 4, 2, 2, EPI_F16, 4>(a, st);
    case W4_96X128: return launch_w4<1, 4, 6, 2, 2, EPI_F16, 3>(a, st);
    case W4_TAIL: return launch_w4_tail(a, c.first_tiles, st);
    case W4_GROUPS2:
        if (scratch < groups_scratch(a, 2))   // asked for by value: refused as the other values are
            return fail(QL_ERR_WORKSPACE, "split-K needs %zu bytes of workspace", groups_scratch(a, 2));
        return launch_w4<1, 4, 4, 2, 2, EPI_F16, 1, 2>(a, st);
    case W4_GROUPS4: return launch_w4<1, 4, 4, 2, 2, EPI_F16, 1, 4>(a, st);
    default:
        if (c.shape < W4_SPLIT256) return launch_w4<1, 4, 8, 2, 2, EPI_PART, 3>(a, st, c.splits);
        return launch_w4<1, 8, 8, 2, 2, EPI_PART, 1>(a, st, c.splits);
    }
}

}  // namespace ql
