// Prefill GEMM + dequantization epilogue of the W8A8 linear layer for gfx950, for shapes that the large tiles of gemm_prefill.hip
// fill badly: workgroups of four wavefronts (1 x 4, each 16 TB tokens x 16 CB channels), two to four of them per CU, each with
// barriers of its own, or two groups of four that take half of K each where 64 or 96 x 128 tiles fit one pass (their int32 sums meet in LDS).
//
// A stage is 128 k.  Tokens go through LDS (global -> LDS loads, three stages); weights, which no other wavefront of the
// workgroup wants, straight to registers, one or two stages ahead of the multiply.  The matrix instruction is 16x16x64 with the tokens as its
// first operand, so a lane ends up with four tokens of one channel.
//
// What bounds it: what a CU can pull when the weights come from HBM, whatever the number of groups or of stages ahead: 45..57 GB/s over
// whole launches, 49..64 in the fastest, so about 70 in the loop (96 channels and fewer; 128 x 256 and 96 x 256 less).  So the tile is chosen by
// the bytes per product and by how evenly the tiles fill the CUs.  Calls that take them, us before and now (tokens x K x N, weights from
// HBM): 260 x 4096 x 12288 31.8 / 25.5, 512 x 4096 x 4096 18.8 / 15.3, 640 x 11008 x 4096 48.2 / 39.0, 900 x 4096 x 6144 34.3 / 29.1, 768 x
// 8192 x 8192 65.5 / 51.8; 492 shapes of 65 tokens and more where a form is the choice 1.23 times on average, 2 % slower at worst.
// Above 1024 tokens nearly none: the other kernels are estimated there by rates of warm weights, too low by up to a quarter, and forms that
// would be ahead are passed over (1300 x 11008 x 4096: taken 84, form 56 65; 1900 x 6144 x 1536: taken 23.3, form 53 21.4).
// Not faster with the weights' or tokens' loads non-temporal, or with every channel tile starting at another k.
#include "gemm_tiles.h"
#include <algorithm>
#include <type_traits>

namespace ql {
namespace {

struct W8Params {
    const int8_t *xq;
    const void *wq;
    const float *sx, *sw;
    const __half *bias;
    __half *y;
    int64_t ldy;
    int32_t *acc;
    int64_t ldacc;
    int M, N, K;
    int tiles_m, tiles_n, group_m;
    int stages_per_group;
    unsigned x_bytes, w_bytes;
};

// A workgroup: KG groups of four wavefronts, one part of K each.  WPF: stages that the weights are requested ahead.
template <int TB, int CB, int WPF, int KG>
struct W8Tile {
    static constexpr int NW = 4, THREADS = KG * NW * 64, TM = TB * 16, TN = NW * CB * 16, STAGES = 3;
    static constexpr int STAGE_BYTES = TM / 32 * 4096, GROUP_BYTES = STAGES * STAGE_BYTES;
    static constexpr int ROW_BYTES = CB * 32 + 16;
    static constexpr int SUMS = KG == 1 ? 0 : KG * NW * TB * CB * 1024;
    static constexpr int PATCH = KG * NW * 16 * ROW_BYTES;
    static constexpr int MAIN = KG * GROUP_BYTES > SUMS + PATCH ? KG * GROUP_BYTES : SUMS + PATCH;
    static constexpr int SXI = (TM + THREADS - 1) / THREADS, SWI = (TN + THREADS - 1) / THREADS;
    static constexpr int LDS = MAIN + (SXI + 2 * SWI) * THREADS * 4;
};

template <int TB, int CB, int WPF, int KG, int EPI>
__device__ __forceinline__ void w8_tile(const W8Params &p, int tm, int tn, char *smem)
{
    using T = W8Tile<TB, CB, WPF, KG>;
    constexpr int NW = T::NW, TM = T::TM, TN = T::TN, STAGES = T::STAGES, XL = TM / 32;
    static_assert(TB % 2 == 0 && CB % 2 == 0 && TB % KG == 0, "whole 32-row blocks, equal shares");
    float *side_sx = reinterpret_cast<float *>(smem + T::MAIN), *side_sw = side_sx + T::SXI * T::THREADS, *side_b = side_sw + T::SWI * T::THREADS;
    const int lane = threadIdx.x & 63;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6) % NW, group = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6) / NW;
    // epilogue operands: requested in front of the first stages, stored to LDS behind them (range-checked: no branch)
    int r_sx[T::SXI], r_sw[T::SWI];
    short r_b[T::SWI];
    if (EPI == EPI_F16) {
        const __amdgpu_buffer_rsrc_t rx = make_rsrc(p.sx, (unsigned)p.M * 4u), rw = make_rsrc(p.sw, (unsigned)p.N * 4u);
        const __amdgpu_buffer_rsrc_t rb = make_rsrc(p.bias, p.bias ? (unsigned)p.N * 2u : 0u);
#pragma unroll
        for (int it = 0; it < T::SXI; ++it)
            r_sx[it] = __builtin_amdgcn_raw_buffer_load_b32(rx, (unsigned)(tm * TM + threadIdx.x + it * T::THREADS) * 4u, 0, 0);
#pragma unroll
        for (int it = 0; it < T::SWI; ++it) {
            const unsigned n = (unsigned)(tn * TN + threadIdx.x + it * T::THREADS);
            r_sw[it] = __builtin_amdgcn_raw_buffer_load_b32(rw, n * 4u, 0, 0);
            r_b[it] = __builtin_amdgcn_raw_buffer_load_b16(rb, n * 2u, 0, 0);
        }
    }
    // This wavefront's stages: own of them from stage0 on; both groups of a workgroup make the same number of steps.
    const int all = p.K / 128, stage0 = group * p.stages_per_group, own = min(p.stages_per_group, all - stage0), steps = p.stages_per_group;
    const unsigned KB = p.K / 32;
    const int ch = lane >> 4, r = lane & 15;
    char *ring = smem + group * T::GROUP_BYTES;
    // Range checking: row-blocks beyond ceil32(M) / ceil32(N) return nothing (their offset alone is behind the buffer); stages behind
    // the last one are requested as the last one again, into buffers that nobody reads.
    unsigned xoff[XL], woff[CB / 2];
#pragma unroll
    for (int i = 0; i < XL; ++i) xoff[i] = lane * 16 + ((unsigned)(tm * (TM / 32) + i) * KB + wave) * 1024u;
#pragma unroll
    for (int i = 0; i < CB / 2; ++i)
        woff[i] = ((unsigned)(tn * (TN / 32) + wave * (CB / 2) + i) * KB + ch / 2) * 1024u + (r + 32 * (ch % 2)) * 16;
    auto issue_tokens = [&](int s) {
        const int k = min(stage0 + s, all - 1);
        const __amdgpu_buffer_rsrc_t xr = make_rsrc(p.xq, p.x_bytes);
        char *buf = ring + (s % STAGES) * T::STAGE_BYTES + wave * 1024;
#pragma unroll
        for (int i = 0; i < XL; ++i) {
            const unsigned off = xoff[i];
            __builtin_amdgcn_raw_ptr_buffer_load_lds(xr, LDS_PTR(buf + i * 4096), 16, off, k * 4096, 0, 0);
        }
    };
    v4i wf[WPF + 1][CB][2];
    auto issue_weights = [&](int s, v4i (&w)[CB][2]) {
        const int k = min(stage0 + s, all - 1);
        const __amdgpu_buffer_rsrc_t wr = make_rsrc(p.wq, p.w_bytes);
#pragma unroll
        for (int i = 0; i < CB; ++i)
#pragma unroll
            for (int t = 0; t < 2; ++t) {
                const unsigned off = woff[i / 2] + (i % 2) * 256 + t * 2048;
                w[i][t] = __builtin_bit_cast(v4i, __builtin_amdgcn_raw_buffer_load_b128(wr, off, k * 4096, 0));
            }
    };
    v4i acc[CB][TB];
#pragma unroll
    for (int i = 0; i < CB; ++i)
#pragma unroll
        for (int j = 0; j < TB; ++j) acc[i][j] = v4i{0, 0, 0, 0};
    issue_tokens(0);
    issue_tokens(1);
#pragma unroll
    for (int s = 0; s < WPF; ++s) issue_weights(s, wf[s]);
    issue_tokens(2);
    if (EPI == EPI_F16) {
#pragma unroll
        for (int it = 0; it < T::SXI; ++it) side_sx[threadIdx.x + it * T::THREADS] = __int_as_float(r_sx[it]);
#pragma unroll
        for (int it = 0; it < T::SWI; ++it) {
            side_sw[threadIdx.x + it * T::THREADS] = __int_as_float(r_sw[it]);
            side_b[threadIdx.x + it * T::THREADS] = __half2float(__ushort_as_half((unsigned short)r_b[it]));
        }
    }
    const int xl = (ch / 2) * 1024 + (r + 32 * (ch % 2)) * 16;
    v4i xf[2][2];
    auto read_tokens = [&](int s, int j) {
        const char *buf = ring + (s % STAGES) * T::STAGE_BYTES + xl;
#pragma unroll
        for (int t = 0; t < 2; ++t)
            xf[j & 1][t] = *reinterpret_cast<const v4i *>(buf + (j / 2) * 4096 + (j % 2) * 256 + t * 2048);
    };
    // loads issued behind a stage's weights: the tokens of one stage, the weights of WPF - 1
    constexpr int NEWER = XL + (WPF - 1) * 2 * CB;
    auto stage = [&](int it, v4i (&w)[CB][2], v4i (&next)[CB][2]) {
        wait_vmcnt<NEWER>();
        __builtin_amdgcn_sched_barrier(0);
        issue_weights(it + WPF, next);
        if (KG > 1 && it >= own) {                       // a group that has fewer stages than the other
#pragma unroll
            for (int i = 0; i < CB; ++i) w[i][0] = w[i][1] = v4i{0, 0, 0, 0};
        }
        __builtin_amdgcn_sched_barrier(0);
#pragma unroll
        for (int j = 0; j < TB; ++j) {
            if (j + 1 < TB) {
                read_tokens(it, j + 1);
            } else {
                __builtin_amdgcn_s_waitcnt(0xC07F);      // lgkmcnt(0): own reads done; everyone's at the barrier, next stage landed
                __builtin_amdgcn_s_barrier();
                issue_tokens(it + STAGES);
                read_tokens(it + 1, 0);
            }
            __builtin_amdgcn_sched_barrier(0);
#pragma unroll
            for (int t = 0; t < 2; ++t)
#pragma unroll
                for (int i = 0; i < CB; ++i) acc[i][j] = __builtin_amdgcn_mfma_i32_16x16x64_i8(xf[j & 1][t], w[i][t], acc[i][j], 0, 0, 0);
            __builtin_amdgcn_sched_barrier(0);
        }
    };
    wait_vmcnt<NEWER>();
    __builtin_amdgcn_s_barrier();
    read_tokens(0, 0);
    {
        constexpr int R = WPF + 1;
        int it = 0;
        for (; it + R <= steps; it += R) {
#pragma unroll
            for (int u = 0; u < R; ++u) stage(it + u, wf[u], wf[(u + WPF) % R]);
        }
#pragma unroll
        for (int u = 0; u < R - 1; ++u)
            if (it + u < steps) stage(it + u, wf[u], wf[(u + WPF) % R]);
    }
    wait_vmcnt<0>();   // drain the loads behind the last stage before the LDS is reused
    __syncthreads();
    char *stg = smem + T::SUMS + (group * NW + wave) * (16 * T::ROW_BYTES);
    const int n_wave0 = tn * TN + wave * CB * 16;
    const bool odd = lane & 1;
    char *at = stg + (4 * ch + (odd ? 2 : 0)) * T::ROW_BYTES + (r & ~1) * 2;
    float sw_r[CB], b_r[CB];
#pragma unroll
    for (int i = 0; i < CB; ++i) sw_r[i] = side_sw[(wave * CB + i) * 16 + r], b_r[i] = side_b[(wave * CB + i) * 16 + r];
    auto finish = [&](int j, const v4i (&s)[CB]) {
        const float4 s4 = *reinterpret_cast<const float4 *>(side_sx + j * 16 + 4 * ch);
        const float sx4[4] = {s4.x, s4.y, s4.z, s4.w};
#pragma unroll
        for (int i = 0; i < CB; ++i) {
            if constexpr (EPI == EPI_ACC) {
#pragma unroll
                for (int e = 0; e < 4; ++e) {
                    const int m = tm * TM + j * 16 + 4 * ch + e, n = n_wave0 + i * 16 + r;
                    if (m < p.M && n < p.N) p.acc[(size_t)m * p.ldacc + n] = s[i][e];
                }
            } else {
                float v[4];
#pragma unroll
                for (int e = 0; e < 4; ++e) {
                    v[e] = __builtin_fmaf((float)s[i][e] * sx4[e], sw_r[i], b_r[i]);
                    asm("" : "+v"(v[e]));   // rounded to fp32, then to fp16, in every kernel variant
                }
                patch_quad(at + i * 32, T::ROW_BYTES, odd, v);
            }
        }
        if constexpr (EPI != EPI_ACC) store_rows<CB * 2, 16>(p.y, p.ldy, p.M, p.N, stg, T::ROW_BYTES, tm * TM + j * 16, n_wave0, lane);
    };
    if constexpr (KG == 1) {
#pragma unroll
        for (int j = 0; j < TB; ++j) {
            v4i s[CB];
#pragma unroll
            for (int i = 0; i < CB; ++i) s[i] = acc[i][j];
            finish(j, s);
        }
    } else {                        // the groups' sums meet in LDS; each finishes its share of the token blocks
#pragma unroll
        for (int j = 0; j < TB; ++j)
#pragma unroll
            for (int i = 0; i < CB; ++i) *reinterpret_cast<v4i *>(smem + (((group * NW + wave) * TB + j) * CB + i) * 1024 + lane * 16) = acc[i][j];
        __syncthreads();
#pragma unroll
        for (int b = 0; b < TB / KG; ++b) {
            const int j = group * (TB / KG) + b;
            v4i s[CB];
#pragma unroll
            for (int i = 0; i < CB; ++i) {
                s[i] = v4i{0, 0, 0, 0};
#pragma unroll
                for (int g = 0; g < KG; ++g) s[i] += *reinterpret_cast<const v4i *>(smem + (((g * NW + wave) * TB + j) * CB + i) * 1024 + lane * 16);
            }
            finish(j, s);
        }
    }
}

template <int TB, int CB, int WPF, int KG, int EPI, int WPS>
__global__ __launch_bounds__(KG * 256, WPS) void gemm_w8_groups_kernel(W8Params p)
{
    extern __shared__ __attribute__((aligned(1024))) char smem[];
    int tm, tn;
    tile_coords(blockIdx.x, p.tiles_m, p.tiles_n, p.group_m, tm, tn);
    w8_tile<TB, CB, WPF, KG, EPI>(p, tm, tn, smem);
}

// OCC: workgroups per CU
template <int TB, int CB, int WPF, int KG, int EPI, int OCC>
int launch(const GemmArgs &a, hipStream_t st)
{
    using T = W8Tile<TB, CB, WPF, KG>;
    static_assert(T::LDS * OCC <= 160 * 1024, "LDS budget");
    auto kern = gemm_w8_groups_kernel<TB, CB, WPF, KG, EPI, OCC * KG>;
    static const hipError_t attr_status = hipFuncSetAttribute(reinterpret_cast<const void *>(kern), hipFuncAttributeMaxDynamicSharedMemorySize, T::LDS);
    QL_TRY(check_hip(attr_status, "hipFuncSetAttribute(max dynamic LDS)"));
    W8Params p = {a.xq, a.wq, a.sx, a.sw, a.bias, a.y, a.ldy, a.acc, a.ldacc ? a.ldacc : a.N, a.M, a.N, a.K};
    p.x_bytes = (unsigned)act_kernel_bytes(a.M, a.K), p.w_bytes = (unsigned)w8_kernel_bytes(a.N, a.K);
    p.tiles_m = ceil_div(a.M, T::TM), p.tiles_n = ceil_div(a.N, T::TN);
    p.group_m = strip_height(p.tiles_m, p.tiles_n, T::TM, T::TN, OCC);
    p.stages_per_group = ceil_div(a.K / 128, KG);
    hipLaunchKernelGGL(kern, dim3(p.tiles_m * p.tiles_n), dim3(T::THREADS), T::LDS, st, p);
    return check_hip(hipGetLastError(), "gemm_w8_groups launch");
}


// The forms and their estimated time: 3 us + the weights at 20 TB/s + the output at 7 TB/s + what the busiest CU does, in
// rounds of as many workgroups as fit it together (a round of n takes o[n - 1] + stages x c[n - 1], groups: their steps), but not
// less than the weights take to arrive (5.5 us + 3.6 TB/s).  128 x 256 is rarely the choice (5 of 60000 shapes), though measured the fastest at 470 x 6016
// x 13745 (45.2 us, taken 51.4) and 1342 x 6272 x 4800 (48.4, taken 51.5).  Fitted to 180 shapes (48..4096 tokens, N 1536..22016, K 1536..11008,
// weights from HBM), within 3 to 10 % on average each on the card they were fitted on; other cards are slower by up to a tenth, hence the factor.
struct W8Form {
    int variant, tm, tn, per_cu, groups;
    double o[4], c[4];
};
constexpr W8Form W8_FORMS[] = {
    {51, 64, 128, 4, 1, {0.0, 0.0, 0.0, 0.0}, {0.320, 0.562, 0.896, 1.214}},
    {52, 64, 128, 1, 2, {0.8}, {0.588}},
    {53, 96, 128, 3, 1, {0.5, 0.2, 0.2}, {0.372, 0.676, 1.052}},
    {54, 96, 128, 1, 2, {1.5}, {0.691}},
    {55, 128, 256, 2, 1, {2.9, 1.4}, {0.735, 1.417}},
    {56, 96, 256, 2, 1, {1.8, 1.9}, {0.645, 1.066}},
};

template <int EPI>
int launch_form(const GemmArgs &a, int variant, hipStream_t st)
{
    switch (variant) {
    case 51: return launch<4, 2, 2, 1, EPI, 4>(a, st);
    case 52: return launch<4, 2, 2, 2, EPI, 1>(a, st);
    case 53: return launch<6, 2, 2, 1, EPI, 3>(a, st);
    case 54: return launch<6, 2, 2, 2, EPI, 1>(a, st);
    case 55: return launch<8, 4, 1, 1, EPI, 2>(a, st);
    default: return launch<6, 4, 1, 1, EPI, 2>(a, st);
    }
}

}  // namespace

int choose_w8_form(const GemmArgs &a, double *us)
{
    int best = 0;
    *us = 1e30;
    if (a.K % 128 || a.M <= 64) return 0;
    for (const W8Form &f : W8_FORMS) {
        const long tiles = (long)ceil_div(a.M, f.tm) * ceil_div(a.N, f.tn), busiest = (tiles + 255) / 256;
        if (f.groups > 1 && tiles > 256) continue;
        const int steps = ceil_div(a.K / 128, f.groups);
        auto round = [&](long n) { return f.o[n - 1] + f.c[n - 1] * steps; };
        const double nk = (double)a.N * a.K;
        const double t = std::max(1.1 * (3.0 + nk / 20e6 + 2.0 * a.M * a.N / 7e6 + (double)(busiest / f.per_cu) * round(f.per_cu) +
                                         (busiest % f.per_cu ? round(busiest % f.per_cu) : 0.0)),
                                  5.5 + nk / 3.6e6);
        if (t < *us) best = f.variant, *us = t;
    }
    return best;
}

bool w8_form_tile(int variant, int *tile_tokens, int *tile_channels)
{
    for (const W8Form &f : W8_FORMS)
        if (f.variant == variant) {
            *tile_tokens = f.tm, *tile_channels = f.tn;
            return true;
        }
    return false;
}

int launch_gemm_w8_form(const GemmArgs &a, int variant, hipStream_t st)
{
    return a.acc ? launch_form<EPI_ACC>(a, variant, st) : launch_form<EPI_F16>(a, variant, st);
}

}  // namespace ql
