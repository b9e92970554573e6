// Pieces the two prefill GEMM kernels (int8 weights: gemm_prefill.hip, int4 weights: gemm_prefill_w4.hip) share:
// range-checked buffers, counted waits, the order in which workgroups take output tiles, and the split-K plan.
#pragma once

#include "common.h"

namespace ql {

typedef int v4i __attribute__((ext_vector_type(4)));
typedef _Float16 h4 __attribute__((ext_vector_type(4)));

enum { EPI_F16 = 0, EPI_ACC = 1, EPI_PART = 2 };   // EPI_PART: split-K, raw partial sums to the workspace

#define LDS_PTR(p) ((__attribute__((address_space(3))) void *)(p))

template <int N>
__device__ inline void wait_vmcnt()
{
    asm volatile("s_waitcnt vmcnt(%0)" ::"n"(N) : "memory");
}

__device__ inline __amdgpu_buffer_rsrc_t make_rsrc(const void *p, unsigned bytes)
{
    return __builtin_amdgcn_make_buffer_rsrc(const_cast<void *>(p), 0, (int)bytes, 0x00020000);
}

// Writes a wavefront's staged block of ROWS tokens to y, 16 bytes per lane (LPR lanes per row).
template <int LPR, int ROWS>
__device__ __forceinline__ void store_rows(__half *y, int64_t ldy, int M, int N, const char *stg, int row_bytes, int m0, int n0, int lane)
{
    constexpr int RPI = 64 / LPR;
    static_assert(64 % LPR == 0 && ROWS % RPI == 0, "whole rows per read-back instruction");
    asm volatile("" ::: "memory");   // (same wavefront, LDS operations complete in order: only the compiler must keep them so)
    __builtin_amdgcn_wave_barrier();
#pragma unroll
    for (int t = 0; t < ROWS / RPI; ++t) {
        const int row = t * RPI + lane / LPR, c = lane % LPR;
        const uint4 v = *reinterpret_cast<const uint4 *>(stg + row * row_bytes + c * 16);
        const int mm = m0 + row, nn = n0 + c * 8;
        if (mm < M && nn < N) {
            __half *dst = y + (size_t)mm * ldy + nn;
            if (nn + 7 < N) {
                *reinterpret_cast<uint4 *>(dst) = v;
            } else {   // the last N % 8 channels: four, two and one of them (as up to seven stores in a loop: 620 x 256 x 191,
                       // int4, 5.6 us against 4.1; 4097 x 1152 x 3487 in 128 x 256 tiles 32.7 against 28.0)
                const int left = N - nn;
                const bool four = left & 4;
                if (four) *reinterpret_cast<uint2 *>(dst) = make_uint2(v.x, v.y);
                const unsigned lo = four ? v.z : v.x, hi = four ? v.w : v.y;
                if (left & 2) *reinterpret_cast<unsigned *>(dst + (left & 4)) = lo;
                if (left & 1) dst[left & 6] = __ushort_as_half((unsigned short)(left & 2 ? hi : lo));
            }
        }
    }
    asm volatile("" ::: "memory");
    __builtin_amdgcn_wave_barrier();
}

// Four tokens of one channel per lane -> a patch in LDS as fp16 [token][channel]: neighbouring lanes exchange half of their
// values, so that each writes two channels of two tokens.  `at`: the lane's first row, its pair of channels.
__device__ __forceinline__ void patch_quad(char *at, int row_bytes, bool odd, const float (&v)[4])
{
    typedef _Float16 h2 __attribute__((ext_vector_type(2)));
    const unsigned p01 = __builtin_bit_cast(unsigned, h2{(_Float16)v[0], (_Float16)v[1]}), p23 = __builtin_bit_cast(unsigned, h2{(_Float16)v[2], (_Float16)v[3]});
    const unsigned kept = odd ? p23 : p01, got = (unsigned)__builtin_amdgcn_mov_dpp((int)(odd ? p01 : p23), 0xB1, 0xf, 0xf, true);
    *reinterpret_cast<unsigned *>(at) = __builtin_amdgcn_perm(got, kept, odd ? 0x01000504u : 0x05040100u);
    *reinterpret_cast<unsigned *>(at + row_bytes) = __builtin_amdgcn_perm(got, kept, odd ? 0x03020706u : 0x07060302u);
}

// Hardware hands consecutive workgroup ids to the 8 XCDs in turn; give every XCD one contiguous
// range of logical tiles, ordered (strips of `group` token tiles, channel tile by channel tile) so that the
// tiles an XCD runs together form a block that shares activation and weight strips in that XCD's L2.
__device__ inline void tile_coords(int bid, int tiles_m, int tiles_n, int group, int &tm, int &tn)
{
    const int nt = tiles_m * tiles_n;
    const int xcd = bid % 8, idx = bid / 8;
    const int per = nt / 8, rem = nt % 8;
    const int logical = xcd * per + (xcd < rem ? xcd : rem) + idx;
    const int per_group = group * tiles_n;
    const int g = logical / per_group, in_g = logical % per_group;
    const int first_m = g * group;
    const int gsize = (tiles_m - first_m) < group ? (tiles_m - first_m) : group;
    tm = first_m + in_g % gsize;
    tn = in_g / gsize;
}

// Strip height: the tiles resident on one XCD together (32 CUs x occupancy, or all of its tiles if fewer) should
// form the block that fetches the fewest operand bytes -- a x b tiles cost a*TM + b*TN rows of K bytes.  Only
// divisors of tiles_m are considered (equal strips; a ragged last strip costs more than it saves), ties go to
// the shorter strip (measured: fewer bytes fetched when the block does not fit the 4 MB L2 anyway).
inline int strip_height(int tiles_m, int tiles_n, int TM, int TN, int occupancy)
{
    const long per_xcd = ((long)tiles_m * tiles_n + 7) / 8;
    const long together = per_xcd < 32L * occupancy ? per_xcd : 32L * occupancy;
    int best = 1;
    long best_cost = -1;
    for (int d = 1; d <= tiles_m; ++d) {
        if (tiles_m % d) continue;
        const long cost = (long)d * TM + ((together + d - 1) / d) * TN;
        if (best_cost < 0 || cost < best_cost) best = d, best_cost = cost;
    }
    return best;
}

}  // namespace ql
