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
