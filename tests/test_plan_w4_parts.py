"""Host logic: when the int4 tile kernels take K in parts by groups of wavefronts (no GPU call is made)."""
import pytest

from paper_2512_23367_amd import binding as ql


@pytest.mark.parametrize("M,N,K,variant", [(200, 8192, 11008, 304), (512, 4096, 8192, 304), (1024, 2048, 6144, 202), (1280, 1536, 6144, 202)])
def test_groups_fit_one_pass_and_need_the_callers_leave(M, N, K, variant):
    p = ql.ql_plan_gemm(M, N, K, 4, 128, 64 << 20)
    assert (p.variant, p.splits, p.tile_tokens, p.tile_channels) == (variant, variant % 100, 64, 128)
    assert M > 64 and -(-M // 64) * -(-N // 128) <= 256
    bare = ql.ql_plan_gemm(M, N, K, 4, 128, 0)
    assert bare.splits == 1 and bare.est_us >= p.est_us


def test_long_k_takes_four_groups_and_short_k_two():
    assert [ql.ql_plan_gemm(512, 4096, K, 4, 128, 64 << 20).variant for K in (2048, 4096, 11008, 16384)] == [202, 202, 304, 304]
    assert ql.ql_plan_gemm(513, 4096, 11008, 4, 128, 64 << 20).variant not in (202, 304)      # 288 tiles: not one pass


@pytest.mark.parametrize("M,N,K", [(512, 4096, 4096), (512, 4096, 11008), (1280, 1536, 6144), (768, 2048, 8192)])
def test_k_is_taken_in_parts_only_where_the_scratch_holds_the_split(M, N, K):
    """Parts of K are another order of the fp32 sums: a caller has them by offering the bytes of the split, and by no less."""
    def plan(scratch):
        return ql.ql_plan_gemm(M, N, K, 4, 128, scratch)

    def need(p):
        rows, channels = -(-M // 128) * 128, 256 if p.variant > 300 else 128
        return p.splits * rows * -(-N // channels) * channels * 4

    whole = plan(64 << 20)
    assert whole.splits > 1 and need(whole) <= 64 << 20
    assert (plan(need(whole)).variant, plan(need(whole)).splits) == (whole.variant, whole.splits)
    below = plan(need(whole) - 1)
    assert below.splits == 1 or need(below) < need(whole)
    unsplit = plan(0)
    for scratch in (16, 256, 4096, 65536):
        p = plan(scratch)
        assert (p.family, p.variant, p.splits, p.est_us) == (unsplit.family, unsplit.variant, 1, unsplit.est_us), scratch
