"""Host logic: when the int4 tile kernels take K in parts by groups of wavefronts (no GPU call is made)."""
import pytest

from paper_2512_23367_amd import binding as ql


@pytest.mark.parametrize("M,N,K", [(65, 4096, 4096), (200, 4096, 11008), (512, 4096, 8192), (300, 1536, 16384), (1024, 2048, 6144)])
def test_groups_fit_one_pass_and_need_the_callers_leave(M, N, K):
    p = ql.ql_plan_gemm(M, N, K, 4, 128, 64 << 20)
    if p.variant in (202, 304):
        assert M > 64 and -(-M // 64) * -(-N // 128) <= 256 and p.splits == p.variant % 100
        assert p.tile_tokens * p.tile_channels == p.splits * 64 * 128
    bare = ql.ql_plan_gemm(M, N, K, 4, 128, 0)
    assert bare.splits == 1 and bare.est_us >= p.est_us


def test_long_k_takes_four_groups_and_short_k_two():
    assert [ql.ql_plan_gemm(512, 4096, K, 4, 128, 64 << 20).variant for K in (2048, 4096, 11008, 16384)] == [202, 202, 304, 304]
    assert ql.ql_plan_gemm(513, 4096, 11008, 4, 128, 64 << 20).variant not in (202, 304)      # 288 tiles: not one pass
