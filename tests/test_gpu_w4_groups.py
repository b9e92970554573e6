"""int4 prefill kernels: the tile forms that test_gpu_w4_tiles does not select, and K taken in parts by groups of wavefronts of one
workgroup (202: two, 304: four), at edges of tiles and with fewer stages (128 k) than parts."""
import numpy as np
import pytest

import oracle
from paper_2512_23367_amd import binding as ql
from paper_2512_23367_amd import synth

pytestmark = pytest.mark.gpu
TOL = 1e-3      # the parity bar: max|y - ref| / max|ref|; the fp16 rounding alone is up to 4.9e-4


@pytest.fixture(scope="module")
def G():
    import gpu_util
    return gpu_util


# stages: 1, 2, 3, 5, 9, 22 (parts of unequal length, empty parts); tokens around 64, 96, 128; channels around 32, 128, 256
@pytest.mark.parametrize("M,K,N", [(1, 128, 32), (65, 256, 129), (97, 384, 33), (63, 640, 260), (129, 1152, 127), (200, 2816, 520), (256, 4096, 128)])
@pytest.mark.parametrize("bias", [False, True])
def test_forms_and_parts_of_k(G, M, K, N, bias):
    x, w = synth.activations(M, K, 0, "single"), synth.weights(N, K, 0, "single")
    b = synth.bias(N, 0, "single") if bias else None
    g = G.gpu_quant_weight(w, 4, 128)
    ref = oracle.linear_w4a8(x, g["canon"], g["scales"], 128, b)["y64"]
    outs = {}
    try:
        for v in (26, 4, 17, 19, 202, 304):
            ql.ql_set_kernel_variant(v)
            outs[v] = G.gpu_linear(x, g, b, extra_ws=64 << 20)
            assert G.norm_err(outs[v], ref) <= TOL, v
            assert (G.gpu_linear(x, g, b, extra_ws=64 << 20).view(np.uint16) == outs[v].view(np.uint16)).all(), v
    finally:
        ql.ql_set_kernel_variant(0)
    for v in (4, 17, 19) + ((202, 304) if K == 128 else ()):       # the same order of the sums: the same bits
        assert (outs[v].view(np.uint16) == outs[26].view(np.uint16)).all(), v


@pytest.mark.parametrize("M,K,N", [(512, 2048, 1024), (200, 4096, 520)])
def test_a_little_scratch_does_not_change_the_sums(G, M, K, N):
    """Too little scratch for a split is as good as none: the same order of the sums, the same bits."""
    import torch
    x, w = synth.activations(M, K, 0, "single"), synth.weights(N, K, 0, "single")
    g = G.gpu_quant_weight(w, 4, 128)
    _, sx, xk = G.gpu_quant_act(x)
    sx, outs = G.dev(sx), []
    for ws in (None, G.empty_bytes(16), G.empty_bytes(4096)):
        y = torch.zeros((M, N), dtype=torch.float16, device=G.DEV)
        ql.ql_w4a8_gemm(xk, sx, M, K, g["kernel"], 128, None, N, y, ws)
        outs.append(y)
    assert torch.equal(outs[0], outs[1]) and torch.equal(outs[0], outs[2])
