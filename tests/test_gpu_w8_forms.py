"""int8 prefill in workgroups of four wavefronts (variants 51..56) at edges of tiles, with one, few and unevenly halved stages of 128 k:
accumulators bit for bit against the oracle, fp16 outputs against another kernel's bits."""
import numpy as np
import pytest

import oracle
from paper_2512_23367_amd import binding as ql
from paper_2512_23367_amd import synth

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def G():
    import gpu_util
    return gpu_util


# tokens around 16 / 64 / 96 / 128, channels around 32 / 128 / 256; K 192: no whole stages, another kernel takes it
@pytest.mark.parametrize("M,K,N", [(1, 128, 32), (63, 256, 129), (97, 384, 31), (129, 640, 257), (200, 1152, 600), (257, 2816, 136), (70, 192, 96)])
def test_forms(G, M, K, N):
    x, w = synth.activations(M, K, 0, "single"), synth.weights(N, K, 0, "single")
    b = synth.bias(N, 0, "single")
    g = G.gpu_quant_weight(w, 8, 0)
    xq = np.random.default_rng(M + K + N).integers(-127, 128, (M, K), dtype=np.int8)
    acc_o = oracle.igemm(xq, g["canon"])
    y = {}
    try:
        for v in (13, 51, 52, 53, 54, 55, 56):
            ql.ql_set_kernel_variant(v)
            assert (G.gpu_acc(xq, g)[0] == acc_o).all(), v
            y[v] = G.gpu_linear(x, g, b)
            assert (y[v].view(np.uint16) == y[13].view(np.uint16)).all(), v
    finally:
        ql.ql_set_kernel_variant(0)
