"""The int4 prefill kernel's tile forms (tokens x channels: 26 128x256, 35 96x256, 37 128x256 by eight wavefronts, 4 128x128, 13 64x128,
19 96x128, 43 128x256 with 128x128 tiles for the last channels; split-K) at edges of tiles and stages: against the oracle, and bit
for bit against each other where K is not split (every form folds the groups in the same order)."""
import numpy as np
import pytest

import oracle
from paper_2512_23367_amd import binding as ql
from paper_2512_23367_amd import synth

pytestmark = pytest.mark.gpu
TOL = 1e-3      # the parity bar: max|y - ref| / max|ref|; the fp16 rounding alone is up to 4.9e-4
UNSPLIT = [26, 35, 37, 4, 13, 19, 43]


@pytest.fixture(scope="module")
def G():
    import gpu_util
    return gpu_util


# tokens: one, around 32 / 64 / 96 / 128 and two tiles of them; channels: around 32 / 128 / 256 / 768 (43: two regions); K: 1, 2, 3, 4 and
# more stages
@pytest.mark.parametrize("M,K,N", [(1, 128, 32), (33, 256, 31), (191, 384, 257), (193, 512, 600), (257, 640, 769), (300, 1152, 1000),
                                   (513, 128, 520), (64, 4096, 264), (95, 256, 127), (97, 640, 255), (127, 384, 129), (129, 896, 513), (65, 128, 128)])
@pytest.mark.parametrize("bias", [False, True])
def test_shapes_agree_with_the_oracle(G, M, K, N, bias):
    x, w = synth.activations(M, K, 0, "single"), synth.weights(N, K, 0, "single")
    b = synth.bias(N, 0, "single") if bias else None
    g = G.gpu_quant_weight(w, 4, 128)
    ref = oracle.linear_w4a8(x, g["canon"], g["scales"], 128, b)["y64"]
    outs = {}
    try:
        for v in UNSPLIT + [0, 2, 202, 203, 302, 303]:
            if v > 200 and K < 1024:
                continue                                   # (at least one stage per split)
            ql.ql_set_kernel_variant(v)
            outs[v] = G.gpu_linear(x, g, b, extra_ws=64 << 20)
    finally:
        ql.ql_set_kernel_variant(0)
    for v, y in outs.items():
        assert G.norm_err(y, ref) <= TOL, v
        if v in UNSPLIT:
            assert (y.view(np.uint16) == outs[26].view(np.uint16)).all(), v
