"""The last N % 8 channels of the kernels with four-wavefront workgroups (stored in pieces of four, two and one): every remainder, against the
oracle, and nothing written behind them."""
import numpy as np
import pytest
import torch

import oracle
from paper_2512_23367_amd import binding as ql
from paper_2512_23367_amd import synth

pytestmark = pytest.mark.gpu
TOL = 1e-3      # the parity bar: max|y - ref| / max|ref|; the fp16 rounding alone is up to 4.9e-4


@pytest.mark.parametrize("bits,variants", [(8, (51, 54, 56)), (4, (26, 13, 304, 203))])   # one workgroup form of each epilogue
@pytest.mark.parametrize("N", [1, 2, 3, 132, 133, 134, 135])
def test_every_remainder(bits, variants, N):
    import gpu_util as G
    M, K = 70, 1536
    x, w = synth.activations(M, K, 0, "single"), synth.weights(N, K, 0, "single")
    g = G.gpu_quant_weight(w, bits, 0 if bits == 8 else 128)
    ref = oracle.linear_w8a8(x, g["canon"], g["scales"], None) if bits == 8 else oracle.linear_w4a8(x, g["canon"], g["scales"], 128, None)
    ws = G.empty_bytes(ql.ql_workspace_bytes(M, N, K, bits) + (8 << 20))
    xd = G.dev(x)
    try:
        for v in variants:
            buf = torch.full((M, 144), 7.0, dtype=torch.float16, device=G.DEV)
            ql.ql_set_kernel_variant(v)
            if bits == 8:
                ql.ql_w8a8_linear(xd, g["kernel"], g["scales_dev"].view(torch.float32), None, N, buf[:, :N], ws)
            else:
                ql.ql_w4a8_linear(xd, g["kernel"], 128, None, N, buf[:, :N], ws)
            out = buf.cpu().numpy()
            assert G.norm_err(out[:, :N], ref["y64"]) <= TOL, v
            assert (out[:, N:] == 7.0).all(), v
    finally:
        ql.ql_set_kernel_variant(0)
