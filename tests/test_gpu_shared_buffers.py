"""Results that take the place of inputs: y written over x (a linear that quantizes its tokens inside the GEMM must have read
all of them first), x and y as column ranges of one buffer, and transformed weight codes over the fp16 weights.  Every case
against the same call on separate buffers, bit for bit."""
import numpy as np
import pytest

from paper_2512_23367_amd import binding as ql, synth

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def G():
    from tests import gpu_util
    return gpu_util


def _linear(x, g, y, M, K, N, bits):
    import torch
    ws = torch.empty(ql.ql_workspace_bytes(M, N, K, bits), dtype=torch.uint8, device="cuda:0")
    if bits == 8:
        ql.ql_w8a8_linear(x, g["kernel"], g["scales_dev"].view(torch.float32), None, N, y, ws)
    else:
        ql.ql_w4a8_linear(x, g["kernel"], 128, None, N, y, ws)
    torch.cuda.synchronize()


@pytest.mark.parametrize("bits", [8, 4])
@pytest.mark.parametrize("M,K,N", [(1, 2048, 2048), (4, 1536, 1536), (8, 1536, 1536), (8, 2048, 1024), (16, 1024, 1024),
                                   (33, 1536, 1536)])
def test_linear_output_over_its_input(G, bits, M, K, N):
    import torch
    x = torch.from_numpy(synth.activations(M, K, 3, "qkv")).to("cuda:0")
    g = G.gpu_quant_weight(synth.weights(N, K, 3, "qkv"), bits, 0 if bits == 8 else 128)
    ref = torch.empty((M, N), dtype=torch.float16, device="cuda:0")
    _linear(x, g, ref, M, K, N, bits)
    for _ in range(3):                                     # y over x, the same rows
        buf = x.clone()
        _linear(buf, g, buf[:, :N], M, K, N, bits)
        assert torch.equal(buf[:, :N], ref)
    wide = torch.zeros((M, K + N), dtype=torch.float16, device="cuda:0")   # side by side: no byte shared
    wide[:, :K] = x
    _linear(wide[:, :K], g, wide[:, K:], M, K, N, bits)
    assert torch.equal(wide[:, K:], ref) and torch.equal(wide[:, :K], x)
    wide[:, N:] = x                                        # y in front of x
    _linear(wide[:, N:], g, wide[:, :N], M, K, N, bits)
    assert torch.equal(wide[:, :N], ref) and torch.equal(wide[:, N:], x)


@pytest.mark.parametrize("M,K,N,never_fused", [(1, 2048, 2048, False), (4, 1536, 1536, False), (4, 4096, 4096, False),
                                                (8, 1536, 1536, False), (8, 4096, 4096, True)])
def test_int4_sums_do_not_depend_on_the_route(G, M, K, N, never_fused):
    """fp16 rounding hides the order in which the wavefronts' fp32 sums are added; large codes of one sign and a bias that
    cancels the result leave its last bits.  Fused quantizer and y over x (two launches) have one order; with four pieces
    per lane it is also that of the quantizer that is never fused."""
    import torch
    rng = np.random.default_rng(K)
    x = torch.from_numpy(rng.uniform(0.5, 1, (1, K)).astype(np.float16)).to("cuda:0").repeat(M, 1)
    g = G.gpu_quant_weight(rng.uniform(-0.2, 1, (N, K)).astype(np.float16), 4, 128)
    ws = torch.empty(ql.ql_workspace_bytes(M, N, K, 4), dtype=torch.uint8, device="cuda:0")

    def linear(x, bias, y):
        ql.ql_w4a8_linear(x, g["kernel"], 128, bias, N, y, ws)
        torch.cuda.synchronize()
        return y

    fresh = lambda: torch.empty((M, N), dtype=torch.float16, device="cuda:0")
    bias = -linear(x, None, fresh())[0].clone()
    ref = linear(x, bias, fresh())
    assert (ref != 0).float().mean() > 0.5                  # the residues are what is compared
    buf = x.clone()
    assert torch.equal(linear(buf, bias, buf[:, :N]), ref)
    if never_fused:
        try:
            ql.ql_set_kernel_variant(130)
            assert torch.equal(linear(x, bias, fresh()), ref)
        finally:
            ql.ql_set_kernel_variant(0)


@pytest.mark.parametrize("bits", [8, 4])
@pytest.mark.parametrize("N,K,block", [(200, 1536, 512), (64, 11008, 256), (100, 4096, 0), (33, 16384, 4096)])
def test_transformed_weight_codes_over_the_weights(G, bits, N, K, block):
    import torch
    w = torch.from_numpy(synth.weights(N, K, 3, "qkv")).to("cuda:0")
    smooth = torch.from_numpy(np.linspace(0.5, 2.0, K).astype(np.float32)).to("cuda:0")
    group = 0 if bits == 8 else 128
    cb, sb, kb = ql.ql_weight_bytes(N, K, bits, group)

    def quantize(w16, canon):
        w32 = torch.empty((N, K), dtype=torch.float32, device="cuda:0")
        scales, kern = G.empty_bytes(sb), torch.zeros(kb, dtype=torch.uint8, device="cuda:0")
        ql.ql_quant_weight_transformed(w16, bits, group, smooth, block, w32, canon, scales, kern)
        torch.cuda.synchronize()
        return w32, scales, kern

    canon = G.empty_bytes(cb)
    ref = quantize(w, canon)
    buf = w.clone()
    over = buf.view(torch.uint8).view(-1)[:cb]
    out = quantize(buf, over)
    assert torch.equal(over, canon) and all(torch.equal(a, b) for a, b in zip(out, ref))
