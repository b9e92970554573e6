"""The transform kernels at the edges of their forms: every Hadamard block size (inside a lane, inside a row of 16 lanes,
across rows, across wavefronts) with rows that end inside a wavefront, and the column maxima over ragged row counts."""
import numpy as np
import pytest
import torch

import oracle
from paper_2512_23367_amd import binding as ql
from paper_2512_23367_amd import synth
from test_gpu_transforms import gpu_act, gpu_weight

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def G():
    import gpu_util
    return gpu_util


BLOCKS = [(64, 16), (192, 32), (1088, 64), (1152, 128), (2304, 256), (1536, 512), (3072, 1024), (1024, 1024), (6144, 2048), (2048, 2048),
          (12288, 4096), (16384, 4096), (4096, 16)]


@pytest.mark.parametrize("K,block", BLOCKS)
@pytest.mark.parametrize("M", [1, 67])
def test_activations_every_block(G, M, K, block):
    x = synth.activations(M, K, 0, "single")
    inv = np.random.default_rng(K).uniform(0.2, 3, K).astype(np.float32)
    for inv_s in (None, inv):
        t = x.astype(np.float32) if inv_s is None else oracle.smooth_act(x, inv_s)
        q_o, s_o = oracle.quant_act_per_token(oracle.fwht_blocks(t, block))
        q, s, xk, _ = gpu_act(G, x, inv_s, block)
        assert (s == s_o).all() and (q == q_o).all()
        rows = (np.arange((M + 31) // 32 * 32 * K) // 1024 // (K // 32)) * 32 + (np.arange((M + 31) // 32 * 32 * K) % 1024 // 16) % 32
        assert (G.repack_act(q_o).cpu().numpy()[rows < M] == xk.cpu().numpy()[rows < M]).all()


# (from K = 15424 on with blocks up to 1024 sixteen wavefronts stage 64 KB, beside the static LDS)
@pytest.mark.parametrize("K,block", [b for b in BLOCKS if b[0] % 128 == 0] + [(1024, 0), (11008, 256), (15488, 128), (16384, 64), (16384, 1024), (16384, 0)])
@pytest.mark.parametrize("bits", [8, 4])
def test_weights_every_block(G, bits, K, block):
    N = 37                                                # rows 37 .. 63 are padding of the kernel layout
    w = synth.weights(N, K, 0, "single")
    w[3] = 0
    smooth = np.random.default_rng(K).uniform(0.2, 3, K).astype(np.float32)
    t = oracle.smooth_weight(w, smooth)
    t = oracle.fwht_blocks(t, block) if block else t
    g = gpu_weight(G, w, bits, smooth, block)
    assert (g["w32"] == t).all()
    if bits == 8:
        q_o, s_o = oracle.quant_weight_int8(t)
    else:
        q_o, _, s_o = oracle.quant_weight_int4(t, 128)
    assert (g["scales"] == s_o).all() and (g["canon"] == q_o).all()
    c, s = G.gpu_export(g["kernel"], N, K, bits, g["group"])
    assert (c == q_o).all() and (bits == 8 or (s == s_o).all())
    # the padding rows hold zero codes, as those of the plain quantizer do
    plain = G.gpu_quant_weight(np.zeros((64, K), np.float16), bits, g["group"], check=False)["kernel"].cpu().numpy()
    codes = 64 * K // (1 if bits == 8 else 2)
    lane_row = 32 + (np.arange(codes // 2) % 1024 // 16) % 32     # second row-block of the blob
    assert (g["kernel"].cpu().numpy()[codes // 2:codes][lane_row >= N] == plain[codes // 2:codes][lane_row >= N]).all()


@pytest.mark.parametrize("factor", [1.0, 1 / 3, 0.7001, 3e-5, 1e-9, 3e-41, 1e36])
@pytest.mark.parametrize("bits", [8, 4])
def test_weight_codes_in_the_middle(G, bits, factor):
    """Weights in the middle between two codes, or an ulp of it away, where a product with the scale's reciprocal and the division
    differ; scales from fp32 subnormal (zero in fp16) to infinite in fp16.  Bit for bit the division's codes."""
    top, K = (127, 384) if bits == 8 else (7, 384)
    k = np.resize(np.arange(-top, top), K)
    w = np.stack([k + 0.5, np.nextafter((k + 0.5).astype(np.float16), np.float16(0)), np.nextafter((k + 0.5).astype(np.float16), np.float16(200)), k]).astype(np.float16)
    w[:, ::128] = top                                     # every group's maximum: scale = factor
    smooth = np.full(K, factor, np.float32)
    with np.errstate(over="ignore"):                      # fp16 scales
        t = oracle.smooth_weight(w, smooth)
        if bits == 8:
            q_o, s_o = oracle.quant_weight_int8(t)
        else:
            q_o, _, s_o = oracle.quant_weight_int4(t, 128)
    g = gpu_weight(G, w, bits, smooth, 0)
    assert (g["w32"] == t).all() and (g["scales"] == s_o).all() and (g["canon"] == q_o).all()
    c, _ = G.gpu_export(g["kernel"], 4, K, bits, g["group"])
    assert (c == q_o).all()


@pytest.mark.parametrize("M,N,K", [(1, 1, 64), (63, 511, 192), (65, 513, 320), (130, 600, 1088), (3, 4100, 192), (2, 2049, 64), (5, 6000, 1088)])   # the last three: several workgroups per strip
def test_column_maxima(G, M, N, K):
    x, w = synth.activations(M, K, 0, "single"), synth.weights(N, K, 0, "single")
    w[-1, 7] = 3                                          # the last row, the last token decide a channel
    x[-1, K - 1] = -50
    xmax = torch.zeros(K, dtype=torch.float32, device=G.DEV)
    ql.ql_smooth_calibrate(G.dev(x), xmax)
    assert (xmax.cpu().numpy() == oracle.channel_absmax(x)).all()
    s, inv = torch.empty_like(xmax), torch.empty_like(xmax)
    ql.ql_smooth_scales(xmax, G.dev(w), 0.5, s, inv)
    s_o, inv_o = oracle.smooth_scales(oracle.channel_absmax(x), w, 0.5)
    np.testing.assert_allclose(s.cpu().numpy(), s_o, rtol=3e-7)
    inv_1, other = inv.clone(), xmax.clone()
    ql.ql_smooth_scales(xmax, G.dev(w), 0.5, xmax, inv)   # in place: every lane reads its maximum before it writes
    assert (xmax == s).all() and (inv == inv_1).all()
    ql.ql_smooth_scales(other, G.dev(w), 0.5, s, other)
    assert (xmax == s).all() and (other == inv_1).all()
