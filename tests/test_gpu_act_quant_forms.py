"""The activation quantizer's kernel forms (a workgroup per token with 1, 2, 4 or 8 chunks per lane, 8 tokens per workgroup
above 3072 tokens, rows read twice where registers do not hold them) at their edges: codes and scales bit for bit against
the oracle, every mode."""
import numpy as np
import pytest
import torch

import oracle
from paper_2512_23367_amd import binding as ql

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def G():
    import gpu_util
    return gpu_util


def _reference(mode, x, vec):
    """(codes, scales) of the oracle; vec: inverse smoothing scales or gamma."""
    if mode == "plain":
        return oracle.quant_act_per_token(x)
    if mode == "smooth":
        return oracle.quant_act_per_token(oracle.smooth_act(x, vec))
    if mode == "rmsnorm":
        return oracle.quant_act_per_token(oracle.rmsnorm_act(x, vec, 1e-5))
    return oracle.quant_act_per_token(oracle.swiglu_act(x))


def _run(G, mode, x, vec, K):
    M = x.shape[0]
    xd = G.dev(x)
    xq = torch.full((M, K), 99, dtype=torch.int8, device=G.DEV)
    sx = torch.full((M,), -1.0, dtype=torch.float32, device=G.DEV)
    xk = G.empty_bytes(ql.ql_act_kernel_bytes(M, K))
    if mode == "plain":
        ql.ql_quant_act_per_token(xd, xq, xk, sx)
    elif mode == "smooth":
        ql.ql_quant_act_per_token_transformed(xd, G.dev(vec), 0, xq, xk, sx)
    elif mode == "rmsnorm":
        ql.ql_quant_act_rmsnorm(xd, G.dev(vec), 1e-5, xq, xk, sx)
    else:
        ql.ql_quant_act_swiglu(xd, xq, xk, sx)
    torch.cuda.synchronize()
    return xq.cpu().numpy(), sx.cpu().numpy(), xk


# K: one chunk row short of / at / past a wavefront (1024), the last row the per-token kernel takes and the first it does
# not, the last the 8-token kernel takes and the first it does not; M: around a group of 8, of 64, and the rule's line
@pytest.mark.parametrize("M,K", [(1, 64), (7, 1024), (9, 1088), (65, 960), (3, 16384), (3, 16448), (3072, 128), (3073, 128),
                                 (3075, 1088), (3081, 12288), (3073, 12352)])
@pytest.mark.parametrize("mode", ["plain", "smooth", "rmsnorm", "swiglu"])
def test_forms_bit_exact(G, mode, M, K):
    _check_form(G, mode, M, K)


# long rows: the last K of 1, 2 and 4 chunks per lane and the first beyond, the longest K there is; SmoothQuant also around
# the token counts where its 8-token form begins (2048, 513) and the last K of its 12-chunk form
@pytest.mark.parametrize("M,K", [(9, 16448), (65, 28672), (3, 32768), (9, 32832), (2, 65536), (9, 65600), (1, 131072)])
@pytest.mark.parametrize("mode", ["plain", "smooth", "rmsnorm", "swiglu"])
def test_long_rows_bit_exact(G, mode, M, K):
    _check_form(G, mode, M, K)


@pytest.mark.parametrize("M,K", [(2047, 16448), (2048, 16448), (2051, 20480), (1, 65600), (17, 98304), (17, 98368), (513, 98368)])
def test_long_smooth_rows_bit_exact(G, M, K):
    _check_form(G, "smooth", M, K)


def _check_form(G, mode, M, K):
    rng = np.random.default_rng(M * 7 + K)
    x = rng.standard_normal((M, 2 * K if mode == "swiglu" else K)).astype(np.float32)
    x[:, rng.integers(0, x.shape[1], 4)] *= 20
    x = x.astype(np.float16)
    if M > 2:
        x[1] = 0
    vec = {"smooth": rng.uniform(0.1, 3, K).astype(np.float32), "rmsnorm": rng.uniform(0.5, 2, K).astype(np.float16)}.get(mode)
    rows = slice(None) if M * K < 4e6 else np.unique(np.r_[0:40, M // 2:M // 2 + 40, M - 80:M])
    q_o, s_o = _reference(mode, x[rows], vec)
    q, s, xk = _run(G, mode, x, vec, K)
    assert (s[rows].view(np.uint32) == s_o.view(np.uint32)).all()
    assert (q[rows] == q_o).all()
    valid = (np.arange((M + 31) // 32 * 32 * K) // 1024 // (K // 32)) * 32 + (np.arange((M + 31) // 32 * 32 * K) % 1024 // 16) % 32 < M
    assert (G.repack_act(q).cpu().numpy()[valid] == xk.cpu().numpy()[valid]).all()


def test_swiglu_of_every_gate(G):
    """One finite fp16 gate per token and u = 1: the token scale is |silu(g)| / 127 itself, so every value of the stated
    step sequence (its reciprocal taken by one Newton step, its power of two by an exponent addition) shows."""
    bits = np.arange(65536, dtype=np.uint32).astype(np.uint16)
    g = bits.view(np.float16)
    g = g[np.isfinite(g)]
    F = 64
    gu = np.zeros((len(g), 2 * F), dtype=np.float16)
    gu[:, 5] = g
    gu[:, F + 5] = 1
    q_o, s_o = oracle.quant_act_per_token(oracle.swiglu_act(gu))
    q, s, _ = _run(G, "swiglu", gu, None, F)
    assert (s.view(np.uint32) == s_o.view(np.uint32)).all()
    assert (q == q_o).all()


@pytest.mark.parametrize("mode", ["plain", "smooth", "rmsnorm", "swiglu", "hadamard"])
def test_nan_reaches_the_scale(G, mode):
    """Codes of a token that holds a NaN are unspecified, but its scale (hence its output) must not look finite."""
    x = np.ones((9, 256 if mode == "swiglu" else 128), dtype=np.float16)
    x[4, 100] = np.nan
    s = _non_finite(G, mode, x)[1]
    assert np.isnan(s[4]) and np.isfinite(np.delete(s, 4)).all()


def _non_finite(G, mode, x, K=128):
    vec = {"smooth": np.ones(K, np.float32), "rmsnorm": np.ones(K, np.float16)}.get(mode)
    if mode != "hadamard":
        return _run(G, mode, x, vec, K)
    xq = torch.empty((x.shape[0], K), dtype=torch.int8, device=G.DEV)
    sx = torch.empty(x.shape[0], dtype=torch.float32, device=G.DEV)
    ql.ql_quant_act_per_token_transformed(G.dev(x), None, 16, xq, None, sx)
    return xq.cpu().numpy(), sx.cpu().numpy(), None


@pytest.mark.parametrize("M,K", [(9, 128), (9, 20480), (3073, 128)])
@pytest.mark.parametrize("mode", ["plain", "smooth"])
def test_infinity_keeps_its_code(G, mode, M, K):
    """A token with an infinity has an infinite scale; its infinite elements have code -127 and the others 0 (the clamp of
    0 * inf), so that its outputs are infinite where such a channel has weight, not NaN throughout."""
    x = np.ones((M, K), dtype=np.float16)
    x[4, 100], x[7, 3] = np.inf, -np.inf
    q, s, _ = _non_finite(G, mode, x, K)
    want = np.full((M, K), 127, dtype=np.int8)
    want[[4, 7]] = 0
    want[4, 100] = want[7, 3] = -127
    assert np.isposinf(s[[4, 7]]).all() and np.isfinite(np.delete(s, [4, 7])).all()
    assert (q == want).all()


@pytest.mark.parametrize("bits", [8, 4])
@pytest.mark.parametrize("M", [1, 4, 8])
def test_infinity_through_the_fused_quantizer(G, bits, M):
    """The decode GEMM that quantizes its tokens itself decides as the stand-alone quantizer does."""
    K, N = 1024, 64
    x = np.ones((M, K), dtype=np.float16)
    x[M - 1, 5] = np.inf
    w = np.ones((N, K), dtype=np.float16)
    w[1::2] = -1
    y = G.gpu_linear(x, G.gpu_quant_weight(w, bits, 0 if bits == 8 else 128))
    assert np.isneginf(y[M - 1, 0::2]).all() and np.isposinf(y[M - 1, 1::2]).all() and np.isfinite(y[:M - 1]).all()
