"""Native argument marshalling (csrc/pycall.cpp) against the Python of binding.py: it makes a call only where binding.py would make
the same one, and whatever is wrong is reported by binding.py as without it."""
import numpy as np
import pytest
import torch

import oracle  # noqa: F401  (the package's path)
from paper_2512_23367_amd import binding as ql


def _outcome(f):
    try:
        return ("returned", f())
    except Exception as e:                                            # noqa: BLE001  (any exception is an outcome)
        return (type(e).__name__, str(e))


def _half(*s):
    return torch.zeros(s, dtype=torch.float16)


def bad_calls():
    x, y, b = _half(2, 128), _half(2, 64), torch.zeros(1 << 16, dtype=torch.uint8)
    f = torch.zeros(64)
    return {
        "host tensors": lambda: ql.ql_w8a8_linear(x, b, f, None, 64, y, b),
        "x type": lambda: ql.ql_w8a8_linear(x.float(), b, f, None, 64, y, b),
        "x dimensions": lambda: ql.ql_w8a8_linear(x[0], b, f, None, 64, y, b),
        "y shape": lambda: ql.ql_w8a8_linear(x, b, f, None, 64, y[:, :32], b),
        "short blob": lambda: ql.ql_w8a8_linear(x, b[:100], f, None, 64, y, b),
        "sw type": lambda: ql.ql_w8a8_linear(x, b, f.double(), None, 64, y, b),
        "sw None": lambda: ql.ql_w8a8_gemm(b, f, 2, 128, b, None, None, 64, y, b),
        "bias type": lambda: ql.ql_w4a8_linear(x, b, 128, f, 64, y, b),
        "group": lambda: ql.ql_w4a8_linear(x, b, 64, None, 64, y, b),
        "N float": lambda: ql.ql_w4a8_linear(x, b, 128, None, 64.0, y, b),
        "short codes": lambda: ql.ql_w4a8_gemm(b[:10], f, 2, 128, b, 128, None, 64, y, b),
        "K": lambda: ql.ql_w8a8_gemm(b, f, 2, 100, b, f, None, 64, y, b),
        "no sx": lambda: ql.ql_quant_act_per_token(x, None, b, None),
        "columns": lambda: ql.ql_quant_act_swiglu(_half(2, 129), None, b, f),
        "gamma type": lambda: ql.ql_quant_act_rmsnorm(x, f, 1e-5, None, b, f),
        "eps text": lambda: ql.ql_quant_act_rmsnorm(x, x[0], "eps", None, b, f),
        "block": lambda: ql.ql_quant_act_per_token_transformed(x, None, 3, None, b, f),
        "not a tensor": lambda: ql.ql_quant_act_per_token(np.zeros((2, 128), np.float16), None, b, f),
    }


@pytest.mark.parametrize("name", sorted(bad_calls()))
def test_what_is_wrong_is_reported_as_before(name, monkeypatch):
    ql.lib()
    assert ql._native is not None
    with_native = _outcome(bad_calls()[name])
    monkeypatch.setattr(ql, "_native", None)
    assert with_native == _outcome(bad_calls()[name]) and with_native[0] != "returned"


@pytest.mark.gpu
@pytest.mark.parametrize("M,K,N", [(1, 256, 64), (3, 512, 72), (40, 256, 520)])
def test_same_results_and_errors_on_the_gpu(M, K, N, monkeypatch):
    import gpu_util as G
    from paper_2512_23367_amd import synth
    ql.lib()
    x = G.dev(synth.activations(M, 2 * K, 0, "single"))
    w = synth.weights(N, K, 0, "single")
    g8, g4 = G.gpu_quant_weight(w, 8, 0), G.gpu_quant_weight(w, 4, 128)
    bias = G.dev(synth.bias(N, 0, "single"))
    gamma = x[0, :K].contiguous()
    sw = G.dev(g8["scales"])

    class Sub(torch.Tensor):
        pass

    def results():
        ws = G.empty_bytes(ql.ql_workspace_bytes(M, N, K, 8))
        out = []
        for xx in (x[:, :K], x[:, K:].contiguous(), torch.nn.Parameter(x[:, :K].contiguous()), x[:, :K].as_subclass(Sub)):
            for b in (None, bias):
                y = torch.zeros((M, (N + 15) // 8 * 8), dtype=torch.float16, device=G.DEV)
                ql.ql_w8a8_linear(xx, g8["kernel"], sw, b, N, y[:, :N], ws)
                out.append(y)
                y = torch.zeros_like(y)
                ql.ql_w4a8_linear(xx, g4["kernel"], 128, b, np.int64(N).item(), y[:, :N], ws)
                out.append(y)
        rm, xk, sx = torch.zeros((M, K), dtype=torch.int8, device=G.DEV), G.empty_bytes(ql.ql_act_kernel_bytes(M, K)), torch.zeros(M, device=G.DEV)
        for f in (lambda: ql.ql_quant_act_per_token(x[:, :K], rm, xk, sx), lambda: ql.ql_quant_act_rmsnorm(x[:, :K], gamma, 1e-5, rm, xk, sx),
                  lambda: ql.ql_quant_act_swiglu(x, rm, xk, sx), lambda: ql.ql_quant_act_per_token_transformed(x[:, :K], None, 64, rm, xk, sx)):
            xk.zero_()
            f()
            out += [rm.clone(), xk.clone(), sx.clone()]
        y = torch.zeros((M, (N + 7) // 8 * 8), dtype=torch.float16, device=G.DEV)
        ql.ql_w8a8_gemm(xk, sx, M, K, g8["kernel"], sw, bias, N, y[:, :N])
        out.append(y.clone())
        ql.ql_w4a8_gemm(xk, sx, M, K, g4["kernel"], 128, None, N, y[:, :N], ws)
        out.append(y.clone())
        ql.ql_w8a8_linear(x[:0, :K], g8["kernel"], sw, None, N, y[:0, :N], ws)                 # no tokens: nothing to do
        torch.cuda.synchronize()
        errors = [_outcome(f) for f in (lambda: ql.ql_w8a8_linear(x[:, :K], g8["kernel"], sw, None, N, y[:, :N], ws[:16]),
                                        lambda: ql.ql_w8a8_linear(x[:, :K], g8["kernel"], sw, None, N, y[:, :N], None),
                                        lambda: ql.ql_quant_act_per_token(x[:, 1:K + 1], rm, xk, sx),
                                        lambda: ql.ql_quant_act_rmsnorm(x[:, :K], gamma, -1.0, rm, xk, sx))]
        return out, errors

    native, native_errors = results()
    monkeypatch.setattr(ql, "_native", None)
    python, python_errors = results()
    assert all(torch.equal(p.view(torch.uint8), q.view(torch.uint8)) for p, q in zip(native, python))
    assert native_errors == python_errors and all(e[0] in ("QlError", "ValueError", "TypeError") for e in native_errors)
