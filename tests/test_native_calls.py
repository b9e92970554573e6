"""Native argument marshalling (csrc/pycall.cpp) against the Python of binding.py: it makes a call only where binding.py would make
the same one, and whatever is wrong is reported by binding.py as without it."""
import ctypes

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


# ---- On the device, where every check of the native code is reached.  The native code is bound to stand-ins that only note the call: a wrong
# argument that it lets through is a failed test and no launch.
K, N, M, GROUP = 128, 64, 2, 128
PYTHON = {"w8a8_linear": "ql_w8a8_linear", "w4a8_linear": "ql_w4a8_linear", "w8a8_gemm": "ql_w8a8_gemm", "w4a8_gemm": "ql_w4a8_gemm",
          "quant_act": "ql_quant_act_per_token", "quant_rmsnorm": "ql_quant_act_rmsnorm", "quant_swiglu": "ql_quant_act_swiglu",
          "quant_transformed": "ql_quant_act_per_token_transformed"}
BOUND = ("ql_weight_bytes", "ql_act_kernel_bytes", "ql_w8a8_linear", "ql_w4a8_linear", "ql_w8a8_gemm", "ql_w4a8_gemm", "ql_quant_act_per_token",
         "ql_quant_act_rmsnorm", "ql_quant_act_swiglu", "ql_quant_act_per_token_transformed")


def bind_stand_ins(module):
    """Binds the native module to functions that note their name and return QL_OK (size queries: the library's).  Returns the notes, and
    what has to be kept alive while it is bound."""
    lib, called, kept, addresses = ql.lib(), [], [], []
    for name in BOUND:
        f = getattr(lib, name)
        if not name.endswith("_bytes"):
            f = ctypes.CFUNCTYPE(ctypes.c_int, *f.argtypes)(lambda *a, name=name: called.append(name) or 0)
            kept.append(f)
        addresses.append(ctypes.cast(f, ctypes.c_void_p).value)
    module.bind(tuple(addresses))
    return called, kept


def good_arguments():
    def dev(*shape, dtype=torch.float16):
        return torch.zeros(shape, dtype=dtype, device="cuda:0")
    x, y, bias, gamma, f = dev(M, K), dev(M, N), dev(N), dev(K), dev(K, dtype=torch.float32)
    b8, b4 = (dev(ql.ql_weight_bytes(N, K, b, g)[2], dtype=torch.uint8) for b, g in ((8, 0), (4, GROUP)))
    xq, rm, ws = dev(ql.ql_act_kernel_bytes(M, K), dtype=torch.uint8), dev(M, K, dtype=torch.int8), dev(1 << 16, dtype=torch.uint8)
    sw, sx = f[:N], f[:M]
    return {"w8a8_linear": [x, b8, sw, bias, N, y, ws], "w4a8_linear": [x, b4, GROUP, bias, N, y, ws],
            "w8a8_gemm": [xq, sx, M, K, b8, sw, bias, N, y, ws], "w4a8_gemm": [xq, sx, M, K, b4, GROUP, bias, N, y, ws],
            "quant_act": [x, rm, xq, sx], "quant_rmsnorm": [x, gamma, 1e-5, rm, xq, sx], "quant_swiglu": [dev(M, 2 * K), rm, xq, sx],
            "quant_transformed": [x, f, 64, rm, xq, sx]}


def _strided(t):
    return torch.zeros((t.shape[0], 2 * t.shape[1]), dtype=t.dtype, device=t.device)[:, ::2]


# function, argument, what is wrong with it, the wrong argument made of the right one
WRONG = [(f, i, what, make) for f, i, kinds in [
    ("w8a8_linear", 0, "matrix"), ("w8a8_linear", 1, "blob"), ("w8a8_linear", 2, "floats"), ("w8a8_linear", 3, "bias"), ("w8a8_linear", 4, "number"),
    ("w8a8_linear", 5, "output"), ("w8a8_linear", 6, "host"), ("w4a8_linear", 0, "matrix"), ("w4a8_linear", 1, "blob"), ("w4a8_linear", 2, "group"),
    ("w4a8_linear", 3, "bias"), ("w4a8_linear", 4, "number"), ("w4a8_linear", 5, "output"), ("w4a8_linear", 6, "host"),
    ("w8a8_gemm", 0, "codes"), ("w8a8_gemm", 1, "sx"), ("w8a8_gemm", 2, "number"), ("w8a8_gemm", 3, "size"), ("w8a8_gemm", 4, "blob"), ("w8a8_gemm", 5, "count"),
    ("w8a8_gemm", 6, "bias"), ("w8a8_gemm", 7, "number"), ("w8a8_gemm", 8, "output"), ("w8a8_gemm", 9, "host"),
    ("w4a8_gemm", 0, "codes"), ("w4a8_gemm", 1, "sx"), ("w4a8_gemm", 2, "number"), ("w4a8_gemm", 3, "size"), ("w4a8_gemm", 4, "blob"), ("w4a8_gemm", 5, "group"),
    ("w4a8_gemm", 6, "bias"), ("w4a8_gemm", 7, "number"), ("w4a8_gemm", 8, "output"), ("w4a8_gemm", 9, "host"),
    ("quant_act", 0, "matrix"), ("quant_act", 1, "host"), ("quant_act", 2, "host"), ("quant_act", 3, "host"),
    ("quant_rmsnorm", 0, "matrix"), ("quant_rmsnorm", 1, "half"), ("quant_rmsnorm", 2, "text"), ("quant_rmsnorm", 3, "host"), ("quant_rmsnorm", 5, "host"),
    ("quant_swiglu", 0, "matrix"), ("quant_swiglu", 0, "odd"), ("quant_swiglu", 2, "host"),
    ("quant_transformed", 0, "matrix"), ("quant_transformed", 1, "host"), ("quant_transformed", 2, "size"), ("quant_transformed", 5, "host")]
    for what, make in {
        "matrix": {"fp32": lambda t: t.float(), "flat": lambda t: t[0], "strided": _strided, "host": lambda t: t.cpu()},
        "output": {"fp32": lambda t: t.float(), "narrow": lambda t: t[:, :32], "short": lambda t: t[:1], "strided": _strided, "host": lambda t: t.cpu()},
        "blob": {"a byte short": lambda t: t[:-1], "None": lambda t: None, "host": lambda t: t.cpu()},
        "codes": {"a byte short": lambda t: t[:-1], "host": lambda t: t.cpu()},
        "floats": {"fp64": lambda t: t.double(), "one short": lambda t: t[:-1], "None": lambda t: None, "host": lambda t: t.cpu()},
        "count": {"one short": lambda t: t[:-1], "None": lambda t: None, "host": lambda t: t.cpu()},
        "sx": {"fp64": lambda t: t.double(), "one short": lambda t: t[:-1], "host": lambda t: t.cpu()},
        "bias": {"fp32": lambda t: t.float(), "one short": lambda t: t[:-1], "host": lambda t: t.cpu()},
        "half": {"fp32": lambda t: t.float(), "host": lambda t: t.cpu()},
        "group": {"64": lambda n: 64, "float": float},
        "number": {"float": float, "text": str, "too many bits": lambda n: n + (1 << 40)},
        "size": {"float": float, "text": str},               # (one of too many bits loses them in ctypes)
        "text": {"text": lambda v: "eps", "None": lambda n: None},
        "odd": {"odd": lambda t: torch.zeros((M, 2 * K + 1), dtype=t.dtype, device=t.device)},
        "host": {"host": lambda t: t.cpu()},
    }[kinds].items()]


def not_refused(module):
    """What a native module does not hand back to binding.py of the table above, as texts."""
    called, kept = bind_stand_ins(module)
    stream, good, let_through = (lambda: 0), good_arguments(), []
    for f, args in good.items():
        assert getattr(module, f)(*args, stream) == 0 and called == [PYTHON[f]], f
        called.clear()
    for f, i, what, make in WRONG:
        args = list(good[f])
        args[i] = make(args[i])
        if getattr(module, f)(*args, stream) is not None or called:
            let_through.append(f"{f}, argument {i}: {what}")
        called.clear()
    del kept
    return let_through


@pytest.mark.gpu
def test_no_wrong_argument_passes_the_native_checks(monkeypatch):
    ql.lib()
    try:
        assert not_refused(ql._native) == []
        called, kept = bind_stand_ins(ql._native)
        for f, i, what, make in WRONG:                    # and binding.py says what is wrong with it, as without the native code
            args = list(good_arguments()[f])
            args[i] = make(args[i])
            call = getattr(ql, PYTHON[f])
            with_native = _outcome(lambda: call(*args))
            with monkeypatch.context() as m:
                m.setattr(ql, "_native", None)
                assert with_native == _outcome(lambda: call(*args)) and with_native[0] != "returned", (f, i, what)
        assert called == []
    finally:
        ql._bind_native(ql.lib())


@pytest.mark.gpu
def test_an_exception_while_the_stream_is_asked_for_is_passed_on():
    """A keyboard interrupt may arrive wherever Python code runs; here that is the function that knows the stream."""
    def interrupted():
        raise KeyboardInterrupt

    ql.lib()
    try:
        called, kept = bind_stand_ins(ql._native)
        with pytest.raises(KeyboardInterrupt):
            ql._native.quant_act(*good_arguments()["quant_act"], interrupted)
        assert called == [] and ql._native.quant_act(*good_arguments()["quant_act"], lambda: "no stream") is None
    finally:
        ql._bind_native(ql.lib())
