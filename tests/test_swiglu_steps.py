"""The shortened step sequence of the SwiGLU kernels (fused operations, adjusted coefficients) against the oracle's, bit for bit
for every finite fp16 gate, with the constants read from the source."""
import ctypes
import ctypes.util
import os
import re

import numpy as np

import oracle

CSRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_2512_23367_amd", "csrc")


def test_every_gate():
    src = open(os.path.join(CSRC, "quant_math.h")).read()
    body = src[src.index("exp_steps(float t)"):src.index("reciprocal_of_sum(float d)")]
    c = [float.fromhex(h) for h in re.findall(r"(0x1\.[0-9a-f]+p-\d+)f", body)]
    assert len(c) == 3 and body.count("__builtin_fmaf") == 7
    libm = ctypes.CDLL(ctypes.util.find_library("m"))
    libm.fmaf.restype, libm.fmaf.argtypes = ctypes.c_float, [ctypes.c_float] * 3
    F = np.float32

    def fma(a, b, c):
        a, b, c = np.broadcast_arrays(a, b, c)
        return np.array([libm.fmaf(*v) for v in zip(a.tolist(), b.tolist(), c.tolist())], F)

    g = np.arange(65536, dtype=np.uint32).astype(np.uint16).view(np.float16)
    g = g[np.isfinite(g)]
    gu = np.stack([g, np.ones_like(g)], axis=1)
    want = oracle.swiglu_act(gu)[:, 0]
    t = np.clip(-g.astype(F), F(-80), F(80))
    z = fma(t, F(1.4426950408889634), F(12582912))
    n = z - F(12582912)
    r = fma(-n, F(0.693359375), t)
    r = r - n * F(-2.12194440e-4)
    p = F(c[0])
    for k in (F(c[1]), F(c[2]), F(1 / 24), F(1 / 6), F(0.5)):
        p = fma(p, r, k)
    p = p * r + F(1)
    p = p * r + F(1)
    e = ((z.view(np.uint32) << np.uint32(23)) + p.view(np.uint32)).view(F)
    got = g.astype(F) * (F(1) / (F(1) + e)) * F(1)
    assert got.dtype == F and (got.view(np.uint32) == want.view(np.uint32)).all()
