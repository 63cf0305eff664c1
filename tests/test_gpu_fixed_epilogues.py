"""bf16 products on the 64x64 tile that is copied straight to LDS: kernels made for one epilogue each, against the oracle.

Operands are small integers, so that sums are exact in fp32: results of every epilogue without a gelu are the sums after one rounding to C's
type, those with one stay within the bars of tests/util.py."""
import numpy as np
import pytest
import torch

from oracle import oracle as O
from paper_1908_00213_amd import binding as B
from tests.util import TOL_BF16, TOL_SUM, bf16r, check, dev, host

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("epilogue", ["none", "bias", "bias_relu", "bias_gelu", "relu_bwd", "gelu_bwd"])
@pytest.mark.parametrize("c_type", ["bf16", "f32"])
@pytest.mark.parametrize("layout", ["kk", "km", "mk", "mm"])
@pytest.mark.parametrize("shape", [(64, 64, 64), (1, 8, 8), (72, 200, 136), (256, 67, 64), (130, 129, 328)])      # whole tiles, edges, columns behind the last four
def test_each_epilogue(shape, layout, c_type, epilogue):
    m, n, k = shape                                          # (an operand that lies along M or N is copied straight in pieces of eight)
    m, n = m if layout[0] == "k" else (m + 7) // 8 * 8, n if layout[1] == "k" else (n + 7) // 8 * 8
    rng = np.random.default_rng(m + n + k)
    a, b = (rng.integers(-4, 5, size=(r, k)).astype(np.float32) for r in (m, n))
    bias, aux = rng.integers(-9, 10, size=n).astype(np.float32), rng.integers(-3, 4, size=(m, n)).astype(np.float32)

    def operand(v, along_k):                                 # rows on the 16-byte grid
        stored = v if along_k else v.T
        buf = torch.zeros(stored.shape[0], (stored.shape[1] + 7) // 8 * 8, device="cuda", dtype=torch.bfloat16)[:, :stored.shape[1]]
        buf.copy_(dev(stored, "bf16"))
        return buf if along_k else buf.t()
    A, Bm = operand(a, layout[0] == "k"), operand(b, layout[1] == "k").t()
    dtype, tol = (torch.bfloat16, TOL_BF16) if c_type == "bf16" else (torch.float32, TOL_SUM)
    C = torch.full((m, n + 4), 7.0, device="cuda", dtype=dtype)
    pre = torch.zeros(m, n, device="cuda", dtype=dtype) if epilogue == "bias_gelu" else None
    B.gemm_plan_override(0, 1, 1)                            # uncut, on the 64x64 tile, copied straight to LDS
    try:
        assert B.gemm_plan_kernel(A, Bm, C[:, :n], True) == "direct4" and B.gemm_plan(A, Bm, C[:, :n], True)[::2] == (0, 1)
        B.gemm(A, Bm, C[:, :n], alpha=2.0, epilogue=epilogue, bias=dev(bias) if epilogue.startswith("bias") else None,
               aux=dev(aux, c_type) if epilogue.endswith("bwd") else None, preact_out=pre)
    finally:
        B.gemm_plan_override()
    rounded = lambda v: (bf16r(v) if c_type == "bf16" else v).astype(np.float64)
    lin = 2.0 * (a.astype(np.float64) @ b.T.astype(np.float64))
    z = lin + bias if epilogue.startswith("bias") else lin
    assert bool((C[:, n:] == 7.0).all())
    got = host(C[:, :n])
    if epilogue == "bias_gelu":
        assert np.array_equal(host(pre), rounded(z))
        check(got, O.elementwise("gelu", [z]), tol, np.abs(z), epilogue)
    elif epilogue == "gelu_bwd":
        check(got, O.elementwise("gelu_bwd", [lin, aux.astype(np.float64)]), tol, np.abs(lin), epilogue)
    else:
        want = np.maximum(z, 0) if epilogue == "bias_relu" else np.where(aux > 0, z, 0) if epilogue == "relu_bwd" else z
        assert np.array_equal(got, rounded(want))
