"""The kernel for few blocks and a short contraction takes 513 to 639 k like its neighbours on either side."""
import pytest
import torch

from paper_1908_00213_amd import binding as B
from tests.test_gpu_gemm_parts import operand
from tests.util import empty, host

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("layout", ["km", "mk", "mm"])
@pytest.mark.parametrize("shape", [(44, 15, 512), (44, 15, 513), (44, 15, 568), (129, 65, 577), (64, 33, 639), (64, 384, 640), (24, 40, 1024)])
@pytest.mark.parametrize("pad", [0, 3])
def test_every_k_up_to_1024(layout, shape, pad):
    m, n, k = shape
    gen = torch.Generator().manual_seed(m + n + k)
    a, b = (torch.randint(-9, 10, s, generator=gen).float().numpy() for s in ((m, k), (n, k)))
    A, Bm, C = operand(a, layout[0] == "k", pad), operand(b, layout[1] == "k", pad).t(), empty((m, n))
    assert B.gemm_plan_kernel(A, Bm, C, True) == "small" and B.gemm_workspace_bytes(A, Bm, C) == 0
    assert (host(B.gemm(A, Bm, C)) == a.astype("f8") @ b.T.astype("f8")).all()
