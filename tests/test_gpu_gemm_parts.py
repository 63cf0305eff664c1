"""fp32 products on the bfloat16 matrix cores: every operand value as the sum of three bfloat16 parts.

Small integers come out bit for bit (their parts beyond the first are zero), random operands with an error
against 64 bits no larger than the fp32 matrix instruction's, element by element down to subnormal numbers, and operands
whose sums overflow when scaled by 2^48 (infinities and NaN among them) exactly as the instruction computes them."""
import numpy as np
import pytest
import torch

from paper_1908_00213_amd import binding as B
from oracle import oracle as O
from tests.util import TOL_SUM, check, dev, empty, host, ws

pytestmark = pytest.mark.gpu
RNG = np.random.default_rng(19080)


def operand(a, unit_along_k, pad):
    """`a` (rows, k) as a device view with the wanted unit stride; pad: extra elements per stored row"""
    stored = a if unit_along_k else a.T
    buf = torch.full((stored.shape[0], stored.shape[1] + pad), float("nan"), device="cuda")
    view = buf[:, :stored.shape[1]]
    view.copy_(torch.from_numpy(np.ascontiguousarray(stored)))
    return view if unit_along_k else view.t()


def product(a, b, layout, tile, splits=1, pad=0, **kw):
    """a (m, k) @ b (n, k).T on the three-part kernel (tile 0 / 1) or, tile None, off it"""
    A, Bm = operand(a, layout[0] == "k", pad), operand(b, layout[1] == "k", pad).t()
    B.gemm_plan_override(-1 if tile is None else tile, splits, 0 if tile is None else 4)
    try:
        C = kw.pop("C", None)
        C = empty((a.shape[0], b.shape[0])) if C is None else C
        need = B.gemm_workspace_bytes(A, Bm, C)
        assert (need > 0) == (splits > 1)
        return host(B.gemm(A, Bm, C, ws=ws(need), **kw))
    finally:
        B.gemm_plan_override()


@pytest.mark.parametrize("tile", [0, 1])
@pytest.mark.parametrize("layout", ["kk", "km", "mk", "mm"])
@pytest.mark.parametrize("shape", [(1, 1, 1), (64, 64, 64), (65, 63, 33), (128, 128, 32), (130, 260, 95), (129, 127, 260), (200, 72, 129)])
@pytest.mark.parametrize("pad", [0, 1, 2, 4])
def test_exact_integers(tile, layout, shape, pad):
    # edges of tiles, one to five tile steps with and without a remainder, rows that allow 16-, 8- and 4-byte
    # pieces; the padding holds NaN, which must never reach C
    m, n, k = shape
    a, b = (RNG.integers(-9, 10, size=s).astype(np.float32) for s in ((m, k), (n, k)))
    got = product(a, b, layout, tile, pad=pad)
    assert np.array_equal(got, a.astype(np.float64) @ b.T.astype(np.float64))
    if k >= 129:
        assert np.array_equal(product(a, b, layout, tile, splits=2, pad=pad), got)


@pytest.mark.parametrize("tile", [0, 1])
@pytest.mark.parametrize("layout", ["kk", "km", "mm"])
@pytest.mark.parametrize("k", [64, 650, 3000])
def test_error_no_larger_than_the_instruction(tile, layout, k):
    # wide spread of magnitudes along k, so that large and small terms meet in one sum
    a, b = (RNG.standard_normal(s).astype(np.float32) * np.exp2(RNG.integers(-12, 13, size=(1, k))).astype(np.float32) for s in ((150, k), (140, k)))
    ref = a.astype(np.float64) @ b.T.astype(np.float64)
    err = lambda x: np.linalg.norm(x - ref) / np.linalg.norm(ref)
    got = product(a, b, layout, tile)
    assert err(got) <= err(product(a, b, layout, None))
    check(got, O.gemm(a, b.T), TOL_SUM, O.gemm(np.abs(a), np.abs(b).T), "against the oracle")


@pytest.mark.parametrize("tile", [0, 1])
@pytest.mark.parametrize("layout", ["kk", "km", "mk", "mm"])
def test_errors_have_no_preferred_sign(tile, layout):
    # the gradient of a softmax (one -1, the rest small and positive) times weights, a product whose results are summed over
    # rows afterwards: n independent errors of relative size e average to e / sqrt(n), here within six of those
    m, n, k = 2048, 640, 10000
    g = torch.Generator(device="cuda").manual_seed(5)
    d = torch.softmax(torch.randn(m, k, generator=g, device="cuda"), 1)
    d[torch.arange(m, device="cuda"), torch.randint(0, k, (m,), generator=g, device="cuda")] -= 1
    w = torch.randn(n, k, generator=g, device="cuda")
    A, Bm = (x if l == "k" else x.t().contiguous().t() for x, l in zip((d, w), layout))
    ref = d.double() @ w.double().t()
    B.gemm_plan_override(tile, 1, 4)
    try:
        err = B.gemm(A, Bm.t(), empty((m, n))).double() - ref
    finally:
        B.gemm_plan_override()
    e = float(err.norm() / ref.norm())
    assert e < 8e-7                                   # (the fp32 instruction's)
    assert abs(float(err.mean() / ref.square().mean().sqrt())) < 6 * e / (m * n) ** 0.5


@pytest.mark.parametrize("tile", [0, 1])
@pytest.mark.parametrize("layout", ["kk", "km", "mk", "mm"])
def test_values_the_parts_cannot_carry(tile, layout):
    a, b = RNG.standard_normal((200, 100)).astype(np.float32), RNG.standard_normal((150, 100)).astype(np.float32)
    b[:, 7] = np.float32(1.5)                       # exact in bfloat16: its lower parts are zero
    for place in ("inf", "nan", "both", "huge", "tiny row", "tiny", "zero row"):
        x = a.copy()
        if place in ("inf", "both"):
            x[3, 7], x[150, 0] = np.inf, -np.inf
        if place in ("nan", "both"):
            x[70, 5] = np.nan
        if place == "huge":
            x[199, 99], x[10, 3] = 3.4e38, -1e30
        if place == "tiny row":
            x[5] *= np.float32(1e-36)
        if place == "tiny":
            x *= np.float32(1e-30)
        if place == "zero row":
            x[140] = 0
        got, want = product(x, b, layout, tile), product(x, b, layout, None)
        assert np.array_equal(np.isnan(got), np.isnan(want)), place
        assert np.array_equal(got[np.isinf(want)], want[np.isinf(want)]) and np.array_equal(np.isinf(got), np.isinf(want)), place
        fin = np.isfinite(want) & np.isfinite(got)
        # both sum 100 terms in fp32: each within 100 * 2^-24 of the sum of magnitudes
        xs = np.nan_to_num(np.abs(x), nan=0.0, posinf=0.0).astype(np.float64)
        S = xs @ np.abs(b).T.astype(np.float64)
        assert np.all(np.abs(got[fin] - want[fin]) <= 2 * 100 * 2.0 ** -24 * S[fin]), place


@pytest.mark.parametrize("tile", [0, 1])
@pytest.mark.parametrize("layout", ["kk", "km", "mk", "mm"])
@pytest.mark.parametrize("exponent", [-90, -112, -120, -126, -135, -149])
def test_small_values_beside_large_ones(tile, layout, exponent):
    # a row that holds a 1 and a small value, against a row that is zero where the 1 stands: one product is the whole
    # result.  Its error: the three partial products left out, 2 * 2^-8 * 2^-17 = 2^-24 of it at most (plus 2^-34), the
    # rounding of the five small ones' sum, 5 * 2^-8 * 2^-24, and of the result, 2^-24 or half a step of 2^-149
    m, n, k = 70, 66, 50
    small = (np.float64(2.0) ** exponent * RNG.uniform(1, 2, m)).astype(np.float32)
    a, b = np.zeros((m, k), np.float32), np.zeros((n, k), np.float32)
    a[:, 0], a[:, 19] = 1, small
    b[:, 19] = RNG.uniform(1, 2, n)
    ref = a[:, 19:20].astype(np.float64) * b[:, 19].astype(np.float64)
    bound = (2 + 5 * 2.0 ** -8 + 2.0 ** -10) * 2.0 ** -24 * ref + 2.0 ** -150
    assert np.all(np.abs(product(a, b, layout, tile) - ref) <= bound)
    assert np.all(np.abs(product(b, a, layout, tile) - ref.T) <= bound.T)


@pytest.mark.parametrize("tile", [0, 1])
@pytest.mark.parametrize("layout", ["kk", "km", "mk", "mm"])
@pytest.mark.parametrize("ea,eb", [(-60, -60), (-20, -100), (-75, -75), (-130, 10), (30, 30), (33, 33), (36, 36), (40, -40), (60, 60)])
def test_scaled_operands(tile, layout, ea, eb):
    # operands far from 1 on both sides of the sums that the scaled parts take (2^80); a sum of 100 terms is within
    # 100 * 2^-24 of the sum of magnitudes, and no step loses more than a subnormal one
    a, b = (np.ldexp(RNG.standard_normal(s), e).astype(np.float32) for s, e in (((90, 100), ea), ((80, 100), eb)))
    ref, S = a.astype(np.float64) @ b.T.astype(np.float64), np.abs(a).astype(np.float64) @ np.abs(b).T.astype(np.float64)
    assert np.all(np.abs(product(a, b, layout, tile) - ref) <= 100 * 2.0 ** -24 * S + 100 * 2.0 ** -149)


@pytest.mark.parametrize("tile", [0, 1])
@pytest.mark.parametrize("layout", ["kk", "mm"])
@pytest.mark.parametrize("k", [1, 129, 4096])
def test_largest_sums(tile, layout, k):
    # every value the same, sums on both sides of 2^80 (where the scaled ones overflow) and of fp32's own limit
    for e in (30, 39.9, 40, 40.1, 48, 63.9, 90, 103, 104, 127):
        a, b = np.full((70, k), 2.0 ** e, np.float32), np.full((66, k), -(2.0 ** e), np.float32)
        got, ref = product(a, b, layout, tile), -k * np.float64(a[0, 0]) ** 2
        if ref < -3.4028235e38:
            assert np.all(np.isneginf(got)), e
        else:
            assert np.all(np.abs(got - ref) <= k * 2.0 ** -24 * -ref), e


@pytest.mark.parametrize("tile", [0, 1])
def test_one_tile_is_computed_again(tile):
    # a sum beyond the scaled range in one tile (and one half of K) of a larger product, split or not; the others keep theirs
    a, b = RNG.standard_normal((300, 700)).astype(np.float32), RNG.standard_normal((290, 700)).astype(np.float32)
    a[140, 650], b[133, 650] = 2.0 ** 45, 2.0 ** 45
    ref, S = a.astype(np.float64) @ b.T.astype(np.float64), np.abs(a).astype(np.float64) @ np.abs(b).T.astype(np.float64)
    for splits in (1, 2):
        assert np.all(np.abs(product(a, b, "km", tile, splits) - ref) <= 700 * 2.0 ** -24 * S)


@pytest.mark.parametrize("tile", [0, 1])
@pytest.mark.parametrize("splits", [1, 3])
def test_epilogues(tile, splits):
    # vector and element-wise epilogue paths (an interior of full 16-byte groups and ragged edges), cut along K or not
    m, n, k = 190, 205, 800
    a, b = RNG.standard_normal((m, k)).astype(np.float32), RNG.standard_normal((n, k)).astype(np.float32) / 28
    bias, aux, c0 = (RNG.standard_normal(s).astype(np.float32) for s in ((n,), (m, n), (m, n)))
    lin, S = O.gemm(a, b.T), O.gemm(np.abs(a), np.abs(b).T)
    run = lambda **kw: product(a, b, "km", tile, splits, **kw)
    for C in (lambda: empty((m, n)), lambda: empty((m, n + 3))[:, :n]):
        pre = C()
        z = lin + bias
        check(run(C=C(), epilogue="bias_gelu", bias=dev(bias), preact_out=pre), O.elementwise("gelu", [z]), TOL_SUM, S + np.abs(bias), "bias_gelu")
        check(host(pre), z, TOL_SUM, S + np.abs(bias), "pre-activation")
        check(run(C=C(), epilogue="bias_relu", bias=dev(bias)), np.maximum(z, 0), TOL_SUM, S + np.abs(bias), "bias_relu")
        check(run(C=C(), epilogue="relu_bwd", aux=dev(aux)), np.where(aux > 0, lin, 0.0), TOL_SUM, S, "relu_bwd")
        old = C()
        old.copy_(dev(c0))
        check(run(C=old, alpha=0.5, beta=-2.0), 0.5 * lin - 2.0 * c0, TOL_SUM, S + 2 * np.abs(c0), "alpha beta")


def test_planner_leaves_few_tiles_to_the_instruction():
    # one or two tiles and a long K: cut along K on the fp32 instruction (44x15x568 9.2 us, here 15.7; 36x80x5127 17.7 and 29.3)
    for m, n, k, pad in ((44, 15, 568, 0), (36, 80, 5127, 2), (336, 53, 578, 0)):
        A, Bm = (torch.empty(r, k + pad, device="cuda")[:, :k] for r in (m, n))
        assert not B.gemm_plan_eight_waves(A, Bm.t(), empty((m, n)), True) and B.gemm_plan(A, Bm.t(), empty((m, n)), True)[2] > 1


def test_planner_takes_the_kernel_and_results_repeat():
    # mid-size and large products without any override; the same call twice gives the same bits
    for m, n, k in ((1024, 1000, 1000), (1100, 1300, 700)):
        A, Bm = torch.randn(m, k, device="cuda"), torch.randn(n, k, device="cuda").t()
        assert B.gemm_plan_eight_waves(A, Bm, empty((m, n)), True) and B.gemm_plan_kernel(A, Bm, empty((m, n)), True) == "parts"
        need = B.gemm_workspace_bytes(A, Bm, empty((m, n)))
        x, y = (B.gemm(A, Bm, empty((m, n)), ws=ws(need)) for _ in range(2))
        assert torch.equal(x, y)
        ref = A.double() @ Bm.double()
        assert float((x.double() - ref).norm() / ref.norm()) < 6e-7


@pytest.mark.parametrize("layout", ["kk", "km", "mk", "mm"])
@pytest.mark.parametrize("shape", [(1, 1, 1), (31, 33, 7), (32, 10, 100), (33, 65, 255), (100, 64, 256), (64, 70, 257), (500, 512, 512), (32, 100, 784), (33, 65, 641), (420, 400, 1021)])
@pytest.mark.parametrize("pad", [0, 3])
def test_small_products(layout, shape, pad):
    # few blocks and a short contraction: edges of the 32x32 block and of the chunks and batches along K, any alignment
    m, n, k = shape
    a, b = (RNG.integers(-9, 10, size=s).astype(np.float32) for s in ((m, k), (n, k)))
    bias, aux, c0 = (RNG.integers(-9, 10, size=s).astype(np.float32) for s in ((n,), (m, n), (m, n)))
    A, Bm = operand(a, layout[0] == "k", pad), operand(b, layout[1] == "k", pad).t()
    assert B.gemm_plan_kernel(A, Bm, empty((m, n)), True) == "small"
    assert B.gemm_plan(A, Bm, empty((m, n)), True) == (0, False, 1) and B.gemm_workspace_bytes(A, Bm, empty((m, n))) == 0
    lin = a.astype(np.float64) @ b.T.astype(np.float64)
    new = lambda: operand(c0, True, 1 + pad)
    assert np.array_equal(host(B.gemm(A, Bm, new())), lin)
    assert np.array_equal(host(B.gemm(A, Bm, new(), alpha=2.0, beta=-1.0)), 2 * lin - c0)
    assert np.array_equal(host(B.gemm(A, Bm, new(), epilogue="bias_relu", bias=dev(bias))), np.maximum(lin + bias, 0))
    assert np.array_equal(host(B.gemm(A, Bm, new(), epilogue="relu_bwd", aux=dev(aux))), np.where(aux > 0, lin, 0))
    low = torch.empty(m, n, device="cuda", dtype=torch.bfloat16)
    got = B.gemm(A, Bm, new(), epilogue="bf16_copy", preact_out=low)
    assert np.array_equal(host(got), lin) and torch.equal(low, got.to(torch.bfloat16))
    scale = np.float32(0.01)
    z = lin * 1e-4 + bias
    pre = empty((m, n))
    out = B.gemm(operand(a * scale, layout[0] == "k", pad), operand(b * scale, layout[1] == "k", pad).t(), new(), epilogue="bias_gelu", bias=dev(bias), preact_out=pre)
    S = np.abs(a).astype(np.float64) @ np.abs(b).T * 1e-4 + np.abs(bias)
    check(host(pre), z, TOL_SUM, S, "pre-activation")
    check(host(out), O.elementwise("gelu", [z]), TOL_SUM, S, "bias_gelu")
