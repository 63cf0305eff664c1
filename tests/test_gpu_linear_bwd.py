"""chn_linear_bwd -- weight, bias and input gradient of a fully connected layer in one call -- against numpy.

The inputs are small integers: every product and every sum is exact in fp32, in whatever order, and results are compared as they are
(bfloat16 input gradients after the one rounding that both sides make).  Sizes: edges of the 16- and 64-blocks, remainders of
the chunks along the contraction (whose length is the batch for dW, the outputs for dx), and sizes of each kernel's range and beyond."""
import numpy as np
import pytest
import torch

from paper_1908_00213_amd import binding as B

pytestmark = pytest.mark.gpu
RNG = np.random.default_rng(77)

SHAPES = [(1, 1, 1), (2, 3, 5), (32, 10, 100), (32, 100, 784), (33, 17, 65), (31, 15, 16), (64, 64, 64), (257, 16, 48), (600, 24, 40), (1000, 20, 33),   # small kernel
          (1024, 1000, 1000), (1023, 997, 1001), (1025, 200, 1030), (700, 260, 520), (2000, 129, 190), (640, 1000, 784),                    # one 64x64 tile a unit or two
          (1024, 10, 1000), (2500, 70, 3000), (1100, 1030, 1300), (4100, 515, 260), (3000, 650, 1999)]                                    # sums in parts, or none


def _dev(a, dt):
    """On the GPU, rows 16 bytes aligned in bfloat16 (where the direct-copy kernel wants them), packed in fp32."""
    t = torch.from_numpy(a).cuda()
    if dt is torch.float32:
        return t
    m, n = a.shape
    buf = torch.zeros(m, (n + 7) // 8 * 8, dtype=dt, device="cuda")
    buf[:, :n] = t.to(dt)
    return buf[:, :n]


@pytest.mark.parametrize("w_layout", ["rows", "columns"])
@pytest.mark.parametrize("dt", [torch.float32, torch.bfloat16])
@pytest.mark.parametrize("shape", SHAPES)
def test_gradients_are_exact(shape, dt, w_layout):
    M, N, K = shape
    dv, W, x, aux = (RNG.integers(-4, 5, size=s).astype(np.float32) for s in ((M, N), (N, K), (M, K), (M, K)))
    d, h, a = _dev(dv, dt), _dev(x, dt), _dev(aux, dt)
    w = _dev(W, dt) if w_layout == "rows" else _dev(np.ascontiguousarray(W.T), dt).t()
    want_dx = np.where(aux > 0, dv.astype(np.float64) @ W, 0.0)
    for with_dx in (True, False):
        for with_db in (True, False):
            dW, db = torch.full((N, K), 7.0, device="cuda"), torch.full((N,), 7.0, device="cuda") if with_db else None
            dx = torch.full((M, K), 7.0, device="cuda", dtype=dt) if with_dx else None
            ws = torch.empty(max(256, B.linear_bwd_workspace_bytes(d, w, h, dx, dW)), dtype=torch.uint8, device="cuda")
            B.linear_bwd(d, w if with_dx else None, h, dW, db, dx, "relu_bwd" if with_dx else "none", a if with_dx else None, ws=ws)
            assert np.array_equal(dW.cpu().numpy(), dv.T.astype(np.float64) @ x), "dW"
            if with_db:
                assert np.array_equal(db.cpu().numpy(), dv.astype(np.float64).sum(0)), "db"
            if with_dx:
                assert torch.equal(dx.cpu(), torch.from_numpy(want_dx).float().to(dt)), "dx"


@pytest.mark.parametrize("dt", [torch.float32, torch.bfloat16])
@pytest.mark.parametrize("shape", SHAPES)
def test_weight_gradient_stored_by_columns(shape, dt):
    # the gradient of weights kept as (inputs, outputs); with too little workspace as with enough
    M, N, K = shape
    dv, x = (RNG.integers(-4, 5, size=s).astype(np.float32) for s in ((M, N), (M, K)))
    d, h = _dev(dv, dt), _dev(x, dt)
    dW, db = torch.empty(K, N, device="cuda"), torch.empty(N, device="cuda")
    need = B.linear_bwd_workspace_bytes(d, None, h, None, dW.t())
    for size in {max(256, need), B.reduce_axis_workspace_bytes(d, 0) + 256}:
        dW.fill_(7.0), db.fill_(7.0)
        B.linear_bwd(d, None, h, dW.t(), db, ws=torch.empty(size, dtype=torch.uint8, device="cuda"))
        assert np.array_equal(dW.cpu().numpy(), x.T.astype(np.float64) @ dv), "dW"
        assert np.array_equal(db.cpu().numpy(), dv.astype(np.float64).sum(0)), "db"


@pytest.mark.parametrize("shape", [(32, 100, 784), (1024, 1000, 1000)])
def test_values_that_the_three_parts_cannot_hold(shape):
    # infinities and values beyond 2^80 have a tile of the large kernel multiplied again; every row sum is its own
    M, N, K = shape
    dv, W, x = (RNG.integers(-4, 5, size=s).astype(np.float32) for s in ((M, N), (N, K), (M, K)))
    dv[3, 5], x[7, 9] = np.inf, 2.0 ** 100
    d, w, h = (torch.from_numpy(v).cuda() for v in (dv, W, x))
    dW, db, dx = torch.empty(N, K, device="cuda"), torch.empty(N, device="cuda"), torch.empty(M, K, device="cuda")
    B.linear_bwd(d, w, h, dW, db, dx)
    with np.errstate(invalid="ignore"):
        for got, want in ((dW, dv.T.astype(np.float64) @ x), (db, dv.astype(np.float64).sum(0)), (dx, dv.astype(np.float64) @ W)):
            got = got.cpu().numpy()
            assert np.array_equal(np.isnan(got), np.isnan(want))
            ok = ~np.isnan(want)
            # 2^100 times a small integer beside integers: the fp32 sum keeps the large term alone
            big = np.isfinite(want) & (np.abs(want) > 2.0 ** 50)
            assert np.array_equal(got[ok & ~big], want[ok & ~big]) and np.allclose(got[big], want[big], rtol=1e-6)


@pytest.mark.parametrize("shape", [(32, 100, 100), (1024, 1000, 1000)])
def test_outputs_over_inputs_are_written_in_order(shape):
    # dx may take x's place, as with the three separate calls: dW is made from x before
    M, N, K = shape
    dv, W, x = (torch.from_numpy(RNG.integers(-4, 5, size=s).astype(np.float32)).cuda() for s in ((M, N), (N, K), (M, K)))
    want_dW, want_dx = dv.double().t() @ x.double(), dv.double() @ W.double()
    dW, db = torch.empty(N, K, device="cuda"), torch.empty(N, device="cuda")
    B.linear_bwd(dv, W, x, dW, db, x)
    assert torch.equal(dW.double(), want_dW) and torch.equal(x.double(), want_dx) and torch.equal(db.double(), dv.double().sum(0))


def test_refused_calls():
    f = lambda *s: torch.empty(*s, device="cuda")
    for args, kw in (((f(4, 3), f(3, 5), f(4, 5), f(3, 5), f(4)), {}), ((f(4, 3), f(3, 5), f(4, 5), f(5, 3)), {}), ((f(4, 3), None, f(4, 5), f(3, 5), None, f(4, 5)), {}),
                     ((f(4, 3), f(3, 5), f(4, 5), f(3, 5), None, f(4, 5)), {"epilogue": "relu_bwd"}), ((f(4, 3), f(3, 5), f(4, 5), f(3, 5), None, f(4, 5)), {"epilogue": "bias"})):
        with pytest.raises(B.ChnError):
            B.linear_bwd(*args, **kw)
