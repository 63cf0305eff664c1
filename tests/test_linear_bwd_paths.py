"""chn_linear_bwd kernel by kernel: which one a call takes (queries of the library, no GPU), and on a GPU its results at those sizes.

Every row is on the 16-byte grid, where the kernels that leave the bias gradient's sums beside the weight gradient are chosen.  Inputs
are small integers: products and sums are exact in fp32 in whatever order, bfloat16 input gradients after one rounding."""
import pytest
import torch

from paper_1908_00213_amd import binding as B

F32, BF16 = torch.float32, torch.bfloat16

# (M, N, K): is it one launch with an input gradient and W by rows, by columns, and without input gradient; fp32 and bf16
ONE_LAUNCH = {
    (32, 10, 100): ((True, True, True), (False, False, False)),          # blocks of 16x16 (fp32)
    (600, 24, 40): ((True, True, True), (True, True, True)),             # ... and one 64x64 tile or two, copied straight to LDS (bf16)
    (64, 64, 64): ((True, True, True), (True, True, True)),
    (1024, 1000, 1000): ((True, False, True), (True, True, True)),       # 64x64 tiles: straight to the registers (fp32), to LDS (bf16)
    (1024, 400, 1000): ((True, True, True), (True, True, True)),
    (1024, 512, 512): ((False, False, False), (True, True, True)),       # the weight gradient on 32x32 blocks (fp32)
    (4096, 1024, 1024): ((False, False, False), (False, False, True)),   # the input gradient on 128x128 tiles (bf16)
    (2048, 512, 512): ((False, False, False), (False, False, False)),    # a cut product
    (1, 1, 1): ((False, False, False), (False, False, False)),
}
# (M, N, K): tile and K splits of a weight gradient that leaves the sums in parts; fp32 and bf16
IN_PARTS = {
    (2048, 512, 512): ((64, 4), (64, 4)),
    (4096, 520, 264): ((64, 5), (64, 5)),                    # ragged last tiles
    (16384, 264, 136): ((64, 16), (64, 16)),
    (1104, 1032, 1304): ((128, 2), (64, 1)),
    (4096, 1024, 1024): ((128, 4), (64, 1)),
    (8192, 784, 1000): ((128, 4), (128, 4)),
    (640, 1672, 2008): ((128, 1), (128, 1)),
    (2048, 2048, 2048): ((128, 1), (128, 1)),
}


def _up(n, b):
    return (n + b - 1) // b * b


def _desc(rows, cols, dt, pad=8):
    p = _up(cols, pad)
    return B.raw_desc(1 << 20, (rows, cols), (p * dt.itemsize, dt.itemsize), B._DTYPES[dt])


def _by_columns(rows, cols):
    d = _desc(cols, rows, F32)
    return B.raw_desc(d.data, (rows, cols), (d.strides[1], d.strides[0]), d.dtype)


@pytest.mark.parametrize("dt", [F32, BF16])
@pytest.mark.parametrize("shape", ONE_LAUNCH)
def test_which_calls_are_one_launch(shape, dt):
    M, N, K = shape
    dv, x, dx, dW = _desc(M, N, dt), _desc(M, K, dt), _desc(M, K, dt), _desc(N, K, F32)
    w_rows, w_columns = _desc(N, K, dt), _desc(K, N, dt)
    w_columns = B.raw_desc(w_columns.data, (N, K), (w_columns.strides[1], w_columns.strides[0]), w_columns.dtype)
    by_rows, by_columns, without = ONE_LAUNCH[shape][dt is BF16]
    assert B.linear_bwd_in_one_launch(dv, w_rows, x, dx, dW) == by_rows
    assert B.linear_bwd_in_one_launch(dv, w_columns, x, dx, dW) == by_columns
    assert B.linear_bwd_in_one_launch(dv, None, x, None, dW) == without
    if N > 1:
        assert not B.linear_bwd_in_one_launch(dv, None, x, None, _by_columns(N, K))


@pytest.mark.parametrize("columns", [False, True])
@pytest.mark.parametrize("dt", [F32, BF16])
@pytest.mark.parametrize("shape", IN_PARTS)
def test_which_weight_gradients_leave_the_sums(shape, dt, columns):
    # the workspace says it: slabs of a cut product, then one row of parts for every tile that shares an operand and every cut
    M, N, K = shape
    tile, splits = IN_PARTS[shape][dt is BF16]
    dv, x, dW = _desc(M, N, dt), _desc(M, K, dt), _by_columns(N, K) if columns else _desc(N, K, F32)
    m, n = (K, N) if columns else (N, K)
    rows = splits * (((m if columns else n) + tile - 1) // tile)
    need = (_up(splits * m * _up(n, 4) * 4, 256) if splits > 1 else 0) + _up(rows * N * 4, 256)
    need += B.lib().chn_reduce_axis_workspace_bytes(B._ref(_desc(rows, N, F32, 1)), 0)
    assert B.linear_bwd_workspace_bytes(dv, None, x, None, dW) == max(need, B.lib().chn_reduce_axis_workspace_bytes(B._ref(dv), 0))


@pytest.mark.gpu
@pytest.mark.parametrize("columns", [False, True])
@pytest.mark.parametrize("dt", [F32, BF16])
@pytest.mark.parametrize("shape", list(IN_PARTS) + [s for s in ONE_LAUNCH if s not in IN_PARTS])
def test_gradients_are_exact(shape, dt, columns):
    M, N, K = shape
    gen = torch.Generator(device="cuda").manual_seed(M + N + K)

    def ints(r, c):                                          # |sum| <= 16 max(M, N, K) < 2^24
        t = torch.zeros(r, _up(c, 8), device="cuda", dtype=dt)
        t[:, :c] = torch.randint(-4, 5, (r, c), generator=gen, device="cuda").to(dt)
        return t[:, :c]
    dv, x, W = ints(M, N), ints(M, K), ints(N, K)
    want_dW, want_db, want_dx = dv.double().t() @ x.double(), dv.double().sum(0), (dv.double() @ W.double()).float().to(dt)
    by_columns = torch.empty(K, _up(N, 8), device="cuda", dtype=dt)[:, :N]
    by_columns.copy_(W.t())
    for w in (None, W, by_columns.t()):
        with_dx = w is not None
        dW = torch.full((K, N), 7.0, device="cuda").t() if columns else torch.full((N, K), 7.0, device="cuda")
        db = torch.full((N,), 7.0, device="cuda")
        dx = torch.full((M, K), 7.0, device="cuda", dtype=dt) if with_dx else None
        need = B.linear_bwd_workspace_bytes(dv, w, x, dx, dW)
        ws = torch.full((max(need, 256),), 0xff, dtype=torch.uint8, device="cuda")
        B.linear_bwd(dv, w, x, dW, db, dx, ws=ws)
        assert torch.equal(dW.double(), want_dW), "dW"
        assert torch.equal(db.double(), want_db), "db"
        assert not with_dx or torch.equal(dx, want_dx), "dx"
