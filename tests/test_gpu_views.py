"""Element-wise maps and reductions over views whose rows do not start on 16-byte boundaries or end in partial
vectors, against NumPy in fp64 on the same values."""
import numpy as np
import pytest
import torch

from oracle import oracle as O
from paper_1908_00213_amd import binding as B
from tests.util import TOL_EW, TOL_SUM, bf16r, check, dev, host, ws

pytestmark = pytest.mark.gpu
RNG = np.random.default_rng(82)
TDT = {"f32": torch.float32, "bf16": torch.bfloat16}


def view(a, dt, layout, guard=float("nan")):
    """`a` on the device as a column slice ("slice"), a transposed slice ("t") or contiguous, inside a guarded buffer"""
    m, n = a.shape
    shape = {"plain": (m, n), "slice": (m, n + 5), "t": (n, m + 3)}[layout]
    buf = torch.full(shape, guard, dtype=TDT[dt], device="cuda")
    v = {"plain": lambda: buf, "slice": lambda: buf[:, 3:n + 3], "t": lambda: buf[:, 1:m + 1].t()}[layout]()
    v.copy_(dev(a, dt))
    return buf, v


@pytest.mark.parametrize("dt,odt", [("f32", "f32"), ("bf16", "bf16"), ("f32", "bf16"), ("bf16", "f32")])
@pytest.mark.parametrize("layouts", [("slice", "plain"), ("t", "slice"), ("t", "t"), ("plain", "t")])
@pytest.mark.parametrize("shape", [(1, 1), (3, 7), (64, 64), (65, 129), (127, 9), (5, 2051), (300, 515)])
def test_elementwise_views(dt, odt, layouts, shape):
    a, b = (bf16r(RNG.uniform(-1, 1, shape)) for _ in range(2))
    c = bf16r(RNG.uniform(-1, 1, (1, shape[1])))
    col = bf16r(RNG.uniform(-1, 1, (shape[0], 1)))
    A, Bm = view(a, dt, layouts[0])[1], view(b, dt, layouts[1])[1]
    tol = TOL_EW if odt == "f32" else 2.0 ** -8
    for z in (c, col):
        obuf, out = view(np.zeros(shape, np.float32), odt, "slice")
        before = obuf.clone()
        B.elementwise_broadcast("mad", [A, Bm, dev(z, dt)], out)
        check(host(out), O.elementwise("mad", [a, b, z]), tol, np.abs(a * b) + np.abs(z), "mad %s" % (layouts,))
        obuf[:, 3:shape[1] + 3] = before[:, 3:shape[1] + 3]
        assert torch.equal(torch.isnan(obuf), torch.isnan(before))          # nothing outside the view was written
    if dt == odt:                                                           # in place
        buf, x = view(a, dt, "slice")
        B.elementwise_broadcast("mul", [x, Bm], x)
        check(host(x), O.elementwise("mul", [a, b]), tol, np.abs(a * b), "in place")
        assert torch.isnan(buf[:, :3]).all() and torch.isnan(buf[:, shape[1] + 3:]).all()


def test_elementwise_three_dimensions_unaligned():
    a = RNG.standard_normal((3, 5, 70)).astype(np.float32)
    buf = torch.full((3, 7, 73), float("nan"), device="cuda")
    v = buf[:, 1:6, 2:72]
    v.copy_(dev(a))
    row = RNG.standard_normal((5, 1)).astype(np.float32)
    out = torch.empty(3, 5, 70, device="cuda")
    B.elementwise_broadcast("add", [v, dev(row)], out)
    check(host(out), a.astype(np.float64) + row, TOL_EW, np.abs(a) + np.abs(row), "3-d")


@pytest.mark.parametrize("dt", ["f32", "bf16"])
@pytest.mark.parametrize("layout", ["plain", "slice", "t"])
@pytest.mark.parametrize("shape", [(1, 1), (2, 9), (70, 33), (65, 1001), (2500, 77), (4099, 1027)])
def test_reductions_of_views(dt, layout, shape):
    a = bf16r(RNG.standard_normal(shape))
    x = view(a, dt, layout)[1]
    for axis in (0, 1, None):
        for op, f in (("sum", np.sum), ("max", np.max)):
            ref = f(a.astype(np.float64), axis=axis)
            out = torch.empty(np.shape(ref), device="cuda")
            got = host(B.reduce_axis(op, x, axis, out, ws=ws(B.reduce_axis_workspace_bytes(x, axis))))
            check(got, ref, TOL_SUM, np.abs(a.astype(np.float64)).sum(axis=axis), "%s axis %s" % (op, axis))
    ints = np.round(a * 4).astype(np.float32)
    x = view(ints, dt, layout)[1]
    for axis in (0, 1):
        out = torch.empty(shape[1 - axis], device="cuda")
        got = host(B.reduce_axis("sum", x, axis, out, ws=ws(B.reduce_axis_workspace_bytes(x, axis))))
        assert np.array_equal(got, ints.astype(np.float64).sum(axis=axis))


@pytest.mark.parametrize("dt", ["f32", "bf16"])
@pytest.mark.parametrize("shape", [(1, 32767), (1, 32768), (3, 100001), (255, 33000), (256, 33000), (1, 3000001), (1, 57343), (8, 57344), (9, 45055), (16, 45056),
                                   (17, 40000), (5, 65535), (200, 65536)])
def test_few_long_rows(dt, shape):
    # rows that are cut in slices: with the workspace asked for, without any (one block per row) and with the built-in scratch
    a = RNG.integers(-4, 5, size=shape).astype(np.float32)
    x = view(a, dt, "slice")[1]
    ref = a.astype(np.float64).sum(axis=1)
    need = B.reduce_axis_workspace_bytes(x, 1)
    assert (need > 0) == (shape[0] < 256 and shape[1] >= 32768)
    new = lambda: torch.full((shape[0],), float("nan"), device="cuda")
    for kw in ({"ws": ws(need)}, {}, {"ws": ws(need)[256:]}):
        assert np.array_equal(host(B.reduce_axis("sum", x, 1, new(), **kw)), ref)
    assert np.array_equal(host(B.reduce_axis_static("sum", x, 1, new())), ref)
    # the same bits with and without it (values whose sums round)
    y = torch.randn(shape, device="cuda").to(TDT[dt])
    first = B.reduce_axis("sum", y, 1, new(), ws=ws(need))
    assert torch.equal(first, B.reduce_axis("sum", y, 1, new())) and torch.equal(first, B.reduce_axis_static("sum", y, 1, new()))
    low = lambda **kw: B.reduce_axis("sum", y, 1, new().to(torch.bfloat16), **kw)
    assert torch.equal(low(ws=ws(need)), low())
    top = torch.empty((), device="cuda")
    assert host(B.reduce_axis("max", x, None, top, ws=ws(B.reduce_axis_workspace_bytes(x, None)))) == a.max()
    assert host(B.reduce_axis("max", dev(a, dt), None, top, ws=ws(256))) == a.max()
    # everything of a contiguous array is one row: no workspace is required, and the bits do not depend on it
    total = lambda **kw: B.reduce_axis("sum", y, None, torch.empty((), device="cuda"), **kw)
    assert torch.equal(total(ws=ws(B.reduce_axis_workspace_bytes(y, None))), total())


@pytest.mark.parametrize("dt", ["f32", "bf16"])
@pytest.mark.parametrize("rows", [2, 63, 64, 65, 128, 1000, 1023, 1024, 1025, 2048, 70000])
@pytest.mark.parametrize("cols", [3, 8, 33, 1000])
def test_stacks_of_rows(dt, rows, cols):
    # column folds around the batch of 16 x 64 rows that one block has in flight, whole and partial vectors; a column of
    # nothing but negative values, one of -inf, one with a NaN (which max drops and sum keeps)
    rows = min(rows, (1 << 22) // cols)
    a = RNG.integers(-4, 5, size=(rows, cols)).astype(np.float32)
    a[:, 0] = -np.abs(a[:, 0]) - 1
    top = a.copy()
    top[:, 1], top[rows // 2, 2] = -np.inf, np.nan
    x, out = view(a, dt, "slice")[1], torch.empty(cols, device="cuda")
    w = ws(B.reduce_axis_workspace_bytes(x, 0))
    assert np.array_equal(host(B.reduce_axis("sum", x, 0, out, ws=w)), a.astype(np.float64).sum(axis=0))
    x[:, 1], x[rows // 2, 2] = float("-inf"), float("nan")
    assert np.array_equal(host(B.reduce_axis("max", x, 0, out, ws=w)), np.fmax.reduce(top, axis=0))
    got = host(B.reduce_axis("sum", x, 0, out, ws=w))
    assert np.isneginf(got[1]) and np.isnan(got[2]) and np.array_equal(got[3:], a[:, 3:].astype(np.float64).sum(axis=0))


@pytest.mark.parametrize("shape,step,axis", [((1 << 22,), 2, None), ((1 << 22,), 2, (0,)), ((3, 1 << 20), 3, (1,)), (((1 << 20) + 4096, 3), 1, (0,)),
                                             ((1 << 22,), 1, None), ((2, 2, 1 << 20), 2, (0, 2))])
def test_long_axes_of_few_results(shape, step, axis):
    # no result is one serial chain over a long axis, whatever its stride: chains of at most 8192 elements whose results are
    # folded in turn (2^22 equal values added one after the other would be off by several per cent)
    x = torch.full(shape[:-1] + (shape[-1] * step,), 0.1, device="cuda")[..., ::step]
    ax = tuple(range(len(shape))) if axis is None else axis
    n = int(np.prod([shape[a] for a in ax]))
    out = torch.empty([s for i, s in enumerate(shape) if i not in ax], device="cuda")
    got = host(B.reduce_axis("sum", x, axis, out, ws=ws(B.reduce_axis_workspace_bytes(x, axis))))
    ref = n * np.float64(np.float32(0.1))
    assert np.all(np.abs(got - ref) <= (8192 + n // 1024) * 2.0 ** -24 * ref)
    assert np.all(host(B.reduce_axis_static("sum", x, axis, out)) == got)


@pytest.mark.parametrize("dt", ["f32", "bf16"])
@pytest.mark.parametrize("V,D,N", [(1, 3, 5), (9, 8, 1), (10, 13, 4095), (7, 650, 4096), (40, 1031, 4097), (3000, 33, 9000)])
def test_embedding_any_width(dt, V, D, N):
    # rows off the 16-byte grid; one id list shorter than a scan, exactly one, and several; many and few matches per row
    ids = RNG.integers(-1, V + 1, N).astype(np.int32)                       # (a stray id gathers zeros and receives nothing)
    table = bf16r(RNG.standard_normal((V, D)))
    buf, t = view(table, dt, "slice")
    obuf, out = view(np.zeros((N, D), np.float32), dt, "slice")
    B.embed_fwd(t, dev(ids), out)
    ok = (ids >= 0) & (ids < V)
    want = np.where(ok[:, None], table[np.where(ok, ids, 0)], 0)
    assert np.array_equal(host(out), want)
    assert torch.isnan(obuf[:, :3]).all() and torch.isnan(obuf[:, D + 3:]).all()
    dout = RNG.integers(-3, 4, (N, D)).astype(np.float32)
    ref = np.zeros((V, D))
    np.add.at(ref, ids[ok], dout[ok])
    g = view(np.zeros((V, D), np.float32), "f32", "slice")[1]
    assert np.array_equal(host(B.embed_bwd(dev(ids), view(dout, "f32", "slice")[1], g)), ref)
    assert np.array_equal(host(B.embed_bwd(dev(ids), dev(dout), g, accumulate=True)), 2 * ref)


@pytest.mark.parametrize("wide", [False, True])
@pytest.mark.parametrize("N", [1, 3, 256, 257, 1024, 1025, 4097])
@pytest.mark.parametrize("D", [1, 256, 257, 513, 769, 1025])
def test_embedding_gradient_scan_lengths(N, D, wide):
    # both sides of the id list lengths and widths at which the kernel changes its scan and its columns per thread; ids
    # outside the table, the extremes of their type among them, match nothing
    V = 21
    ids = RNG.integers(0, V, N).astype(np.int64 if wide else np.int32)
    stray = [-1, -2 ** 31, 2 ** 31 - 1, V, -8] + ([-2 ** 63, 2 ** 63 - 1, 2 ** 32, -2 ** 32 + 3] if wide else [])
    ids[::5] = [stray[i % len(stray)] for i in range(len(ids[::5]))]
    dout = RNG.integers(-3, 4, (N, D)).astype(np.float32)
    ok = (ids >= 0) & (ids < V)
    ref = np.zeros((V, D))
    np.add.at(ref, ids[ok], dout[ok])
    g = torch.full((V, D), float("nan"), device="cuda")
    assert np.array_equal(host(B.embed_bwd(dev(ids), dev(dout), g)), ref)
    assert np.array_equal(host(B.embed_bwd(dev(ids), dev(dout), g, accumulate=True)), 2 * ref)


@pytest.mark.parametrize("dt", ["f32", "bf16"])
@pytest.mark.parametrize("shape", [(3, 5), (129, 65), (130, 449), (65, 577), (1001, 515), (300, 1027), (1027, 1100)])
@pytest.mark.parametrize("pitch", [0, 3])
def test_tiles_of_transposed_views_off_the_vector_grid(dt, shape, pitch):
    # one tile to several hundred, numbers of tiles that the eight XCDs share evenly and not; the transposed operand with and
    # without a gap between its rows, whole kilobytes of pitch among them (513 + 511, 1025 + 1023: another order of tiles)
    m, n = shape
    gen = torch.Generator(device="cuda").manual_seed(m * n)
    ints = lambda *s: torch.randint(-8, 9, s, generator=gen, device="cuda").to(TDT[dt])
    for gap in (pitch, -m % 512):
        a, b, c = ints(n, m + gap)[:, :m].t(), ints(m, n + 5)[:, 2:n + 2], ints(1, n)
        out = torch.full((m, n + gap), float("nan"), device="cuda", dtype=TDT[dt])
        B.elementwise_broadcast("mad_relu", [a, b, c], out[:, :n])
        assert torch.equal(out[:, :n].float(), (a.float() * b.float() + c.float()).clamp(min=0))
        assert bool(out[:, n:].isnan().all())
