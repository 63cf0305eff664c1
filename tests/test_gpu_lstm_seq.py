"""GPU parity of the whole-sequence recurrent forward (one launch for all time steps) against the CPU oracle,
step by step from the GPU's own previous state, and against the chain of per-step calls."""
import numpy as np
import pytest
import torch

from oracle import oracle as O
from paper_1908_00213_amd import binding as B
from tests.util import TOL_BF16, TOL_EW, TOL_SUM, bf16r, check, dev, empty, host, ws

pytestmark = pytest.mark.gpu

CASES = [(128, 672, 35, "f32"), (128, 672, 35, "bf16"),      # the language-model workload: 84 x 2 workgroups
         (70, 40, 4, "f32"), (5, 8, 3, "f32"),               # ragged batch block, one partial chunk
         (33, 144, 6, "bf16"), (200, 256, 3, "f32"),         # four batch blocks, two chunks
         (64, 1536, 2, "bf16"), (128, 768, 2, "f32"),        # the widest rows: Ut in registers, five stages, six chunks
         (64, 640, 3, "f32"),                                # ... five chunks
         (64, 512, 3, "f32"), (40, 352, 3, "f32")]           # four chunks through three stages (one reused); three, the last one partial


def inputs(Bn, H, T, dt, seed):
    rng = np.random.default_rng(seed)
    q = (lambda a: a) if dt == "f32" else bf16r
    u = lambda shape, lo, hi: rng.uniform(lo, hi, size=shape).astype(np.float32)
    s = 1.5 / np.sqrt(H)
    return u((T * Bn, 4 * H), -2, 2), u((4 * H,), -1, 1), q(u((Bn, H), -1, 1)), u((Bn, H), -2, 2), q(u((H, 4 * H), -s, s))


def run(zx, bias, h0, c0, U, T, dt, Hs=None, Cs=None, gates=None, work=None):
    Bn, H = h0.shape
    Hs = empty(((T + 1) * Bn, H), dt) if Hs is None else Hs
    Cs = empty(((T + 1) * Bn, H)) if Cs is None else Cs
    gates = empty((T * Bn, 4 * H)) if gates is None else gates
    work = ws(B.lstm_seq_workspace_bytes(Bn)) if work is None else work
    Hs[:Bn].copy_(dev(h0, dt))
    Cs[:Bn].copy_(dev(c0))
    print("lstm_seq_fwd B=%d H=%d T=%d %s" % (Bn, H, T, dt), flush=True)
    B.lstm_seq_fwd(dev(zx), dev(np.ascontiguousarray(U.T), dt), None if bias is None else dev(bias), Hs, Cs, gates, T, work)
    torch.cuda.synchronize()
    return Hs, Cs, gates, work


def status_word(work):
    return int(work[:4].view(torch.int32).item())


def check_against_oracle(zx, bias, U, T, dt, Hs, Cs, gates):
    """Every step from the state the GPU itself left for it: one product and one cell of error per check."""
    Bn, H = Hs.shape[0] // (T + 1), Hs.shape[1]
    Hh, Ch, Gh = host(Hs), host(Cs), host(gates)
    tol = TOL_SUM if dt == "f32" else TOL_BF16
    for t in range(T):
        hp, cp, z0 = Hh[t * Bn:(t + 1) * Bn], Ch[t * Bn:(t + 1) * Bn], zx[t * Bn:(t + 1) * Bn]
        rc, rh, rg = O.lstm_fwd(O.gemm(hp, U, z0, 1.0, 1.0), bias, cp)
        Sz = O.gemm(np.abs(hp), np.abs(U)) + np.abs(z0) + (0 if bias is None else np.abs(bias))
        Sg = np.concatenate([0.25 * Sz[:, :H], 0.25 * Sz[:, H:2 * H], Sz[:, 2 * H:3 * H], 0.25 * Sz[:, 3 * H:]], axis=1)
        check(Gh[t * Bn:(t + 1) * Bn], rg, TOL_SUM, Sg + 1e-1, "gates of step %d" % t)
        Sc = np.abs(rg[:, H:2 * H] * cp) + np.abs(rg[:, :H] * rg[:, 2 * H:3 * H]) + Sg[:, :H] + Sg[:, H:2 * H] * np.abs(cp) + Sg[:, 2 * H:3 * H]
        check(Ch[(t + 1) * Bn:(t + 2) * Bn], rc, TOL_SUM, Sc, "c of step %d" % t)
        check(Hh[(t + 1) * Bn:(t + 2) * Bn], rh, tol, Sc + Sg[:, 3 * H:], "h of step %d" % t)


@pytest.mark.parametrize("Bn,H,T,dt", CASES)
def test_whole_sequence_forward(Bn, H, T, dt):
    zx, bias, h0, c0, U = inputs(Bn, H, T, dt, 7)
    Hs, Cs, gates, work = run(zx, bias, h0, c0, U, T, dt)
    assert status_word(work) == 0
    check_against_oracle(zx, bias, U, T, dt, Hs, Cs, gates)
    assert np.array_equal(host(Hs[:Bn]), h0.astype(np.float64)) and np.array_equal(host(Cs[:Bn]), c0.astype(np.float64))
    # the per-step calls on the same operands walk the same trajectory (another order of the fp32 sums)
    if H % 32 == 0:
        H2, C2, G2 = empty(((T + 1) * Bn, H), dt), empty(((T + 1) * Bn, H)), empty((T * Bn, 4 * H))
        H2[:Bn].copy_(dev(h0, dt)); C2[:Bn].copy_(dev(c0))
        B.lstm_step_fwd_seq(dev(zx), H2, dev(np.ascontiguousarray(U.T), dt), dev(bias), C2, G2, T)
        loose = (1e-4 if dt == "f32" else 4e-2) * max(1, T // 4)
        check(host(Cs), host(C2), loose, 1.0, "c whole sequence vs per step")
        check(host(Hs), host(H2), loose, 1.0, "h whole sequence vs per step")
    # the same buffers again with other inputs: nothing of the first call may be read back from a cache
    zx, bias, h0, c0, U = inputs(Bn, H, T, dt, 8)
    run(zx, None, h0, c0, U, T, dt, Hs, Cs, gates, work)
    assert status_word(work) == 0
    check_against_oracle(zx, None, U, T, dt, Hs, Cs, gates)


def test_whole_sequence_without_gates_and_pitched_buffers():
    Bn, H, T = 40, 64, 3
    zx, bias, h0, c0, U = inputs(Bn, H, T, "f32", 9)
    wide_z = dev(np.concatenate([zx, zx], axis=1))[:, :4 * H]
    wide_h = torch.zeros((T + 1) * Bn, 2 * H, device="cuda")[:, :H]
    Cs = empty(((T + 1) * Bn, H))
    wide_h[:Bn].copy_(dev(h0)); Cs[:Bn].copy_(dev(c0))
    work = ws(B.lstm_seq_workspace_bytes(Bn))
    B.lstm_seq_fwd(wide_z, dev(np.ascontiguousarray(U.T)), dev(bias), wide_h, Cs, None, T, work)
    Hs, C2, gates, _ = run(zx, bias, h0, c0, U, T, "f32")
    assert torch.equal(wide_h, Hs) and torch.equal(Cs, C2)


def test_whole_sequence_refusals():
    def call(Bn, H, T, dt="f32", work=None, hs_rows=None):
        tdt = torch.float32 if dt == "f32" else torch.bfloat16
        z = torch.zeros(T * Bn, 4 * H, device="cuda")
        Hs = torch.zeros((T + 1) * Bn if hs_rows is None else hs_rows, H, dtype=tdt, device="cuda")
        Cs = torch.zeros((T + 1) * Bn, H, device="cuda")
        B.lstm_seq_fwd(z, torch.zeros(4 * H, H, dtype=tdt, device="cuda"), None, Hs, Cs, None, T,
                       ws(B.lstm_seq_workspace_bytes(Bn)) if work is None else work)
    for args, status in [((4, 44, 2), -4),                     # hidden width not a multiple of 8
                         ((4, 40, 2, "bf16"), -4),             # ... of 16 for bfloat16
                         ((4, 776, 2), -4),                    # rows wider than the resident slice holds
                         ((256, 768, 2), -4),                  # 96 x 4 workgroups: more than compute units
                         ((4, 64, 2, "f32", None, 8), -4)]:    # Hs with too few rows
        with pytest.raises(B.ChnError) as e:
            call(*args)
        assert e.value.status == status, args
    with pytest.raises(B.ChnError):
        call(4, 64, 2, work=torch.empty(16, dtype=torch.uint8, device="cuda"))
    call(4, 64, 0)                                              # no steps: nothing to do
    torch.cuda.synchronize()


def test_a_wait_that_runs_out_ends_the_kernel_and_raises_the_status_word():
    """Spin limit 0: the first wait (before step 1) gives up without looking, in every workgroup.  The kernel
    ends after its first step with the status word set; the next call, with the default limit, is complete."""
    Bn, H, T, dt = 128, 672, 35, "f32"
    zx, bias, h0, c0, U = inputs(Bn, H, T, dt, 11)
    B.lstm_seq_spin_limit(0)
    try:
        Hs, Cs, gates, work = run(zx, bias, h0, c0, U, T, dt)
    finally:
        B.lstm_seq_spin_limit(1 << 20)
    assert status_word(work) == 1
    Hs, Cs, gates, work = run(zx, bias, h0, c0, U, T, dt, Hs, Cs, gates, work)
    assert status_word(work) == 0
    check_against_oracle(zx, bias, U, T, dt, Hs, Cs, gates)


# ------------------------------------------------------------------------------------ backward through time
BWD_CASES = [(128, 672, 35, "f32"), (128, 672, 35, "bf16"),  # the language-model workload: 42 x 4 workgroups
             (40, 48, 4, "f32"), (5, 16, 3, "f32"),          # ragged batch block, a partial 32-unit tile; one workgroup
             (33, 144, 5, "bf16"), (200, 256, 3, "f32"),
             (40, 96, 4, "bf16"), (250, 512, 2, "bf16"),     # ragged batch block; 32 x 8 = 256 workgroups, every compute unit
             (96, 768, 2, "f32"), (32, 1536, 2, "bf16")]     # the widest U the registers hold (bf16: two batches of partial sums)


def bwd_inputs(Bn, H, T, dt, seed):
    rng = np.random.default_rng(seed)
    q = (lambda a: a) if dt == "f32" else bf16r
    u = lambda shape, lo, hi: rng.uniform(lo, hi, size=shape).astype(np.float32)
    s = 1.5 / np.sqrt(H)
    gates = np.concatenate([u((T * Bn, 2 * H), 0.05, 0.95), u((T * Bn, H), -0.95, 0.95), u((T * Bn, H), 0.05, 0.95)], axis=1)
    return q(u((H, 4 * H), -s, s)), q(u((T * Bn, H), -1, 1)), gates, u(((T + 1) * Bn, H), -1.5, 1.5), u((Bn, H), -1, 1)


def run_bwd(U, dh_in, gates, Cs, dc_last, T, dt, bufs=None):
    Bn, H = Cs.shape[0] // (T + 1), Cs.shape[1]
    dHs, dZ, dc0, work = bufs or (empty((T * Bn, H), dt), empty((T * Bn, 4 * H), dt), empty((Bn, H)),
                                  ws(B.lstm_seq_bwd_workspace_bytes(Bn, H)))
    dHs.copy_(dev(dh_in, dt))
    print("lstm_seq_bwd B=%d H=%d T=%d %s" % (Bn, H, T, dt), flush=True)
    B.lstm_seq_bwd(dev(U, dt), dHs, dev(gates), dev(Cs), None if dc_last is None else dev(dc_last), dZ, dc0, T, work)
    torch.cuda.synchronize()
    return dHs, dZ, dc0, work


def check_bwd_against_oracle(U, dh_in, gates, Cs, dc_last, T, dt, dHs, dZ, dc0):
    """Last step first; the product of every step from the dz the GPU itself stored for the step after it, the
    cell from the dh the GPU stored; only dc is carried along by the oracle."""
    Bn, H = Cs.shape[0] // (T + 1), Cs.shape[1]
    dH, dz_gpu = host(dHs), host(dZ)
    tol = TOL_SUM if dt == "f32" else TOL_BF16
    dc = None if dc_last is None else dc_last.astype(np.float64)
    for t in range(T - 1, -1, -1):
        sl = slice(t * Bn, (t + 1) * Bn)
        if t == T - 1:
            assert np.array_equal(dH[sl], dh_in[sl].astype(np.float64))
        else:
            nx = slice((t + 1) * Bn, (t + 2) * Bn)
            check(dH[sl], O.gemm(dz_gpu[nx], U.T, dh_in[sl], 1.0, 1.0), tol, O.gemm(np.abs(dz_gpu[nx]), np.abs(U.T)) + np.abs(dh_in[sl]), "dh total %d" % t)
        cp, c = Cs[sl].astype(np.float64), Cs[(t + 1) * Bn:(t + 2) * Bn].astype(np.float64)
        rdz, dc = O.lstm_bwd(gates[sl], cp, c, dH[sl], dc)
        Sdc = np.abs(dc) + np.abs(dH[sl]) + 1e-3
        Sdz = np.concatenate([Sdc, Sdc * (1 + np.abs(cp)), Sdc, np.abs(dH[sl])], axis=1)
        check(dz_gpu[sl], rdz, TOL_EW * 10 * (T - t) if dt == "f32" else TOL_BF16, Sdz, "dz %d" % t)
    check(host(dc0), dc, TOL_EW * 10 * T, 1.0, "dc0")


@pytest.mark.parametrize("Bn,H,T,dt", BWD_CASES)
def test_whole_sequence_backward(Bn, H, T, dt):
    U, dh_in, gates, Cs, dc_last = bwd_inputs(Bn, H, T, dt, 21)
    dHs, dZ, dc0, work = run_bwd(U, dh_in, gates, Cs, dc_last, T, dt)
    assert status_word(work) == 0
    check_bwd_against_oracle(U, dh_in, gates, Cs, dc_last, T, dt, dHs, dZ, dc0)
    if H % 32 == 0:      # the chain of per-step calls walks the same trajectory
        d2, z2, dcs = dev(dh_in, dt), empty((T * Bn, 4 * H), dt), [empty((Bn, H)), empty((Bn, H))]
        B.lstm_step_bwd_seq(z2, dev(U, dt), d2, dev(gates), dev(Cs), dev(dc_last), dcs, T)
        loose = (1e-4 if dt == "f32" else 4e-2) * max(1, T // 4)
        check(host(dZ), host(z2), loose, 1.0, "dz whole sequence vs per step")
        check(host(dc0), host(dcs[0]), loose, 1.0, "dc0 whole sequence vs per step")
    # the same buffers and workspace again with other values, no gradient into the last cell state
    U, dh_in, gates, Cs, _ = bwd_inputs(Bn, H, T, dt, 22)
    run_bwd(U, dh_in, gates, Cs, None, T, dt, (dHs, dZ, dc0, work))
    assert status_word(work) == 0
    check_bwd_against_oracle(U, dh_in, gates, Cs, None, T, dt, dHs, dZ, dc0)


def test_whole_sequence_backward_refusals_and_give_up():
    def call(Bn, H, T, dt="f32", work=None):
        tdt = torch.float32 if dt == "f32" else torch.bfloat16
        z = lambda *s: torch.zeros(*s, device="cuda")
        B.lstm_seq_bwd(torch.zeros(H, 4 * H, dtype=tdt, device="cuda"), torch.zeros(T * Bn, H, dtype=tdt, device="cuda"), z(T * Bn, 4 * H),
                       z((T + 1) * Bn, H), None, torch.zeros(T * Bn, 4 * H, dtype=tdt, device="cuda"), z(Bn, H), T,
                       ws(B.lstm_seq_bwd_workspace_bytes(Bn, H)) if work is None else work)
    for args in [(4, 40, 2), (4, 784, 2), (4, 1552, 2, "bf16"), (288, 512, 2)]:      # width not a multiple of 16; too wide; 9 x 32 workgroups
        with pytest.raises(B.ChnError) as e:
            call(*args)
        assert e.value.status == -4, args
        assert not B.lstm_seq_bwd_supported(args[0], args[1], torch.float32 if len(args) < 4 else torch.bfloat16)
    with pytest.raises(B.ChnError):
        call(4, 64, 2, work=torch.empty(4096, dtype=torch.uint8, device="cuda"))
    call(4, 64, 0)
    torch.cuda.synchronize()
    # spin limit 0: the first exchange gives up without looking; the kernel ends, the status word says so
    Bn, H, T, dt = 128, 672, 35, "f32"
    U, dh_in, gates, Cs, dc_last = bwd_inputs(Bn, H, T, dt, 23)
    B.lstm_seq_spin_limit(0)
    try:
        bufs = run_bwd(U, dh_in, gates, Cs, dc_last, T, dt)
    finally:
        B.lstm_seq_spin_limit(1 << 20)
    assert status_word(bufs[3]) == 1
    dHs, dZ, dc0, work = run_bwd(U, dh_in, gates, Cs, dc_last, T, dt, bufs)
    assert status_word(work) == 0
    check_bwd_against_oracle(U, dh_in, gates, Cs, dc_last, T, dt, dHs, dZ, dc0)


@pytest.mark.parametrize("dt", ["f32", "bf16"])
def test_whole_sequence_kernels_are_reproducible_bit_for_bit(dt):
    """Every sum is taken in a fixed order (partial tiles in wave order, partial dh in sender order): two runs of
    the same launch agree in every bit, whatever order the workgroups arrive in."""
    Bn, H, T = 128, 672, 35
    zx, bias, h0, c0, U = inputs(Bn, H, T, dt, 31)
    first = [t.clone() for t in run(zx, bias, h0, c0, U, T, dt)[:3]]
    for _ in range(2):
        again = run(zx, bias, h0, c0, U, T, dt)[:3]
        assert all(torch.equal(a, b) for a, b in zip(first, again))
    Ub, dh_in, gates, Cs, dc_last = bwd_inputs(Bn, H, T, dt, 32)
    first = [t.clone() for t in run_bwd(Ub, dh_in, gates, Cs, dc_last, T, dt)[:3]]
    for _ in range(2):
        again = run_bwd(Ub, dh_in, gates, Cs, dc_last, T, dt)[:3]
        assert all(torch.equal(a, b) for a, b in zip(first, again))


# ------------------------------------------------------------- the kernels that exchange inside an XCD: where their tiles end
# batches around sixteen rows and 128, widths around 8, 16 and 24 units a workgroup and 32 k, one to five steps (marks run three ahead)
EDGES = [(1, 16, 1), (15, 24, 2), (16, 32, 3), (17, 40, 4), (33, 248, 5), (127, 256, 2), (128, 264, 3), (16, 504, 4), (64, 512, 2),
         (31, 520, 5), (128, 528, 2), (48, 744, 3), (113, 760, 2), (128, 768, 5)]


@pytest.mark.parametrize("dt", ["f32", "bf16"])
@pytest.mark.parametrize("Bn,H,T", EDGES)
def test_sequence_edges(Bn, H, T, dt):
    if H % (8 if dt == "f32" else 16) == 0:
        zx, bias, h0, c0, U = inputs(Bn, H, T, dt, 41)
        Hs, Cs, gates, work = run(zx, bias, h0, c0, U, T, dt)
        assert status_word(work) == 0
        check_against_oracle(zx, bias, U, T, dt, Hs, Cs, gates)
        # a workspace that holds no messages: the kernels that exchange through device memory, the same results but for the order of sums
        small = ws(256 + 256 + 256)
        H2, C2, G2, small = run(zx, bias, h0, c0, U, T, dt, work=small)
        assert status_word(small) == 0
        check_against_oracle(zx, bias, U, T, dt, H2, C2, G2)
    if H % 16 == 0:
        U, dh_in, gates, Cs, dc_last = bwd_inputs(Bn, H, T, dt, 42)
        dHs, dZ, dc0, work = run_bwd(U, dh_in, gates, Cs, dc_last, T, dt)
        assert status_word(work) == 0
        check_bwd_against_oracle(U, dh_in, gates, Cs, dc_last, T, dt, dHs, dZ, dc0)


def test_sequence_values_that_three_parts_do_not_hold():
    """fp32: infinities, NaN and values whose scaled parts overflow are multiplied again as they are."""
    Bn, H, T = 40, 272, 3
    zx, bias, h0, c0, U = inputs(Bn, H, T, "f32", 43)
    h0 = np.abs(h0) + 0.25
    U[5, 7] = np.inf                       # gate i of unit 7: 1 in every row whose h is positive
    U[11, H + 30] = -np.inf                # gate f of unit 30: 0
    h0[3] *= np.float32(2.0 ** -112)       # against 2^110: a product of about one, each factor scaled out of range or far from its row
    h0[3, 5] = h0[3, 11] = 1.0
    U[:, 3 * H + 100] *= np.float32(2.0 ** 110)
    h0[20, 9] = np.nan                     # this row and no other
    Hs, Cs, gates, work = run(zx, bias, h0, c0, U, T, "f32")
    assert status_word(work) == 0
    with np.errstate(all="ignore"):
        z = zx[:Bn].astype(np.float64) + bias + h0.astype(np.float64) @ U.astype(np.float64)
        want = 1.0 / (1.0 + np.exp(-z))
        want[:, 2 * H:3 * H] = np.tanh(z[:, 2 * H:3 * H])
        S = np.abs(zx[:Bn]) + np.abs(bias) + np.abs(h0).astype(np.float64) @ np.abs(U).astype(np.float64)
    got = host(gates)[:Bn]
    assert np.isnan(got[20]).all() and not np.isnan(np.delete(got, 20, 0)).any()
    rows = [b for b in range(Bn) if b != 20]
    assert (got[rows, 7] == 1.0).all() and (got[rows, H + 30] == 0.0).all()
    cols = [j for j in range(4 * H) if j not in (7, H + 30, 3 * H + 100)]
    check(got[np.ix_(rows, cols)], want[np.ix_(rows, cols)], TOL_SUM, S[np.ix_(rows, cols)] + 1e-1, "gates")
    check(got[3, 3 * H + 100], want[3, 3 * H + 100], TOL_SUM, 1.0, "a product of 2^110 and 2^-112")
    # backward: dz scaled out of range against a small U
    U, dh_in, gates, Cs, _ = bwd_inputs(Bn, H, T, "f32", 44)
    U *= np.float32(2.0 ** -100)
    dh_in *= np.float32(2.0 ** 106)
    dHs, dZ, dc0, work = run_bwd(U, dh_in, gates, Cs, None, T, "f32")
    assert status_word(work) == 0 and torch.isfinite(dHs).all()
    dz = host(dZ)
    for t in range(T - 1):
        nx = slice((t + 1) * Bn, (t + 2) * Bn)
        back = host(dHs)[t * Bn:(t + 1) * Bn] - dh_in[t * Bn:(t + 1) * Bn].astype(np.float64)
        S = np.abs(dz[nx]) @ np.abs(U.T).astype(np.float64) + np.abs(dh_in[t * Bn:(t + 1) * Bn])
        check(back, dz[nx] @ U.T.astype(np.float64), TOL_SUM, S, "dh of step %d" % t)


@pytest.mark.parametrize("Bn,H,T", [(40, 272, 9), (128, 656, 12), (17, 40, 10)])
def test_sequence_of_sums_taken_again(Bn, H, T):
    """fp32, more steps than blocks of h: infinities and entries of 2^90 to 2^100 in U make the sums of a few units, in one or two
    workgroups, overflow in every step, which read h again while the other workgroups go on.  Every step from the state that
    the GPU left for it."""
    zx, bias, h0, c0, U = inputs(Bn, H, T, "f32", 45)
    odd = {"i": 7, "f": H // 2, "g": H - 3, "o": H - 9}
    U[5, odd["i"]] = np.inf
    U[11, H + odd["f"]] = -np.inf
    U[13, 2 * H + odd["g"]] = np.float32(2.0 ** 90)
    U[:, 3 * H + odd["o"]] *= np.float32(2.0 ** 100)
    Hs, Cs, gates, work = run(zx, bias, h0, c0, U, T, "f32")
    assert status_word(work) == 0
    # four columns: saturated gates, in every step; all others as ever
    special = [odd["i"], H + odd["f"], 2 * H + odd["g"], 3 * H + odd["o"]]
    Hh, Ch, Gh = host(Hs), host(Cs), host(gates)
    assert np.isfinite(Hh).all() and np.isfinite(Ch).all() and np.isfinite(Gh).all()
    plain = U.copy()
    plain[:, special] = 0
    for t in range(T):
        hp, cp, z0 = Hh[t * Bn:(t + 1) * Bn], Ch[t * Bn:(t + 1) * Bn], zx[t * Bn:(t + 1) * Bn]
        z = (z0 + bias).astype(np.float64) + hp @ plain.astype(np.float64)
        S = np.abs(z0) + np.abs(bias) + np.abs(hp) @ np.abs(plain).astype(np.float64)
        want = 1.0 / (1.0 + np.exp(-z))
        want[:, 2 * H:3 * H] = np.tanh(z[:, 2 * H:3 * H])
        for col in special:
            with np.errstate(all="ignore"):
                zc = hp @ U[:, col].astype(np.float64) if np.isfinite(U[:, col]).all() else U[:, col][~np.isfinite(U[:, col])][0] * hp[:, 5 if col == special[0] else 11]
            assert (np.abs(zc) > 1e3).all()
            want[:, col] = np.sign(zc) if col == special[2] else (zc > 0).astype(np.float64)
        got = Gh[t * Bn:(t + 1) * Bn]
        check(got, want, TOL_SUM, S + 1e-1, "gates of step %d" % t)
        c = got[:, H:2 * H] * cp + got[:, :H] * got[:, 2 * H:3 * H]
        check(Ch[(t + 1) * Bn:(t + 2) * Bn], c, TOL_SUM, np.abs(cp) + 1, "c of step %d" % t)
        check(Hh[(t + 1) * Bn:(t + 2) * Bn], got[:, 3 * H:] * np.tanh(c), TOL_SUM, 1.0, "h of step %d" % t)


# ------------------------------------------------------------- how the kernels that exchange inside an XCD come to run, and end
@pytest.fixture
def meeting():
    yield B.lstm_seq_meeting
    B.lstm_seq_meeting()
    B.lstm_seq_spin_limit(1 << 20)


PATHS = [(33, 64, 5), (128, 272, 9), (70, 528, 6), (128, 672, 12)]


@pytest.mark.parametrize("dt", ["f32", "bf16"])
@pytest.mark.parametrize("Bn,H,T", PATHS)
def test_sequences_that_are_called_off_are_done_by_the_other_kernels(Bn, H, T, dt, meeting):
    """Nobody waits for the others: the walk is called off before its first step, with marks where h will be, and the kernels launched
    behind do the whole of it, bit for bit what they do by themselves."""
    zx, bias, h0, c0, U = inputs(Bn, H, T, dt, 51)
    alone = run(zx, bias, h0, c0, U, T, dt, work=ws(256 + 256 + 256))     # (no room for the messages of the first kind)
    meeting(patience=0)
    Hs, Cs, gates, work = run(zx, bias, h0, c0, U, T, dt)
    assert status_word(work) == 0
    check_against_oracle(zx, bias, U, T, dt, Hs, Cs, gates)
    assert all(torch.equal(a, b) for a, b in zip((Hs, Cs, gates), alone))
    U, dh_in, gates, Cs, dc_last = bwd_inputs(Bn, H, T, dt, 52)
    dHs, dZ, dc0, work = run_bwd(U, dh_in, gates, Cs, dc_last, T, dt)
    assert status_word(work) == 0
    check_bwd_against_oracle(U, dh_in, gates, Cs, dc_last, T, dt, dHs, dZ, dc0)


@pytest.mark.parametrize("dt", ["f32", "bf16"])
@pytest.mark.parametrize("Bn,H,T", PATHS)
def test_sequences_that_exchange_at_device_scope(Bn, H, T, dt, meeting):
    """As where a group's workgroups do not share an XCD: the same values another way, so the same bits."""
    zx, bias, h0, c0, U = inputs(Bn, H, T, dt, 53)
    through_l2 = run(zx, bias, h0, c0, U, T, dt)
    bwd = bwd_inputs(Bn, H, T, dt, 54)
    back = run_bwd(*bwd, T, dt)
    meeting(share_l2=False)
    for _ in range(2):
        Hs, Cs, gates, work = run(zx, bias, h0, c0, U, T, dt)
        assert status_word(work) == 0
        assert all(torch.equal(a, b) for a, b in zip((Hs, Cs, gates), through_l2))
        dHs, dZ, dc0, work = run_bwd(*bwd, T, dt)
        assert status_word(work) == 0
        assert all(torch.equal(a, b) for a, b in zip((dHs, dZ, dc0), back))
    check_against_oracle(zx, bias, U, T, dt, Hs, Cs, gates)
    check_bwd_against_oracle(*bwd, T, dt, dHs, dZ, dc0)


@pytest.mark.parametrize("share_l2", [True, False])
@pytest.mark.parametrize("dt", ["f32", "bf16"])
def test_a_walk_that_gives_up_on_its_way_ends(dt, share_l2, meeting):
    """The walk has begun, then its first wait runs out (spin limit 0) or one does somewhere (1): every workgroup leaves, the status word
    is up and the kernels behind do not touch the outputs; the next call is complete."""
    Bn, H, T = 128, 528, 9
    zx, bias, h0, c0, U = inputs(Bn, H, T, dt, 55)
    bwd = bwd_inputs(Bn, H, T, dt, 56)
    for polls in (0, 1):
        meeting(patience=1 << 14, share_l2=share_l2)
        B.lstm_seq_spin_limit(polls)
        Hs, Cs, gates, work = run(zx, bias, h0, c0, U, T, dt)
        bufs = run_bwd(*bwd, T, dt)
        if polls == 0:
            assert status_word(work) == 1 and status_word(bufs[3]) == 1
        meeting()
        B.lstm_seq_spin_limit(1 << 20)
        Hs, Cs, gates, work = run(zx, bias, h0, c0, U, T, dt, Hs, Cs, gates, work)
        assert status_word(work) == 0
        check_against_oracle(zx, bias, U, T, dt, Hs, Cs, gates)
        dHs, dZ, dc0, work = run_bwd(*bwd, T, dt, bufs)
        assert status_word(work) == 0
        check_bwd_against_oracle(*bwd, T, dt, dHs, dZ, dc0)


def test_the_library_says_where_the_backward_pass_stays_inside_the_xcds():
    """The answer follows the device (32 workgroups on each of eight XCDs need 256 compute units), the sizes and the steps."""
    whole = torch.cuda.get_device_properties(0).multi_processor_count >= 256
    for Bn, H, fits in [(1, 16, True), (128, 672, True), (128, 768, True), (129, 672, False), (128, 784, False), (128, 1536, False), (16, 40, False)]:
        for dt in (torch.float32, torch.bfloat16):
            assert B.lstm_seq_bwd_in_xcd(Bn, H, 6, dt) == (fits and whole), (Bn, H)
            assert not B.lstm_seq_bwd_in_xcd(Bn, H, 2, dt)


@pytest.mark.parametrize("dt", ["f32", "bf16"])
@pytest.mark.parametrize("Bn,H,T", EDGES)
def test_sequence_edges_inside_the_xcds(Bn, H, T, dt, meeting):
    """As test_sequence_edges, where few steps are left to the other kernels otherwise; those do the same to the last roundings."""
    def both(call, check_it):
        meeting(patience=1 << 14)
        first = call()
        assert status_word(first[-1]) == 0
        check_it(*first[:-1])
        meeting()
        usual = call()
        assert status_word(usual[-1]) == 0
        check_it(*usual[:-1])
    if H % (8 if dt == "f32" else 16) == 0:
        zx, bias, h0, c0, U = inputs(Bn, H, T, dt, 61)
        both(lambda: run(zx, bias, h0, c0, U, T, dt), lambda Hs, Cs, gates: check_against_oracle(zx, bias, U, T, dt, Hs, Cs, gates))
    if H % 16 == 0:
        bwd = bwd_inputs(Bn, H, T, dt, 62)
        both(lambda: run_bwd(*bwd, T, dt), lambda dHs, dZ, dc0: check_bwd_against_oracle(*bwd, T, dt, dHs, dZ, dc0))


def test_overflowing_products_inside_the_xcds(meeting):
    """As test_sequence_values_that_three_parts_do_not_hold, whose three steps are left to the other kernels otherwise."""
    meeting(patience=1 << 14)
    test_sequence_values_that_three_parts_do_not_hold()


@pytest.mark.parametrize("share_l2", [True, False])
@pytest.mark.parametrize("Bn,H,T", [(17, 64, 10), (40, 272, 9), (70, 528, 8), (33, 640, 9), (128, 656, 12)])
def test_backward_sums_taken_again_while_others_go_on(Bn, H, T, share_l2, meeting):
    """fp32, more steps than blocks of messages: dz of three units of every third row exceeds what the parts hold, against small columns
    of U, so that two squares at most multiply again in every step, from a block of dz that is marked for its next use two steps on, while
    the others go on.  Every step from the dz that the GPU left for it."""
    assert B.lstm_seq_bwd_in_xcd(Bn, H, T, torch.float32)
    U, dh_in, gates, Cs, dc_last = bwd_inputs(Bn, H, T, "f32", 57)
    for unit in (7, H // 2, H // 2 + 1):
        dh_in[::3, unit] *= np.float32(2.0 ** 106)
        U[:, unit::H] *= np.float32(2.0 ** -100)
    meeting(share_l2=share_l2)
    dHs, dZ, dc0, work = run_bwd(U, dh_in, gates, Cs, dc_last, T, "f32")
    assert status_word(work) == 0 and torch.isfinite(dHs).all()
    dH, dz, dc = host(dHs), host(dZ), dc_last.astype(np.float64)
    for t in range(T - 1, -1, -1):
        sl, nx = slice(t * Bn, (t + 1) * Bn), slice((t + 1) * Bn, (t + 2) * Bn)
        if t < T - 1:
            check(dH[sl], O.gemm(dz[nx], U.T, dh_in[sl], 1.0, 1.0), TOL_SUM, O.gemm(np.abs(dz[nx]), np.abs(U.T)) + np.abs(dh_in[sl]), "dh total %d" % t)
        rdz, dc = O.lstm_bwd(gates[sl], Cs[sl].astype(np.float64), Cs[nx].astype(np.float64), dH[sl], dc)
        Sdc = np.abs(dc) + np.abs(dH[sl]) + 1e-3
        check(dz[sl], rdz, TOL_EW * 10 * (T - t), np.concatenate([Sdc, Sdc * (1 + np.abs(Cs[sl])), Sdc, np.abs(dH[sl])], axis=1), "dz %d" % t)
    check(host(dc0), dc, TOL_EW * 10 * T, np.abs(dc) + 1.0, "dc0")
