"""The work that programs give this framework, as cases that can be timed and compared.

A case is a dict of plain values.  `prepare` builds what a program holds before the call (inputs drawn from the
seed, parameters, buffers, workspaces), `run` is one pass through the public entry points, `work` the bytes and
operations that the pass cannot do without, `exact` the same results from plain torch in 64 bits.

Kinds:
  mlp_step   one training step of a three-layer classifier (forward, loss, backward, SGD) by `steps.MLPTrainer`
  lm_step    one training step of the LSTM language model by `steps.LSTMTrainer`
  dense      one fully connected layer through `binding.gemm`: forward with bias and activation, gradient of its
             input through the activation of the layer before, weight gradient, and the bias gradient
  lstm       the recurrent layer of a whole sequence, forward and backward, as a function of the tape
  loss       softmax cross-entropy, loss and gradient in one call
  array      relu(a * b + c) over arrays and views of the ndarray layer, by the built-in operation or a user-defined kernel
  reduce     column sums, row sums and the largest element of a matrix
  embedding  lookup, gradient of the table, and the table's Adam update
"""
import math

import torch

from paper_1908_00213_amd import binding as B, steps, tape, workloads

F32, BF16, F64 = torch.float32, torch.bfloat16, torch.float64


def listed():
    return [
        # The smallest whole program: the tiny classifier at batch 32, where every launch counts.
        {"name": "mlp_step_f32_b32", "kind": "mlp_step", "batch": 32, "n_in": 784, "hidden": 100, "classes": 10, "dtype": "f32"},
        # The classifier of the paper's MNIST example at its benchmark size.
        {"name": "mlp_step_f32_b1024", "kind": "mlp_step", "batch": 1024, "n_in": 784, "hidden": 1000, "classes": 10, "dtype": "f32"},
        # The recurrent language model: vocabulary 10000, 650 units, batch 128, 35 steps.
        {"name": "lm_step_f32", "kind": "lm_step", "vocab": 10000, "hidden": 650, "batch": 128, "steps": 35, "dtype": "f32"},
        # A hidden layer of the wide MLP in mixed precision: the largest products.
        {"name": "dense_bf16_8192", "kind": "dense", "batch": 8192, "n_in": 4096, "n_out": 4096, "act": "gelu", "dtype": "bf16"},
        # The first layer of the classifier in mixed precision: a product far too small to fill the chip for long.
        {"name": "dense_bf16_1024", "kind": "dense", "batch": 1024, "n_in": 784, "n_out": 1000, "act": "relu", "dtype": "bf16"},
        # The language model's input projection at its own, unpadded width: rows that start off 16-byte boundaries.
        {"name": "dense_f32_4480", "kind": "dense", "batch": 4480, "n_in": 650, "n_out": 2600, "act": "relu", "dtype": "f32"},
        # The recurrent layer by itself in mixed precision, driven by the tape.
        {"name": "lstm_bf16_35", "kind": "lstm", "batch": 128, "hidden": 672, "steps": 35, "dtype": "bf16"},
        # The loss over the language model's vocabulary.
        {"name": "loss_f32_10000", "kind": "loss", "rows": 4480, "classes": 10000, "dtype": "f32", "grad": "f32"},
        # The array benchmark: large contiguous operands, a broadcast row.
        {"name": "array_f32_8192", "kind": "array", "rows": 8192, "cols": 8192, "layout": "plain", "api": "op", "dtype": "f32"},
        # Views as array programs meet them: a transposed operand and a column slice, sizes that divide nothing.
        {"name": "array_bf16_views", "kind": "array", "rows": 4999, "cols": 3001, "layout": "views", "api": "op", "dtype": "bf16"},
        # Reductions of a matrix whose rows are not whole vectors.
        {"name": "reduce_bf16_10000", "kind": "reduce", "rows": 10000, "cols": 4001, "dtype": "bf16"},
        # The language model's embedding layer and its optimiser.
        {"name": "embedding_f32", "kind": "embedding", "vocab": 10000, "width": 650, "tokens": 4480},
    ]


def _log(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def _size(rng, lo, hi):
    """A size spread over the logarithm of its range: a third as drawn, a third multiples of 8, a third of 64."""
    n, step = _log(rng, lo, hi), rng.choice((1, 8, 64))
    return max(lo, min(hi, (n + step - 1) // step * step))


def draw(rng):
    kind = rng.choice(("mlp_step", "lm_step", "dense", "dense", "dense", "lstm", "loss", "array", "reduce", "embedding"))
    dtype = rng.choice(("f32", "bf16"))
    if kind == "mlp_step":
        return {"kind": kind, "batch": _size(rng, 16, 2048), "n_in": _size(rng, 64, 2048), "hidden": _size(rng, 64, 2048),
                "classes": _log(rng, 2, 1000), "dtype": dtype}
    if kind == "lm_step":
        return {"kind": kind, "vocab": _size(rng, 500, 10000), "hidden": _size(rng, 100, 672), "batch": _size(rng, 8, 128),
                "steps": rng.randint(5, 35), "dtype": dtype}
    if kind == "dense":
        n_in, n_out = _size(rng, 64, 4096), _size(rng, 64, 4096)
        most = (2 ** 35 if dtype == "f32" else 2 ** 37) // (n_in * n_out)          # (no longer than the largest listed cases)
        return {"kind": kind, "batch": min(most, _size(rng, 32, 8192)), "n_in": n_in, "n_out": n_out,
                "act": rng.choice(("relu", "gelu")), "dtype": dtype}
    if kind == "lstm":
        return {"kind": kind, "batch": _size(rng, 8, 128), "hidden": 32 * rng.randint(2, 24) + rng.choice((0, 0, 10)),
                "steps": rng.randint(5, 35), "dtype": dtype}
    if kind == "loss":
        rows = _size(rng, 64, 4480)
        return {"kind": kind, "rows": rows, "classes": _size(rng, 2, min(32768, 44800000 // rows)), "dtype": dtype, "grad": rng.choice(("f32", "bf16"))}
    if kind == "array":
        return {"kind": kind, "rows": _size(rng, 64, 8192), "cols": _size(rng, 64, 8192), "layout": rng.choice(("plain", "views", "slice", "column")),
                "api": rng.choice(("op", "op", "user")), "dtype": dtype}
    if kind == "reduce":
        return {"kind": kind, "rows": _size(rng, 16, 16384), "cols": _size(rng, 16, 16384), "dtype": dtype}
    return {"kind": kind, "vocab": _size(rng, 100, 40000), "width": _size(rng, 16, 1024), "tokens": _size(rng, 32, 16384)}


# ---- inputs -------------------------------------------------------------------------------------------------
class _Draw:
    """Seeded normal, uniform and integer tensors on the GPU, the same for `prepare` and `exact`."""

    def __init__(self, seed):
        self.g = torch.Generator(device="cuda")
        self.g.manual_seed(int(seed))

    def normal(self, *shape, std=1.0, dtype=F32):
        return (torch.randn(*shape, generator=self.g, device="cuda") * std).to(dtype)

    def uniform(self, *shape, dtype=F32):
        return (torch.rand(*shape, generator=self.g, device="cuda") * 2 - 1).to(dtype)

    def ints(self, high, *shape):
        return torch.randint(0, high, shape, generator=self.g, device="cuda", dtype=torch.int32)


def _dt(case, key="dtype"):
    return BF16 if case[key] == "bf16" else F32


def _mlp_inputs(case, seed):
    return workloads.make_mlp("classifier", (case["n_in"], case["hidden"], case["hidden"], case["classes"]), case["batch"], "gelu", int(seed))


def _lm_inputs(case, seed):
    return workloads.config4(int(seed), vocab=case["vocab"], embed=case["hidden"], hidden=case["hidden"], batch=case["batch"], bptt=case["steps"])


def _dense_inputs(case, seed):
    d, dt = _Draw(seed), _dt(case)
    M, K, N = case["batch"], case["n_in"], case["n_out"]
    return {"x": d.normal(M, K, dtype=dt), "W": d.normal(N, K, std=math.sqrt(2.0 / K), dtype=dt), "b": d.normal(N, std=0.1),
            "dv": d.normal(M, N, std=1.0 / M, dtype=dt), "aux": d.normal(M, K, dtype=dt)}


def _lstm_inputs(case, seed):
    d, n, H = _Draw(seed), case["batch"], case["hidden"]
    return {"c0": d.normal(n, H, std=0.5), "h0": d.uniform(n, H) * 0.5, "zx": d.normal(case["steps"] * n, 4 * H),
            "U": d.normal(H, 4 * H, std=math.sqrt(1.0 / H)), "b": d.normal(4 * H, std=0.1),
            "ghs": d.normal(case["steps"] * n, H, std=1e-3, dtype=_dt(case))}


def _loss_inputs(case, seed):
    d = _Draw(seed)
    return {"z": d.normal(case["rows"], case["classes"], std=2.0, dtype=_dt(case)), "t": d.ints(case["classes"], case["rows"])}


def _array_inputs(case, seed):
    d, dt, m, n = _Draw(seed), _dt(case), case["rows"], case["cols"]
    layout = case["layout"]
    a = d.uniform(n, m, dtype=dt).t() if layout == "views" else d.uniform(m, n, dtype=dt)
    b = d.uniform(m, n + 5, dtype=dt)[:, 2:n + 2] if layout in ("views", "slice") else d.uniform(m, n, dtype=dt)
    c = d.uniform(m, 1, dtype=dt) if layout == "column" else d.uniform(1, n, dtype=dt)
    return {"a": a, "b": b, "c": c}


def _embedding_inputs(case, seed):
    d = _Draw(seed)
    return {"table": d.normal(case["vocab"], case["width"]), "ids": d.ints(case["vocab"], case["tokens"]),
            "dout": d.normal(case["tokens"], case["width"], std=1e-3)}


# ---- what a program holds before the call ---------------------------------------------------------------------
def _bytes(n):
    return torch.empty(max(256, int(n)), dtype=torch.uint8, device="cuda")


def prepare(case, seed):
    kind = case["kind"]
    s = {"case": case}
    empty = lambda *shape, dtype=F32: torch.empty(*shape, dtype=dtype, device="cuda")
    if kind == "mlp_step":
        w = _mlp_inputs(case, seed)
        s["trainer"] = steps.MLPTrainer(w.params, w.batch, w.act, w.lr, lowp=case["dtype"] == "bf16")
        x = torch.from_numpy(w.xs[0]).cuda()
        s["x"] = B.cast(x, BF16) if case["dtype"] == "bf16" else x
        s["t"] = torch.from_numpy(w.ts[0]).cuda()
    elif kind == "lm_step":
        w = _lm_inputs(case, seed)
        s["trainer"] = steps.LSTMTrainer(w.params, w.bptt, w.batch, w.lr, lowp=case["dtype"] == "bf16")
        s["ids"], s["targets"] = torch.from_numpy(w.ids).cuda(), torch.from_numpy(w.targets).cuda()
    elif kind == "dense":
        s.update(_dense_inputs(case, seed))
        M, K, N, dt = case["batch"], case["n_in"], case["n_out"], _dt(case)
        s.update(y=empty(M, N, dtype=dt), pre=empty(M, N, dtype=dt) if case["act"] == "gelu" else None,
                 dx=empty(M, K, dtype=dt), dW=empty(N, K), db=empty(N))
        s["ws"] = _bytes(max(B.gemm_workspace_bytes(s["x"], s["W"].t(), s["y"]), B.gemm_workspace_bytes(s["dv"], s["W"], s["dx"]),
                             B.gemm_workspace_bytes(s["dv"].t(), s["x"], s["dW"])))
        s["ws_red"] = _bytes(B.reduce_axis_workspace_bytes(s["dv"], 0))
    elif kind == "lstm":
        i = _lstm_inputs(case, seed)
        s["lowp"] = case["dtype"] == "bf16"
        s["c0"], s["h0"] = (tape.Variable(i[k], requires_grad=False) for k in ("c0", "h0"))
        s["zx"], s["b"] = tape.Parameter(i["zx"], None, "zx"), tape.Parameter(i["b"], None, "b")
        s["U"] = tape.Parameter(i["U"], B.cast(i["U"], BF16) if s["lowp"] else None, "U")
        s["ghs"] = i["ghs"]
    elif kind == "loss":
        s.update(_loss_inputs(case, seed))
        s.update(loss=empty(()), lse=empty(case["rows"]), dz=empty(case["rows"], case["classes"], dtype=_dt(case, "grad")))
        s["ws"] = _bytes(B.softmax_ce_workspace_bytes(case["rows"]))
    elif kind == "array":
        s.update(_array_inputs(case, seed))
        s["out"] = empty(case["rows"], case["cols"], dtype=_dt(case))
        if case["api"] == "user":
            s["kernel"] = B.ElementwiseKernel("T x, T y, T z", "T w", "w = max(x * y + z, (T)0)", "mad_relu")
            s["kernel"].prepare(s["a"], s["b"], s["c"], s["out"])
    elif kind == "reduce":
        m, n = case["rows"], case["cols"]
        s["x"] = _Draw(seed).normal(m, n, dtype=_dt(case))
        s.update(cols=empty(n), rows=empty(m), top=empty(()))
        s["ws"] = _bytes(max(B.reduce_axis_workspace_bytes(s["x"], axis) for axis in (0, 1, None)))
    elif kind == "embedding":
        s.update(_embedding_inputs(case, seed))
        V, D = case["vocab"], case["width"]
        s.update(out=empty(case["tokens"], D), grad=empty(V, D), m=torch.zeros(V, D, device="cuda"), v=torch.zeros(V, D, device="cuda"), step=0)
    else:
        raise ValueError("unknown kind %r" % kind)
    return s


# ---- one pass ---------------------------------------------------------------------------------------------------
def run(s):
    case = s["case"]
    kind = case["kind"]
    if kind == "mlp_step":
        tr = s["trainer"]
        loss = tr.step(s["x"], s["t"])
        return {"loss": loss, "logits": tr.logits, "dW": tr.dW, "db": tr.db}
    if kind == "lm_step":
        tr = s["trainer"]
        loss = tr.step(s["ids"], s["targets"])
        return {"loss": loss, "lse": tr.lse, "h": tr.Hs, "grads": tr.g}
    if kind == "dense":
        gelu, ws = case["act"] == "gelu", s["ws"]
        B.gemm(s["x"], s["W"].t(), s["y"], epilogue="bias_gelu" if gelu else "bias_relu", bias=s["b"], preact_out=s["pre"], ws=ws)
        B.gemm(s["dv"], s["W"], s["dx"], epilogue="gelu_bwd" if gelu else "relu_bwd", aux=s["aux"], ws=ws)
        B.gemm(s["dv"].t(), s["x"], s["dW"], ws=ws)
        B.reduce_axis("sum", s["dv"], 0, s["db"], ws=s["ws_red"])
        return {"y": s["y"], "dx": s["dx"], "dW": s["dW"], "db": s["db"]}
    if kind == "lstm":
        for p in (s["zx"], s["U"], s["b"]):
            p.cleargrad()
        c, h, hs = tape.n_step_lstm(s["c0"], s["h0"], s["zx"], s["U"], s["b"], case["steps"], s["lowp"])
        hs.grad = s["ghs"]
        hs.backward()
        return {"hs": hs.array, "c": c.array, "dz": s["zx"].grad, "dU": s["U"].grad, "db": s["b"].grad}
    if kind == "loss":
        B.softmax_ce_fwd_bwd(s["z"], s["t"], s["loss"], s["dz"], lse=s["lse"], ws=s["ws"])
        return {"loss": s["loss"], "lse": s["lse"], "dz": s["dz"]}
    if kind == "array":
        if case["api"] == "user":
            return s["kernel"](s["a"], s["b"], s["c"], s["out"])
        return B.elementwise_broadcast("mad_relu", [s["a"], s["b"], s["c"]], s["out"])
    if kind == "reduce":
        B.reduce_axis("sum", s["x"], 0, s["cols"], ws=s["ws"])
        B.reduce_axis("sum", s["x"], 1, s["rows"], ws=s["ws"])
        B.reduce_axis("max", s["x"], None, s["top"], ws=s["ws"])
        return {"cols": s["cols"], "rows": s["rows"], "top": s["top"]}
    s["step"] += 1
    B.embed_fwd(s["table"], s["ids"], s["out"])
    B.embed_bwd(s["ids"], s["dout"], s["grad"])
    B.adam_update_multi([s["table"]], [s["grad"]], [s["m"]], [s["v"]], 1e-3, s["step"])
    return {"out": s["out"], "grad": s["grad"], "table": s["table"], "m": s["m"], "v": s["v"]}


# ---- bytes and operations a pass cannot do without ------------------------------------------------------------------
def work(case):
    kind = case["kind"]
    e = 2 if case.get("dtype") == "bf16" else 4
    if kind == "mlp_step":
        M, sizes = case["batch"], (case["n_in"], case["hidden"], case["hidden"], case["classes"])
        params = sum(a * b + b for a, b in zip(sizes, sizes[1:]))
        acts = M * sum(sizes)
        flops = sum(2.0 * M * a * b * (2 if l == 0 else 3) for l, (a, b) in enumerate(zip(sizes, sizes[1:])))
        # parameters read, gradients written, parameters updated (and their bf16 copies); activations written once and read once
        return {"bytes": params * (12 + (4 if e == 2 else 0)) + 2 * acts * e, "flops": flops}
    if kind == "lm_step":
        T, n, H, V = case["steps"], case["batch"], case["hidden"], case["vocab"]
        N = T * n
        params = 2 * V * H + 8 * H * H + 4 * H + V
        flops = 2.0 * N * H * 4 * H * 6 + 2.0 * N * H * V * 3
        return {"bytes": params * (12 + (4 if e == 2 else 0)) + N * (V * (4 + e) + 8 * H * 4 + 6 * H * e), "flops": flops}
    if kind == "dense":
        M, K, N = case["batch"], case["n_in"], case["n_out"]
        acts = M * K * 3 + M * N * 2 + N * K + (M * N if case["act"] == "gelu" else 0)
        return {"bytes": acts * e + N * K * 4 + 2 * N * 4, "flops": 6.0 * M * K * N}
    if kind == "lstm":
        N, H = case["steps"] * case["batch"], case["hidden"]
        # zx, gates (written and read), cell states, hidden states, their gradients, dz; U and its gradient
        return {"bytes": N * H * (4 * 4 + 2 * 4 * 4 + 2 * 4 + 3 * e + 4 * e) + 4 * H * H * (4 + 2 * e), "flops": 2.0 * N * H * 4 * H * 3}
    if kind == "loss":
        n = case["rows"] * case["classes"]
        return {"bytes": n * (e + (2 if case["grad"] == "bf16" else 4)) + case["rows"] * 8, "flops": 6.0 * n}
    if kind == "array":
        m, n = case["rows"], case["cols"]
        return {"bytes": e * (3 * m * n + (m if case["layout"] == "column" else n)), "flops": 3.0 * m * n}
    if kind == "reduce":
        m, n = case["rows"], case["cols"]
        return {"bytes": 3 * m * n * e + 4 * (m + n), "flops": 3.0 * m * n}
    V, D, N = case["vocab"], case["width"], case["tokens"]
    return {"bytes": 4 * (min(N, V) * D + 2 * N * D + V * D + 7 * V * D) + 8 * N, "flops": float(N * D + 12 * V * D)}


# Each bound is about four times the largest difference seen between this framework and 64-bit results.
def tolerance(case):
    kind, low = case["kind"], case.get("dtype") == "bf16"
    if kind in ("mlp_step", "lm_step", "lstm"):
        return {"rel": 1.5e-2 if low else 5e-6}
    if kind == "dense":
        return {"rel": 8e-3 if low else 4e-6}
    if kind == "loss":
        return {"rel": 8e-3 if case["grad"] == "bf16" else 1e-6}
    if kind == "array":
        return {"rel": 8e-3 if low else 1.5e-7}
    return {"rel": 5e-7}


# ---- the same in 64 bits ------------------------------------------------------------------------------------------------
def _gelu(x):
    return 0.5 * x * (1.0 + torch.erf(x / math.sqrt(2.0)))


def _gelu_grad(x):
    return 0.5 * (1.0 + torch.erf(x / math.sqrt(2.0))) + x * torch.exp(-0.5 * x * x) / math.sqrt(2.0 * math.pi)


def _softmax_grad(z, t):
    """(mean loss, log-sum-exp, gradient of the mean loss)"""
    n = z.shape[0]
    lse = torch.logsumexp(z, 1)
    idx = torch.arange(n, device=z.device)
    loss = (lse - z[idx, t.long()]).mean()
    g = torch.exp(z - lse[:, None])
    g[idx, t.long()] -= 1.0
    return loss, lse, g / n


def _cell_forward(zx, U, b, c, h, n_steps):
    n, H = c.shape
    hs, cs, gates = [h], [c], []
    for t in range(n_steps):
        z = zx[t * n:(t + 1) * n] + h @ U + b
        i, f, g, o = (torch.sigmoid(z[:, :H]), torch.sigmoid(z[:, H:2 * H]), torch.tanh(z[:, 2 * H:3 * H]), torch.sigmoid(z[:, 3 * H:]))
        c = f * c + i * g
        h = o * torch.tanh(c)
        hs.append(h), cs.append(c), gates.append((i, f, g, o))
    return hs, cs, gates


def _cell_backward(dhs, U, cs, gates, n_steps):
    """dz (T*n, 4H) for the gradient `dhs` (T*n, H) that reaches every h from outside"""
    n = cs[0].shape[0]
    dz, dc, back = [None] * n_steps, torch.zeros_like(cs[0]), torch.zeros_like(cs[0])
    for t in range(n_steps - 1, -1, -1):
        i, f, g, o = gates[t]
        tc = torch.tanh(cs[t + 1])
        dh = dhs[t * n:(t + 1) * n] + back
        dc = dc + dh * o * (1 - tc * tc)
        dz[t] = torch.cat([dc * g * i * (1 - i), dc * cs[t] * f * (1 - f), dc * i * (1 - g * g), dh * tc * o * (1 - o)], 1)
        back, dc = dz[t] @ U.t(), dc * f
    return torch.cat(dz)


def exact(case, seed):
    kind, low = case["kind"], case.get("dtype") == "bf16"
    if kind == "mlp_step":
        w = _mlp_inputs(case, seed)
        q = lambda a: (torch.from_numpy(a).cuda().to(BF16) if low else torch.from_numpy(a).cuda()).to(F64)
        Ws, bs, t = [q(W) for W, _ in w.params], [torch.from_numpy(b).cuda().to(F64) for _, b in w.params], torch.from_numpy(w.ts[0]).cuda()
        hs, zs = [q(w.xs[0])], []
        for l, (W, b) in enumerate(zip(Ws, bs)):
            zs.append(hs[-1] @ W.t() + b)
            hs.append(_gelu(zs[-1]) if l + 1 < len(Ws) else zs[-1])
        loss, _, d = _softmax_grad(zs[-1], t)
        dW, db = [None] * len(Ws), [None] * len(Ws)
        for l in range(len(Ws) - 1, -1, -1):
            dW[l], db[l] = d.t() @ hs[l], d.sum(0)
            if l > 0:
                d = (d @ Ws[l]) * _gelu_grad(zs[l - 1])
        return {"loss": loss, "logits": zs[-1], "dW": dW, "db": db}
    if kind == "lm_step":
        w = _lm_inputs(case, seed)
        q = lambda k: (torch.from_numpy(w.params[k]).cuda().to(BF16) if low and k in ("E", "W", "U", "W_out") else torch.from_numpy(w.params[k]).cuda()).to(F64)
        E, W, U, b, Wo, bo = (q(k) for k in ("E", "W", "U", "b", "W_out", "b_out"))
        ids, tg = torch.from_numpy(w.ids).cuda().reshape(-1).long(), torch.from_numpy(w.targets).cuda().reshape(-1)
        n, T, H = w.batch, w.bptt, w.hidden
        zero = torch.zeros(n, H, dtype=F64, device="cuda")
        X = E[ids]
        hs, cs, gates = _cell_forward(X @ W, U, b, zero, zero, T)
        h_all = torch.cat(hs[1:])
        loss, lse, d = _softmax_grad(h_all @ Wo.t() + bo, tg)
        dz = _cell_backward(d @ Wo, U, cs, gates, T)
        dE = torch.zeros_like(E).index_add_(0, ids, dz @ W.t())
        grads = {"E": dE, "W": X.t() @ dz, "U": torch.cat(hs[:-1]).t() @ dz, "b": dz.sum(0), "W_out": d.t() @ h_all, "b_out": d.sum(0)}
        return {"loss": loss, "lse": lse, "h": torch.cat(hs), "grads": grads}
    if kind == "dense":
        i = {k: v.to(F64) for k, v in _dense_inputs(case, seed).items()}
        z = i["x"] @ i["W"].t() + i["b"]
        dx = i["dv"] @ i["W"]
        y, dx = (_gelu(z), dx * _gelu_grad(i["aux"])) if case["act"] == "gelu" else (z.clamp(min=0), dx * (i["aux"] > 0))
        return {"y": y, "dx": dx, "dW": i["dv"].t() @ i["x"], "db": i["dv"].sum(0)}
    if kind == "lstm":
        i = _lstm_inputs(case, seed)
        U = (i["U"].to(BF16) if low else i["U"]).to(F64)
        c0, h0, zx, b, ghs = (i[k].to(F64) for k in ("c0", "h0", "zx", "b", "ghs"))
        hs, cs, gates = _cell_forward(zx, U, b, c0, h0, case["steps"])
        dz = _cell_backward(ghs, U, cs, gates, case["steps"])
        return {"hs": torch.cat(hs[1:]), "c": cs[-1], "dz": dz, "dU": torch.cat(hs[:-1]).t() @ dz, "db": dz.sum(0)}
    if kind == "loss":
        i = _loss_inputs(case, seed)
        loss, lse, g = _softmax_grad(i["z"].to(F64), i["t"])
        return {"loss": loss, "lse": lse, "dz": g}
    if kind == "array":
        i = {k: v.to(F64) for k, v in _array_inputs(case, seed).items()}
        return (i["a"] * i["b"] + i["c"]).clamp(min=0)
    if kind == "reduce":
        x = _Draw(seed).normal(case["rows"], case["cols"], dtype=_dt(case)).to(F64)
        return {"cols": x.sum(0), "rows": x.sum(1), "top": x.max()}
    i = _embedding_inputs(case, seed)
    ids, table = i["ids"].long(), i["table"].to(F64)
    g = torch.zeros_like(table).index_add_(0, ids, i["dout"].to(F64))
    m, v = 0.1 * g, 0.001 * g * g                                  # first step of Adam: betas 0.9 and 0.999
    table2 = table - 1e-3 * (m / 0.1) / (torch.sqrt(v / 0.001) + 1e-8)
    return {"out": table[ids], "grad": g, "table": table2, "m": m, "v": v}
