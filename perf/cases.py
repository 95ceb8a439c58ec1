"""The calls whose speed this repository is judged by, as a program that uses the library makes them.

Three kinds of case cover the entry points a training program calls:

* ``step``: one optimizer step of one or more FP8 linears through a stage context: the forward of
  every linear and microbatch, the backward (split dI / deferred dW, or the full backward), finalize
  and commit.  Sizes run from the single 256 x 256 linear with 128 tokens up to the four linears of a
  Llama-3-70B-shaped stage with 8192 tokens.
* ``gemm``: ``qe_fp8_gemm_tn`` on FP8 codes, as a program that keeps its own tapes calls it.
* ``cast``: the FP8 cast with its transpose and scale update (delayed or current scaling).

Inputs are seeded and made on the GPU: X ~ N(0, 1), W ~ N(0, 0.02), dY ~ N(0, 0.01); the outlier
option multiplies 0.1% of X's channels by 300 and draws dY as sign * exp(2 z).
"""
import math

import torch

from paper_2609_23536_amd import qe

FMAX = {qe.E4M3: 448.0, qe.E5M2: 57344.0}
FEMAX = {qe.E4M3: 8, qe.E5M2: 15}
TORCH_FP8 = {qe.E4M3: torch.float8_e4m3fn, qe.E5M2: torch.float8_e5m2}

# (K in-features, N out-features) of the linears of one stage layer: QKV, O, gate+up, down
STAGES = {
    "llama3_8b": ((4096, 6144), (4096, 4096), (4096, 28672), (14336, 4096)),
    "llama3_70b": ((8192, 10240), (8192, 8192), (8192, 57344), (28672, 8192)),
}


def _step(**kw):
    case = {"kind": "step", "stage": "", "k": 0, "n": 0, "tokens": 0, "microbatches": 1, "dtype": "bf16", "out": "bf16",
            "history": 16, "margin": 0, "scaling": "delayed", "backward": "split", "executor": "graph_caller",
            "outliers": False}
    case.update(kw)
    return case


def listed():
    return [
        # One small linear, fp32: the latency of the calls themselves (launches, graph replays, host work).
        _step(name="step_256x256_128tok", k=256, n=256, tokens=128, microbatches=2, dtype="f32", out="f32", history=4),
        # Ragged sizes (nothing a multiple of 16, rows not 16-byte aligned), direct launches, full backward.
        _step(name="step_ragged_1000tok", k=1365, n=2730, tokens=1000, microbatches=2, backward="full",
              executor="eager"),
        # A square projection fed with small microbatches, as a deep pipeline does; the library's default executor.
        _step(name="step_4096x4096_256tok", k=4096, n=4096, tokens=256, microbatches=4, executor="graph_stream"),
        # The zero-bubble microbatch: long reduction, dW initialised by the first microbatch and accumulated by the second.
        _step(name="step_down_8b_2048tok", k=14336, n=4096, tokens=2048, microbatches=2),
        # The whole Llama-3-8B-shaped stage, one 4096-token microbatch.
        _step(name="stage_8b_4096tok", stage="llama3_8b", tokens=4096, history=1024),
        # The whole Llama-3-70B-shaped stage, one 8192-token microbatch: the benchmark's step.
        _step(name="stage_70b_8192tok", stage="llama3_70b", tokens=8192, history=1024),
        # Outlier activations and log-normal gradients, fp32 in and out, current scaling, full backward.
        _step(name="step_8192_current_f32", k=8192, n=8192, tokens=8192, dtype="f32", out="f32", history=1, margin=1,
              scaling="current", backward="full", executor="eager", outliers=True),
        # dI of a small microbatch: few rows, long reduction.
        {"kind": "gemm", "name": "gemm_dgrad_512x4096x14336", "m": 512, "n": 4096, "k": 14336, "fmt_a": "e5m2",
         "fmt_b": "e4m3", "out": "bf16", "accumulate": False, "pad": 0},
        # dW accumulated into an odd-strided view at sizes that divide by no tile.
        {"kind": "gemm", "name": "gemm_wgrad_4100x4100x1040", "m": 4100, "n": 4100, "k": 1040, "fmt_a": "e5m2",
         "fmt_b": "e4m3", "out": "f32", "accumulate": True, "pad": 3},
        # An activation cast with delayed scaling and its scale update, an ordinary size.
        {"kind": "cast", "name": "cast_4096x4096_bf16", "rows": 4096, "cols": 4096, "dtype": "bf16", "fmt": "e4m3",
         "scaling": "delayed", "history": 1024},
        # A gradient cast with current scaling, ragged, through the allocation-free entry.
        {"kind": "cast", "name": "cast_1500x4099_f32_current", "rows": 1500, "cols": 4099, "dtype": "f32",
         "fmt": "e5m2", "scaling": "current_noalloc", "history": 1},
        # The largest weight of the 70B stage, cast once per optimizer step.
        {"kind": "cast", "name": "cast_57344x8192_bf16", "rows": 57344, "cols": 8192, "dtype": "bf16", "fmt": "e4m3",
         "scaling": "delayed", "history": 16},
    ]


def _log_int(rng, lo, hi, odd=0.4):
    """A size spread over the logarithm of [lo, hi]: any integer, or (more often) a multiple of 64 where that fits."""
    v = int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))
    if rng.random() >= odd and v >= 96:
        v = (v + 32) // 64 * 64
    return max(lo, min(hi, v))


def draw(rng):
    kind = rng.choice(("step", "step", "gemm", "cast"))
    if kind == "step":
        while True:
            k, n = _log_int(rng, 128, 16384), _log_int(rng, 128, 28672)
            tokens, mbs = _log_int(rng, 64, 8192), rng.choice((1, 1, 2, 4, 8))
            if 6.0 * k * n * tokens * mbs <= 1.0e13 and 4 * n * k <= 2 ** 31:
                break
        dtype = rng.choice(("bf16", "bf16", "f32"))
        scaling = rng.choice(("delayed", "delayed", "delayed", "current"))
        return _step(k=k, n=n, tokens=tokens, microbatches=mbs, dtype=dtype,
                     out=rng.choice((dtype, "bf16", "f32")),
                     history=1 if scaling == "current" else rng.choice((8, 16, 1024)), margin=rng.choice((0, 0, 1)),
                     scaling=scaling, backward=rng.choice(("split", "split", "full")),
                     executor=rng.choice(("graph_caller", "graph_stream", "eager")), outliers=rng.random() < 0.2)
    if kind == "gemm":
        while True:
            m, n, k = _log_int(rng, 32, 8192), _log_int(rng, 32, 28672), _log_int(rng, 64, 28672)
            if 2.0 * m * n * k <= 5.0e12:
                break
        out = rng.choice(("bf16", "f32"))
        return {"kind": "gemm", "m": m, "n": n, "k": k, "fmt_a": rng.choice(("e4m3", "e5m2")),
                "fmt_b": "e4m3", "out": out, "accumulate": out == "f32" and rng.random() < 0.5,
                "pad": rng.choice((0, 0, 0, 3, 16))}
    while True:
        rows, cols = _log_int(rng, 64, 57344), _log_int(rng, 64, 28672)
        if rows * cols <= 57344 * 8192:
            break
    scaling = rng.choice(("delayed", "delayed", "current", "current_noalloc"))
    return {"kind": "cast", "rows": rows, "cols": cols, "dtype": rng.choice(("bf16", "bf16", "f32")),
            "fmt": rng.choice(("e4m3", "e5m2")), "scaling": scaling,
            "history": rng.choice((4, 16, 1024)) if scaling == "delayed" else 1}


# ------------------------------------------------------------------ inputs
FMT = {"e4m3": qe.E4M3, "e5m2": qe.E5M2}
DT = {"f32": qe.F32, "bf16": qe.BF16}
TDT = {"f32": torch.float32, "bf16": torch.bfloat16}
ESIZE = {"f32": 4, "bf16": 2}


def _gen(seed):
    g = torch.Generator(device="cuda")
    g.manual_seed(int(seed))
    return g


def _normal(g, rows, cols, sigma, dtype):
    x = torch.empty((rows, cols), dtype=TDT[dtype], device="cuda")
    chunk = max(1, (1 << 27) // cols)  # rows at a time, drawn in fp32 and rounded
    for r in range(0, rows, chunk):
        n = min(chunk, rows - r)
        x[r:r + n] = torch.randn((n, cols), generator=g, device="cuda") * sigma
    return x


def _activations(g, rows, cols, dtype, outliers):
    x = _normal(g, rows, cols, 1.0, dtype)
    if outliers:
        ch = torch.randperm(cols, generator=g, device="cuda")[:max(1, round(0.001 * cols))]
        x[:, ch] *= 300
    return x


def _gradients(g, rows, cols, dtype, outliers):
    if not outliers:
        return _normal(g, rows, cols, 0.01, dtype)
    z = torch.randn((rows, cols), generator=g, device="cuda")
    s = torch.randint(0, 2, (rows, cols), generator=g, device="cuda") * 2 - 1
    return (s * torch.exp(2.0 * z)).to(TDT[dtype])


def _linears(case):
    return STAGES[case["stage"]] if case["stage"] else ((case["k"], case["n"]),)


def _step_inputs(case, seed):
    """Weights, and X and dY of every (linear, microbatch)."""
    g = _gen(seed)
    dt, t, out = case["dtype"], case["tokens"], []
    for k, n in _linears(case):
        w = _normal(g, n, k, 0.02, dt)
        xs = [_activations(g, t, k, dt, case["outliers"]) for _ in range(case["microbatches"])]
        dys = [_gradients(g, t, n, dt, case["outliers"]) for _ in range(case["microbatches"])]
        out.append((w, xs, dys))
    return out


def _codes(g, rows, k, fmt):
    """FP8 codes of normal values at the scale the delayed update would give them, row stride a multiple of 16."""
    ld = (k + 15) // 16 * 16
    q = torch.zeros((rows, ld), dtype=torch.uint8, device="cuda")
    x = torch.randn((rows, k), generator=g, device="cuda")
    scale = 2.0 ** _exponent(float(x.abs().max()), fmt, 0)
    q[:, :k] = (x * scale).clamp(-FMAX[fmt], FMAX[fmt]).to(TORCH_FP8[fmt]).view(torch.uint8)
    return q, 1.0 / scale


def _exponent(amax, fmt, margin):
    """floor(log2(fmax / amax)) - margin: fmax = 1.75 * 2^emax, amax = m * 2^e."""
    if not (0.0 < amax < math.inf):
        return 0
    m, e = math.frexp(amax)  # amax = (2 m) * 2^(e - 1)
    v = FEMAX[fmt] - (e - 1) - (1 if 2 * m > 1.75 else 0) - margin
    return max(-126, min(126, v))


# ------------------------------------------------------------------ the program's state
class _Memory:
    """The context's FP8 state as tensors (it stays alive as long as they do)."""

    def __init__(self, ctx, pointer, count):
        self.ctx = ctx
        self.__cuda_array_interface__ = {"shape": (count,), "typestr": "<f4", "data": (int(pointer), False),
                                         "version": 2, "strides": None}


def _state_tensors(ctx, layer):
    got = {}
    for role, name in ((qe.ROLE_X, "x"), (qe.ROLE_W, "w"), (qe.ROLE_DY, "dy")):
        m = ctx.qe_layer_meta(layer, role)
        for what, p, c in (("history", m.amax_history, m.history_len), ("scale", m.scale, 1)):
            got["%s_%s" % (name, what)] = torch.as_tensor(_Memory(ctx, p, c), device="cuda")
    return got


def _ok(status):
    if status != "OK":
        raise RuntimeError(status)


class _Step:
    """A training program: its tensors, its context, and one optimizer step on them."""

    def __init__(self, case, seed):
        self.case = case
        t, mbs = case["tokens"], case["microbatches"]
        self.data = _step_inputs(case, seed)
        ex = case["executor"]
        self.ctx = qe.Context(mbs, use_graphs=ex != "eager", replay_on_caller=ex != "graph_stream")
        scaling = qe.SCALING_CURRENT if case["scaling"] == "current" else qe.SCALING_DELAYED
        lins = _linears(case)
        self.flat = torch.zeros(sum(k * n for k, n in lins), dtype=torch.float32, device="cuda")
        self.layers, self.y, self.dx, self.views, off = [], [], [], [], 0
        for u, (k, n) in enumerate(lins):
            st, layer = self.ctx.qe_layer_register(0, u, n, k, t, self.data[u][0], DT[case["dtype"]], case["history"],
                                                   case["margin"], scaling=scaling)
            _ok(st)
            for m in range(mbs):
                _ok(self.ctx.qe_arena_bind(layer, m, self.flat, self.flat.numel(), off, k))
            self.layers.append(layer)
            self.views.append((off, k))
            self.y.append([torch.zeros((t, n), dtype=TDT[case["out"]], device="cuda") for _ in range(mbs)])
            self.dx.append([torch.zeros((t, k), dtype=TDT[case["out"]], device="cuda") for _ in range(mbs)])
            off += k * n
        if ex != "eager":
            o, i = DT[case["out"]], DT[case["dtype"]]
            _ok(self.ctx.qe_prebuild_graphs(t, i, o, i, o))
        self.epoch = 0
        self.out = {"y": self.y, "dx": self.dx, "grad": [self.flat[o:o + k * n] for (o, _), (k, n) in zip(self.views, lins)],
                    "state": [_state_tensors(self.ctx, layer) for layer in self.layers]}
        self.run()  # the step before: the scales come from its amaxes

    def run(self):
        c, ctx, e = self.case, self.ctx, self.epoch
        i, o, t, mbs = DT[c["dtype"]], DT[c["out"]], c["tokens"], c["microbatches"]
        refs = {}
        for m in range(mbs):
            for u, layer in enumerate(self.layers):
                st, refs[m, u] = ctx.qe_fp8_linear_fwd(layer, qe.key(e, 0, m, u), self.data[u][1][m], i, t, self.y[u][m], o)
                _ok(st)
        for m in range(mbs):
            mode = qe.INIT if m == 0 else qe.ACCUM
            for u in reversed(range(len(self.layers))):
                layer, key, (off, ld), dy, dx = self.layers[u], qe.key(e, 0, m, u), self.views[u], self.data[u][2][m], self.dx[u][m]
                if c["backward"] == "full":
                    _ok(ctx.qe_fp8_linear_bwd_full(layer, key, refs[m, u], dy, i, dx, o, self.flat, off, ld, mode))
                else:
                    _ok(ctx.qe_fp8_linear_dgrad(layer, key, refs[m, u], dy, i, dx, o))
                    _ok(ctx.qe_fp8_linear_wgrad_place(layer, key, refs[m, u], self.flat, off, ld, mode))
        _ok(ctx.qe_arena_finalize())
        _ok(ctx.qe_optimizer_commit())
        self.epoch += 1
        return self.out


class _Gemm:
    def __init__(self, case, seed):
        g = _gen(seed)
        self.case = case
        m, n, k = case["m"], case["n"], case["k"]
        self.a, sa = _codes(g, m, k, FMT[case["fmt_a"]])
        self.b, sb = _codes(g, n, k, FMT[case["fmt_b"]])
        self.inv = torch.tensor([sa, sb], dtype=torch.float32, device="cuda")
        self.c = torch.zeros((m, n + case["pad"]), dtype=TDT[case["out"]], device="cuda")
        if case["accumulate"]:
            self.c.copy_(torch.randn(self.c.shape, generator=g, device="cuda") * math.sqrt(k))

    def run(self):
        c, a, b = self.case, self.a, self.b
        _ok(qe.qe_fp8_gemm_tn(a, FMT[c["fmt_a"]], a.shape[1], b, FMT[c["fmt_b"]], b.shape[1], c["m"], c["n"], c["k"],
                              self.inv[0:1], self.inv[1:2], self.c, DT[c["out"]], self.c.shape[1],
                              qe.ACCUM if c["accumulate"] else qe.INIT))
        return self.c


def _cast_input(case, seed):
    if case["fmt"] == "e5m2":
        return _gradients(_gen(seed), case["rows"], case["cols"], case["dtype"], False)
    return _activations(_gen(seed), case["rows"], case["cols"], case["dtype"], False)


class _Cast:
    def __init__(self, case, seed):
        self.case = case
        r, c, h = case["rows"], case["cols"], case["history"]
        self.x = _cast_input(case, seed)
        self.q_row = torch.zeros((r, (c + 15) // 16 * 16), dtype=torch.uint8, device="cuda")
        self.q_col = torch.zeros((c, (r + 15) // 16 * 16), dtype=torch.uint8, device="cuda")
        self.hist = torch.zeros(h, dtype=torch.float32, device="cuda")
        self.scales = torch.ones(3, dtype=torch.float32, device="cuda")  # scale, its inverse, the cast's snapshot
        self.token = torch.zeros(1, dtype=torch.int64, device="cuda")
        accum = None
        if case["scaling"] != "current_noalloc":
            accum = torch.zeros(qe.AMAX_LINES * qe.AMAX_STRIDE, dtype=torch.float32, device="cuda")
        self.accum = accum
        self.meta = qe.make_meta(self.hist, self.scales[0:1], self.scales[1:2], FMT[case["fmt"]], 0, accum)
        self.out = {"q_row": self.q_row, "q_col": self.q_col, "hist": self.hist, "scales": self.scales, "token": self.token}
        if case["scaling"] == "delayed":
            self.run()  # the cast before: the scale comes from its amax

    def run(self):
        c, s = self.case, self.scales
        args = (self.x, DT[c["dtype"]], c["rows"], c["cols"], self.meta, self.q_row, self.q_row.shape[1], self.q_col,
                self.q_col.shape[1], s[2:3])
        if c["scaling"] == "delayed":
            _ok(qe.qe_quantize_fp8(*args))
            _ok(qe.qe_amax_scale_update([self.meta], self.token))
        elif c["scaling"] == "current":
            _ok(qe.qe_quantize_fp8_current(*args, self.token))
        else:
            _ok(qe.qe_quantize_fp8_current_noalloc(*args, self.token))
        return self.out


def prepare(case, seed):
    return {"step": _Step, "gemm": _Gemm, "cast": _Cast}[case["kind"]](case, seed)


def run(state):
    return state.run()


# ------------------------------------------------------------------ what a pass cannot do without
def work(case):
    if case["kind"] == "step":
        b, f, i, o = 0, 0, ESIZE[case["dtype"]], ESIZE[case["out"]]
        t = case["tokens"] * case["microbatches"]
        for k, n in _linears(case):
            f += 3 * 2 * t * k * n
            b += n * k * i + t * k * i + t * n * i  # W, X, dY in
            b += t * n * o + t * k * o + n * k * 4  # Y, dX, dW out
        return {"bytes": b, "flops": f}
    if case["kind"] == "gemm":
        m, n, k = case["m"], case["n"], case["k"]
        return {"bytes": m * k + n * k + m * n * ESIZE[case["out"]] * (2 if case["accumulate"] else 1),
                "flops": 2 * m * n * k}
    e = case["rows"] * case["cols"]
    return {"bytes": e * (ESIZE[case["dtype"]] + 2) + 8 * case["history"], "flops": 0}


def tolerance(case):
    """Codes, scales and histories are whole or power-of-two values and exact.  Sums are FP32 inside the matrix
    instructions, then rounded once to the output type: about four times the error measured against 64 bits
    (fp32 out 1.2e-5, with outliers 8.5e-5; bf16 out 1.7e-3)."""
    if case["kind"] == "cast":
        return "exact"
    if case["out"] == "bf16":
        return {"rel": 7e-3, "max": 3e-2}
    return {"rel": 3e-4, "max": 1e-2} if case.get("outliers") else {"rel": 5e-5, "max": 2e-3}


# ------------------------------------------------------------------ the same in 64 bits
def _encode(x, exponent, fmt):
    """The FP8 codes of x * 2^exponent, as torch's own cast gives them after clamping."""
    return (x.float() * 2.0 ** exponent).clamp(-FMAX[fmt], FMAX[fmt]).to(TORCH_FP8[fmt])


def _amax(x):
    return float(x.abs().max())


def _quantized(x, amax, fmt, margin):
    """x after its FP8 cast at the scale of `amax`, in 64 bits."""
    e = _exponent(amax, fmt, margin)
    return _encode(x, e, fmt).double() * 2.0 ** -e


def _exact_step(case, seed):
    own = case["scaling"] == "current"
    ys, dxs, grads = [], [], []
    for w, xs, dys in _step_inputs(case, seed):
        ax, ady = max(_amax(x) for x in xs), max(_amax(d) for d in dys)
        wq = _quantized(w, _amax(w), qe.E4M3, case["margin"])
        y, dx, grad = [], [], None
        for x, dy in zip(xs, dys):
            xq = _quantized(x, _amax(x) if own else ax, qe.E4M3, case["margin"])
            dq = _quantized(dy, _amax(dy) if own else ady, qe.E5M2, case["margin"])
            y.append(xq @ wq.t())
            dx.append(dq @ wq)
            g = dq.t() @ xq
            grad = g if grad is None else grad.add_(g)
        ys.append(y)
        dxs.append(dx)
        grads.append(grad.reshape(-1))
    return {"y": ys, "dx": dxs, "grad": grads, "state": None}


def _exact_gemm(case, seed):
    s = _Gemm(case, seed)
    a = s.a[:, :case["k"]].contiguous().view(TORCH_FP8[FMT[case["fmt_a"]]]).double()
    b = s.b[:, :case["k"]].contiguous().view(TORCH_FP8[FMT[case["fmt_b"]]]).double()
    out = s.c.double()
    d = (a @ b.t()) * (s.inv[0].double() * s.inv[1].double())
    if case["accumulate"]:
        out[:, :case["n"]] += d
    else:
        out[:, :case["n"]] = d
    return out


def exact(case, seed):
    if case["kind"] == "step":
        return _exact_step(case, seed)
    if case["kind"] == "gemm":
        return _exact_gemm(case, seed)
    x, fmt, h = _cast_input(case, seed), FMT[case["fmt"]], case["history"]
    a = _amax(x)
    e = _exponent(a, fmt, 0)
    hist = torch.zeros(h, dtype=torch.float64, device="cuda")
    if h > 1:  # two casts recorded; the newest is in the last place
        hist[max(1, h - 2):] = a
    scales = torch.tensor([2.0 ** e, 2.0 ** -e, 2.0 ** -e], dtype=torch.float64, device="cuda")
    return {"q_row": None, "q_col": None, "hist": hist, "scales": scales, "token": None}
