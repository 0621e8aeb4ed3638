"""The work that users of this library have it do, as timed cases.

A case is a dict of plain values. Four kinds, each through the public calls of
paper_1805_08939_amd.api:

  fc         one fully connected layer of a training step under row patterns:
             the weight compaction (where the layer keeps its weights
             output-major and its inputs are dropped), forward, backward and,
             where asked, the momentum update
  mlp        a whole training step of a ReLU MLP: every layer's forward,
             backward and update
  tile       one layer under a tile pattern: the plan, forward and backward
  lstm       one or more stacked LSTM layers under row patterns on the hidden
             units: forward and (for training) backward through time
  lstm_tile  one LSTM layer under a tile pattern on its weights

A pattern's period is part of the case (it sets the work); its offset, like
every input, comes from the seed. Inputs are drawn on the GPU. As in the
library's own benchmark, device addresses and the stream are looked up once,
in prepare.
"""

import math
import random

import torch

from paper_1805_08939_amd import api

DEV = "cuda:0"
LR, MOMENTUM = 1e-4, 0.9


def listed():
    return [
        # the smallest layer of the benchmark: MNIST inputs, one hidden layer, batch 64
        dict(name="fc-784x512-f32-b64", kind="fc", dtype="f32", batch=64, inputs=784, outputs=512, period_in=1,
             period_out=2, layout="full", relu=True, zero=False, update=False),
        # the three-layer MNIST MLP, the whole training step, both hidden layers at half rate
        dict(name="mlp-784-2048-2048-10-f32-b128", kind="mlp", dtype="f32", batch=128, d0=784, d1=2048, d2=2048,
             d3=10, period1=2, period2=2),
        # a layer whose sizes fit no tile and whose rows fit no 16 bytes, dropped entries written zero
        dict(name="fc-1023x1537-bf16-b100", kind="fc", dtype="bf16", batch=100, inputs=1023, outputs=1537, period_in=3,
             period_out=2, layout="full", relu=True, zero=True, update=False),
        # the output layer of a language model (1500 hidden units at half rate, 8800 words, 35 steps of batch 20)
        dict(name="fc-head-1500x8800-f32-b700", kind="fc", dtype="f32", batch=700, inputs=1500, outputs=8800,
             period_in=2, period_out=1, layout="input_major", relu=False, zero=False, update=False),
        # first layer of the wide MLP: all inputs kept, half of the outputs
        dict(name="fc-8192x8192-bf16-b2048-half", kind="fc", dtype="bf16", batch=2048, inputs=8192, outputs=8192,
             period_in=1, period_out=2, layout="full", relu=True, zero=False, update=True),
        # its middle layer at a high rate: both sides dropped, compact weights
        dict(name="fc-8192x8192-bf16-b2048-high", kind="fc", dtype="bf16", batch=2048, inputs=8192, outputs=8192,
             period_in=4, period_out=3, layout="compact", relu=True, zero=False, update=True),
        # the tile-pattern layer of the benchmark
        dict(name="tile-4096x4096-bf16-b512-t64", kind="tile", dtype="bf16", batch=512, inputs=4096, outputs=4096,
             tile=64, p=0.5, zero=False),
        # the hidden layer of the MNIST MLP under 32 x 32 tiles, the paper's tile size
        dict(name="tile-2048x2048-f32-b128-t32", kind="tile", dtype="f32", batch=128, inputs=2048, outputs=2048,
             tile=32, p=0.5, zero=False),
        # evaluation of a medium LSTM: forward only, nothing dropped, a batch whose rows fit no 16 bytes
        dict(name="lstm-fwd-t35-b10-650", kind="lstm", seq=35, batch=10, inputs=650, hidden=650, layers=1, period=1,
             train=False),
        # one LSTM layer of the benchmark in training, half of the hidden units
        dict(name="lstm-t35-b64-1024", kind="lstm", seq=35, batch=64, inputs=1024, hidden=1024, layers=1, period=2,
             train=True),
        # the stacked language model in training, half of the hidden units
        dict(name="lstm-2x1500-t35-b20", kind="lstm", seq=35, batch=20, inputs=1500, hidden=1500, layers=2, period=2,
             train=True),
        # the LSTM layer with a tile pattern on its weights in training
        dict(name="lstm-tile-t35-b64-1024", kind="lstm_tile", seq=35, batch=64, inputs=1024, hidden=1024, tile=64,
             period=2),
    ]


def _log(rng, lo, hi):
    return max(lo, min(hi, round(math.exp(rng.uniform(math.log(lo), math.log(hi))))))


def draw(rng):
    """One more case of the same ranges; never more work than the largest listed one of its kind."""
    kind = rng.choice(["fc", "fc", "fc", "mlp", "tile", "tile", "lstm", "lstm", "lstm_tile"])
    while True:
        if kind == "fc":
            c = dict(kind="fc", dtype=rng.choice(["f32", "bf16"]), batch=_log(rng, 16, 2048),
                     inputs=_log(rng, 64, 8192), outputs=_log(rng, 64, 8192), period_in=rng.choice([1, 1, 2, 3, 4, 8]),
                     period_out=rng.choice([1, 2, 2, 3, 5]), layout="full", relu=rng.random() < 0.7,
                     zero=rng.random() < 0.3, update=rng.random() < 0.5)
            if rng.random() < 0.5:  # the sizes that networks are usually given; the others are odd ones too
                for k in ("batch", "inputs", "outputs"):
                    c[k] = (c[k] + 15) // 16 * 16
            if c["period_out"] == 1:
                c["layout"] = rng.choice(["full", "input_major"])
            elif c["period_in"] > 1:
                c["layout"] = rng.choice(["full", "compact"])
            if work(c)["flops"] <= (3.5e10 if c["dtype"] == "f32" else 8e10):
                return c
        elif kind == "mlp":
            return dict(kind="mlp", dtype="f32", batch=_log(rng, 16, 256), d0=_log(rng, 256, 1024),
                        d1=_log(rng, 256, 3072), d2=_log(rng, 256, 3072), d3=rng.choice([10, 26, 100]),
                        period1=rng.choice([1, 2, 3, 4]), period2=rng.choice([1, 2, 3, 4]))
        elif kind == "tile":
            tile = rng.choice([32, 64])
            c = dict(kind="tile", dtype=rng.choice(["f32", "bf16"]), batch=_log(rng, 16, 512),
                     inputs=tile * _log(rng, 4, 4096 // tile), outputs=tile * _log(rng, 4, 4096 // tile), tile=tile,
                     p=rng.choice([0.3, 0.5, 0.7]), zero=rng.random() < 0.3)
            if rng.random() < 0.6:
                c["batch"] = (c["batch"] + 15) // 16 * 16
            if work(c)["flops"] <= (8e9 if c["dtype"] == "f32" else 3e10):
                return c
        elif kind == "lstm":
            c = dict(kind="lstm", seq=_log(rng, 8, 35), batch=_log(rng, 4, 64), inputs=_log(rng, 128, 1500),
                     hidden=_log(rng, 128, 1500), layers=rng.choice([1, 1, 2]), period=rng.choice([1, 2, 2, 3, 4]),
                     train=rng.random() < 0.8)
            if rng.random() < 0.6:
                for k in ("batch", "inputs", "hidden"):
                    c[k] = (c[k] + 3) // 4 * 4
            odd = any(c[k] % 4 for k in ("batch", "inputs", "hidden"))
            if work(c)["flops"] <= (1e10 if odd else 4e10):
                return c
        else:
            tile = rng.choice([32, 64])
            c = dict(kind="lstm_tile", seq=_log(rng, 8, 35 if tile == 64 else 16), batch=_log(rng, 8, 64),
                     inputs=tile * _log(rng, 4, 1024 // tile), hidden=tile * _log(rng, 4, 1024 // tile), tile=tile,
                     period=rng.choice([1, 2, 3]))
            if rng.random() < 0.6:
                c["batch"] = (c["batch"] + 3) // 4 * 4
            if work(c)["flops"] <= (5e10 if c["batch"] % 4 == 0 else 1e10):
                return c


# --------------------------------------------------------------------- shared

def _cdiv(a, b):
    return -(-a // b)


class _Draws:
    """Seeded draws on the GPU, and the pattern offsets of the seed."""

    def __init__(self, seed):
        self.g = torch.Generator(device=DEV)
        self.g.manual_seed(int(seed))
        self.rng = random.Random(int(seed) * 7919 + 1)

    def normal(self, *shape, std=1.0):
        return torch.randn(*shape, generator=self.g, device=DEV) * std

    def uniform(self, a, *shape):
        return (torch.rand(*shape, generator=self.g, device=DEV) * 2 - 1) * a

    def offset(self, period):
        return self.rng.randrange(period)


def _dtype(c):
    return torch.float32 if c["dtype"] == "f32" else torch.bfloat16


def _ard_dtype(c):
    return api.ARD_F32 if c["dtype"] == "f32" else api.ARD_BF16


def _workspace(nbytes):
    t = torch.empty(max(nbytes, 16) // 4 + 4, device=DEV)
    return t, (t.data_ptr(), t.numel() * 4)


def _dropped(c):
    return api.ARD_DROPPED_ZERO if c["zero"] else api.ARD_DROPPED_SKIP


# ------------------------------------------------------------------- fc layer

class _Fc:
    """One layer's buffers. x and dx may be given (an MLP's layers share them)."""

    def __init__(self, d, dtype, batch, n_in, n_out, pin, pout, layout, relu, zero, w_std, x=None, dx=None, gate=True):
        sdt = torch.float32 if dtype == "f32" else torch.bfloat16
        self.layout, self.batch, self.n_in, self.n_out = layout, batch, n_in, n_out
        self.gate = gate
        self.pin, self.pout = pin, pout  # (period, offset)
        # a hidden layer's input is a ReLU's output, whose dropped rows are zero
        if x is None:
            x = torch.relu(d.normal(n_in, batch)).to(sdt)
        self.x = x
        w = d.normal(n_out, n_in, std=w_std).to(sdt)
        self.w = w.t().contiguous() if layout == "input_major" else w
        del w
        self.bias = d.normal(n_out, std=0.02)
        self.y = torch.zeros(n_out, batch, dtype=sdt, device=DEV)
        dy = d.normal(n_out, batch, std=1.0 / batch)
        if relu:  # the layer above writes the output derivative already gated
            dy = dy * (d.normal(n_out, batch) > 0)
        self.dy = dy.to(sdt)
        self.dx = torch.zeros(n_in, batch, dtype=sdt, device=DEV) if dx is None else dx
        plans = [api.ard_row_plan() for _ in range(2)]
        self.plans = plans
        api.ard_plan_rows(n_in, pin[0], pin[1], None, plan=plans[0])
        api.ard_plan_rows(n_out, pout[0], pout[1], None, plan=plans[1])
        code = {"full": api.ARD_WEIGHTS_FULL, "compact": api.ARD_WEIGHTS_COMPACT_GRAD,
                "input_major": api.ARD_WEIGHTS_INPUT_MAJOR}[layout]
        self.desc = api.fc_desc(api.ARD_F32 if dtype == "f32" else api.ARD_BF16, batch, n_in, n_out, plans[0], plans[1],
                                1.0, api.ARD_ACT_RELU if relu else api.ARD_ACT_NONE,
                                api.ARD_DROPPED_ZERO if zero else api.ARD_DROPPED_SKIP, code)
        if layout == "compact":
            # buffers for any offset of the pattern; this one's matrix [kept][ld] is at their start
            self.ld = api.ard_fc_compact_ld(self.desc)
            size = _cdiv(n_out, pout[0]) * ((_cdiv(n_in, pin[0]) + 7) // 8 * 8)
            self.wc = torch.zeros(size, dtype=sdt, device=DEV)
            self.dw = torch.zeros(size, device=DEV)
        else:
            self.wc = None
            self.dw = torch.zeros_like(self.w, dtype=torch.float32)
        self.db = torch.zeros(n_out, device=DEV)
        self.v = self.vb = None
        self.ws, self.ws_arg = _workspace(api.ard_fc_workspace_bytes(self.desc))
        self.stream = torch.cuda.current_stream().cuda_stream
        self.p = {k: getattr(self, k).data_ptr() for k in ("x", "w", "bias", "y", "dy", "dx", "dw", "db")}
        self.p["wt"] = self.wc.data_ptr() if self.wc is not None else self.p["w"]

    def momentum(self):
        self.v, self.vb = torch.zeros(self.w.shape, device=DEV), torch.zeros(self.n_out, device=DEV)
        self.p["v"], self.p["vb"] = self.v.data_ptr(), self.vb.data_ptr()

    def plan(self):
        """A step's row patterns: list-free plans (the kept rows are strided views)."""
        api.ard_plan_rows(self.n_in, self.pin[0], self.pin[1], None, self.stream, plan=self.plans[0])
        api.ard_plan_rows(self.n_out, self.pout[0], self.pout[1], None, self.stream, plan=self.plans[1])

    def compact(self):
        if self.wc is not None:
            api.ard_fc_compact_weights(self.desc, self.p["w"], self.p["wt"], self.stream)

    def forward(self):
        p = self.p
        api.ard_fc_fwd(self.desc, p["x"], p["wt"], p["bias"], p["y"], self.ws_arg, self.stream)

    def backward(self, data=True):
        p = self.p
        if data:
            api.ard_fc_bwd(self.desc, p["x"], p["dy"], None, p["wt"], p["dx"], p["dw"], p["db"], self.ws_arg,
                           self.stream, Xgate=p["x"] if self.gate else None)
        else:
            api.ard_fc_bwd_weight(self.desc, p["x"], p["dy"], None, p["dw"], p["db"], self.ws_arg, self.stream)

    def update(self):
        p = self.p
        api.ard_fc_sgd_momentum(self.desc, p["w"], p["v"], p["dw"], p["bias"], p["vb"], p["db"], LR, MOMENTUM,
                                self.stream)


def _kept(n, pat):
    return list(range(pat[1], n, pat[0]))


def _fc_prepare(c, seed):
    d = _Draws(seed)
    pin, pout = (c["period_in"], d.offset(c["period_in"])), (c["period_out"], d.offset(c["period_out"]))
    f = _Fc(d, c["dtype"], c["batch"], c["inputs"], c["outputs"], pin, pout, c["layout"], c["relu"], c["zero"],
            math.sqrt(2.0 / c["inputs"]))
    if c["update"]:
        f.momentum()
    return f


def _fc_run(c, f):
    f.plan()
    f.compact()
    f.forward()
    f.backward()
    out = {"y": f.y, "dx": f.dx, "dw": f.dw, "db": f.db}
    if c["update"]:
        f.update()
        out.update(w=f.w, v=f.v, bias=f.bias, vb=f.vb)
    return out


def _fc_exact(c, seed):
    f = _fc_prepare(c, seed)
    si, so = _kept(c["inputs"], f.pin), _kept(c["outputs"], f.pout)
    si, so = torch.tensor(si, device=DEV), torch.tensor(so, device=DEV)
    w = (f.w.t() if c["layout"] == "input_major" else f.w).double()
    x, dy = f.x.double()[si], f.dy.double()[so]
    ws = w[so][:, si]
    y = torch.zeros(f.y.shape, dtype=torch.float64, device=DEV)
    yk = ws @ x + f.bias.double()[so, None]
    y[so] = yk.clamp(min=0) if c["relu"] else yk
    dx = torch.zeros(f.dx.shape, dtype=torch.float64, device=DEV)
    dx[si] = (ws.t() @ dy) * (x > 0)
    dwk = dy @ x.t()
    dw = torch.zeros(f.dw.shape, dtype=torch.float64, device=DEV)
    full = torch.zeros(w.shape, dtype=torch.float64, device=DEV)
    full[so[:, None], si[None, :]] = dwk
    if c["layout"] == "compact":
        dw[:len(so) * f.ld].view(len(so), f.ld)[:, :len(si)] = dwk
    else:
        dw.copy_(full.t() if c["layout"] == "input_major" else full)
    db = torch.zeros(c["outputs"], dtype=torch.float64, device=DEV)
    db[so] = dy.sum(1)
    out = {"y": y, "dx": dx, "dw": dw, "db": db}
    if c["update"]:
        v, w2 = full, w - LR * full
        if c["layout"] == "input_major":
            v, w2 = v.t(), w2.t()
        out.update(w=w2, v=v, bias=f.bias.double() - LR * db, vb=db)
    return out


def _fc_work(c):
    e = 4 if c["dtype"] == "f32" else 2
    k, n, b = _cdiv(c["inputs"], c["period_in"]), _cdiv(c["outputs"], c["period_out"]), c["batch"]
    nbytes = e * (k * n + 2 * k * b + 2 * n * b) + 4 * (k * n + 2 * n)  # w, x, dx, y, dy, dw, bias, db
    if c["zero"]:  # the zeros of y, dx, dw and db
        nbytes += e * b * (c["inputs"] - k + c["outputs"] - n) + 4 * (c["inputs"] * c["outputs"] - k * n)
    if c["update"]:
        nbytes += k * n * (e + 8) + 12 * n  # w written, v read and written
    return {"bytes": nbytes, "flops": 6.0 * k * n * b}


# ------------------------------------------------------------------------ mlp

def _mlp_prepare(c, seed):
    d = _Draws(seed)
    dims = [c["d0"], c["d1"], c["d2"], c["d3"]]
    pats = [(1, 0), (c["period1"], d.offset(c["period1"])), (c["period2"], d.offset(c["period2"])), (1, 0)]
    layers = []
    for l in range(3):
        # Xavier weights; the first input is plain data, the last layer keeps every output and stores its
        # weights input-major
        below = layers[-1] if layers else None
        x = below.y if below else d.normal(dims[0], c["batch"])
        layout = "input_major" if l == 2 else "compact" if pats[l][0] > 1 else "full"
        layers.append(_Fc(d, c["dtype"], c["batch"], dims[l], dims[l + 1], pats[l], pats[l + 1], layout, l < 2, False,
                          math.sqrt(2.0 / (dims[l] + dims[l + 1])), x=x, dx=below.dy if below else None))
        layers[-1].momentum()
    return layers


def _mlp_run(layers):
    for f in layers:
        f.plan()
    for f in layers:
        f.compact()
    for f in layers:
        f.forward()
    for l in (2, 1, 0):
        layers[l].backward(data=l > 0)
    for f in layers:
        f.update()
    return [{"y": layers[2].y}] + [{"dw": f.dw, "db": f.db, "w": f.w, "v": f.v, "bias": f.bias} for f in layers]


def _mlp_exact(c, seed):
    """The logits and the top layer's gradients. Those below pass the ReLU gates
    of 32-bit activations, where a value next to zero may go either way: they
    have no one true value."""
    layers = _mlp_prepare(c, seed)
    x, f = layers[0].x.double(), layers[0]
    for f in layers[:2]:
        si, so = torch.tensor(_kept(f.n_in, f.pin), device=DEV), torch.tensor(_kept(f.n_out, f.pout), device=DEV)
        y = torch.zeros(f.n_out, f.batch, dtype=torch.float64, device=DEV)
        y[so] = (f.w.double()[so][:, si] @ x[si] + f.bias.double()[so, None]).clamp(min=0)
        x = y
    f = layers[2]
    si = torch.tensor(_kept(f.n_in, f.pin), device=DEV)
    w, dy = f.w.double(), f.dy.double()
    y = w[si].t() @ x[si] + f.bias.double()[:, None]
    dw = torch.zeros(f.dw.shape, dtype=torch.float64, device=DEV)
    dw[si] = x[si] @ dy.t()
    db = dy.sum(1)
    none = dict.fromkeys(("dw", "db", "w", "v", "bias"))
    return [{"y": y}, none, none, {"dw": dw, "db": db, "w": w - LR * dw, "v": dw, "bias": f.bias.double() - LR * db}]


def _mlp_work(c):
    dims = [c["d0"], _cdiv(c["d1"], c["period1"]), _cdiv(c["d2"], c["period2"]), c["d3"]]
    b, nbytes, flops = c["batch"], 4 * dims[0] * c["batch"], 0.0
    for l in range(3):
        k, n = dims[l], dims[l + 1]
        flops += (6.0 if l else 4.0) * k * n * b
        nbytes += 4 * (5 * k * n + 5 * n) + 8 * n * b  # w and v read and written, dw; y and dy
    return {"bytes": nbytes, "flops": flops}


# ----------------------------------------------------------------- tile layer

class _Tile:
    pass


def _tile_prepare(c, seed):
    d, s = _Draws(seed), _Tile()
    n, k, b, t = c["outputs"], c["inputs"], c["batch"], c["tile"]
    sdt = _dtype(c)
    s.seed, s.x, s.w = int(seed), d.normal(k, b).to(sdt), d.normal(n, k, std=0.02).to(sdt)
    s.dy = d.normal(n, b).to(sdt)
    s.y, s.dx = torch.zeros(n, b, dtype=sdt, device=DEV), torch.zeros(k, b, dtype=sdt, device=DEV)
    s.dw = torch.zeros(n, k, device=DEV)
    s.bits = torch.zeros(_cdiv((n // t) * (k // t), 32), dtype=torch.int32, device=DEV)
    s.plan_ws = torch.zeros(max(api.ard_tile_plan_workspace_bytes(n // t, k // t), 16) // 4, dtype=torch.int32,
                            device=DEV)
    s.desc = api.tile_desc(_ard_dtype(c), b, k, n, 1.0, _dropped(c))
    s.stream = torch.cuda.current_stream().cuda_stream
    s.p = [v.data_ptr() for v in (s.x, s.w, s.y, s.dy, s.dx, s.dw)]
    return s


def _tile_run(c, s):
    x, w, y, dy, dx, dw = s.p
    plan = api.ard_plan_tiles_bernoulli(c["outputs"], c["inputs"], c["tile"], c["p"], s.seed, 0, 0, s.bits, s.plan_ws,
                                        s.stream)
    api.ard_tile_fwd(s.desc, plan, x, w, y, s.stream)
    api.ard_tile_bwd(s.desc, plan, x, dy, w, dx, dw, s.stream)
    return {"y": s.y, "dx": s.dx, "dw": s.dw, "bits": s.bits}


_MASK64 = (1 << 64) - 1


def _bernoulli(total, p, seed):
    """Keep bits of the tile sampler: draw e of the SplitMix64 stream from state seed, as a 53-bit uniform, is >= p."""
    keep, state = [], seed & _MASK64
    for _ in range(total):
        state = (state + 0x9E3779B97F4A7C15) & _MASK64
        z = state
        z = ((z ^ (z >> 30)) * 0xBF58476D1CE4E5B9) & _MASK64
        z = ((z ^ (z >> 27)) * 0x94D049BB133111EB) & _MASK64
        keep.append(((z ^ (z >> 31)) >> 11) * 2.0 ** -53 >= p)
    return keep


def _expand(keep, tn, tk, tile):
    m = torch.tensor(keep, dtype=torch.float64, device=DEV).view(tn, tk)
    return m.repeat_interleave(tile, 0).repeat_interleave(tile, 1)


def _tile_exact(c, seed):
    s = _tile_prepare(c, seed)
    tn, tk = c["outputs"] // c["tile"], c["inputs"] // c["tile"]
    m = _expand(_bernoulli(tn * tk, c["p"], s.seed), tn, tk, c["tile"])
    w = s.w.double() * m
    return {"y": w @ s.x.double(), "dx": w.t() @ s.dy.double(), "dw": (s.dy.double() @ s.x.double().t()) * m,
            "bits": None}


def _tile_work(c):
    e = 4 if c["dtype"] == "f32" else 2
    n, k, b = c["outputs"], c["inputs"], c["batch"]
    kept = n * k * (1 - c["p"])
    return {"bytes": e * (kept + 2 * (n + k) * b) + 4 * (n * k if c["zero"] else kept), "flops": 6.0 * kept * b}


# ----------------------------------------------------------------------- lstm

class _Lstm:
    pass


def _lstm_prepare(c, seed):
    d, s = _Draws(seed), _Lstm()
    t, b, h = c["seq"], c["batch"], c["hidden"]
    s.layers, s.train = [], c["train"]
    s.x = d.uniform(0.1, t, c["inputs"], b)
    s.pats = [(c["period"], d.offset(c["period"])) for _ in range(c["layers"])]
    s.stream = torch.cuda.current_stream().cuda_stream
    for l in range(c["layers"]):
        q = _Lstm()
        i = c["inputs"] if l == 0 else h
        q.i, q.w, q.b = i, d.uniform(0.1, 4 * h, i + h), d.uniform(0.1, 4 * h)
        q.h0, q.c0 = d.uniform(0.1, h, b), d.uniform(0.1, h, b)
        q.hs, q.ht, q.ct = (torch.zeros(*shape, device=DEV) for shape in ((t, h, b), (h, b), (h, b)))
        q.idx = torch.zeros(h, dtype=torch.int32, device=DEV)
        q.plan = api.ard_plan_rows(h, s.pats[l][0], s.pats[l][1], q.idx, s.stream)
        q.desc = api.lstm_desc(api.ARD_F32, t, b, i, h, q.plan, s.layers[-1].plan if l else None)
        q.ws = torch.zeros(max(api.ard_lstm_workspace_bytes(q.desc), 16) // 4 + 4, device=DEV)
        if s.train:
            q.dx, q.dw, q.db = (torch.zeros(*shape, device=DEV) for shape in ((t, i, b), (4 * h, i + h), (4 * h,)))
            q.dh0, q.dc0 = torch.zeros(h, b, device=DEV), torch.zeros(h, b, device=DEV)
        s.layers.append(q)
    s.dhs = d.normal(t, h, b, std=1.0 / (t * b)) if s.train else None
    return s


def _lstm_run(c, s):
    x, outs = s.x, []
    for q, pat in zip(s.layers, s.pats):
        api.ard_plan_rows(c["hidden"], pat[0], pat[1], q.idx, s.stream, plan=q.plan)
    for q in s.layers:
        q.x = x
        api.ard_lstm_fwd(q.desc, x, q.w, q.b, q.h0, q.c0, q.hs, q.ht, q.ct, q.ws, s.stream)
        x = q.hs
        outs.append({"hs": q.hs, "ht": q.ht, "ct": q.ct})
    if s.train:
        dh = s.dhs
        for l in reversed(range(len(s.layers))):
            q = s.layers[l]
            api.ard_lstm_bwd(q.desc, q.x, dh, None, None, q.ws, q.dx, q.dw, q.db, q.dh0, q.dc0, s.stream)
            dh = q.dx
            outs[l].update(dx=q.dx, dw=q.dw, db=q.db, dh0=q.dh0, dc0=q.dc0)
    return outs


def _lstm_exact_fwd(x, w, b, m, h, c):
    i_, hid, saved, hs = x.shape[1], m.shape[0], [], []
    h, c = h * m, c * m
    for t in range(x.shape[0]):
        z = w[:, :i_] @ x[t] + w[:, i_:] @ h + b[:, None]
        i, f, g, o = z[:hid].sigmoid(), z[hid:2 * hid].sigmoid(), z[2 * hid:3 * hid].tanh(), z[3 * hid:].sigmoid()
        saved.append((h, c, i, f, g, o))
        c = m * (f * c + i * g)
        h = m * (o * c.tanh())
        saved[-1] += (c,)
        hs.append(h)
    return torch.stack(hs), h, c, saved


def _lstm_exact_bwd(x, w, m, saved, dhs):
    i_ = x.shape[1]
    dh, dc = torch.zeros_like(dhs[0]), torch.zeros_like(dhs[0])
    dx, dw, db = torch.zeros_like(x), torch.zeros_like(w), torch.zeros_like(w[:, 0])
    for t in reversed(range(x.shape[0])):
        hp, cp, i, f, g, o, c = saved[t]
        dh = m * (dhs[t] + dh)
        tc = c.tanh()
        dc = m * (dc + dh * o * (1 - tc * tc))
        dz = torch.cat([dc * g * i * (1 - i), dc * cp * f * (1 - f), dc * i * (1 - g * g), dh * tc * o * (1 - o)])
        dx[t] = w[:, :i_].t() @ dz
        dw += dz @ torch.cat([x[t], hp]).t()
        db += dz.sum(1)
        dh, dc = m * (w[:, i_:].t() @ dz), dc * f
    return dx, dw, db, dh, dc


def _row_mask(n, pat):
    m = torch.zeros(n, 1, dtype=torch.float64, device=DEV)
    m[pat[1]::pat[0]] = 1
    return m


def _lstm_exact(c, seed):
    s = _lstm_prepare(c, seed)
    x, outs, kept = s.x.double(), [], []
    for q, pat in zip(s.layers, s.pats):
        m = _row_mask(c["hidden"], pat)
        hs, ht, ct, saved = _lstm_exact_fwd(x, q.w.double(), q.b.double(), m, q.h0.double(), q.c0.double())
        outs.append({"hs": hs, "ht": ht, "ct": ct})
        kept.append((x, m, saved))
        x = hs
    if s.train:
        dh = s.dhs.double()
        for l in reversed(range(len(s.layers))):
            x, m, saved = kept[l]
            dx, dw, db, dh0, dc0 = _lstm_exact_bwd(x, s.layers[l].w.double(), m, saved, dh)
            if l:
                dx = dx * kept[l - 1][1]  # inputs that the layer below dropped
            outs[l].update(dx=dx, dw=dw, db=db, dh0=dh0, dc0=dc0)
            dh = dx
    return outs


def _lstm_work(c):
    t, b, h, k = c["seq"], c["batch"], c["hidden"], _cdiv(c["hidden"], c["period"])
    nbytes, flops = 0.0, 0.0
    for l in range(c["layers"]):
        i, ik = (c["inputs"], c["inputs"]) if l == 0 else (h, k)
        mult = 3.0 if c["train"] else 1.0
        flops += mult * 2.0 * t * b * (ik + k) * 4 * k
        nbytes += 4 * (4 * k * (ik + k) + t * b * (ik + h) + 2 * b * (k + h))  # w, x, hs, the states
        if c["train"]:  # dhs, dx, dw
            nbytes += 4 * (t * b * (k + i) + 4 * h * (i + h) + 2 * b * h)
    return {"bytes": nbytes, "flops": flops}


# ------------------------------------------------------------------ lstm_tile

def _lstm_tile_prepare(c, seed):
    d, s = _Draws(seed), _Lstm()
    t, b, i, h, tile = c["seq"], c["batch"], c["inputs"], c["hidden"], c["tile"]
    s.tn, s.tk, s.off = 4 * h // tile, (i + h) // tile, d.offset(c["period"])
    s.x, s.w, s.b = d.uniform(0.1, t, i, b), d.uniform(0.1, 4 * h, i + h), d.uniform(0.1, 4 * h)
    s.h0, s.c0, s.dhs = d.uniform(0.1, h, b), d.uniform(0.1, h, b), d.normal(t, h, b, std=1.0 / (t * b))
    s.hs, s.ht, s.ct = (torch.zeros(*shape, device=DEV) for shape in ((t, h, b), (h, b), (h, b)))
    s.dx, s.dw, s.db = (torch.zeros(*shape, device=DEV) for shape in ((t, i, b), (4 * h, i + h), (4 * h,)))
    s.dh0, s.dc0 = torch.zeros(h, b, device=DEV), torch.zeros(h, b, device=DEV)
    bits = api.ard_tile_bitmap_tdp(s.tn, s.tk, c["period"], s.off)
    s.nnz = api.ard_bitmap_popcount(bits, s.tn * s.tk)
    s.bits = torch.from_numpy(bits.view("int32").copy()).to(DEV)
    s.plan_ws = torch.zeros(max(api.ard_tile_plan_workspace_bytes(s.tn, s.tk), 16) // 4, dtype=torch.int32, device=DEV)
    s.stream = torch.cuda.current_stream().cuda_stream
    s.plan = api.ard_plan_tiles(4 * h, i + h, tile, s.bits, s.nnz, s.plan_ws, s.stream)
    s.desc = api.lstm_tile_desc(api.ARD_F32, t, b, i, h, s.plan)
    s.ws = torch.zeros(max(api.ard_lstm_tile_workspace_bytes(s.desc), 16) // 4 + 4, device=DEV)
    return s


def _lstm_tile_run(c, s):
    t, b, i, h = c["seq"], c["batch"], c["inputs"], c["hidden"]
    # a sequence's pattern: its bitmap is resident, the lists are built on the device
    plan = api.ard_plan_tiles(4 * h, i + h, c["tile"], s.bits, s.nnz, s.plan_ws, s.stream)
    desc = api.lstm_tile_desc(api.ARD_F32, t, b, i, h, plan)
    api.ard_lstm_tile_fwd(desc, s.x, s.w, s.b, s.h0, s.c0, s.hs, s.ht, s.ct, s.ws, s.stream)
    api.ard_lstm_tile_bwd(desc, s.w, s.dhs, None, None, s.ws, s.dx, s.dw, s.db, s.dh0, s.dc0, s.stream)
    return {"hs": s.hs, "ht": s.ht, "ct": s.ct, "dx": s.dx, "dw": s.dw, "db": s.db, "dh0": s.dh0, "dc0": s.dc0}


def _lstm_tile_exact(c, seed):
    s = _lstm_tile_prepare(c, seed)
    m = _expand([e % c["period"] == s.off for e in range(s.tn * s.tk)], s.tn, s.tk, c["tile"])
    w, ones = s.w.double() * m, torch.ones(c["hidden"], 1, dtype=torch.float64, device=DEV)
    hs, ht, ct, saved = _lstm_exact_fwd(s.x.double(), w, s.b.double(), ones, s.h0.double(), s.c0.double())
    dx, dw, db, dh0, dc0 = _lstm_exact_bwd(s.x.double(), w, ones, saved, s.dhs.double())
    return {"hs": hs, "ht": ht, "ct": ct, "dx": dx, "dw": dw * m, "db": db, "dh0": dh0, "dc0": dc0}


def _lstm_tile_work(c):
    t, b, i, h = c["seq"], c["batch"], c["inputs"], c["hidden"]
    kept = 4 * h * (i + h) / c["period"]
    nbytes = 4 * (kept + 4 * h * (i + h) + 2 * t * b * (i + h) + 6 * b * h)  # w, dw, x, hs, dhs, dx, the states
    return {"bytes": nbytes, "flops": 6.0 * t * b * kept}


# ----------------------------------------------------------------------------

def prepare(case, seed):
    k = case["kind"]
    state = {"fc": _fc_prepare, "mlp": _mlp_prepare, "tile": _tile_prepare, "lstm": _lstm_prepare,
             "lstm_tile": _lstm_tile_prepare}[k](case, seed)
    return case, state


def run(state):
    case, s = state
    k = case["kind"]
    if k == "fc":
        return _fc_run(case, s)
    if k == "mlp":
        return _mlp_run(s)
    if k == "tile":
        return _tile_run(case, s)
    if k == "lstm":
        return _lstm_run(case, s)
    return _lstm_tile_run(case, s)


def work(case):
    return {"fc": _fc_work, "mlp": _mlp_work, "tile": _tile_work, "lstm": _lstm_work,
            "lstm_tile": _lstm_tile_work}[case["kind"]](case)


def tolerance(case):
    if case["kind"] == "mlp":
        # a ReLU gate of an activation next to zero that goes the other way changes one gradient entry of
        # about 1e5: 1 / sqrt(1e5) of the norm, and much of one weight gradient row's element
        return {"rel": 1e-2, "max": 0.99}
    if case.get("dtype") == "bf16":
        # outputs rounded to 8 bits: sums of another order round a few of them the other way
        return {"rel": 4e-3, "max": 1.6e-2}
    # 32-bit sums: each side is up to 9e-7 off the 64-bit value (the deepest products and the LSTMs)
    return {"rel": 4e-6, "max": 2e-4}


def exact(case, seed):
    return {"fc": _fc_exact, "mlp": _mlp_exact, "tile": _tile_exact, "lstm": _lstm_exact,
            "lstm_tile": _lstm_tile_exact}[case["kind"]](case, seed)
