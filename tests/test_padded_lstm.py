"""The LSTM's products over all steps at once at batches that are padded inside
(no multiple of 4), and the fp32 tile configurations and splits of the FC
products, with the reported workspace and the smallest accepted one."""
import pytest
import torch

from gpu_util import device
from native_plan import planner  # noqa: F401  (fixture)
from paper_1805_08939_amd import api, synth
from test_lstm_parity import run_lstm

# (T, B, I, H), hidden pattern, input pattern: padded batches of one sample to
# more than one tile; tiles of T * Bp columns that end inside a step; flat
# contractions over T * Bp with remainders of a slab, in the gathered and the
# identity layout; rows of X that are no multiple of 16 bytes. With the shapes
# below them every tile in each product (test_lstm_shapes_reach_every_tile).
LSTM = [((1, 1, 3, 5), (1, 0), (1, 0)), ((7, 1, 40, 64), (2, 1), (1, 0)), ((35, 5, 96, 130), (2, 0), (3, 1)),
        ((9, 10, 300, 512), (2, 1), (1, 0)), ((5, 20, 256, 1024), (2, 1), (2, 0)), ((3, 66, 130, 96), (3, 2), (1, 0)),
        ((2, 129, 512, 256), (1, 0), (4, 1)), ((20, 64, 768, 640), (2, 0), (1, 0))]
LSTM += [(shape, (1, 0), (1, 0)) for shape in
         [(8, 121, 658, 25), (20, 72, 2278, 5), (11, 10, 1718, 5), (7, 13, 2476, 19), (14, 132, 74, 35),
          (18, 65, 114, 122), (18, 103, 6, 402), (17, 121, 13, 28), (17, 1, 5, 272), (13, 6, 6, 398), (1, 1, 4, 861),
          (1, 1, 5, 264), (20, 1, 2238, 6), (9, 10, 2497, 13), (1, 1, 1801, 420), (3, 1, 2360, 5), (1, 5, 33, 5125),
          (1, 30, 20490, 16)]]


def test_lstm_shapes_reach_every_tile(planner):
    reached = set()
    for (T, B, I, H), pattern, in_pattern in LSTM:
        n, cols = len(range(pattern[1], H, pattern[0])), T * ((B + 3) // 4 * 4)
        k = len(range(in_pattern[1], I, in_pattern[0]))
        # input projection, dX, and the two parts of dW (four gates in one launch), none split
        for name, m, w, depth, batch in (("zx", 4 * n, cols, k, 1), ("dx", k, cols, 4 * n, 1), ("dw", n, k, cols, 4),
                                         ("dwh", n, n, cols, 4)):
            reached.add((name, planner.f32(m, w, depth, 1, batch, 0)[0][0]))
    want = {(p, t) for p in ("zx", "dx", "dw", "dwh") for t in ("HUGE", "BIG", "DUO", "MID", "SMALL")}
    want |= {("zx", "NARROW"), ("dx", "NARROW")}
    assert want <= reached, want - reached


@pytest.mark.gpu
@pytest.mark.parametrize("shape,pattern,in_pattern", LSTM)
@pytest.mark.parametrize("states", [True, False])
def test_products_over_all_steps(shape, pattern, in_pattern, states):
    print(shape, pattern, in_pattern, states, flush=True)
    run_lstm(*shape, pattern, seed=sum(shape), with_state=states, with_final_grads=states, in_pattern=in_pattern)


# (batch, inputs, outputs): every tile, with and without a split contraction, remainders of each
FC = [(2048, 1536, 2240), (1028, 2052, 1028), (260, 4100, 516), (20, 9000, 1500), (700, 3004, 1500), (64, 8200, 68)]


def test_fc_shapes_reach_every_tile(planner):
    plans = [planner.f32(*p)[0] for B, K, N in FC for p in ((N, B, K), (K, B, N), (N, K, B))]
    assert {k for k, _ in plans} >= {"HUGE", "BIG", "DUO", "MID", "SMALL"}
    assert {k for k, s in plans if s > 1} >= {"DUO", "MID", "SMALL"}


@pytest.mark.gpu
@pytest.mark.parametrize("shape", FC)
def test_f32_tiles_and_workspaces(shape):
    B, K, N = shape
    g = synth.generator(41)
    X, W = synth.normal(g, (K, B)).to(device()), synth.normal(g, (N, K)).to(device())
    dY, b = synth.normal(g, (N, B)).to(device()), synth.normal(g, (N,)).to(device())
    plan = [api.ard_plan_rows(n, 1, 0, None) for n in (K, N)]
    desc = api.fc_desc(api.ARD_F32, B, K, N, plan[0], plan[1], 1.0, api.ARD_ACT_NONE, api.ARD_DROPPED_SKIP,
                       api.ARD_WEIGHTS_FULL)
    full = api.ard_fc_workspace_bytes(desc)
    sizes = [full] + [s for s in (full * 3 // 4, full // 2, full // 4, full // 8, 0) if s < full]
    x, w, dy = X.double(), W.double(), dY.double()
    want = [(w @ x + b.double()[:, None], w.abs() @ x.abs()), (w.t() @ dy, w.abs().t() @ dy.abs()),
            (dy @ x.t(), dy.abs() @ x.abs().t()), (dy.sum(1), dy.abs().sum(1))]
    ran = 0
    for size in sizes:
        print(shape, size, flush=True)
        ws = torch.full((size // 16 * 4 + 64,), float("nan"), device=device())  # 256 bytes more than are named
        use = ws[:size // 16 * 4] if size >= 16 else None
        Y, dX = torch.full((N, B), 7.0, device=device()), torch.full((K, B), 7.0, device=device())
        dW, db = torch.full((N, K), 7.0, device=device()), torch.full((N,), 7.0, device=device())
        try:
            api.ard_fc_fwd(desc, X, W, b, Y, use)
            api.ard_fc_bwd(desc, X, dY, None, W, dX, dW, db, use)
        except api.ArdError:
            assert size < full  # a smaller one may be refused, but never overrun
            continue
        finally:
            torch.cuda.synchronize()
            assert torch.isnan(ws[size // 16 * 4:]).all()
        ran += 1
        for got, (v, norm) in zip((Y, dX, dW, db), want):
            # fp32 sums of up to 9000 terms in at least 8 chains: (9000 / 8) 2^-24 = 7e-5 at the most, typically its
            # square root's worth (2e-6); the bias is one term more
            assert ((got.double() - v).abs() <= 1e-5 * norm + 1e-6).all()
    assert ran > 0


@pytest.mark.gpu
def test_initial_state_gradient_precision():
    """dh0 through the one-kernel backward step, 1640 gate rows deep."""
    import numpy as np
    from oracle import lstm as olstm
    T, B, I, H = 14, 9, 200, 410
    g = torch.Generator(device=device())
    g.manual_seed(8)

    def u(a, *shape):
        return (torch.rand(*shape, generator=g, device=device()) * 2 - 1) * a
    X, W, b, h0, c0 = u(0.1, T, I, B), u(0.1, 4 * H, I + H), u(0.1, 4 * H), u(0.1, H, B), u(0.1, H, B)
    dHs = u(1.0, T, H, B)
    desc = api.lstm_desc(api.ARD_F32, T, B, I, H, None, None)
    ws = torch.empty(api.ard_lstm_workspace_bytes(desc) // 4 + 4, device=device())
    Hs, hT, cT = torch.empty(T, H, B, device=device()), torch.empty(H, B, device=device()), torch.empty(H, B, device=device())
    dX, dW, db = torch.empty(T, I, B, device=device()), torch.empty(4 * H, I + H, device=device()), torch.empty(4 * H, device=device())
    dh0, dc0 = torch.empty(H, B, device=device()), torch.empty(H, B, device=device())
    api.ard_lstm_fwd(desc, X, W, b, h0, c0, Hs, hT, cT, ws)
    api.ard_lstm_bwd(desc, X, dHs, None, None, ws, dX, dW, db, dh0, dc0)
    torch.cuda.synchronize()

    def n(t):
        return t.transpose(-1, -2).double().cpu().numpy()
    w, ones = W.double().cpu().numpy(), np.ones(H)
    _, _, _, cache = olstm.lstm_forward(n(X), w, b.double().cpu().numpy(), ones, n(h0), n(c0))
    want = olstm.lstm_backward(n(X), w, ones, cache, n(dHs), None, None)[3]
    err = np.linalg.norm(n(dh0) - want) / np.linalg.norm(want)
    # each step adds its product's error: chains of L additions in C accumulators leave 2^-24 sqrt((L + C) / 6) of a sum;
    # L = 13 slabs and C = 4 waves x 8: 1.6e-7 and as much from the gates; L = 52 and C = 8: 1.9e-7 and that. Measured
    # 1.8e-7, and 2.9e-7 with two accumulators per wave
    assert err <= 2.3e-7, err
