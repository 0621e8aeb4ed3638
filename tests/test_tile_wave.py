"""The tile layer on the wave kernels (32 x 32 tiles, batch rows of any length,
grids that do not fill the chip) against float64 torch: every batch block
width, remainders of the batch, empty and full tile rows, lists longer than one
64-entry window, and the one-call backward bit for bit the two calls."""
import numpy as np
import pytest
import torch

from gpu_util import ard_dtype, device
from paper_1805_08939_amd import api, synth

pytestmark = pytest.mark.gpu

# largest |error| over |A| |B|: fp32 partial sums, bf16 outputs rounded by 2^-9
TOL = {"f32": 1e-5, "bf16": 2.0 ** -8}


def close(got, a, b, tol):
    want, norm = a @ b, a.abs() @ b.abs()
    assert torch.isfinite(got).all()
    err = (got.double() - want).abs()
    assert (err <= tol * norm + 1e-30).all(), float((err / (norm + 1e-30)).max())


# (tile, tiles_n, tiles_k, batch): one tile; batch blocks of 32, 64 and 128 columns with remainders; lists of
# more than 64 entries; rows that start at any element; the pipeline's rows and groups beside the wave kernels
CASES = [(32, 1, 1, 1), (32, 3, 5, 31), (32, 9, 130, 33), (32, 70, 6, 200), (32, 140, 5, 129), (64, 2, 3, 7),
         (64, 5, 70, 64), (64, 33, 9, 100), (64, 66, 3, 257), (64, 40, 40, 96), (64, 3, 100, 128), (64, 24, 24, 516)]


@pytest.mark.parametrize("dtype", ["f32", "bf16"])
@pytest.mark.parametrize("case", CASES)
@pytest.mark.parametrize("known", [True, False])
def test_wave_kernels(dtype, case, known):
    tile, tn, tk, B = case
    print(dtype, case, known, flush=True)
    N, K = tn * tile, tk * tile
    sdt = synth.storage_dtype(dtype)
    g = synth.generator(5)
    X, W, dY = synth.normal(g, (K, B)).to(sdt), synth.normal(g, (N, K)).to(sdt), synth.normal(g, (N, B)).to(sdt)
    X, W, dY = X.to(device()), W.to(device()), dY.to(device())
    ws = torch.empty(max(api.ard_tile_plan_workspace_bytes(tn, tk), 16) // 4, dtype=torch.int32, device=device())
    p = 0.4
    bits = api.ard_tile_bitmap_bernoulli(tn, tk, p, 11, 0, 3)
    keep = np.array([(int(bits[t // 32]) >> (t % 32)) & 1 for t in range(tn * tk)]).reshape(tn, tk)
    if known:  # a full and an empty tile row (and column)
        if tn > 2 and tk > 2:
            keep[0], keep[1], keep[:, 1] = 1, 0, 0
        flat = keep.reshape(-1)
        words = np.zeros((tn * tk + 31) // 32, dtype=np.uint32)
        for t in np.nonzero(flat)[0]:
            words[t // 32] |= np.uint32(1 << (t % 32))
        dbits = torch.from_numpy(words.view("int32").copy()).to(device())
        plan = api.ard_plan_tiles(N, K, tile, dbits, int(flat.sum()), ws)
    else:
        dbits = torch.zeros((tn * tk + 31) // 32, dtype=torch.int32, device=device())
        plan = api.ard_plan_tiles_bernoulli(N, K, tile, p, 11, 0, 3, dbits, ws)
    M = torch.from_numpy(np.kron(keep, np.ones((tile, tile)))).to(device())
    W = torch.where(M > 0, W, torch.full_like(W, float("nan")))  # dropped tiles are never read
    desc = api.tile_desc(ard_dtype(dtype), B, K, N, 0.5, api.ARD_DROPPED_SKIP)
    Y, dX = torch.full((N, B), 7.0, dtype=sdt, device=device()), torch.full((K, B), 7.0, dtype=sdt, device=device())
    dW = torch.full((N, K), 7.0, device=device())
    dX2, dW2 = dX.clone(), dW.clone()
    api.ard_tile_fwd(desc, plan, X, W, Y)
    api.ard_tile_bwd_data(desc, plan, dY, W, dX)
    api.ard_tile_bwd_weight(desc, plan, X, dY, dW)
    api.ard_tile_bwd(desc, plan, X, dY, W, dX2, dW2)
    torch.cuda.synchronize()
    Wm = torch.where(M > 0, W.double(), torch.zeros_like(M))
    close(Y, 0.5 * Wm, X.double(), TOL[dtype])
    close(dX, 0.5 * Wm.t(), dY.double(), TOL[dtype])
    kept = M > 0
    want = 0.5 * (dY.double() @ X.double().t())
    norm = 0.5 * (dY.double().abs() @ X.double().abs().t())
    assert ((dW.double() - want).abs()[kept] <= TOL["f32"] * norm[kept] + 1e-30).all()
    assert (dW[~kept] == 7.0).all()
    assert torch.equal(dX, dX2) and torch.equal(dW, dW2)


@pytest.mark.parametrize("T,B,I,H,tile", [(3, 5, 64, 32, 32), (2, 1, 40, 24, 32), (4, 66, 128, 192, 64),
                                          (2, 64, 96, 160, 64), (1, 7, 32, 32, 32), (3, 16, 1024, 128, 32)])
@pytest.mark.parametrize("outs", ["all", "some"])
def test_lstm_tile_padded_batch(T, B, I, H, tile, outs):
    """The tile-pattern LSTM with a batch that is padded inside, with the input
    tiles' products hoisted out of the steps (I a multiple of the tile) and not."""
    from oracle import lstm as olstm
    print(T, B, I, H, tile, outs, flush=True)
    tn, tk = 4 * H // tile, (I + H) // tile
    g = synth.generator(9)
    X, W = synth.uniform(g, (T, B, I), 0.5), synth.uniform(g, (4 * H, I + H), 0.2)
    b, dHs = synth.uniform(g, (4 * H,), 0.1), synth.normal(g, (T, B, H))
    h0, c0, dhT, dcT = (synth.normal(g, (B, H), 0.3) for _ in range(4))
    bits = api.ard_tile_bitmap_bernoulli(tn, tk, 0.5, 3, 0, 1)
    keep = np.array([(int(bits[t // 32]) >> (t % 32)) & 1 for t in range(tn * tk)]).reshape(tn, tk)
    M = np.kron(keep, np.ones((tile, tile)))
    ws = torch.empty(max(api.ard_tile_plan_workspace_bytes(tn, tk), 16) // 4, dtype=torch.int32, device=device())
    plan = api.ard_plan_tiles(4 * H, I + H, tile, torch.from_numpy(bits.view("int32").copy()).to(device()),
                              int(keep.sum()), ws)
    desc = api.lstm_tile_desc(api.ARD_F32, T, B, I, H, plan)

    def dev(t):
        return t.permute(*range(t.dim() - 2), -1, -2).contiguous().to(device())

    Wd = torch.where(torch.from_numpy(M).bool(), W, torch.full_like(W, float("nan"))).to(device())
    lw = torch.full((api.ard_lstm_tile_workspace_bytes(desc) // 4 + 4,), float("nan"), device=device())
    Hs = torch.full((T, H, B), 7.0, device=device())
    hT, cT = torch.empty(H, B, device=device()), torch.empty(H, B, device=device())
    full = outs == "all"
    api.ard_lstm_tile_fwd(desc, dev(X), Wd, b.to(device()), dev(h0) if full else None, dev(c0) if full else None, Hs,
                          hT if full else None, cT if full else None, lw)
    dX, dW = torch.full((T, I, B), 7.0, device=device()), torch.full((4 * H, I + H), 7.0, device=device())
    db, dh0, dc0 = torch.empty(4 * H, device=device()), hT.clone(), cT.clone()
    for _ in range(2):  # the forward's workspace serves a second backward too
        api.ard_lstm_tile_bwd(desc, Wd, dev(dHs), dev(dhT) if full else None, dev(dcT) if full else None, lw,
                              dX, dW, db, dh0 if full else None, dc0 if full else None)
    torch.cuda.synchronize()
    ones, Wm = np.ones(H), W.double().numpy() * M
    n = (lambda t: t.double().numpy()) if full else (lambda t: None)
    Hs64, hT64, cT64, cache = olstm.lstm_forward(X.double().numpy(), Wm, b.double().numpy(), ones, n(h0), n(c0))
    dX64, dW64, db64, dh64, dc64 = olstm.lstm_backward(X.double().numpy(), Wm, ones, cache, dHs.double().numpy(),
                                                       n(dhT), n(dcT))
    want = [(Hs, Hs64.transpose(0, 2, 1)), (dX, dX64.transpose(0, 2, 1)), (dW, dW64 * M), (db, db64)]
    if full:
        want += [(hT, hT64.T), (cT, cT64.T), (dh0, dh64.T), (dc0, dc64.T)]
    for got, w in want:
        got = got.double().cpu().numpy()
        assert np.isfinite(got).all()
        # fp32 gates and sums over a few steps: some tens of roundings of 2^-24 of the largest value
        assert np.abs(got - w).max() <= 1e-5 * max(np.abs(w).max(), 1e-3)


def test_lstm_tile_input_gradient_precision():
    """dX of the tile-pattern LSTM, one product over all steps, as close to 64
    bits as a sum in sixteen chains: every tile kept, 4096 terms an output."""
    T, B, I, H, tile = 6, 24, 512, 1024, 64
    g = torch.Generator(device=device())
    g.manual_seed(21)

    def u(a, *shape):
        return (torch.rand(*shape, generator=g, device=device()) * 2 - 1) * a
    X, W, b, dHs = u(0.1, T, I, B), u(0.1, 4 * H, I + H), u(0.1, 4 * H), u(1.0, T, H, B)
    tn, tk = 4 * H // tile, (I + H) // tile
    bits = torch.full(((tn * tk + 31) // 32,), -1, dtype=torch.int32, device=device())
    pw = torch.empty(api.ard_tile_plan_workspace_bytes(tn, tk) // 4, dtype=torch.int32, device=device())
    plan = api.ard_plan_tiles(4 * H, I + H, tile, bits, tn * tk, pw)
    desc = api.lstm_tile_desc(api.ARD_F32, T, B, I, H, plan)
    ws = torch.empty(api.ard_lstm_tile_workspace_bytes(desc) // 4 + 4, device=device())
    Hs, dX = torch.empty(T, H, B, device=device()), torch.empty(T, I, B, device=device())
    api.ard_lstm_tile_fwd(desc, X, W, b, None, None, Hs, None, None, ws)
    api.ard_lstm_tile_bwd(desc, W, dHs, None, None, ws, dX, None, None, None, None)
    torch.cuda.synchronize()
    # 64-bit reference on the GPU
    w, x, h, c, saved = W.double(), X.double(), torch.zeros(H, B, dtype=torch.float64, device=device()), None, []
    c = torch.zeros_like(h)
    for t in range(T):
        z = w[:, :I] @ x[t] + w[:, I:] @ h + b.double()[:, None]
        i, f, gg, o = z[:H].sigmoid(), z[H:2 * H].sigmoid(), z[2 * H:3 * H].tanh(), z[3 * H:].sigmoid()
        saved.append((i, f, gg, o, c))
        c = f * c + i * gg
        h = o * c.tanh()
        saved[-1] += (c,)
    want, dh, dc = torch.zeros_like(x), torch.zeros_like(h), torch.zeros_like(h)
    for t in reversed(range(T)):
        i, f, gg, o, cp, ct = saved[t]
        dh = dh + dHs[t].double()
        tc = ct.tanh()
        dc = dc + dh * o * (1 - tc * tc)
        dz = torch.cat([dc * gg * i * (1 - i), dc * cp * f * (1 - f), dc * i * (1 - gg * gg), dh * tc * o * (1 - o)])
        want[t], dh, dc = w[:, :I].t() @ dz, w[:, I:].t() @ dz, dc * f
    err = ((dX.double() - want).norm() / want.norm()).item()
    # a chain of L additions of equal terms: rms error 2^-24 sqrt(L / 6) of the sum. Sixteen chains have L = 4096 / 16 /
    # 2 MFMAs = 128, joined by sixteen more additions; dZ's own rounding adds as much again at the most (measured:
    # 3.0e-7 in sixteen chains, 5.2e-7 in four)
    assert err <= 2.0 ** -24 * (2 * (128 + 16) / 6) ** 0.5, err
