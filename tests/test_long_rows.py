"""Calls whose rows are too long for 32-bit load offsets, at the true sizes: the
paths with 64-bit addresses. The batch is the long side; each sample stands
alone, so chosen samples (the last ones among them) are compared with the
oracle on those samples only."""
import numpy as np
import pytest
import torch

from gpu_util import device
from oracle import lstm as olstm
from paper_1805_08939_amd import api

pytestmark = pytest.mark.gpu


def some_columns(B):
    """The first, some middle and the last 300 columns of B."""
    c = sorted(set(range(5)) | set(range(B // 2, B // 2 + 70)) | set(range(B - 300, B)))
    return torch.tensor(c, device=device())


def random_on_gpu(seed, *shape):
    g = torch.Generator(device=device())
    g.manual_seed(seed)
    return torch.empty(*shape, device=device()).uniform_(-0.5, 0.5, generator=g)


def lstm_reference(X, W, b, h0, c0, dHs, cols, mask=None):
    """The oracle's forward and backward (without weight gradients) of the samples
    cols of X[T][I][B] and the others, in the library's layouts."""
    def take(t):
        return t[..., cols].transpose(-1, -2).double().cpu().numpy()
    w = W.double().cpu().numpy() * (1.0 if mask is None else mask)
    ones = np.ones(w.shape[0] // 4)
    Hs, hT, cT, cache = olstm.lstm_forward(take(X), w, b.double().cpu().numpy(), ones, take(h0), take(c0))
    dX, _, _, dh0, dc0 = olstm.lstm_backward(take(X), w, ones, cache, take(dHs), None, None)
    return {"Hs": Hs.transpose(0, 2, 1), "hT": hT.T, "cT": cT.T, "dX": dX.transpose(0, 2, 1), "dh0": dh0.T,
            "dc0": dc0.T}


def check(got, want, cols):
    for name, w in want.items():
        v = got[name][..., cols].double().cpu().numpy()
        # fp32 gates and sums of at most some tens of terms: a few roundings of 2^-24 of the largest value
        assert np.abs(v - w).max() <= 1e-5 * max(np.abs(w).max(), 1e-3), name


# Step products on contiguous copies of a step's columns, whose rows are Bp
# floats: row 31 of a tile passes 2^31 bytes from Bp = 2^24 on, and 2^32 bytes
# at the last columns of 2^25 + 8.
@pytest.mark.parametrize("T,B", [(1, (1 << 25) + 6)])
def test_lstm_tile_long_rows(T, B):
    I, H, tile = 24, 8, 32
    print(T, B, I, H, tile, flush=True)
    W, b = random_on_gpu(1, 4 * H, I + H), random_on_gpu(2, 4 * H)
    X, dHs = random_on_gpu(3, T, I, B), random_on_gpu(4, T, H, B)
    h0, c0 = random_on_gpu(5, H, B), random_on_gpu(6, H, B)
    bits = torch.ones(1, dtype=torch.int32, device=device())
    plan_ws = torch.empty(api.ard_tile_plan_workspace_bytes(1, 1) // 4, dtype=torch.int32, device=device())
    plan = api.ard_plan_tiles(4 * H, I + H, tile, bits, 1, plan_ws)
    desc = api.lstm_tile_desc(api.ARD_F32, T, B, I, H, plan)
    ws = torch.empty(api.ard_lstm_tile_workspace_bytes(desc) // 4 + 4, device=device())
    got = {"Hs": torch.empty(T, H, B, device=device()), "dX": torch.empty(T, I, B, device=device())}
    for n in ("hT", "cT", "dh0", "dc0"):
        got[n] = torch.empty(H, B, device=device())
    api.ard_lstm_tile_fwd(desc, X, W, b, h0, c0, got["Hs"], got["hT"], got["cT"], ws)
    api.ard_lstm_tile_bwd(desc, W, dHs, None, None, ws, got["dX"], None, None, got["dh0"], got["dc0"])
    torch.cuda.synchronize()
    cols = some_columns(B)
    check(got, lstm_reference(X, W, b, h0, c0, dHs, cols), cols)
