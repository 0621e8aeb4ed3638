"""Layers whose backward runs as one launch although one of its products alone
would take larger tiles: the plan, and ard_fc_bwd bit for bit the two calls."""
import pytest
import torch

from gpu_util import device, workspace
from native_plan import planner  # noqa: F401  (fixture)
from paper_1805_08939_amd import api, synth
from test_any_rows import close

# (batch, inputs, outputs), all kept
LAYERS = [(184, 364, 832), (704, 512, 688), (20, 624, 452), (392, 620, 960), (140, 748, 508)]


@pytest.mark.parametrize("layer", LAYERS)
def test_one_launch_is_planned(planner, layer):
    B, K, N = layer
    alone = [planner.f32(M, n, k)[0] for M, n, k in ((K, B, N), (N, K, B))]
    assert planner.pair(B, K, N) and alone != [("SMALL", 1)] * 2, alone


@pytest.mark.gpu
@pytest.mark.parametrize("off", [0, 1])
@pytest.mark.parametrize("layer", LAYERS)
def test_one_call_is_the_two_calls(layer, off):
    """off: rows off 16 bytes, on register loads."""
    B, K, N = (v + off for v in layer)
    print(B, K, N, flush=True)
    g = synth.generator(3)
    X, W, dY = synth.normal(g, (K, B)).to(device()), synth.normal(g, (N, K)).to(device()), synth.normal(g, (N, B)).to(device())
    plans = [api.ard_plan_rows(n, 1, 0, None) for n in (K, N)]
    desc = api.fc_desc(api.ARD_F32, B, K, N, plans[0], plans[1], 1.0, api.ARD_ACT_NONE, api.ARD_DROPPED_SKIP,
                       api.ARD_WEIGHTS_FULL)
    ws = workspace(api.ard_fc_workspace_bytes(desc))
    dX, dW, db = torch.empty(K, B, device=device()), torch.empty(N, K, device=device()), torch.empty(N, device=device())
    dX2, dW2, db2 = torch.empty_like(dX), torch.empty_like(dW), torch.empty_like(db)
    api.ard_fc_bwd(desc, X, dY, None, W, dX, dW, db, ws)
    api.ard_fc_bwd_data(desc, dY, None, W, dX2, ws)
    api.ard_fc_bwd_weight(desc, X, dY, None, dW2, db2, ws)
    torch.cuda.synchronize()
    assert torch.equal(dX, dX2) and torch.equal(dW, dW2) and torch.equal(db, db2)
    close(dX, W.double().t(), dY.double(), 1e-5)  # fp32 sums in eight chains: far below 2^-24 K / 16
    close(dW, dY.double(), X.double().t(), 1e-5)
    close(db[:, None], dY.double(), torch.ones(B, 1, dtype=torch.float64, device=device()), 1e-5)
