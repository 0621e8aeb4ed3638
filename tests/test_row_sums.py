"""The bias gradient, which the weight-gradient kernels take from the rows of dY
that they read, on rows whose sum is lost by one 32-bit chain of additions: a
large first value, then ones, which round away one by one when added to it."""
import pytest
import torch

from gpu_util import ard_dtype, device, workspace
from paper_1805_08939_amd import api

pytestmark = pytest.mark.gpu


# (batch, inputs, outputs): rows on and off 16 bytes; large tiles without a split contraction, and the smallest tile.
# bf16 off 16 bytes only: on direct loads it keeps one 32-bit chain.
@pytest.mark.parametrize("dtype,shape", [("f32", (8192, 1000, 2048)), ("f32", (8191, 1001, 2049)),
                                         ("f32", (2048, 256, 256)), ("f32", (2047, 256, 255)),
                                         ("bf16", (8191, 1001, 2049)), ("bf16", (2047, 256, 255))])
def test_bias_gradient_of_long_rows(dtype, shape):
    B, K, N = shape
    print(dtype, shape, flush=True)
    sdt = torch.float32 if dtype == "f32" else torch.bfloat16
    dY = torch.ones(N, B, dtype=sdt, device=device())
    dY[:, 0] = 2.0 ** 26
    X = torch.zeros(K, B, dtype=sdt, device=device())
    dW, db = torch.empty(N, K, device=device()), torch.full((N,), 7.0, device=device())
    plans = [api.ard_plan_rows(n, 1, 0, None) for n in (K, N)]
    desc = api.fc_desc(ard_dtype(dtype), B, K, N, plans[0], plans[1], 1.0, api.ARD_ACT_NONE, api.ARD_DROPPED_SKIP,
                       api.ARD_WEIGHTS_FULL)
    api.ard_fc_bwd_weight(desc, X, dY, None, dW, db, workspace(api.ard_fc_workspace_bytes(desc)))
    torch.cuda.synchronize()
    # a step's four or eight values are added in 32 bits (at most 4 roundings of 2^-24 of 2^26), the steps in 64, and
    # at most 10 more 32-bit additions join the lanes and waves. Where a kernel of its own takes the sums (split
    # contractions), 64 lanes add B / 64 values each, and one of them loses its ones. A 32-bit
    # chain through the matrix kernel loses B / 8 (the smallest tile: B / 16) or more.
    assert ((db.double() - (2.0 ** 26 + B - 1)).abs() <= 14 * 4 + B // 64).all(), float(db[0]) - 2.0 ** 26 - B + 1


def test_infinities_stay_infinite():
    B, K, N = 1030, 70, 66
    dY = torch.ones(N, B, device=device())
    dY[0, 5], dY[1, 700], dY[2, 3], dY[3, 1] = float("inf"), float("-inf"), float("nan"), 3e38
    dY[3, 900] = 3e38
    plans = [api.ard_plan_rows(n, 1, 0, None) for n in (K, N)]
    desc = api.fc_desc(api.ARD_F32, B, K, N, plans[0], plans[1], 1.0, api.ARD_ACT_NONE, api.ARD_DROPPED_SKIP,
                       api.ARD_WEIGHTS_FULL)
    dW, db = torch.empty(N, K, device=device()), torch.empty(N, device=device())
    api.ard_fc_bwd_weight(desc, torch.zeros(K, B, device=device()), dY, None, dW, db,
                          workspace(api.ard_fc_workspace_bytes(desc)))
    torch.cuda.synchronize()
    assert db[0] == float("inf") and db[1] == float("-inf") and torch.isnan(db[2]) and db[3] == float("inf")
    assert (db[4:] == B).all()
