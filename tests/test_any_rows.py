"""FC products whose operand rows start at any element (batches and row lengths
that are no multiple of 16 bytes), against float64 torch: every tile
configuration of the register-load variant, its remainders and a split
contraction. The operands end at NaNs, so that a chunk read past a row's last
valid element into the arithmetic shows."""
import pytest
import torch

from gpu_util import ard_dtype, device, workspace
from native_plan import planner  # noqa: F401  (fixture)
from paper_1805_08939_amd import api, synth

# largest |error| over |A| |B| of one product: fp32 sums of K terms round each
# partial sum by 2^-24 of the terms so far (K / 8 sequential steps of the matrix
# cores at the most here: 2560 * 2^-24 = 1.6e-4, typically its square root);
# bf16 outputs round by 2^-9
TOL = {"f32": 1e-5, "bf16": 2.0 ** -8}


def nan_ended(t):
    """t on the GPU, directly followed by NaNs."""
    buf = torch.full((t.numel() + 64,), float("nan"), dtype=t.dtype, device=device())
    buf[:t.numel()] = t.reshape(-1).to(device())
    return buf[:t.numel()].view(t.shape)


def close(got, a, b, tol, rows=None):
    want, norm = a @ b, a.abs() @ b.abs()
    err = (got.double() - want).abs()
    assert torch.isfinite(got).all()
    assert (err <= tol * norm + 1e-30).all(), float((err / (norm + 1e-30)).max())


# (batch, inputs, outputs): K of one element to many slabs, and split contractions; with the second part every
# fp32 tile in each of the three products (the full layout; see test_shapes_reach_every_tile)
SHAPES = [(1501, 1700, 1703), (833, 834, 835), (31, 45, 20481), (17, 1501, 33), (1, 1, 1), (129, 33, 65),
          (7, 255, 130),
          (1507, 137, 2071), (582, 5194, 82), (107, 1994, 1547), (274, 70, 3660), (63, 798, 1120), (46, 585, 987),
          (71, 4327, 106), (1190, 781, 33), (33, 522, 1603), (38, 35, 5042), (19, 18, 510)]


def test_shapes_reach_every_tile(planner):
    reached = set()
    for B, K, N in SHAPES:
        if B % 4 and K % 4:  # both operands' rows off 16 bytes in every product
            for form, (m, n, k) in enumerate([(N, B, K), (K, B, N), (N, K, B)]):
                reached.add((form, planner.reg("f32", form, m, n, k)[0]))
    want = {(form, kind) for form in range(3) for kind in ("HUGE", "BIG", "DUO", "MID", "SMALL")} | {(0, "NARROW")}
    assert want <= reached, want - reached


@pytest.mark.gpu
@pytest.mark.parametrize("dtype", ["f32", "bf16"])
@pytest.mark.parametrize("shape", SHAPES)
@pytest.mark.parametrize("layout", ["full", "gathered", "compact_grad", "input_major"])
def test_unaligned_rows(dtype, shape, layout):
    B, K, N = shape
    if layout in ("gathered", "compact_grad") and K < 3:
        pytest.skip("no input to drop")
    print(dtype, shape, layout, flush=True)
    g = synth.generator(77)
    sdt = synth.storage_dtype(dtype)
    X, W = synth.normal(g, (K, B)).to(sdt), synth.normal(g, (N, K)).to(sdt)
    dY = synth.normal(g, (N, B)).to(sdt)
    pin = (3, 1) if layout in ("gathered", "compact_grad") else (1, 0)
    pout = (2, 0) if layout != "input_major" else (1, 0)
    plan_in = api.ard_plan_rows(K, pin[0], pin[1], None)
    plan_out = api.ard_plan_rows(N, pout[0], pout[1], None)
    code = {"full": api.ARD_WEIGHTS_FULL, "gathered": api.ARD_WEIGHTS_FULL,
            "compact_grad": api.ARD_WEIGHTS_COMPACT_GRAD, "input_major": api.ARD_WEIGHTS_INPUT_MAJOR}[layout]
    desc = api.fc_desc(ard_dtype(dtype), B, K, N, plan_in, plan_out, 1.0, api.ARD_ACT_NONE, api.ARD_DROPPED_SKIP, code)
    Xd, dYd = nan_ended(X), nan_ended(dY)
    Wd = nan_ended(W.t().contiguous() if layout == "input_major" else W)
    w = Wd
    ld = api.ard_fc_compact_ld(desc)
    if layout == "compact_grad":
        w = torch.zeros(plan_out.kept, ld, dtype=sdt, device=device())
        api.ard_fc_compact_weights(desc, Wd, w)
    Y = torch.full((N, B), 7.0, dtype=sdt, device=device())
    dX = torch.full((K, B), 7.0, dtype=sdt, device=device())
    dW = torch.full((plan_out.kept, ld) if layout == "compact_grad" else tuple(Wd.shape), 7.0, device=device())
    db = torch.full((N,), 7.0, device=device())
    ws = workspace(api.ard_fc_workspace_bytes(desc))
    api.ard_fc_fwd(desc, Xd, w, None, Y, ws)
    api.ard_fc_bwd(desc, Xd, dYd, None, w, dX, dW, db, ws)
    torch.cuda.synchronize()
    si = torch.arange(pin[1], K, pin[0], device=device())
    so = torch.arange(pout[1], N, pout[0], device=device())
    x, dy = Xd.double()[si], dYd.double()[so]
    wk = (Wd.t() if layout == "input_major" else Wd).double()[so][:, si]
    close(Y[so], wk, x, TOL[dtype])
    close(dX[si], wk.t(), dy, TOL[dtype])
    full = dW.t() if layout == "input_major" else dW
    got = full[:, :len(si)] if layout == "compact_grad" else full[so][:, si]
    close(got, dy, x.t(), TOL["f32"])  # weight gradients are fp32
    close(db[so, None], dy, torch.ones(B, 1, dtype=torch.float64, device=device()), TOL["f32"])
    # dropped rows and entries stay untouched
    if pout[0] > 1:
        assert (Y[1::2] == 7).all() and (db[1::2] == 7).all()
    if pin[0] > 1:
        assert (dX[0::3] == 7).all() and (dX[2::3] == 7).all()
        if layout == "gathered":
            assert (dW[:, 0::3] == 7).all() and (dW[1::2] == 7).all()
