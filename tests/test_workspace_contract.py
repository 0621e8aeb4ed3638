"""What a caller may rely on about the FC workspace: the forward's sums follow
from the descriptor alone, a workspace queried for another pattern of the layer
is accepted where it covers the least, and nothing is written past it."""
import pytest
import torch

from gpu_util import device, row_plan, workspace
from paper_1805_08939_amd import api, synth

pytestmark = pytest.mark.gpu


def operands(B, K, N, seed=5):
    g = synth.generator(seed)
    return (synth.normal(g, (K, B)).to(device()), synth.normal(g, (N, K), 0.05).to(device()),
            synth.normal(g, (N,), 0.1).to(device()))


def full_desc(B, K, N, pin, pout, layout=api.ARD_WEIGHTS_FULL):
    return api.fc_desc(api.ARD_F32, B, K, N, row_plan(K, *pin, with_list=False), row_plan(N, *pout, with_list=False),
                       1.0, api.ARD_ACT_RELU, api.ARD_DROPPED_ZERO, layout)


def test_forward_beside_a_large_compact_copy():
    """The compact weight copy of this layer almost fills the 32 MiB that
    ard_fc_fwd_noalloc admits: the forward splits its contraction all the same,
    so a caller's own compact copy, and the call without a workspace, give the
    same bits."""
    B, K, N = 40, 8180, 2000
    X, W, b = operands(B, K, N)
    desc = full_desc(B, K, N, (2, 1), (1, 0))
    need = api.ard_fc_workspace_bytes(desc)
    assert need > api.ard_fc_compact_bytes(desc) + 4 * 4 * N * B  # room for more than the two splits of the least plan
    Y, Yn, Yc = (torch.full((N, B), v, device=device()) for v in (1.0, 2.0, 3.0))
    api.ard_fc_fwd(desc, X, W, b, Y, workspace(need))
    api.ard_fc_fwd_noalloc(desc, X, W, b, Yn)
    given = full_desc(B, K, N, (2, 1), (1, 0), api.ARD_WEIGHTS_COMPACT)
    wc = torch.empty(api.ard_fc_compact_bytes(given) // 4, device=device())
    api.ard_fc_compact_weights(given, W, wc)
    api.ard_fc_fwd(given, X, wc, b, Yc, workspace(api.ard_fc_workspace_bytes(given)))
    torch.cuda.synchronize()
    assert torch.equal(Y, Yn) and torch.equal(Y, Yc)
    want = (W.double()[:, 1::2] @ X.double()[1::2] + b.double()[:, None]).clamp(min=0)
    norm = W.double().abs()[:, 1::2] @ X.double().abs()[1::2] + b.double().abs()[:, None]
    assert ((Y.double() - want).abs() <= 1e-5 * norm).all()


def test_more_workspace_changes_nothing():
    B, K, N = 40, 4096, 1024
    X, W, b = operands(B, K, N)
    desc = full_desc(B, K, N, (1, 0), (1, 0))
    need = api.ard_fc_workspace_bytes(desc)
    outs = []
    for size in (need, need + (64 << 20)):
        Y = torch.empty(N, B, device=device())
        api.ard_fc_fwd(desc, X, W, b, Y, workspace(size))
        outs.append(Y)
    torch.cuda.synchronize()
    assert torch.equal(*outs)


# (batch, inputs, outputs), the pattern: the size queried for the layer with everything kept is smaller than the
# pattern's own; the call is refused, or right within it
@pytest.mark.parametrize("shape,pin,pout", [((1105, 2166, 828), (1, 0), (3, 0)), ((64, 3000, 700), (1, 0), (3, 1)),
                                            ((700, 4096, 512), (1, 0), (5, 2)), ((36, 1924, 612), (1, 0), (2, 0))])
def test_workspace_of_the_dense_pattern(shape, pin, pout):
    B, K, N = shape
    print(shape, pin, pout, flush=True)
    X, W, b = operands(B, K, N)
    dense = api.ard_fc_workspace_bytes(full_desc(B, K, N, (1, 0), (1, 0)))
    desc = full_desc(B, K, N, pin, pout)
    own = api.ard_fc_workspace_bytes(desc)
    buf = torch.full((dense // 4 + 4096,), float("nan"), device=device())
    use = buf[:dense // 4] if dense else None
    Y, ref = torch.full((N, B), 7.0, device=device()), torch.full((N, B), 8.0, device=device())
    api.ard_fc_fwd(desc, X, W, b, ref, workspace(own))
    try:
        api.ard_fc_fwd(desc, X, W, b, Y, use)
    except api.ArdError as e:
        assert e.status == 5 and dense < own
    else:
        torch.cuda.synchronize()
        norm = (W.double().abs() @ X.double().abs() + b.double().abs()[:, None])
        assert ((Y.double() - ref.double()).abs() <= 2e-5 * norm).all()  # the order of rounding may differ
        assert dense < own or torch.equal(Y, ref)
    torch.cuda.synchronize()
    assert torch.isnan(buf[dense // 4:]).all()
