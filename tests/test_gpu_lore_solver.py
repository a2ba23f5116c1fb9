"""The LoRE fit's GPU eigensolver and solve (more than 48 tokens) where they can go wrong: just past
the host path's limit, sizes that are no multiple of a panel, a wave or a rotation block, the
largest, ranks beyond the token count, targets of low rank (a zero tail), the host path on a
workspace without the solver's buffers, and dependent tokens.  Against the oracle's regression on
the GPU's own targets, with the tolerances of the fit's other tests."""
import numpy as np
import pytest
import torch

from paper_2608_21240_amd import layer as LY, spice, synth, workloads as W
from paper_2608_21240_amd.workloads import MoEShape, Workload

from parity import say

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def orc():
    import oracle
    return oracle


def fit(shape, n, r, x=None, zero_expert_rows=0, spare=0):
    wl = Workload("fit", shape, tokens=n, resident=0, skew=False, seed=n)
    d, dt = shape.d, shape.dtype
    w13, w2 = synth.gen_expert(wl, 0, 1)
    if zero_expert_rows:  # the outputs keep d - zero_expert_rows features: targets of that rank
        w2 = w2.copy()
        w2[d - zero_expert_rows:] = 0
    x = synth.gen_x(wl, 0, 0, n) if x is None else x
    shared = [LY.to_tensor(a, dt, "cuda") for a in synth.gen_shared(wl, 0)] if shape.shared_inter else [None, None]
    cfg = spice.make_cfg(shape, 1)
    A = torch.full((r, d), 7.0, device="cuda")
    B = torch.full((d, r), 7.0, device="cuda")
    Y = torch.empty((n, d), device="cuda")
    size = spice.lib().spice_lore_fit_workspace_bytes(spice.ctypes.byref(cfg), n, r) - spare
    ws = torch.empty(size, dtype=torch.uint8, device="cuda")
    loss = spice.moe_lore_fit(cfg, n, r, LY.to_tensor(x, dt, "cuda"), LY.to_tensor(w13, dt, "cuda"),
                              LY.to_tensor(w2, dt, "cuda"), *shared, A, B, Y, ws, size)
    return synth.as_f32(x, dt).astype(np.float64), *(t.cpu().numpy().astype(np.float64) for t in (A, B, Y)), loss


def check(orc, X, A, B, Y, loss, r):
    A_o, B_o, loss_o = orc.lore_fit(X, Y, min(r, X.shape[1]))
    total = float((Y ** 2).sum())
    ew = np.linalg.norm(B @ A - B_o @ A_o) / np.linalg.norm(B_o @ A_o)
    say(f"loss {loss:.6e} oracle {loss_o:.6e} of {total:.3e}, B A rel err {ew:.2e}")
    assert abs(loss - loss_o) <= 1e-6 * loss_o + 1e-9 * total
    assert ew <= 1e-4
    assert orc.lore_loss(X, Y, A, B) == pytest.approx(loss, rel=1e-4, abs=1e-7 * total)


BF = W.DTYPE_BF16


@pytest.mark.parametrize("shape,n,r", [
    (MoEShape(200, 4, 2, 96, 160, 8, BF), 48, 8), (MoEShape(200, 4, 2, 96, 160, 8, BF), 49, 8),
    (MoEShape(200, 4, 2, 96, 0, 8, W.DTYPE_F32), 97, 1), (MoEShape(256, 4, 2, 64, 96, 8, BF), 65, 80),
    (MoEShape(384, 4, 2, 64, 96, 8, BF), 300, 299), (MoEShape(1024, 4, 2, 64, 96, 8, BF), 1024, 24)])
def test_fit_sizes(orc, shape, n, r):
    say(f"lore fit solver d={shape.d} n={n} r={r} dtype={shape.dtype}")
    X, A, B, Y, loss = fit(shape, n, r)
    check(orc, X, A, B, Y, loss, r)


def test_fit_low_rank_targets(orc):
    say("lore fit solver, targets of rank 12")
    X, A, B, Y, loss = fit(MoEShape(128, 4, 2, 64, 0, 8, BF), 80, 20, zero_expert_rows=116)
    check(orc, X, A, B, Y, loss, 20)
    assert loss <= 1e-9 * (Y ** 2).sum()


def test_fit_without_the_solver_workspace(orc):
    say("lore fit, host path on a workspace without the solver's buffers")
    shape = MoEShape(128, 4, 2, 64, 96, 8, BF)
    X, A, B, Y, loss = fit(shape, 70, 9, spare=256)
    check(orc, X, A, B, Y, loss, 9)
    X, A2, B2, _, loss2 = fit(shape, 70, 9)
    assert loss2 == pytest.approx(loss, rel=1e-10)
    assert np.linalg.norm(B2 @ A2 - B @ A) <= 1e-6 * np.linalg.norm(B @ A)  # fp32 factors


def test_fit_refuses_dependent_tokens():
    say("lore fit solver, a zero token")
    shape = MoEShape(128, 4, 2, 64, 96, 8, BF)
    x = synth.gen_x(Workload("fit", shape, tokens=70, resident=0, skew=False), 0, 0, 70).copy()
    x[33] = 0
    with pytest.raises(spice.SpiceError, match="dependent"):
        fit(shape, 70, 9, x=x)
