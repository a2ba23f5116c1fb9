"""GPU parity of the tiled routing where its dispatch changes: the row-per-wave launch against
the one- and three-launch forms (207 / 208 and 256 / 257 tokens), one contraction part against
several (2048 / 2049 tokens, short rows, the smallest workspace, which has no room for the
partial logits), ragged token and expert tiles, both dtypes, repeated calls on one workspace (the arrival counters are
left at zero).  Every token's routing against the oracle, and its host copies."""
import numpy as np
import pytest
import torch

from paper_2608_21240_amd import layer as LY, spice, workloads as W
from parity import Case, say, to_np

pytestmark = pytest.mark.gpu

BF, F32 = W.DTYPE_BF16, W.DTYPE_F32


def shape(d, N, K, dtype, I=32, Is=32):
    return W.MoEShape(d=d, n_experts=N, top_k=K, inter=I, shared_inter=Is, lore_rank=8, dtype=dtype)


@pytest.mark.parametrize("s,T,R", [
    (shape(1000, 20, 3, BF), 207, 9), (shape(1000, 20, 3, BF), 208, 9), (shape(1000, 20, 3, BF), 223, 20),
    (shape(512, 70, 8, F32), 256, 31), (shape(512, 70, 8, F32), 257, 31), (shape(1024, 256, 6, BF), 250, 100),
    (shape(2048, 64, 6, BF), 300, 32), (shape(256, 33, 2, BF), 2048, 11), (shape(256, 33, 2, BF), 2049, 11),
    (shape(64, 17, 4, BF), 240, 5), (shape(4096, 100, 1, BF, I=8, Is=8), 300, 50)])
def test_tiled_routing(s, T, R):
    say(f"tiled routing d={s.d} N={s.n_experts} K={s.top_k} T={T} R={R} dtype={s.dtype}")
    c = Case(W.Workload("route", s, tokens=T, resident=R, skew=True))
    c.run_gpu(fused=False)
    c.run_oracle(tokens=[0, T - 1])
    c.check_routing()
    c.check_outputs()
    x = torch.from_numpy(c.x if s.dtype == F32 else c.x.view(np.int16)).cuda()
    x = x if s.dtype == F32 else x.view(torch.bfloat16)
    for _ in range(3):
        c.run.route(c.dev, x, torch.from_numpy(c.conf).cuda(), T)
        torch.cuda.synchronize()
        assert np.array_equal(to_np(c.run.topk_idx), c.o["idx"]) and np.array_equal(to_np(c.run.perm), c.o["perm"])
        assert np.array_equal(c.run.idx_host.numpy(), c.o["idx"]) and np.array_equal(c.run.cls_host.numpy(), c.o["cls"])
        assert np.array_equal(to_np(c.run.x_host), c.x)


@pytest.mark.parametrize("s,T", [(shape(4096, 100, 1, BF, I=8, Is=8), 300), (shape(1024, 64, 6, F32), 230)])
def test_routing_on_the_smallest_workspace(s, T):
    say(f"routing on the smallest workspace d={s.d} N={s.n_experts} T={T}")
    c = Case(W.Workload("route", s, tokens=T, resident=30, skew=False))
    dev = LY.DeviceLayer(c.host)
    run = LY.LayerRun(s, T, dev.C, keep_logits=True, layer_call=False)
    full, run.ws_bytes = run.ws_bytes, 1024
    with pytest.raises(spice.SpiceError) as e:
        run.route(dev, run.out, run.topk_w, T)
    run.ws_bytes = int(str(e.value).split("needs ")[1].split()[0].rstrip(")"))
    assert run.ws_bytes < full
    run.ws = torch.zeros(run.ws_bytes, dtype=torch.uint8, device="cuda")
    c.run_gpu(dev=dev, run=run)
    c.run_oracle(tokens=[0, T - 1])
    c.check_routing()
    c.check_outputs()


def test_routing_beside_an_ffn_on_one_workspace():
    """A routing call (its contraction split) on one stream while the FFN of an earlier one runs on
    another, on the same workspace: the FFN's outputs stay what they are alone."""
    s = shape(1024, 64, 6, BF, I=256, Is=512)
    T = 600
    say("routing beside an FFN on one workspace")
    c = Case(W.Workload("route", s, tokens=T, resident=40, skew=False))
    c.run_gpu(exact=False, layer_call=False)
    R, dev = c.run, c.dev
    x = torch.from_numpy(c.x.view(np.int16)).cuda().view(torch.bfloat16)
    conf = torch.from_numpy(c.conf).cuda()
    want = R.y_slots.clone(), R.y_shared.clone()
    other = type(R)(s, T, dev.C)  # buffers of the second routing, but the first one's workspace
    other.ws, other.ws_bytes = R.ws, R.ws_bytes
    side = torch.cuda.Stream()
    torch.cuda.synchronize()
    for _ in range(10):
        R.y_slots.fill_(-1.0)
        R.y_shared.fill_(-1.0)
        torch.cuda.synchronize()
        with torch.cuda.stream(side):
            for _ in range(4):
                other.route(dev, x, conf, T, to_host=False, mark=False)
        R.experts(dev, x, T)
        torch.cuda.synchronize()
        live = R.inv_perm[(R.slot_class.reshape(-1) != 2)].long()
        assert torch.equal(R.y_slots[live], want[0][live]) and torch.equal(R.y_shared, want[1])


# without host copies: few experts, or a contraction split too little for its length, stay on the
# row-per-wave launch up to 256 tokens; one part for a small product
@pytest.mark.parametrize("s,T,R", [
    (shape(2048, 55, 6, BF), 208, 20), (shape(2048, 56, 6, BF, I=512), 208, 20), (shape(2048, 56, 6, BF, I=512), 207, 20),
    (shape(4096, 128, 2, BF), 256, 20), (shape(4096, 128, 2, BF), 257, 20), (shape(1024, 100, 8, F32), 256, 31),
    (shape(200, 20, 10, BF), 256, 8),   # 2560 slots, a row per wave
    (shape(136, 87, 3, BF), 300, 9), (shape(248, 99, 3, F32), 300, 9), (shape(256, 93, 3, F32), 300, 9),
    (shape(256, 94, 3, F32), 300, 9)])
def test_routing_without_host_copies(s, T, R):
    say(f"routing on the device alone d={s.d} N={s.n_experts} K={s.top_k} T={T} R={R} dtype={s.dtype}")
    c = Case(W.Workload("route", s, tokens=T, resident=R, skew=True))
    c.run_gpu(exact=False, layer_call=False)
    c.run_oracle(tokens=[0, T - 1])
    c.check_routing()
