"""GPU parity of the tiled routing where its dispatch changes: the row-per-wave launch against
the one- and three-launch forms (207 / 208 and 256 / 257 tokens), one contraction part against
several (2048 / 2049 tokens, short rows, a workspace too small for the partial logits), ragged
token and expert tiles, both dtypes, repeated calls on one workspace (the arrival counters are
left at zero).  Every token's routing against the oracle, and its host copies."""
import numpy as np
import pytest
import torch

from paper_2608_21240_amd import workloads as W
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


# without host copies: few experts, or a contraction split too little for its length, stay on the
# row-per-wave launch up to 256 tokens; one part for a small product
@pytest.mark.parametrize("s,T,R", [
    (shape(2048, 55, 6, BF), 208, 20), (shape(2048, 56, 6, BF, I=512), 208, 20), (shape(2048, 56, 6, BF, I=512), 207, 20),
    (shape(4096, 128, 2, BF), 256, 20), (shape(4096, 128, 2, BF), 257, 20), (shape(1024, 100, 8, F32), 256, 31),
    (shape(200, 20, 10, BF), 256, 8),   # 2560 slots, a row per wave
    (shape(136, 87, 3, BF), 300, 9), (shape(256, 93, 3, F32, I=256), 300, 9), (shape(256, 95, 3, F32, I=256), 300, 9)])
def test_routing_without_host_copies(s, T, R):
    say(f"routing on the device alone d={s.d} N={s.n_experts} K={s.top_k} T={T} R={R} dtype={s.dtype}")
    c = Case(W.Workload("route", s, tokens=T, resident=R, skew=True))
    c.run_gpu(exact=False, layer_call=False)
    c.run_oracle(tokens=[0, T - 1])
    c.check_routing()
