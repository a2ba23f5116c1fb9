"""GPU parity of moe_layer_gpu on either side of each limit that picks its launches: the slots the
fused launches hold (1024; fp32, MXFP4 whose rows are no multiple of 128, bf16 below 64 tokens), the
tokens and slots up to which a small layer keeps them although the GEMM tiles apply, and the fewest
tokens of the GEMM tiles (64; MXFP4 72).  Every token against the oracle, and the combine inside
the call."""
import numpy as np
import pytest

from paper_2608_21240_amd import workloads as W
from parity import Case, say
from test_gpu_parity import check_combine_in_layer_call

pytestmark = pytest.mark.gpu

BF, F32, MX = W.DTYPE_BF16, W.DTYPE_F32, W.WFMT_MXFP4


def shape(d, N, K, I, Is, r, dtype=BF):
    return W.MoEShape(d=d, n_experts=N, top_k=K, inter=I, shared_inter=Is, lore_rank=r, dtype=dtype)


FP = shape(132, 16, 8, 68, 100, 4, F32)
MX_STREAM = shape(192, 16, 8, 96, 136, 8)
MANY = shape(200, 24, 16, 72, 104, 8)
SMALL = shape(264, 16, 4, 136, 392, 16)        # few slots, short rows: fused from 64 to 96 tokens
LONG = shape(1032, 16, 2, 72, 2008, 16)        # a shared block of long rows: GEMM tiles from 64 on
NO_SHARED = shape(264, 24, 2, 136, 0, 16)
MX_GEMM = shape(256, 12, 3, 128, 1800, 16)


@pytest.mark.parametrize("s,T,R,gate,wfmt", [
    (FP, 128, 6, False, 0), (FP, 129, 6, True, 0), (FP, 256, 9, False, 0),       # 1024, 1032 slots, both launches' end
    (MX_STREAM, 128, 6, False, MX), (MX_STREAM, 129, 9, True, MX),
    (MANY, 63, 9, True, 0), (MANY, 60, 9, False, 0),                              # 1008 and 960 slots of one call
    (SMALL, 64, 7, False, 0), (SMALL, 96, 7, True, 0), (SMALL, 97, 7, True, 0), (SMALL, 130, 7, False, 0),
    (LONG, 63, 7, True, 0), (LONG, 64, 7, True, 0), (NO_SHARED, 128, 9, False, 0), (NO_SHARED, 255, 9, False, 0),
    (NO_SHARED, 257, 9, False, 0), (MX_GEMM, 71, 5, False, MX), (MX_GEMM, 97, 5, True, MX)])
def test_layer_call_limits(s, T, R, gate, wfmt):
    say(f"layer limits d={s.d} K={s.top_k} T={T} R={R} gate={gate} wfmt={wfmt} dtype={s.dtype}")
    c = Case(W.Workload("limits", s, tokens=T, resident=R, skew=False, shared_gate=gate, wfmt=wfmt))
    c.run_gpu(layer_call=True)
    c.run_oracle()
    c.check_routing()
    c.check_outputs()
    assert (np.bincount(c.o["cls"].reshape(-1), minlength=3) > 0).all()  # all three classes
    check_combine_in_layer_call(c)
