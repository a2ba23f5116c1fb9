"""GPU parity of the grouped GEMM tiles where they can go wrong: contractions, rows, ranks and
buckets that are no multiple of a tile, each of the tile shapes (test_dispatch_cpu.py checks that
the layers here reach them), the split of the shared block's down pass (and a workspace without
room for it), k orders that start at other stages (rows of a multiple of 2 KiB), gated and absent
shared blocks, and the separate LoRE call.  Every token against the oracle, but for the tall tiles
every third."""
import pytest
import torch

from paper_2608_21240_amd import layer as LY, workloads as W
from parity import Case, say

pytestmark = pytest.mark.gpu


def shape(d, N, K, I, Is, r):
    return W.MoEShape(d=d, n_experts=N, top_k=K, inter=I, shared_inter=Is, lore_rank=r, dtype=W.DTYPE_BF16)


# Layers of few tiles: 128 x 64 tiles at any bucket size, 64 x 64 for the up pass
SMALL = shape(200, 20, 5, 104, 168, 24)     # buckets of 16-32, k tails of 8 and 40
WIDE = shape(264, 6, 3, 72, 2064, 136)      # buckets of 32-120; shared block split in 8
BIG = shape(520, 4, 2, 136, 264, 40)        # buckets of 150
NO_SHARED = shape(256, 8, 2, 128, 0, 16)
SMALL_UP = shape(200, 64, 6, 168, 328, 24)  # too many tiles for 64 x 64: 128 x 64 in both passes
# rows of 2 KiB (d) and 4 KiB (I_s): rotated k orders in the up pass, and in each of the 8 parts of the
# shared down pass
ROTATED = shape(1024, 8, 2, 256, 2048, 136)
SPARSE = shape(520, 64, 3, 72, 104, 40)     # buckets of 6: LoRE alone stays on the streaming tiles


@pytest.mark.parametrize("layer_call", [True, False])
@pytest.mark.parametrize("s,T,R,gate,fused", [
    (SMALL, 63, 9, False, True), (SMALL, 64, 9, False, True), (SMALL, 65, 20, True, True),
    (SMALL, 130, 3, False, False), (WIDE, 96, 3, True, True), (WIDE, 209, 2, False, True), (BIG, 300, 2, False, True),
    (BIG, 257, 4, True, True), (NO_SHARED, 129, 4, False, True), (NO_SHARED, 64, 1, False, False),
    (SPARSE, 130, 20, False, False), (SMALL_UP, 130, 40, False, True), (SMALL_UP, 203, 40, True, True),
    (ROTATED, 96, 4, True, True), (ROTATED, 65, 4, False, False)])
def test_gemm_edges(s, T, R, gate, fused, layer_call):
    say(f"gemm d={s.d} I={s.inter} Is={s.shared_inter} T={T} R={R} gate={gate} fused={fused}")
    c = Case(W.Workload("gemm", s, tokens=T, resident=R, skew=True, shared_gate=gate))
    c.run_gpu(fused=fused, layer_call=layer_call)
    c.run_oracle()
    c.check_routing()
    c.check_outputs()


# (layer, tokens, residents): enough up tiles for the shapes named, ragged against them
WIDE_TILES = [(shape(136, 20, 3, 104, 8200, 24), 600, 12), (shape(72, 90, 4, 520, 40, 8), 790, 90)]
BIG_TILES = [(shape(136, 4, 2, 104, 10960, 40), 600, 3), (shape(264, 64, 4, 520, 0, 8), 2200, 64)]
MX_WIDE_TILES = [(shape(128, 12, 2, 256, 6920, 24), 705, 10)]


@pytest.mark.parametrize("s,T,R", WIDE_TILES + BIG_TILES)
def test_gemm_tall_tiles(s, T, R):
    say(f"gemm tall tiles d={s.d} I={s.inter} Is={s.shared_inter} T={T} R={R}")
    c = Case(W.Workload("gemm", s, tokens=T, resident=R, skew=False))
    c.run_gpu()
    c.run_oracle(tokens=range(0, T, 3))
    c.check_routing()
    c.check_outputs()


MX_SMALL = shape(256, 12, 3, 128, 168, 24)  # MXFP4: 2 stages up, 1 down; buckets of 24
MX_WIDE = shape(384, 6, 3, 256, 1096, 40)   # buckets of 96 and more, few tiles


@pytest.mark.parametrize("s,T,R", [(MX_SMALL, 71, 12), (MX_SMALL, 72, 5), (MX_SMALL, 97, 12), (MX_WIDE, 200, 3),
                                   (MX_WIDE, 333, 6), (ROTATED, 97, 6)] + MX_WIDE_TILES)
def test_gemm_mxfp4_edges(s, T, R):
    say(f"gemm mxfp4 d={s.d} I={s.inter} T={T} R={R}")
    c = Case(W.Workload("gemm", s, tokens=T, resident=R, skew=True, wfmt=W.WFMT_MXFP4))
    c.run_gpu()
    c.run_oracle()
    c.check_routing()
    c.check_outputs()


def test_workspace_without_room_for_the_split():
    """A workspace of the size every call needs, but not of the split's partial results."""
    say("gemm without the split's workspace")
    c = Case(W.Workload("gemm", WIDE, tokens=96, resident=3, skew=True))
    dev = LY.DeviceLayer(c.host)
    run = LY.LayerRun(WIDE, 96, dev.C, keep_logits=True)
    run.ws_bytes -= 256
    run.ws = torch.zeros(run.ws_bytes, dtype=torch.uint8, device="cuda")
    c.run_gpu(dev=dev, run=run)
    c.run_oracle()
    c.check_routing()
    c.check_outputs()
