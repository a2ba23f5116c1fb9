"""The rules that pick a call's kernels, without a GPU: the inline functions of spice_internal.h
compiled into a small driver (sanitize/dispatch_driver.cpp), on layers whose best choice was
measured on a GPU."""
import os
import shutil
import subprocess

import pytest

from paper_2608_21240_amd import workloads as W

import test_gpu_gemm as G
import test_gpu_layer_limits as LIM

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CSRC = os.path.join(ROOT, "paper_2608_21240_amd", "csrc")
ROCM = os.environ.get("ROCM_PATH", "/opt/rocm")
SMALL, WIDE, BIG = 0, 1, 2


@pytest.fixture(scope="module")
def driver(tmp_path_factory):
    if not shutil.which("g++") or not os.path.exists(os.path.join(ROCM, "include", "hip", "hip_runtime_api.h")):
        pytest.skip("g++ or the HIP headers are not installed")
    exe = str(tmp_path_factory.mktemp("dispatch") / "driver")
    subprocess.run(["g++", "-std=c++17", "-O1", f"-I{ROOT}/include", f"-I{CSRC}", f"-I{ROCM}/include",
                    "-D__HIP_PLATFORM_AMD__", os.path.join(ROOT, "tests", "sanitize", "dispatch_driver.cpp"), "-o", exe],
                   check=True)
    return exe


@pytest.fixture(scope="module")
def rules(driver):
    """rules(T, shape, C, wfmt=0) -> (tile shape, parts of the shared block, fused layer call, GEMM tiles for LoRE
    alone)."""

    def ask(T, s, C, wfmt=0):
        line = f"{T} {s.d} {s.n_experts} {s.top_k} {C} {s.inter} {s.shared_inter} {wfmt}\n"
        r = subprocess.run([driver], input=line, capture_output=True, text=True, check=True)
        return tuple(int(v) for v in r.stdout.split())

    return ask


def layer(d, N, K, I, Is, r=16):
    return W.MoEShape(d=d, n_experts=N, top_k=K, inter=I, shared_inter=Is, lore_rank=r, dtype=W.DTYPE_BF16)


@pytest.fixture(scope="module")
def routing(driver):
    """routing(T, N, d, dtype, part_bytes, x_to_host) -> (contraction parts, row per wave)."""

    def ask(*args):
        r = subprocess.run([driver, "routing"], input=" ".join(str(int(v)) for v in args) + "\n", capture_output=True,
                           text=True, check=True)
        return tuple(int(v) for v in r.stdout.split())

    return ask


# Layers of few tiles, FFN call in us on Small against the shape their buckets' size alone would take:
# 13.1 / 16.7 and 20.0 / 32.0 (Wide), 71.7 / 102.3 and 30.4 / 42.2 (Wide, Big).
@pytest.mark.parametrize("T,s,C", [
    (253, layer(328, 4, 1, 64, 0), 4), (81, layer(1448, 2, 1, 960, 0), 2), (152, layer(1224, 6, 5, 360, 952), 1),
    (128, layer(256, 16, 4, 256, 384), 8), (81, layer(2576, 3, 3, 280, 0), 3), (600, layer(512, 4, 4, 256, 512), 4)])
def test_few_tiles_take_the_small_shape(rules, T, s, C):
    assert T * s.top_k // s.n_experts >= 32
    assert rules(T, s, C)[0] == SMALL


@pytest.mark.parametrize("T,s,C,wfmt,want", [
    (192, W.DSV2, 48, 0, SMALL), (512, W.DSV2, 48, 0, WIDE), (1000, W.DSV2, 32, 0, WIDE), (1000, W.QWEN2, 64, 0, BIG),
    (4096, W.QWEN2, 64, 0, BIG), (600, W.DSV2, 64, W.WFMT_MXFP4, SMALL), (777, W.DSV2, 64, W.WFMT_MXFP4, WIDE),
    (4096, W.QWEN2, 64, W.WFMT_MXFP4, WIDE)])
def test_large_layers_take_the_shape_of_their_buckets(rules, T, s, C, wfmt, want):
    assert rules(T, s, C, wfmt)[0] == want


# Layer calls in us, fused launches / GEMM tiles: 22.1 / 25.8, 30.0 / 34.7, 22.7 / 25.8, 20.7 / 26.4, 28.0 / 31.9,
# 26.0 / 36.2; 92.3 / 60.5, 155 / 142, 31.5 / 28.0, 47.1 / 35.5, 577 / 549.
@pytest.mark.parametrize("T,s,fused", [
    (64, layer(256, 16, 4, 256, 384), 1), (64, layer(1024, 16, 2, 512, 1024), 1), (64, layer(128, 64, 6, 64, 128), 1),
    (128, layer(512, 16, 2, 512, 0), 1), (255, layer(512, 16, 2, 512, 0), 1), (133, layer(896, 21, 1, 1336, 0), 1),
    (128, layer(2048, 16, 2, 1408, 2816), 0), (64, W.DSV2, 0), (128, layer(256, 16, 4, 256, 384), 0),
    (128, layer(1024, 16, 2, 512, 1024), 0), (32, W.QWEN2, 0)])
def test_small_layers_keep_the_fused_launches(rules, T, s, fused):
    assert rules(T, s, s.n_experts // 2)[2] == fused


# lore_surrogate_apply in us, streaming / GEMM tiles: 12.0 / 26.2, 13.0 / 29.9, 13.9 / 30.1, 10.3 / 21.5; 107.4 / 11.8,
# 22.9 / 11.0, 50.6 / 16.7, 243.7 / 65.5.
@pytest.mark.parametrize("T,s,gemm", [
    (71, layer(3968, 49, 1, 64, 64, 16), 0), (120, layer(3496, 99, 3, 64, 64, 40), 0), (193, layer(3968, 51, 3, 64, 64, 56), 0),
    (64, W.DSV2, 0), (182, layer(80, 73, 8, 64, 64, 64), 1), (142, layer(128, 31, 7, 64, 64, 40), 1),
    (108, layer(112, 3, 2, 64, 64, 64), 1), (498, layer(3200, 7, 7, 64, 64, 16), 1)])
def test_lore_alone_takes_the_shorter_tiles(rules, T, s, gemm):
    assert rules(T, s, 1)[3] == gemm


# moe_route_bucket in us, row per wave / tiles: 13.0 / 18.4, 12.1 / 14.5, 49.6 / 94.2 (a workspace with room for one
# part), 197 / 249 (the same, with x to the host), 24.4 / 21.7, 26.0 / 22; with x to the
# host 58 / 43.
@pytest.mark.parametrize("T,N,d,room,x_to_host,rows", [
    (208, 17, 2048, 1 << 30, 0, 1), (208, 8, 256, 1 << 30, 0, 1), (208, 128, 4096, 300000, 0, 1),
    (208, 256, 4096, 700000, 1, 1), (256, 64, 2048, 1 << 30, 0, 0), (256, 64, 3584, 1 << 30, 0, 0), (208, 28, 2040, 1 << 30, 1, 0),
    (207, 64, 2048, 1 << 30, 0, 1), (207, 64, 2048, 1 << 30, 1, 1), (257, 8, 64, 1 << 30, 0, 0)])
def test_routing_keeps_rows_where_they_are_shorter(routing, T, N, d, room, x_to_host, rows):
    assert routing(T, N, d, W.DTYPE_BF16, room, x_to_host)[1] == rows


# Small products stay whole (15.2 / 16.6 us in two parts, 15.6 / 18.1, 22.4 / 24.6,
# 31.1 / 33.0); large ones are split, as far as the
# workspace, the CUs and the passes go.
@pytest.mark.parametrize("T,N,d,dtype,room,parts", [
    (563, 12, 144, W.DTYPE_F32, 1 << 30, 1), (1172, 8, 448, W.DTYPE_BF16, 1 << 30, 1), (388, 35, 1440, W.DTYPE_BF16, 1 << 30, 8),
    (1000, 64, 2048, W.DTYPE_BF16, 1 << 30, 4), (1000, 64, 2048, W.DTYPE_BF16, 3 * 63 * 16 * 64 * 8, 3),
    (1000, 64, 2048, W.DTYPE_BF16, 0, 1), (4096, 64, 2048, W.DTYPE_BF16, 1 << 30, 1), (300, 64, 256, W.DTYPE_BF16, 1 << 30, 1), (300, 128, 256, W.DTYPE_BF16, 1 << 30, 1), (300, 64, 512, W.DTYPE_BF16, 1 << 30, 4)])
def test_routing_parts(routing, T, N, d, dtype, room, parts):
    assert routing(T, N, d, dtype, room, 0)[0] == parts


def test_the_gpu_cases_reach_the_shapes_they_name(rules):
    for cases, wfmt, want in ((G.WIDE_TILES, 0, WIDE), (G.BIG_TILES, 0, BIG), (G.MX_WIDE_TILES, W.WFMT_MXFP4, WIDE)):
        for s, T, R in cases:
            assert rules(T, s, R, wfmt)[0] == want, (s, T, R)
    assert rules(96, G.WIDE, 3)[1] == rules(96, G.ROTATED, 4)[1] == rules(65, G.ROTATED, 4)[1] == 8

    def deep_tiles(T, s, R):  # the launch's bound on its 64 x 64 up tiles; at most 256 take them
        up = lambda n, per: -(-n // per)
        slots = T * s.top_k
        nt_e, nt_l = up(s.inter, 32), up(s.lore_rank, 64)
        return (up(T, 64) * up(s.shared_inter, 32) + slots // 64 * max(nt_e, nt_l) + min(s.n_experts, R, slots) * nt_e +
                min(s.n_experts, slots) * nt_l)

    for T, R in ((130, 40), (203, 40)):
        assert rules(T, G.SMALL_UP, R)[0] == SMALL and deep_tiles(T, G.SMALL_UP, R) > 256
    assert deep_tiles(64, G.SMALL, 9) <= 256
    for s, T, fused in ((LIM.SMALL, 64, 1), (LIM.SMALL, 96, 1), (LIM.SMALL, 97, 0), (LIM.LONG, 64, 0), (LIM.NO_SHARED, 255, 1),
                        (LIM.NO_SHARED, 257, 0), (LIM.MX_GEMM, 97, 0)):
        assert rules(T, s, 7)[2] == fused, (s, T)
    assert [rules(T, s, 1)[3] for s, T in ((G.SMALL, 130), (G.NO_SHARED, 64), (G.SPARSE, 130))] == [1, 1, 0]
