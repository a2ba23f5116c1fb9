// Internal declarations shared by the HIP kernels and the C-ABI layer of libspice_moe.
#pragma once

#include <hip/hip_runtime_api.h>
#include <stddef.h>
#include <stdint.h>

#include "spice_moe.h"

namespace spice {

// Workspace control region (32-bit words at the start of every workspace).
constexpr int kWordFlags = 0;       // device flags, SPICE_FLAG_* (atomic OR)
constexpr int kWordWorkCount = 16;  // [3] non-empty buckets per class (the work lists' lengths)
constexpr int kWordScanCount = 32;  // arrivals of the prefill bucket-scan blocks
constexpr int kWordRouteDone = 33;  // arrivals of the tokens' last routing blocks (decode routing call)
constexpr int kWordWorkList = 1024; // [3][N] int4 work records {expert, pool slot, start, n}
// [T] arrivals of a token's (tiled routing: a 16-token group's) routing blocks, each counter alone in a
// 128-byte line: the atomics of different tokens' blocks do not queue on one line
constexpr int kWordTokCount = 4096;
constexpr int kTokCountStride = 32;  // words between two tokens' counters
static_assert(kWordWorkList + 3 * SPICE_MAX_EXPERTS * 4 <= kWordTokCount, "work lists overlap the counters");

// Largest T whose routing call is one launch.
constexpr int kRouteTokenMaxT = 256;
// Fewest tokens whose logits may be computed as fp64 MFMA tiles of 16 tokens (route_bucket.hip).
constexpr int kRouteTiledMinT = 208;
// Contraction parts per group of 16 tokens of the tiled logits: as many as fill the 256 CUs with a
// block each (a group's logits are bound by its CU's fp64 matrix rate), at least two passes of
// 128 bytes per part, and partial logits that fit part_bytes.  One for small products and short rows,
// whose logits take less time than a group's wait for its parts (whole / split: N = 12, d = 144
// 15.2 / 16.6 us, N = 64, d = 256 22.4 / 24.6, N = 128, d = 256 31.1 / 33.0; N = 5, d = 3736 23.1 / 17.4, N = 35, d = 1440 26.4 / 21.2).
constexpr int kRouteTileTok = 16, kRouteMaxParts = 8;
inline int route_parts(int32_t T, int32_t N, int32_t d, int32_t dtype, size_t part_bytes) {
    const int groups = (T + kRouteTileTok - 1) / kRouteTileTok;
    const int npass = d * (dtype == SPICE_BF16 ? 2 : 4) / 128;
    if (npass < 8 || (int64_t)N * d < (d <= 1024 ? 24000 : 12000)) return 1;
    const size_t per_part = (size_t)groups * kRouteTileTok * N * sizeof(double);
    int p = kRouteMaxParts;
    p = p < 256 / groups ? p : 256 / groups;
    p = p < npass / 2 ? p : npass / 2;
    if ((size_t)(p > 0 ? p : 0) * per_part > part_bytes) p = (int)(part_bytes / per_part);
    return p > 1 ? p : 1;
}
// Whether a routing call of kRouteTiledMinT tokens or more keeps a row per wave (kRouteTokenMaxT at
// most).  The tiles pay for many experts whose contraction is split far enough; copying x to the host
// the last block's 1024 threads take less time than the rows' 256, unless the logits take very long.
// Rows / tiles, us per call of 208 - 256 tokens: N = 17, d = 2048 13.0 / 18.4; N = 64, d = 2048 in 8
// parts 24.4 / 21.7; N = 128, d = 4096 in one part 49.6 / 94.2; with x to the host N = 28, d = 2040
// 58 / 43, N = 256, d = 4096 in one part 197 / 249.
inline bool route_keeps_rows(int32_t T, int32_t N, int32_t d, int parts, bool x_to_host) {
    if (T < kRouteTiledMinT) return true;
    if (T > kRouteTokenMaxT) return false;
    return x_to_host ? N >= 128 && d > 16 * T * parts : N < 56 || d > 4 * T * parts;
}
static_assert((kWordTokCount + kRouteTokenMaxT * kTokCountStride) * 4 <= SPICE_WS_CONTROL_BYTES, "control region too small");
// [T*K] bucket keys (class * N + expert) of the decode routing call's slots, written through
// to the device-coherent level for the block that buckets them (top-K of 64 at most)
constexpr int kWordSlotKeys = 12288;
static_assert(kWordTokCount + kRouteTokenMaxT * kTokCountStride <= kWordSlotKeys, "slot keys overlap the counters");
static_assert((kWordSlotKeys + kRouteTokenMaxT * 64) * 4 <= SPICE_WS_CONTROL_BYTES, "control region too small");
// Most slots T*K of the fused decode-layer launches (layer_decode.hip); larger calls take
// the separate routing, FFN and combine launches.
constexpr int kLayerMaxSlots = 1024;

// Row padding (elements) of the SwiGLU intermediates in the workspace: row strides
// that are multiples of large powers of two put every row of a tile on the same
// HBM channel.
constexpr int kHPad = 64;

// Byte offsets of the workspace regions for one (cfg, T).
struct WsLayout {
    size_t logits;  // fp64 [T][N]
    size_t h;       // SwiGLU intermediate of routed slots [T*K][I + kHPad] (dtype)
    size_t hs;      // shared-block intermediate [T][I_s + kHPad] (dtype)
    size_t u;       // LoRE A x, fp32 [T*K][r]
    size_t sgate;   // output gate of the shared block, fp32 [T]
    size_t base;    // bytes every call needs; the rest is used when the workspace has it
    size_t zpart;   // partial logits of the tiled routing, fp64 (its own: no FFN buffer is touched by a routing call)
    size_t part;    // the shared block's partial results, fp32 [parts][T][d]
    size_t total;
};
WsLayout ws_layout(const spice_moe_cfg_t& c, int32_t T);

// Which expert groups a grouped-FFN launch covers.
enum : int { kDoHit = 1, kDoShared = 2, kDoLore = 4 };

struct RouteArgs {
    int32_t T, d, N, K, C, dtype, norm_topk, conf_mode;
    float tau;
    const void* x;
    const void* wg;
    const float* bias;
    const int32_t* resident_slot;
    const float* conf;
    double* logits_out;   // caller's, nullable
    double* logits_ws;    // workspace copy read by the top-K step
    double* part_ws;      // partial logits of the tiled routing
    size_t part_bytes;    // its size
    int32_t* topk_idx;
    float* topk_w;
    uint8_t* slot_class;
    int32_t* offsets;
    int32_t* perm;
    int32_t* inv_perm;
    uint32_t* ctrl;       // workspace control words
    int32_t* worklist;    // [3][N][4] work records (control region)
    int32_t* wl_count;    // [3] their lengths (control region)
    const void* w_sg;     // nullable: the shared block's gate row [d]; sgate[t] = sigmoid(w_sg . x[t])
    float* sgate;         // [T], written when w_sg is set
    // device-visible addresses of the caller's pinned host copies (each nullable)
    void* hx;
    int32_t* h_idx;
    float* h_w;
    uint8_t* h_cls;
    int32_t* h_counts;
    uint32_t* h_ready;    // nullable: receives ready_value once every host copy has landed
    uint32_t ready_value;
};

// Bytes of one routed expert's W13 [2I][d] and W2 [d][I] in the cfg's weight format.
inline size_t expert_w13_bytes(const spice_moe_cfg_t& c) {
    const size_t n = (size_t)2 * c.inter * c.d;
    return c.wfmt == SPICE_WFMT_MXFP4 ? n / 2 + n / 32 : n * (c.dtype == SPICE_BF16 ? 2 : 4);
}
inline size_t expert_w2_bytes(const spice_moe_cfg_t& c) {
    const size_t n = (size_t)c.inter * c.d;
    return c.wfmt == SPICE_WFMT_MXFP4 ? n / 2 + n / 32 : n * (c.dtype == SPICE_BF16 ? 2 : 4);
}

struct FfnArgs {
    int32_t T, d, N, K, C, I, Is, r, dtype, groups;
    int32_t wfmt;  // SPICE_WFMT_*: the pools hold MXFP4 blobs when SPICE_WFMT_MXFP4
    int32_t ldh, ldhs;  // row strides (elements) of h and hs
    const void* x;
    const int32_t* perm;
    const int32_t* offsets;
    const int32_t* resident_slot;
    const void* w13_pool;
    const void* w2_pool;
    const void* w13s;
    const void* w2s;
    const void* lore_A;
    const void* lore_B;
    float* y_slots;
    float* y_shared;
    const float* sgate;  // nullable: y_shared[t] is scaled by sgate[t] (gated shared block)
    void* h;        // workspace [T*K][I]
    void* hs;       // workspace [T][I_s]
    float* u;       // workspace [T*K][r]
    float* part;    // workspace [parts][T][d], or null: the shared block's down pass is not split
    uint32_t* ctrl;
};

// The fetched-expert FFN (M_fetch of Eq. 12): fetch slot j serves the bucket
// (EXACT, fetch_expert[j]) with the weights in slot j of the fetch pool (passed as
// the FfnArgs pools), and relabels that bucket's slots EXACT -> EXACT_GPU.
struct FetchArgs {
    const int32_t* fetch_expert;  // device [n_slots], -1 = unused slot
    uint8_t* slot_class;          // device [T*K]
    int32_t n_slots;
};

// One depth of the speculative-prefetch draft rollout (spec_draft.hip).
struct SpecArgs {
    int32_t T, d, K, dtype, delta, l_min, last, lore;
    float tau;
    const void* h_in;
    void* h_out;            // may equal h_in
    const int32_t* topk_idx;
    const float* topk_w;
    const int32_t* inv_perm;
    const float* y_slots;
    const float* y_shared;
    int32_t* halted;        // [T], in/out
    int32_t* pred_idx;      // [T][K]
    float* pred_prob;       // [T][K]
    float* conf;            // [T]
    uint32_t* ctrl;
    // device-visible addresses of the caller's pinned host copies (each nullable)
    int32_t* h_pred_idx;
    float* h_pred_prob;
    float* h_conf;
};

struct CombineArgs {
    int32_t T, d, K, dtype;
    const float* topk_w;
    const uint8_t* slot_class;
    const int32_t* inv_perm;
    const float* y_slots;
    const float* y_shared;
    const float* resid;
    void* out;
};

// Grouped MFMA GEMMs of the HIT experts, the shared block and the LoRE correction for many
// tokens (bf16; used by launch_expert_ffn when expert_gemm_applies).
// Fewest tokens of a call that takes them.  Below, the streaming tiles: one pass over the
// shared block's weights per 32 tokens.  Streaming tiles / GEMMs, us per layer call:
// DeepSeek-V2-Lite sizes, 48 experts resident, T = 40 177 / 184, T = 64 204 / 187 (8 resident: 88 /
// 82); Qwen2 sizes, whose shared block is 440 MB, T = 24 310 / 315, T = 32 577 / 549, T = 48
// 677 / 561.  MXFP4 experts, all 64 of DeepSeek-V2-Lite resident: T = 72 145 / 125, T = 96
// 159 / 131; Qwen2 sizes T = 40 424 / 378, T = 64 482 / 391.
// Small layers gain nothing from them at so few tokens: layer_fused_is_shorter.
constexpr int kGemmMinTokens = 64, kGemmMinTokensWide = 32;
inline int gemm_min_tokens(int32_t d, int32_t Is, int32_t wfmt) {
    const int n = (int64_t)3 * Is * d * 2 >= (64 << 20) ? kGemmMinTokensWide : kGemmMinTokens;
    return wfmt == SPICE_WFMT_MXFP4 ? n + 8 : n;
}
// Whether moe_layer_gpu takes the three fused launches where both they and the GEMM tiles could run
// the call.  The fused launches route beside the shared block's up pass but read a weight once per 32
// tokens; the GEMMs wait for the routing, and for a shared gate's own launch.  So few slots in short
// buckets stay fused, as long as the shared block's passes over its rows, T / 32 of d + I_s, are
// short.  Fused / GEMM, us per call: d = 256, N = 16, K = 4, I = 256, I_s = 384 T = 64 22.1 / 25.8,
// T = 96 25.5 / 26.6, T = 128 31.5 / 28.0; d = 1024, K = 2, I = 512, I_s = 1024 T = 64 30.0 / 34.7,
// T = 96 38.0 / 35.4; d = 512, K = 2, I = 512 without a shared block T = 128 20.7 / 26.4, T = 255
// 28.0 / 31.9.
inline bool layer_fused_is_shorter(int32_t T, int32_t d, int32_t N, int32_t K, int32_t Is) {
    const int64_t slots = (int64_t)T * K, n = slots / (N > 0 ? N : 1);
    if (Is == 0) return slots <= 256 ? n < 64 : slots <= 512 && n < 32;
    return T <= 96 && slots <= 512 && n < 48 && (int64_t)T * (d + Is) <= 32 * 6000;
}
// Whether the LoRE corrections alone (lore_surrogate_apply) take the GEMM tiles.  A tile waits for d /
// 64 stages one after the other, the streaming tiles read the factors once per 32 entries of a
// bucket: GEMM / streaming, geometric mean over random layers at d = 2048 - 4096 1.57 times with
// 4 - 8 entries in the mean bucket, 1.00 with 16 - 32, 0.63 with 64 - 128; at d = 256 - 512 1.07,
// 0.83, 0.40.  (Buckets that residents leave short keep the GEMMs, up to twice as long.)
inline bool lore_gemm_is_shorter(int32_t T, int32_t d, int32_t N, int32_t K) {
    const int64_t n = (int64_t)T * K / (N > 0 ? N : 1);
    return n >= 16 && 28 * n >= d;
}
// Tile shape by the mean bucket size: a tile as tall as the buckets are long reads each weight
// once and wastes no token column, and the more weight rows a block takes the more bytes it
// keeps in flight.  Small / Wide / Big, us per call: n = 18 212 / 216 / 258, n = 48 223 / 211 /
// 259, n = 94 293 / 266 / 280 (DeepSeek-V2-Lite sizes), n = 128 1774 / 1403 / 1359 (Qwen2).
// That holds while the tiles fill the GPU (one Wide or Big block per CU); with fewer, a call takes
// as long as one tile, and the smaller is the shorter.  FFN call, geometric mean over random
// layers by the up launch's tiles: Wide / Small 1.57 below 64 tiles, 1.38 to 128, 1.22 to 256,
// about 1.1 to 512; Big / Wide 1.46, 1.34, 1.15, and 1.13 to 384 (at most 3.6 in one layer).
enum : int { kGemmSmall = 0, kGemmWide = 1, kGemmBig = 2 };
// weight rows, tokens
constexpr int kGemmSmallTile[2] = {128, 64}, kGemmWideTile[2] = {256, 128}, kGemmBigTile[2] = {256, 256};
constexpr int kGemmWideMinTiles = 320, kGemmBigMinTiles = 256;
// Up tiles of the shared block and of the HIT buckets, n tokens in each.
inline int64_t gemm_up_tiles(const int* tile, int32_t T, int64_t n, int32_t N, int32_t C, int32_t I, int32_t Is) {
    const int64_t feat = tile[0] / 2, buckets = N < C ? N : C, per = n > 0 ? (n + tile[1] - 1) / tile[1] : 1;
    return ((int64_t)T + tile[1] - 1) / tile[1] * ((Is + feat - 1) / feat) + buckets * per * ((I + feat - 1) / feat);
}
// For MXFP4 experts there is no Big shape (two stages of it would not fit the LDS), and Wide is
// the better from twice the bucket on (Small / Wide, us per call: n = 37 215 / 225, n = 73 294 /
// 261).
inline int gemm_shape(int32_t T, int32_t N, int32_t K, int32_t C, int32_t I, int32_t Is, int32_t wfmt) {
    const int64_t n = (int64_t)T * K / (N > 0 ? N : 1);
    const bool mx = wfmt == SPICE_WFMT_MXFP4;
    int s = n < (mx ? 64 : 32) ? kGemmSmall : mx || n < 120 ? kGemmWide : kGemmBig;
    if (s == kGemmBig && gemm_up_tiles(kGemmBigTile, T, n, N, C, I, Is) < kGemmBigMinTiles) s = kGemmWide;
    if (s == kGemmWide && gemm_up_tiles(kGemmWideTile, T, n, N, C, I, Is) < kGemmWideMinTiles) s = kGemmSmall;
    return s;
}
// Splits of the shared block's down contraction.  Its tiles are Is / I times as long as a
// routed expert's; with few of them (small T) the launch would wait for them at its end (Qwen2,
// T = 96: 738 us whole, 604 in 8 parts).  At most as many as the GPU takes at a time (one Big
// block per CU, two of the others): more only add partial sums (T = 2048: 2117 -> 2166).
constexpr int kMaxSharedParts = 8;
inline int gemm_shared_parts(int32_t T, int32_t d, int32_t N, int32_t K, int32_t C, int32_t I, int32_t Is) {
    const int shape = gemm_shape(T, N, K, C, I, Is, SPICE_WFMT_DTYPE);
    if (T < gemm_min_tokens(d, Is, SPICE_WFMT_DTYPE) || Is <= 0) return 1;
    const int* t = shape == kGemmBig ? kGemmBigTile : shape == kGemmWide ? kGemmWideTile : kGemmSmallTile;
    const int64_t tiles = (int64_t)((T + t[1] - 1) / t[1]) * ((d + t[0] - 1) / t[0]);
    const int64_t most = shape == kGemmBig ? 256 : 512;
    int64_t p = C > 0 ? Is / I : kMaxSharedParts;  // no routed tiles: as many as fill the GPU
    p = p < most / tiles ? p : most / tiles;
    p = p < Is / 256 ? p : Is / 256;
    return (int)(p < 1 ? 1 : p > kMaxSharedParts ? kMaxSharedParts : p);
}

struct GemmArgs {
    int32_t T, d, N, K, C, I, Is, r;
    int32_t do_hit;                    // HIT buckets too (else the shared block and LoRE only)
    int32_t parts;                     // contraction splits of the shared block's down pass
    int32_t super_up[2], super_dn[2];  // shared-block super-tile (weight tiles, token tiles)
    const uint16_t* x;
    const int32_t* perm;
    const int32_t* offsets;
    const int32_t* resident_slot;
    const void* w13_pool;
    const void* w2_pool;
    const uint16_t* w13s;
    const uint16_t* w2s;
    const uint16_t* lore_A;
    const uint16_t* lore_B;
    uint16_t* h;
    uint16_t* hs;
    float* u;
    float* part;                       // [parts][T][d] when parts > 1
    float* y_slots;
    float* y_shared;
    const float* sgate;  // nullable, as in FfnArgs
    uint32_t* ctrl;
};

bool expert_gemm_applies(const FfnArgs& a);
hipError_t launch_expert_gemm(const FfnArgs& a, bool hit, bool shared, hipStream_t s);

hipError_t launch_route_bucket(const RouteArgs& a, hipStream_t s);
// The fused decode layer (routing, bucketing, shared block, HIT and LoRE FFN) in three
// launches; bf16/fp32 or MXFP4 routed experts, T <= kRouteTokenMaxT, T*K <= kLayerMaxSlots.
hipError_t launch_layer_decode(const RouteArgs& r, const FfnArgs& f, hipStream_t s);
hipError_t launch_expert_ffn(const FfnArgs& a, hipStream_t s);
// The same launch with MXFP4 routed experts (expert_ffn_mx.hip).
hipError_t launch_expert_ffn_mx(const FfnArgs& a, hipStream_t s);
// sgate[t] = sigmoid(w_sg . x[t]) for T tokens (fp64 dot products), shared_gate.hip.
hipError_t launch_shared_gate(const void* x, const void* w_sg, int32_t T, int32_t d, int32_t dtype, float* sgate,
                              hipStream_t s);
hipError_t launch_expert_ffn_fetched(const FfnArgs& a, const FetchArgs& f, hipStream_t s);
hipError_t launch_combine(const CombineArgs& a, hipStream_t s);
hipError_t launch_spec_update(const SpecArgs& a, hipStream_t s);

// LoRE calibration fit (lore_fit.hip).
hipError_t launch_fit_setup(int32_t n, int32_t* perm, int32_t* offsets, int32_t* resident, hipStream_t s);
hipError_t launch_fit_residual(size_t count, float* y, const float* shared, hipStream_t s);
hipError_t launch_fit_gram(int32_t n, int32_t d, int dtype, const void* M, double* G, hipStream_t s);
hipError_t launch_fit_project(int32_t n, int32_t d, int32_t r, int dtype, const void* M, const double* C, float* out,
                              bool b_layout, hipStream_t s);
// Eigen-decomposition and SPD solve of the fit, n <= 1024 (device pointers; see the kernels).
hipError_t launch_fit_tridiag(int32_t n, double* A, double* V, double* tau, double* p, double* dv, double* ev, hipStream_t s);
hipError_t launch_fit_rotate(int32_t n, const double* rot, const int32_t* sweeps, int32_t nsweeps, bool first, double* Zt,
                             hipStream_t s);
hipError_t launch_fit_back(int32_t n, int32_t m, const double* Zt, const int32_t* ord, const double* V, const double* tau,
                           double* vec, hipStream_t s);
hipError_t launch_fit_chol(int32_t n, double* G, double* L, uint32_t* bad, hipStream_t s);
hipError_t launch_fit_solve(int32_t n, int32_t r, const double* L, const double* vec, const double* sv, double* ca,
                            double* cb, hipStream_t s);
hipError_t launch_fill_u32(uint32_t* p, size_t words, uint32_t value, hipStream_t s);

}  // namespace spice
