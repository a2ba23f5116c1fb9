// Grouped expert GEMMs for many tokens (prefill and large decode batches), bf16 activations:
// the SwiGLU FFN of Eq. 6 over every HIT expert's bucket and over all tokens for the shared
// block (Sec. 2.1, 4.2), and the LoRE correction of Eq. 9 over every LORE bucket.
//
//   up   : H[pos][f] = silu(sum_k W1[f][k] x[k]) * (sum_k W3[f][k] x[k])   (bf16 out)
//          U[pos][q] = sum_k A[q][k] x[k]                                  (fp32 out)
//   down : Y[pos][j] = sum_k W2[j][k] H[pos][k]                            (fp32 out)
//          D[pos][j] = sum_q B[j][q] U[pos][q]     (fp32 MFMA: U is not rounded; fp32 out)
//
// A block computes a tile of BM weight rows x BT tokens over the whole contraction, 64 k per
// stage (v_mfma_f32_16x16x32_bf16, weights as the A operand, tokens as B).  For `up` the rows
// are BM / 2 W1 rows and the same W3 rows, so a wave holds the gate and up sums of its
// features and applies SwiGLU in registers.  A wave's token sub-tiles are interleaved with the
// other waves' (rows kTStride t + 16 wt), so the ragged last tile of an expert spreads over
// the SIMDs; sub-tiles without a live token are not read and issue no MFMA, and their rows are
// not fetched.
//
// Staging: buffer loads straight to LDS (no staging registers) into a ring of S stages of
// 128-byte rows whose 16-byte chunks are XOR-swizzled by row (chunk c of row r at
// c ^ ((r >> 1) & 7)): free of bank conflicts for the fragment reads and the DMA writes.  A
// chunk past the end of a row, and a row past the end of a matrix or a bucket, reads zero (an
// offset past the buffer), so no size has to be a multiple of the tile.
// Pipeline: the fragments of a stage's two k-steps are read half a stage ahead of their MFMAs,
// so a wave reads LDS while its MFMAs run; one barrier per stage, in the middle of the MFMAs,
// frees the buffer just read for the stage S ahead.
// MXFP4 HIT experts: the codes are staged as they are (a quarter of the bytes) and decoded
// after the read from LDS, once per wave and tile instead of once per 16 tokens as in the
// streaming tiles: DeepSeek-V2-Lite sizes, all resident, T = 777 693 -> 229 us per call; Qwen2
// sizes T = 1000 5609 -> 1116.
// What bounds it: with short buckets, the weight stream from HBM (bytes in flight: S - 1 stages
// per block), with long ones the MFMAs (1030 TFLOP/s at Qwen2 sizes, T = 4096).  Against
// one 256 x 256 two-stage shape for every T, with 32 or more tokens per pass of the streaming
// tiles below T = 256 and separate LoRE launches (us per layer call): DeepSeek-V2-Lite sizes
// with 48 experts resident T = 64 202 -> 185, T = 192 261 -> 207, T = 300 347 -> 220, with 32
// T = 1000 360 -> 245, T = 2000 514 -> 368; Qwen2 sizes, all resident, skewed, T = 96 1062 -> 707,
// T = 300 1310 -> 911 (its shared block split), T = 1000 1700 -> 1429, T = 4096 3743 -> 3490.
// Tiles: the shared block first, then the HIT experts in id order, then the LORE buckets.  In the
// bf16 shapes with one block per CU (Deep, Wide, Big) the reverse: a LORE tile lasts as long as any
// other (its loads' latency, 27 - 36 us at d = 2048) and was the launch's tail on a fifth of the
// CUs, and the shared tiles, which L2 feeds, fill the CUs that the last HIT tiles leave
// (T = 1000 of DeepSeek-V2-Lite 6 % of the call, T = 2000 and Qwen2's T = 4096 1 %).  With two blocks
// per CU, or MXFP4 tiles, whose weights stream at a lower rate, the shared block first is the
// better (3 % at T = 300, MXFP4 4 % at T = 777).  Deep launches have a CU for every tile.
// Inside a group the token tiles of one weight tile are consecutive (the weight tile is then
// served from L2), and consecutive tiles are kept on one XCD.
#include <hip/hip_runtime.h>

#include <algorithm>

#include "mx_decode.h"
#include "spice_internal.h"

namespace spice {
namespace {

// Tile shapes: BM weight rows x BT tokens, a grid of WF x WT waves, S stages in LDS, W waves
// per SIMD the register budget targets, L waves that issue the stages' loads.  Of the big tiles'
// eight waves four load, one per SIMD, so the others' MFMAs never wait behind the load queue
// (Qwen2, T = 4096, Big: 3.5 %; T = 1000 of DeepSeek-V2-Lite, Wide: 1 %).  Deep is Small's rows halved
// with eight stages in flight, for up launches of at most a tile per CU (a draft rollout's shared
// block and LoRE factors): there a tile waits for its own loads, not for the memory's rate (T = 64:
// 18.6 -> 14.0 us).  Measured beside them and slower over their ranges: 128 x 128 (2 or 4 stages),
// 64 x 64 with three stages, 128 x 32 and 256 x 64 tiles.
template <int BM_, int BT_, int WF_, int WT_, int S_, int W_, int L_>
struct Shape {
    static constexpr int BM = BM_, BT = BT_, WF = WF_, WT = WT_, S = S_, W = W_;
    static constexpr int kThreads = 64 * WF * WT;
    static constexpr int kLoaders = 64 * L_;
    static constexpr int RF = BM / WF / 16;      // 16-row sub-tiles per wave
    static constexpr int RT = BT / WT / 16;      // 16-token sub-tiles per wave
    static constexpr int kTStride = 16 * WT;     // tile rows between a wave's token sub-tiles
    static constexpr int kUpFeat = BM / 2;       // features of an up tile (W1 rows = W3 rows)
    static constexpr int kWTile = BM * 128;      // bytes of a stage's weight rows
    static constexpr int kStage = (BM + BT) * 128;
    static constexpr int kRowStep = kLoaders / 8;  // rows one load instruction of the loaders covers
    static constexpr int kWLoads = BM / kRowStep, kXLoads = BT / kRowStep;
    static constexpr bool kOnePerCu = 2 * S * kStage > 163840;
    static constexpr int kXcdBlocks = 32 * std::max(1, 163840 / (S * kStage));  // resident blocks per XCD
    // MXFP4 HIT tiles: 128 k per stage, 64 code bytes and 4 scale bytes per weight row and 256
    // bytes per token row; every wave loads
    static constexpr int kWaves = WF * WT;
    static constexpr int kMxCodes = BM * 64, kMxScales = BM * 4;
    static constexpr int kMxStage = kMxCodes + BT * 256 + kMxScales;
    static constexpr int kMxWLoads = BM / (16 * kWaves), kMxXLoads = BT / (4 * kWaves);  // + 1 of scales
    static constexpr int kLds = S * std::max(kStage, kMxStage);
    // whole load instructions of whole rows: the shape can take MXFP4 tiles
    static constexpr bool kMxOk = kMxWLoads * 16 * kWaves == BM && kMxXLoads * 4 * kWaves == BT &&
                                  kUpFeat % (16 * kWaves) == 0 && (4 * kWaves) % 16 == 0 && BM % 64 == 0 &&
                                  kWaves % (BM / 64) == 0 && kUpFeat % 64 == 0;
    static_assert(kRowStep % 16 == 0 && kUpFeat % kRowStep == 0, "staged rows keep their swizzle");
    static_assert(BM % kRowStep == 0 && BT % kRowStep == 0, "whole load instructions");
    static_assert((S - 2) * (kWLoads + kXLoads) < 64, "vmcnt holds the loads in flight");
};
using Big = Shape<256, 256, 2, 4, 2, 2, 4>;
using Wide = Shape<256, 128, 4, 2, 3, 2, 4>;
using Small = Shape<128, 64, 2, 2, 3, 2, 4>;
using Deep = Shape<64, 64, 2, 2, 8, 2, 4>;
static_assert(Big::BM == kGemmBigTile[0] && Big::BT == kGemmBigTile[1] && Wide::BM == kGemmWideTile[0] &&
                  Wide::BT == kGemmWideTile[1] && Small::BM == kGemmSmallTile[0] && Small::BT == kGemmSmallTile[1],
              "the shapes' tiles as the split rule knows them");

constexpr int kBK = 64;                          // contraction per stage
constexpr int kLoreDown = 4;                     // BM-row blocks of a LORE down tile (short: r is small)
constexpr uint32_t kOutOfRange = 0xFFFFFFF0u;    // an offset past every buffer
constexpr long long kMaxBuffer = 0xFFFF0000ll;   // bytes a buffer may hold
constexpr int kRawBufferWord3 = 0x00020000;      // gfx9 raw buffer: 32-bit data format

typedef __bf16 bf16x8_t __attribute__((ext_vector_type(8)));
typedef float f32x4_t __attribute__((ext_vector_type(4)));

__device__ __forceinline__ uint32_t bf16_rne(float f) {
    const uint32_t u = __float_as_uint(f);
    if ((u & 0x7FFFFFFFu) > 0x7F800000u) return 0x7FC0u;
    return (u + 0x7FFFu + ((u >> 16) & 1u)) >> 16;
}

__device__ __forceinline__ float silu(float u) { return u / (1.0f + __expf(-u)); }

// Logical tile of block b.  The hardware deals blocks to the 8 XCDs round robin (block b to
// XCD b % 8).  Here every round of 8 x per_xcd blocks gives each XCD per_xcd consecutive
// logical tiles (neighbouring tiles share operands in that XCD's L2), and the rounds
// alternate over all XCDs so that long tiles at the front of the order spread over the whole
// chip.  A final partial round keeps block order; the map is a bijection on [0, G).
__device__ __forceinline__ int xcd_tile(int b, int G, int per_xcd) {
    const int round = 8 * per_xcd;
    if (b >= (G / round) * round) return b;
    const int x = b & 7, slot = b >> 3;
    return (slot / per_xcd) * round + x * per_xcd + slot % per_xcd;
}

enum : int { kTileHit = 0, kTileShared = 1, kTileLore = 2 };

struct TileJob {
    int kind;
    const void* w;        // weight matrix of the group (W13, W2, A or B of one expert)
    uint32_t w_bytes;     // its size
    int kdim;             // contraction length
    int nfeat;            // output features of the group
    int up_off;           // up: rows from a tile row of the first half to its partner of the second
    int row0;             // first weight row (= output feature) of the tile
    int k0, k1;           // stages of the contraction this tile takes (all, but for a split shared block)
    int part;             // which of the shared block's partial results it is
    int tok0, ntok;       // tile's first token of the group / token count of the group
    int start;            // group's first bucket position (0 for the shared block)
};

// The bucket of class c holding tile L of nt tiles per token tile, found by a wave's scan of
// the offsets; L is reduced by the class's tiles when it lies past them.
__device__ bool scan_class(const GemmArgs& a, int c, int nt, int BT, int& L, int lane, int& e_, int& st_, int& n_,
                           int& slot_) {
    const int32_t* off = a.offsets + c * (a.N + 1);
    for (int e0 = 0; e0 < a.N; e0 += 64) {
        const int e = e0 + lane;
        int st = 0, n = 0, slot = -1;
        if (e < a.N) {
            st = off[e];
            n = off[e + 1] - st;
            if (c == SPICE_CLASS_HIT) slot = a.resident_slot[e];
        }
        const int tiles = n > 0 ? ((n + BT - 1) / BT) * nt : 0;
        int incl = tiles;
#pragma unroll
        for (int o = 1; o < 64; o <<= 1) {
            const int up = __shfl_up(incl, o);
            if (lane >= o) incl += up;
        }
        const int excl = incl - tiles;
        const unsigned long long bal = __ballot(tiles > 0 && L >= excl && L < incl);
        if (bal) {
            const int src = __builtin_amdgcn_readfirstlane(__ffsll((long long)bal) - 1);
            e_ = e0 + src;
            st_ = __builtin_amdgcn_readlane(st, src);
            n_ = __builtin_amdgcn_readlane(n, src);
            slot_ = __builtin_amdgcn_readlane(slot, src);
            L -= __builtin_amdgcn_readlane(excl, src);
            return true;
        }
        L -= __builtin_amdgcn_readlane(incl, 63);
    }
    return false;
}

// Resolve logical tile L of a launch; every wave does it for itself (uniform values).
// Returns false for tiles past the live work.
template <bool kUp, bool kMx, class C>
__device__ bool resolve(const GemmArgs& a, int L, TileJob& j) {
    const int lane = threadIdx.x & 63;
    constexpr int feat = kUp ? C::kUpFeat : C::BM;
    const int d = a.d, I = a.I, Is = a.Is;
    const int nt_sh = ((kUp ? Is : d) + feat - 1) / feat;  // weight tiles of the shared block
    const int nt_e = ((kUp ? I : d) + feat - 1) / feat;    // of a routed expert
    constexpr int lrows = kUp ? C::BM : C::BM * kLoreDown;
    const int nt_l = ((kUp ? a.r : d) + lrows - 1) / lrows;  // of a LORE expert
    const int mt_sh = (a.T + C::BT - 1) / C::BT;
    const int parts = kUp ? 1 : a.parts, per_part = nt_sh * mt_sh;
    const int tiles_sh = Is > 0 ? per_part * parts : 0;
    j.k0 = 0;
    j.part = 0;
    auto shared_tile = [&](int L) {
        j.part = L / per_part;
        L -= j.part * per_part;
        // groups of sn weight tiles x sm token tiles (about one XCD's worth of blocks)
        // run together and share their operand tiles in that XCD's L2
        const int sn = kUp ? a.super_up[0] : a.super_dn[0], sm = kUp ? a.super_up[1] : a.super_dn[1];
        const int g = L / (sn * sm), in = L - g * (sn * sm);
        const int mg = mt_sh / sm;
        const int n = (g / mg) * sn + in / sm;
        const int m = (g % mg) * sm + in % sm;
        j.kind = kTileShared;
        j.w = kUp ? a.w13s : a.w2s;
        j.w_bytes = (uint32_t)(kUp ? 2 : 1) * (uint32_t)Is * (uint32_t)d * 2u;
        j.kdim = kUp ? d : Is;
        const int nk = (j.kdim + kBK - 1) / kBK;
        j.k0 = j.part * nk / parts;
        j.k1 = (j.part + 1) * nk / parts;
        j.nfeat = kUp ? Is : d;
        j.up_off = Is;
        j.row0 = n * feat;
        j.tok0 = m * C::BT;
        j.ntok = a.T;
        j.start = 0;
        return true;
    };
    constexpr bool kSharedLast = !kMx && C::kOnePerCu;
    if constexpr (!kSharedLast) {
        if (L < tiles_sh) return shared_tile(L);
        L -= tiles_sh;
    }
    int e = 0, st = 0, n = 0, slot = -1;
    int kind = kTileHit, nt = nt_e;
    auto find_lore = [&]() {
        if (a.r <= 0 || !scan_class(a, SPICE_CLASS_LORE, nt_l, C::BT, L, lane, e, st, n, slot)) return false;
        kind = kTileLore;
        nt = nt_l;
        return true;
    };
    bool found = kSharedLast && find_lore();
    if (!found) found = a.do_hit && a.C > 0 && scan_class(a, SPICE_CLASS_HIT, nt_e, C::BT, L, lane, e, st, n, slot);
    if (!found && !kSharedLast) found = find_lore();
    if (!found) return kSharedLast && L < tiles_sh && shared_tile(L);
    if (st < 0 || n <= 0 || st + n > a.T * a.K) {
        if (threadIdx.x == 0) atomicOr(&a.ctrl[kWordFlags], (uint32_t)SPICE_FLAG_BAD_INDEX);
        return false;
    }
    const int mt = (n + C::BT - 1) / C::BT;
    const int nn = L / mt, m = L - nn * mt;
    j.kind = kind;
    j.tok0 = m * C::BT;
    j.ntok = n;
    j.start = st;
    if (kind == kTileHit) {
        if (slot < 0 || slot >= a.C) {
            if (threadIdx.x == 0) atomicOr(&a.ctrl[kWordFlags], (uint32_t)SPICE_FLAG_BAD_SLOT);
            return false;
        }
        // bf16 rows, or a blob of MXFP4 codes followed by the block scales
        const size_t elems = (size_t)(kUp ? 2 : 1) * I * d, bytes = kMx ? elems / 2 + elems / 32 : elems * 2;
        j.w = static_cast<const char*>(kUp ? a.w13_pool : a.w2_pool) + slot * bytes;
        j.w_bytes = (uint32_t)(kMx ? elems / 2 : elems * 2);
        j.kdim = kUp ? d : I;
        j.nfeat = kUp ? I : d;
        j.up_off = I;
        j.row0 = nn * feat;
    } else {
        j.w = (kUp ? a.lore_A : a.lore_B) + (size_t)e * a.r * d;
        j.w_bytes = (uint32_t)a.r * (uint32_t)d * 2u;
        j.kdim = kUp ? d : a.r;
        j.nfeat = kUp ? a.r : d;
        j.up_off = C::kUpFeat;  // BM consecutive rows of A
        j.row0 = nn * lrows;
    }
    j.k1 = (j.kdim + kBK - 1) / kBK;
    return true;
}

// Byte offset of 16-byte chunk c of staged row r inside an operand tile.
__device__ __forceinline__ uint32_t lds_off(int r, int c) {
    return (uint32_t)(r * 128 + ((c ^ ((r >> 1) & 7)) << 4));
}

typedef __amdgpu_buffer_rsrc_t rsrc_t;
__device__ __forceinline__ rsrc_t raw_buffer(const void* p, uint32_t bytes) {
    return __builtin_amdgcn_make_buffer_rsrc(const_cast<void*>(p), 0, (int)bytes, kRawBufferWord3);
}

// 16 bytes (load_lds4: 4) from offset off of a buffer to LDS byte lds + 16 * lane (4 *), lds uniform over the wave
// (counted by vmcnt, not lgkmcnt; an offset past the buffer writes zeros).  Device pass only:
// the host pass of a kernel naming this target builtin would lose its launch stub.
__device__ __forceinline__ void load_lds16(rsrc_t b, uint32_t off, unsigned char* lds) {
#if defined(__HIP_DEVICE_COMPILE__)
    __builtin_amdgcn_raw_ptr_buffer_load_lds(b, (__attribute__((address_space(3))) void*)lds, 16, (int)off, 0, 0, 0);
#endif
}

__device__ __forceinline__ void load_lds4(rsrc_t b, uint32_t off, unsigned char* lds) {
#if defined(__HIP_DEVICE_COMPILE__)
    __builtin_amdgcn_raw_ptr_buffer_load_lds(b, (__attribute__((address_space(3))) void*)lds, 4, (int)off, 0, 0, 0);
#endif
}

// s_waitcnt with vmcnt(n) lgkmcnt(0), then the block's barrier: no wait for loads to LDS
// beyond those the caller names (a __syncthreads would drain them all).
template <int n>
__device__ __forceinline__ void wait_and_barrier() {
    asm volatile("" ::: "memory");
    __builtin_amdgcn_s_waitcnt((n & 15) | ((n >> 4) << 14) | 0x70);
    __builtin_amdgcn_s_barrier();
    asm volatile("" ::: "memory");
}

// Fragments of one 32-k step: RF weight sub-tiles and the NL live token sub-tiles.
template <class C, int NL>
struct Frags {
    u32x4_t a[C::RF], b[NL];
};

// The bf16 main loop of one tile with NL live token sub-tiles in this wave (NL = 0: the wave
// only loads and keeps the barriers).
template <class C, bool kUp, int NL, class Load>
__device__ __forceinline__ void product(unsigned char* s_lds, int nk, uint32_t fbase, uint32_t tbase, Load load,
                                        f32x4_t (&acc)[C::RF][C::RT]) {
    constexpr int N1 = NL > 0 ? NL : 1;
    constexpr int kLoads = (C::S - 2) * (C::kWLoads + C::kXLoads);  // stages in flight past the next one
    auto read = [&](int buf, uint32_t kx, Frags<C, N1>& f) {
        if constexpr (NL > 0) {
            const unsigned char* base = s_lds + buf * C::kStage;
#pragma unroll
            for (int t = 0; t < NL; ++t)
                f.b[t] = *reinterpret_cast<const u32x4_t*>(base + ((tbase + t * C::kTStride * 128) ^ kx));
#pragma unroll
            for (int s = 0; s < C::RF; ++s) {
                const int row = kUp ? (s % (C::RF / 2)) * 16 + (s / (C::RF / 2)) * C::kUpFeat : s * 16;
                f.a[s] = *reinterpret_cast<const u32x4_t*>(base + ((fbase + row * 128) ^ kx));
            }
        }
    };
    auto mma = [&](const Frags<C, N1>& f) {
        if constexpr (NL > 0) {
            __builtin_amdgcn_s_setprio(1);  // favour the wave that is issuing MFMAs
#pragma unroll
            for (int t = 0; t < NL; ++t)
#pragma unroll
                for (int s = 0; s < C::RF; ++s)
                    acc[s][t] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8_t, f.a[s]),
                                                                        __builtin_bit_cast(bf16x8_t, f.b[t]),
                                                                        acc[s][t], 0, 0, 0);
            __builtin_amdgcn_s_setprio(0);
        }
    };
    wait_and_barrier<kLoads + C::kWLoads + C::kXLoads>();  // stage 0 of the S in flight has landed
    Frags<C, N1> f0, f1;
    read(0, 0u, f0);
    int buf = 0;
    for (int kt = 0; kt < nk; ++kt) {
        read(buf, 64u, f1);
        __builtin_amdgcn_sched_barrier(0);
        mma(f0);
        __builtin_amdgcn_sched_barrier(0);
        // stage kt + 1 has landed and every wave has read all of stage kt
        wait_and_barrier<kLoads>();
        load(buf, kt + C::S);
        buf = buf + 1 == C::S ? 0 : buf + 1;
        read(buf, 0u, f0);  // past the last stage: zeros, unused
        __builtin_amdgcn_sched_barrier(0);
        mma(f1);
        __builtin_amdgcn_sched_barrier(0);
    }
    __builtin_amdgcn_s_waitcnt(0x70);  // no load to LDS outlives the block
}

// The main loop of a HIT tile with MXFP4 weights: 128 k per stage.  A lane's 16 code bytes of a
// row are one block of 32 elements, decoded to the A operands of 4 MFMA steps (v_cvt_scalef32,
// exact) after they are read from LDS; step u takes elements 8 u .. 8 u + 7 of the lane's block,
// and the token operand reads the same k (chunk 4 quad + u of its 256-byte row).  load(buf, kt, l)
// issues the l-th load of a stage: a wave's own loads go out between its MFMAs, not in one run
// before its fragment reads, where the MFMAs waited for the load queue (T = 777 of
// DeepSeek-V2-Lite: 5 % of the call; the bf16 loop, whose stages hold four times the
// weight bytes, gains nothing from it).  Reading half a stage ahead, as product() does, gave
// nothing here.
template <class C, bool kUp, int NL, class Load>
__device__ __forceinline__ void mx_product(unsigned char* s_lds, int nk, int frow0, int wt, Load load,
                                           f32x4_t (&acc)[C::RF][C::RT]) {
    constexpr int kPer = C::kMxWLoads + C::kMxXLoads + 1, kLoads = (C::S - 2) * kPer;
    const int lane = threadIdx.x & 63, m = lane & 15, quad = lane >> 4;
    const uint32_t cbase = (uint32_t)((frow0 + m) * 64 + ((quad ^ ((m >> 2) & 3)) << 4));
    const uint32_t tbase = (uint32_t)(C::kMxCodes + (wt * 16 + m) * 256 + (((4 * quad) ^ m) << 4));
    const uint32_t sbase = (uint32_t)(C::kMxCodes + C::BT * 256 + (frow0 + m) * 4 + quad);
#pragma unroll
    for (int s = 0; s < C::S - 1; ++s)
#pragma unroll
        for (int l = 0; l < kPer; ++l) load(s, s, l);
    int buf = 0;
    for (int kt = 0; kt < nk; ++kt) {
        // stage kt has landed and every wave has read all of stage kt - 1
        wait_and_barrier<kLoads>();
        const int freed = buf == 0 ? C::S - 1 : buf - 1;
        if constexpr (NL == 0) {
#pragma unroll
            for (int l = 0; l < kPer; ++l) load(freed, kt + C::S - 1, l);
        } else {
            const unsigned char* base = s_lds + buf * C::kMxStage;
            u32x4_t b[NL][4], raw[C::RF];
            uint32_t sc[C::RF];
#pragma unroll
            for (int s = 0; s < C::RF; ++s) {
                const int row = kUp ? (s % (C::RF / 2)) * 16 + (s / (C::RF / 2)) * C::kUpFeat : s * 16;
                raw[s] = *reinterpret_cast<const u32x4_t*>(base + cbase + row * 64);
                sc[s] = base[sbase + row * 4];
            }
#pragma unroll
            for (int t = 0; t < NL; ++t)
#pragma unroll
                for (int u = 0; u < 4; ++u)
                    b[t][u] = *reinterpret_cast<const u32x4_t*>(base + ((tbase + t * C::kTStride * 256) ^ (u << 4)));
            __builtin_amdgcn_sched_barrier(0);
            __builtin_amdgcn_s_setprio(1);
#pragma unroll
            for (int s = 0; s < C::RF; ++s) {
                u32x4_t op[4];
                mx_decode(raw[s], e8m0(sc[s]), op);
#pragma unroll
                for (int u = 0; u < 4; ++u) {
#pragma unroll
                    for (int l = 0; l < kPer; ++l)
                        if (l * 4 * C::RF / kPer == 4 * s + u) {
                            __builtin_amdgcn_sched_barrier(0);
                            load(freed, kt + C::S - 1, l);
                            __builtin_amdgcn_sched_barrier(0);
                        }
#pragma unroll
                    for (int t = 0; t < NL; ++t)
                        acc[s][t] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8_t, op[u]),
                                                                            __builtin_bit_cast(bf16x8_t, b[t][u]),
                                                                            acc[s][t], 0, 0, 0);
                }
            }
            __builtin_amdgcn_s_setprio(0);
            __builtin_amdgcn_sched_barrier(0);
        }
        buf = buf + 1 == C::S ? 0 : buf + 1;
    }
    __builtin_amdgcn_s_waitcnt(0x70);  // no load to LDS outlives the block
}

// Row of x of a tile row: the token itself (shared block) or that of slot s of the bucket
// (row 0 and a flag for a slot out of range).
__device__ __forceinline__ int token_row(const GemmArgs& a, const TileJob& j, int s) {
    if (j.kind == kTileShared) return s;
    if (s < 0 || s >= a.T * a.K) {
        atomicOr(&a.ctrl[kWordFlags], (uint32_t)SPICE_FLAG_BAD_INDEX);
        return 0;
    }
    return s / a.K;
}

// D = U B_e^T of BM rows of B_e x BT bucket entries (a LORE tile takes kLoreDown such blocks:
// one alone is shorter than the block's start; draft rollout, T = 64: 17.8 -> 12.7 us), contraction
// r.  fp32 MFMAs
// (16x16x4), so that U keeps its 32 bits; operands straight from L2, whose reuse is within the
// block.  A 32-k step gives each lane 8 consecutive k of its row (quad), and MFMA i takes
// element i of every lane; the next step's loads are out before this one's MFMAs.  Rows past d
// and entries past the bucket read the last one.
template <class C>
__device__ __forceinline__ void lore_down(const GemmArgs& a, const TileJob& j) {
    const int lane = threadIdx.x & 63, m = lane & 15, quad = lane >> 4;
    const int w = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int wf = w % C::WF, wt = w / C::WF;
    const int nlive = min(C::RT, max(0, (j.ntok - j.tok0 - 16 * wt + C::kTStride - 1) / C::kTStride));
    if (nlive == 0) return;
    const uint16_t* B = static_cast<const uint16_t*>(j.w);
    f32x4_t acc[C::RF][C::RT];
#pragma unroll
    for (int s = 0; s < C::RF; ++s)
#pragma unroll
        for (int t = 0; t < C::RT; ++t) acc[s][t] = f32x4_t{0.f, 0.f, 0.f, 0.f};
    const uint16_t* brow[C::RF];
    const float* urow[C::RT];
#pragma unroll
    for (int s = 0; s < C::RF; ++s)
        brow[s] = B + (size_t)min(j.row0 + wf * (C::BM / C::WF) + s * 16 + m, a.d - 1) * a.r;
#pragma unroll
    for (int t = 0; t < C::RT; ++t)
        urow[t] = a.u + (size_t)(j.start + min(j.tok0 + t * C::kTStride + wt * 16 + m, j.ntok - 1)) * a.r;
    struct Step {
        u32x4_t b[C::RF];
        f32x4_t u[C::RT][2];
    };
    auto fetch = [&](int k0, Step& st) {
        const int k = k0 + quad * 8;
        const bool in = k < a.r;  // r is a multiple of 8
#pragma unroll
        for (int s = 0; s < C::RF; ++s)
            st.b[s] = in ? *reinterpret_cast<const u32x4_t*>(brow[s] + k) : u32x4_t{0u, 0u, 0u, 0u};
#pragma unroll
        for (int t = 0; t < C::RT; ++t)
#pragma unroll
            for (int h = 0; h < 2; ++h)
                st.u[t][h] = in && t < nlive ? *reinterpret_cast<const f32x4_t*>(urow[t] + k + 4 * h)
                                             : f32x4_t{0.f, 0.f, 0.f, 0.f};
    };
    auto mul = [&](const Step& st) {
#pragma unroll
        for (int s = 0; s < C::RF; ++s) {
#pragma unroll
            for (int i = 0; i < 8; ++i) {
                const uint32_t v = st.b[s][i >> 1];
                const float av = __uint_as_float(i & 1 ? v & 0xFFFF0000u : v << 16);
#pragma unroll
                for (int t = 0; t < C::RT; ++t)
                    if (t < nlive)
                        acc[s][t] = __builtin_amdgcn_mfma_f32_16x16x4f32(av, st.u[t][i >> 2][i & 3], acc[s][t], 0, 0, 0);
            }
        }
    };
    Step cur, nxt;
    fetch(0, cur);
    for (int k0 = 0; k0 < a.r; k0 += 32) {
        if (k0 + 32 < a.r) fetch(k0 + 32, nxt);
        mul(cur);
        cur = nxt;
    }
#pragma unroll
    for (int t = 0; t < C::RT; ++t) {
        const int pos = j.tok0 + t * C::kTStride + wt * 16 + m;
        if (pos >= j.ntok) continue;
        float* dst = a.y_slots + (size_t)(j.start + pos) * a.d;
#pragma unroll
        for (int s = 0; s < C::RF; ++s) {
            const int f = j.row0 + wf * (C::BM / C::WF) + s * 16 + quad * 4;
            if (f < a.d) *reinterpret_cast<f32x4_t*>(dst + f) = acc[s][t];
        }
    }
}

template <bool kUp, bool kMx, class C>
__global__ __launch_bounds__(C::kThreads) __attribute__((amdgpu_waves_per_eu(C::W))) void expert_gemm_kernel(GemmArgs a) {
    static_assert(!kMx || C::kMxOk, "MXFP4 tiles need whole load instructions");
    extern __shared__ __align__(16) unsigned char s_lds[];
    TileJob j;
    if (!resolve<kUp, kMx, C>(a, xcd_tile(blockIdx.x, gridDim.x, C::kXcdBlocks), j)) return;
    if constexpr (!kUp) {
        if (j.kind == kTileLore) {
            for (int b = 0; b < kLoreDown && j.row0 < a.d; ++b, j.row0 += C::BM) lore_down<C>(a, j);
            return;
        }
    }

    const int tid = threadIdx.x, lane = tid & 63;
    const int w = __builtin_amdgcn_readfirstlane(tid >> 6);
    // wave's feature part and token lane group
    const int wf = w % C::WF, wt = w / C::WF;
    const int m = lane & 15, quad = lane >> 4;

    const int S = j.kind == kTileShared ? a.T : a.T * a.K;  // rows of the activations behind the tile
    const int frow0 = wf * ((kUp ? C::kUpFeat : C::BM) / C::WF);
    // token sub-tiles of this wave with a live row
    const int nlive = min(C::RT, max(0, (j.ntok - j.tok0 - 16 * wt + C::kTStride - 1) / C::kTStride));
    f32x4_t acc[C::RF][C::RT];
#pragma unroll
    for (int s = 0; s < C::RF; ++s)
#pragma unroll
        for (int t = 0; t < C::RT; ++t) acc[s][t] = f32x4_t{0.f, 0.f, 0.f, 0.f};

    if (kMx && j.kind == kTileHit) {
        // Staging of an MXFP4 tile.  A wave's load of codes covers 16 rows of four 16-byte chunks
        // (chunk c of row r at c ^ ((r >> 2) & 3)), of tokens 4 rows of 16 chunks (at c ^ (r & 15)),
        // of scales the dword (4 blocks) of 64 rows: all free of bank conflicts.  Waves past the
        // scales' rows load the same ones again, so that every wave counts the same loads.
        const uint32_t rb = (uint32_t)j.kdim / 2, sb = (uint32_t)j.kdim / 32;
        const int cr = w * 16 + (lane >> 2), cc = (lane & 3) ^ ((lane >> 4) & 3);
        const int tr = w * 4 + (lane >> 4), tc = (lane & 15) ^ (tr & 15);
        const int sr = (w % (C::BM / 64)) * 64 + lane;
        const rsrc_t cbuf = raw_buffer(j.w, j.w_bytes);
        const rsrc_t sbuf = raw_buffer(static_cast<const char*>(j.w) + j.w_bytes, j.w_bytes / 16);
        const rsrc_t xbuf = kUp ? raw_buffer(a.x, (uint32_t)a.T * (uint32_t)a.d * 2u)
                                : raw_buffer(a.h, (uint32_t)S * (uint32_t)j.kdim * 2u);
        auto wrow = [&](int r) { return (uint32_t)(j.row0 + (kUp && r >= C::kUpFeat ? j.up_off + r - C::kUpFeat : r)); };
        const uint32_t soff = wrow(sr) * sb;
        const uint32_t xstep = kUp ? 256u : (uint32_t)S * 256u;
        uint32_t xoff[C::kMxXLoads];
#pragma unroll
        for (int i = 0; i < C::kMxXLoads; ++i) {
            const int pos = j.tok0 + tr + 4 * C::kWaves * i;
            xoff[i] = kOutOfRange;
            if (pos < j.ntok)
                xoff[i] = kUp ? (uint32_t)token_row(a, j, a.perm[j.start + pos]) * (uint32_t)a.d * 2u + tc * 16
                              : ((uint32_t)(tc >> 3) * (uint32_t)S + (uint32_t)(j.start + pos)) * 128u + (tc & 7) * 16;
        }
        const int nk = j.kdim / 128;
        auto load = [&](int buf, int kt, int l) {
            unsigned char* st = s_lds + buf * C::kMxStage;
            const bool in = kt < nk;
            if (l < C::kMxWLoads) {
                load_lds16(cbuf, in ? wrow(cr + 16 * C::kWaves * l) * rb + (uint32_t)kt * 64u + cc * 16 : kOutOfRange,
                           st + (w + C::kWaves * l) * 1024);
            } else if (l < C::kMxWLoads + C::kMxXLoads) {
                const int i = l - C::kMxWLoads;
                load_lds16(xbuf, in && xoff[i] != kOutOfRange ? xoff[i] + (uint32_t)kt * xstep : kOutOfRange,
                           st + C::kMxCodes + (w + C::kWaves * i) * 1024);
            } else {
                load_lds4(sbuf, in ? soff + (uint32_t)kt * 4u : kOutOfRange,
                          st + C::kMxCodes + C::BT * 256 + (w % (C::BM / 64)) * 256);
            }
        };
        if (nlive == C::RT) mx_product<C, kUp, C::RT>(s_lds, nk, frow0, wt, load, acc);
        else if (nlive == 0) mx_product<C, kUp, 0>(s_lds, nk, frow0, wt, load, acc);
        else if (nlive == 1) mx_product<C, kUp, 1>(s_lds, nk, frow0, wt, load, acc);
        else if constexpr (C::RT > 2) {
            if (nlive == 2) mx_product<C, kUp, 2>(s_lds, nk, frow0, wt, load, acc);
            else mx_product<C, kUp, 3>(s_lds, nk, frow0, wt, load, acc);
        }
    } else {
    // Staging: a loader wave's load writes 64 x 16 bytes to consecutive LDS, 8 staged rows of 8
    // chunks.  Lane l fills LDS chunk l % 8 of row r0 = tid / 8 (+ kRowStep i), which holds the
    // row's chunk (l % 8) ^ swizzle(row), so that is the chunk it fetches.
    const int r0 = tid / 8;
    const bool loader = C::kLoaders == C::kThreads || tid < C::kLoaders;
    const int c16 = (int)((lds_off(r0, tid & 7) & 127u) >> 4);
    const rsrc_t wbuf = raw_buffer(j.w, j.w_bytes);
    const rsrc_t xbuf = kUp ? raw_buffer(a.x, (uint32_t)a.T * (uint32_t)a.d * 2u)
                            : raw_buffer(j.kind == kTileShared ? a.hs : a.h,
                                         (uint32_t)S * (uint32_t)((j.kdim + kBK - 1) / kBK) * (kBK * 2u));
    const uint32_t wstep = (uint32_t)j.kdim * 2u;
    const uint32_t woff0 = (uint32_t)(j.row0 + r0) * wstep + c16 * 16;
    const uint32_t xstep = kUp ? 128u : (uint32_t)S * 128u;  // bytes from one stage to the next
    const int klim = j.kdim - c16 * 8;  // the lane's chunk of stage kt is in the row while 64 kt < klim
    const int nk = j.k1 - j.k0;
    // Weight rows whose stride is a multiple of 2 KiB start on a few memory channels only, and
    // tiles that march through k together queue there: each weight tile starts its k order at
    // another stage (d = 2048, T = 192: 235 -> 217 us a call; at d = 3584, whose rows spread by
    // themselves, the lost sharing in L2 costs 1-2 %).
    const int rot = wstep % 2048 == 0 ? (int)((uint32_t)(j.row0 / C::kUpFeat) * 5u % (uint32_t)nk) : 0;
    // stage kt of the tile's nk; past the last one, a stage past the row
    auto stage_k = [&](int kt) {
        return kt >= nk ? 0x1000000 : j.k0 + (kt + rot >= nk ? kt + rot - nk : kt + rot);
    };
    auto load_w = [&](int buf, int kt) {
        if (!loader) return;
        unsigned char* run = s_lds + buf * C::kStage + w * 1024;
        kt = stage_k(kt);
        const bool in = kt * kBK < klim;
#pragma unroll
        for (int i = 0; i < C::kWLoads; ++i) {
            const int r = C::kRowStep * i;
            const uint32_t delta = (uint32_t)(kUp && r >= C::kUpFeat ? j.up_off + r - C::kUpFeat : r) * wstep;
            load_lds16(wbuf, in ? woff0 + delta + (uint32_t)kt * 128u : kOutOfRange, run + i * C::kRowStep * 128);
        }
    };
    uint32_t xoff[C::kXLoads];
    auto load_x = [&](int buf, int kt) {
        if (!loader) return;
        unsigned char* run = s_lds + buf * C::kStage + w * 1024 + C::kWTile;
        kt = stage_k(kt);
        const bool in = kt * kBK < klim;
#pragma unroll
        for (int i = 0; i < C::kXLoads; ++i)
            load_lds16(xbuf, in && xoff[i] != kOutOfRange ? xoff[i] + (uint32_t)kt * xstep : kOutOfRange,
                       run + i * C::kRowStep * 128);
    };
    auto load = [&](int buf, int kt) {
        load_w(buf, kt);
        load_x(buf, kt);
    };
    // the slot ids of the tile's rows, the weights of stage 0, then (once the ids are there) its
    // token rows and the other stages of the ring
    int sid[C::kXLoads];
#pragma unroll
    for (int i = 0; i < C::kXLoads; ++i) {
        const int pos = j.tok0 + r0 + C::kRowStep * i;
        sid[i] = -1;
        if (loader && pos < j.ntok) sid[i] = (!kUp || j.kind == kTileShared) ? j.start + pos : a.perm[j.start + pos];
    }
    __builtin_amdgcn_sched_barrier(0);
    load_w(0, 0);
    __builtin_amdgcn_sched_barrier(0);
#pragma unroll
    for (int i = 0; i < C::kXLoads; ++i) {
        const int pos = j.tok0 + r0 + C::kRowStep * i;
        xoff[i] = kOutOfRange;
        if (loader && pos < j.ntok)
            xoff[i] = kUp ? (uint32_t)token_row(a, j, sid[i]) * (uint32_t)a.d * 2u + c16 * 16
                          : (uint32_t)sid[i] * 128u + c16 * 16;
    }
    load_x(0, 0);
#pragma unroll
    for (int s = 1; s < C::S; ++s) load(s, s);

    // LDS addresses of the fragments of k-step 0 (k-step 1 reads chunk c ^ 4: bit 6 flipped).
    // The swizzle of row r depends on (r >> 1) & 7, which steps of 16 rows leave unchanged.
    const uint32_t fbase = lds_off(frow0 + m, quad);
    const uint32_t tbase = C::kWTile + lds_off(wt * 16 + m, quad);
    static_assert(C::RT == 2 || C::RT == 4, "token sub-tiles per wave");
    if (nlive == C::RT) product<C, kUp, C::RT>(s_lds, nk, fbase, tbase, load, acc);
    else if (nlive == 0) product<C, kUp, 0>(s_lds, nk, fbase, tbase, load, acc);
    else if (nlive == 1) product<C, kUp, 1>(s_lds, nk, fbase, tbase, load, acc);
    else if constexpr (C::RT > 2) {
        if (nlive == 2) product<C, kUp, 2>(s_lds, nk, fbase, tbase, load, acc);
        else product<C, kUp, 3>(s_lds, nk, fbase, tbase, load, acc);
    }
    }

    // Epilogue: lane holds features 4 quad .. + 3 of sub-tile s for token m of sub-tile t.
#pragma unroll
    for (int t = 0; t < C::RT; ++t) {
        const int pos = j.tok0 + t * C::kTStride + wt * 16 + m;
        if (pos >= j.ntok) continue;
        if constexpr (kUp) {
            if (j.kind == kTileLore) {
                float* dst = a.u + (size_t)(j.start + pos) * a.r;
#pragma unroll
                for (int s = 0; s < C::RF; ++s) {
                    const int q = j.row0 + frow0 + (s % (C::RF / 2)) * 16 + (s / (C::RF / 2)) * C::kUpFeat + quad * 4;
                    if (q < a.r) *reinterpret_cast<f32x4_t*>(dst + q) = acc[s][t];
                }
                continue;
            }
            // intermediates are k-blocked: element (row, f) at ((f / 64) * rows + row) * 64 + f % 64,
            // so a down-projection stage reads its token rows as one contiguous block
            uint16_t* dst = (j.kind == kTileShared ? a.hs : a.h) + (size_t)(j.start + pos) * kBK;
            const size_t fstride = (size_t)S * kBK;
#pragma unroll
            for (int s = 0; s < C::RF / 2; ++s) {
                const f32x4_t g = acc[s][t], u = acc[s + C::RF / 2][t];
                const int f = j.row0 + frow0 + s * 16 + quad * 4;
                uint2 p;
                p.x = bf16_rne(silu(g.x) * u.x) | (bf16_rne(silu(g.y) * u.y) << 16);
                p.y = bf16_rne(silu(g.z) * u.z) | (bf16_rne(silu(g.w) * u.w) << 16);
                if (f < j.nfeat) *reinterpret_cast<uint2*>(dst + (size_t)(f / kBK) * fstride + (f % kBK)) = p;
            }
        } else {
            const bool shared = j.kind == kTileShared, split = shared && a.parts > 1;
            float* dst = split ? a.part + ((size_t)j.part * a.T + pos) * a.d
                               : (shared ? a.y_shared : a.y_slots) + (size_t)(j.start + pos) * a.d;
            const float gs = (shared && a.sgate && !split) ? a.sgate[pos] : 1.0f;  // gated shared block
#pragma unroll
            for (int s = 0; s < C::RF; ++s) {
                const int f = j.row0 + frow0 + s * 16 + quad * 4;
                if (f < a.d) *reinterpret_cast<f32x4_t*>(dst + f) = acc[s][t] * gs;
            }
        }
    }
}

// y_shared = the sum of the shared block's partial results, in order, times the gate: 4
// features of one token per thread.
__global__ __launch_bounds__(256) void shared_sum_kernel(int T, int d, int parts, const float* part, const float* sgate,
                                                         float* y) {
    const int f = (blockIdx.x * 256 + threadIdx.x) * 4, t = blockIdx.y;
    if (f >= d) return;
    const size_t at = (size_t)t * d + f, step = (size_t)T * d;
    f32x4_t v[kMaxSharedParts];
#pragma unroll
    for (int p = 0; p < kMaxSharedParts; ++p)
        if (p < parts) v[p] = *reinterpret_cast<const f32x4_t*>(part + p * step + at);
    f32x4_t sum = v[0];
#pragma unroll
    for (int p = 1; p < kMaxSharedParts; ++p)
        if (p < parts) sum += v[p];
    if (sgate) sum *= sgate[t];
    *reinterpret_cast<f32x4_t*>(y + at) = sum;
}

// Super-tile of the shared block: sn weight tiles x sm token tiles with sn | nt and
// sm | mt, at most one XCD's resident blocks, as square as possible (the bytes a group
// fetches per stage are proportional to sn + sm).
void super_shape(int mt, int nt, int most, int* out) {
    int best_n = 1, best_m = 1, best_score = -1;
    for (int sm = 1; sm <= mt && sm <= most; ++sm) {
        if (mt % sm) continue;
        for (int sn = 1; sn <= nt && sn * sm <= most; ++sn) {
            if (nt % sn) continue;
            // more blocks per group first, then fewer distinct tiles per block
            const int score = sn * sm * 64 - (sn + sm);
            if (score > best_score) { best_score = score; best_n = sn; best_m = sm; }
        }
    }
    out[0] = best_n;
    out[1] = best_m;
}

long long tiles_of(int n, int per) { return ((long long)n + per - 1) / per; }

// Upper bound of a launch's tiles in shape C: sum_e ceil(n_e / BT) <= slots / BT + buckets, the
// slots of both classes together at most T K; blocks past the live tiles exit.
template <bool kUp, class C>
long long tile_bound(const GemmArgs& a) {
    const long long TK = (long long)a.T * a.K;
    const long long hit_b = a.do_hit ? std::min<long long>(std::min(a.N, a.C), TK) : 0;
    const long long lore_b = a.r > 0 ? std::min<long long>(a.N, TK) : 0;
    const long long nt_sh = kUp ? tiles_of(a.Is, C::kUpFeat) : tiles_of(a.d, C::BM) * a.parts;
    const long long nt_e = hit_b ? (kUp ? tiles_of(a.I, C::kUpFeat) : tiles_of(a.d, C::BM)) : 0;
    const long long nt_l = lore_b ? (kUp ? tiles_of(a.r, C::BM) : tiles_of(a.d, C::BM * kLoreDown)) : 0;
    return (a.Is > 0 ? tiles_of(a.T, C::BT) * nt_sh : 0) + TK / C::BT * std::max(nt_e, nt_l) + hit_b * nt_e + lore_b * nt_l;
}

template <bool kUp, bool kMx, class C>
hipError_t launch_pass(GemmArgs a, hipStream_t s) {
    const long long tiles = tile_bound<kUp, C>(a);
    if (tiles == 0) return hipSuccess;
    if (tiles > 0x7FFFFFFFll) return hipErrorInvalidValue;
    if (a.Is > 0)
        super_shape((int)tiles_of(a.T, C::BT), (int)(kUp ? tiles_of(a.Is, C::kUpFeat) : tiles_of(a.d, C::BM)), C::kXcdBlocks,
                    kUp ? a.super_up : a.super_dn);
    hipLaunchKernelGGL((expert_gemm_kernel<kUp, kMx, C>), dim3((unsigned)tiles), dim3(C::kThreads),
                       kMx ? C::kLds : C::S * C::kStage, s, a);
    return hipGetLastError();
}

template <bool kMx, class Up, class Down>
hipError_t launch_shapes(const GemmArgs& a, hipStream_t s) {
    hipError_t e = launch_pass<true, kMx, Up>(a, s);
    if (e == hipSuccess) e = launch_pass<false, kMx, Down>(a, s);
    if (e != hipSuccess || a.Is <= 0 || a.parts <= 1) return e;
    hipLaunchKernelGGL(shared_sum_kernel, dim3((unsigned)((a.d / 4 + 255) / 256), (unsigned)a.T), dim3(256), 0, s, a.T, a.d,
                       a.parts, a.part, a.sgate, a.y_shared);
    return hipGetLastError();
}

}  // namespace

bool expert_gemm_applies(const FfnArgs& a) {
    if (a.dtype != SPICE_BF16 || a.T < gemm_min_tokens(a.d, a.Is, a.wfmt)) return false;
    if (!(a.groups & (kDoHit | kDoShared)) && !lore_gemm_is_shorter(a.T, a.d, a.N, a.K)) return false;
    // offsets inside one operand are 32-bit
    auto fits = [](long long rows, long long cols) { return rows * ((cols + kBK - 1) / kBK * kBK) * 2 <= kMaxBuffer; };
    // MXFP4 blocks of whole stages and 16-byte rows of codes
    if (a.wfmt == SPICE_WFMT_MXFP4 &&
        (a.d % 128 || a.I % 128 || ((uintptr_t)a.w13_pool | (uintptr_t)a.w2_pool) % 16))
        return false;
    const long long TK = (long long)a.T * a.K;
    if (!fits(a.T, a.d) || !fits(TK, a.I) || !fits(a.T, a.Is) || !fits(2ll * a.I, a.d) || !fits(2ll * a.Is, a.d) ||
        !fits(a.d, a.I) || !fits(a.d, a.Is))
        return false;
    // the staged tiles need more LDS than the 64 KiB every AMD GPU offers
    static int lds_per_block[64] = {0};
    int dev = 0;
    if (hipGetDevice(&dev) != hipSuccess || dev < 0 || dev >= 64) return false;
    if (lds_per_block[dev] == 0) {
        int v = 0;
        if (hipDeviceGetAttribute(&v, hipDeviceAttributeMaxSharedMemoryPerBlock, dev) != hipSuccess) return false;
        lds_per_block[dev] = v;
    }
    return lds_per_block[dev] >= std::max({Big::S * Big::kStage, Wide::kLds, Small::kLds});
}

hipError_t launch_expert_gemm(const FfnArgs& f, bool hit, bool shared, hipStream_t s) {
    const bool lore = (f.groups & kDoLore) != 0;
    GemmArgs a{};
    a.T = f.T; a.d = f.d; a.N = f.N; a.K = f.K; a.C = f.C; a.I = f.I; a.Is = shared ? f.Is : 0;
    a.r = lore ? f.r : 0;
    a.do_hit = hit ? 1 : 0;
    a.x = static_cast<const uint16_t*>(f.x);
    a.perm = f.perm;
    a.offsets = f.offsets;
    a.resident_slot = f.resident_slot;
    a.w13_pool = f.w13_pool;
    a.w2_pool = f.w2_pool;
    a.w13s = static_cast<const uint16_t*>(f.w13s);
    a.w2s = static_cast<const uint16_t*>(f.w2s);
    a.lore_A = static_cast<const uint16_t*>(f.lore_A);
    a.lore_B = static_cast<const uint16_t*>(f.lore_B);
    a.u = f.u;
    a.h = static_cast<uint16_t*>(f.h);
    a.hs = static_cast<uint16_t*>(f.hs);
    a.y_slots = f.y_slots;
    a.y_shared = f.y_shared;
    a.sgate = f.sgate;
    a.ctrl = f.ctrl;
    a.part = f.part;
    a.parts = a.Is > 0 && f.part ? gemm_shared_parts(f.T, f.d, f.N, f.K, f.C, f.I, f.Is) : 1;
    const int shape = gemm_shape(f.T, f.N, f.K, hit ? f.C : 0, f.I, a.Is, f.wfmt);
    if (f.wfmt == SPICE_WFMT_MXFP4)
        return shape == kGemmSmall ? launch_shapes<true, Small, Small>(a, s) : launch_shapes<true, Wide, Wide>(a, s);
    switch (shape) {
        case kGemmBig: return launch_shapes<false, Big, Big>(a, s);
        case kGemmWide: return launch_shapes<false, Wide, Wide>(a, s);
        default:
            // so few tiles that one block per CU holds them all: the deep ring
            return tile_bound<true, Deep>(a) <= 256 ? launch_shapes<false, Deep, Small>(a, s)
                                                    : launch_shapes<false, Small, Small>(a, s);
    }
}

}  // namespace spice
