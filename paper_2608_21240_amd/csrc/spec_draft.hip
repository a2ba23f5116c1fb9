// One depth of the speculative-prefetch draft rollout (Sec. 4.1, Alg. 1 steps 2-4),
// after the routing and the surrogate FFN of that depth have run:
//   the router's top-K of each running token is its prediction (Eq. 2) and is enqueued;
//   its confidence is the top-K probability mass (Eq. 5);
//   a token at depth >= l_min whose confidence is below tau stops (its prediction stays);
//   the others move their draft state one layer on,
//     h <- Attn(h) + sum_k pi_k (S(h) + B_k A_k h),  Ẽ_k = S + B_k A_k (Eq. 11),
//   with the target layer's attention replaced by the identity.
// S(h) comes from the shared block's FFN (y_shared) and B_k A_k h from the LoRE FFN
// of the slots (y_slots at the slot's bucket position); the routing of the depth put
// every slot in the LoRE class, so every predicted expert has its surrogate row.
//
// One block per token.  Thread 0 reads the K predictions, writes the queue entries and
// takes the halting decision; then every thread updates (or copies) 4 features at a time
// of the token's draft state in fp32 and stores it in the activation dtype (bf16 with
// round-to-nearest-even).
#include <hip/hip_runtime.h>

#include "spice_internal.h"

namespace spice {
namespace {

constexpr int kThreads = 256;
constexpr int kMaxK = 64;

__device__ __forceinline__ uint32_t bf16_rne(float f) {
    const uint32_t u = __float_as_uint(f);
    if ((u & 0x7FFFFFFFu) > 0x7F800000u) return 0x7FC0u;  // NaN stays NaN
    return (u + 0x7FFFu + ((u >> 16) & 1u)) >> 16;
}

template <int DT>
__device__ __forceinline__ float4 load4(const void* p, size_t i) {
    if constexpr (DT == SPICE_BF16) {
        const uint2 v = *reinterpret_cast<const uint2*>(static_cast<const uint16_t*>(p) + i);
        return make_float4(__uint_as_float(v.x << 16), __uint_as_float(v.x & 0xFFFF0000u),
                           __uint_as_float(v.y << 16), __uint_as_float(v.y & 0xFFFF0000u));
    } else {
        return *reinterpret_cast<const float4*>(static_cast<const float*>(p) + i);
    }
}

template <int DT>
__device__ __forceinline__ void store4(void* p, size_t i, float4 v) {
    if constexpr (DT == SPICE_BF16) {
        uint2 o;
        o.x = bf16_rne(v.x) | (bf16_rne(v.y) << 16);
        o.y = bf16_rne(v.z) | (bf16_rne(v.w) << 16);
        *reinterpret_cast<uint2*>(static_cast<uint16_t*>(p) + i) = o;
    } else {
        *reinterpret_cast<float4*>(static_cast<float*>(p) + i) = v;
    }
}

// One block per token.  Bound by its chain of round trips (the predictions, then the rows they
// name): wave 0 reads the predictions one per lane, every thread issues its first rows of h and S
// before the decision is known, and the correction rows go out 8 at a time (T = 64, K = 6,
// d = 2048: 8.6 -> 5.3 us; the loads went one after the other before).
template <int DT>
__global__ __launch_bounds__(kThreads) void spec_update_kernel(SpecArgs a) {
    constexpr int kB = 8;  // correction rows in flight
    __shared__ int s_update;
    __shared__ float s_w[kMaxK];
    __shared__ int s_pos[kMaxK];
    const int t = blockIdx.x, K = a.K, lane = threadIdx.x;
    const size_t row = (size_t)t * a.d;
    int i = threadIdx.x * 4;
    float4 h = make_float4(0.f, 0.f, 0.f, 0.f), s = h;
    if (i < a.d) {
        h = load4<DT>(a.h_in, row + i);
        s = *reinterpret_cast<const float4*>(a.y_shared + row + i);
    }
    if (lane < 64) {
        const size_t r = (size_t)t * K + lane;
        const bool mine = lane < K;
        const int e = mine ? a.topk_idx[r] : -1;
        const float w = mine ? a.topk_w[r] : 0.f;
        const int pos = mine ? a.inv_perm[r] : 0;
        const bool halted = a.halted[t] != 0;
        double c = 0.0;
        for (int k = 0; k < K; ++k) c += (double)__uint_as_float(__builtin_amdgcn_readlane(__float_as_uint(w), k));
        const bool ok = __ballot(pos < 0 || pos >= a.T * K) == 0;
        const bool halt = a.delta >= a.l_min && c < (double)a.tau;  // the prediction stays queued
        const float conf = halted ? __builtin_nanf("") : (float)c;
        if (mine) {
            a.pred_idx[r] = halted ? -1 : e;
            a.pred_prob[r] = halted ? 0.f : w;
            if (a.h_pred_idx) a.h_pred_idx[r] = halted ? -1 : e;
            if (a.h_pred_prob) a.h_pred_prob[r] = halted ? 0.f : w;
            s_w[lane] = w;
            s_pos[lane] = pos;
        }
        if (lane == 0) {
            a.conf[t] = conf;
            if (a.h_conf) a.h_conf[t] = conf;
            if (!halted && !ok) atomicOr(&a.ctrl[kWordFlags], (uint32_t)SPICE_FLAG_BAD_INDEX);
            if (!halted && halt) a.halted[t] = 1;  // no deeper speculation
            s_update = !halted && !halt && !a.last && ok;
        }
    }
    __syncthreads();
    if (!s_update && a.h_out == a.h_in) return;
    while (i < a.d) {
        float4 acc = h;
        if (s_update) {
            for (int k0 = 0; k0 < K; k0 += kB) {
                float4 dl[kB];
#pragma unroll
                for (int u = 0; u < kB; ++u)
                    dl[u] = a.lore && k0 + u < K
                                ? *reinterpret_cast<const float4*>(a.y_slots + (size_t)s_pos[k0 + u] * a.d + i)
                                : make_float4(0.f, 0.f, 0.f, 0.f);
#pragma unroll
                for (int u = 0; u < kB; ++u) {
                    if (k0 + u >= K) break;
                    const float w = s_w[k0 + u];
                    acc.x += w * (s.x + dl[u].x); acc.y += w * (s.y + dl[u].y);
                    acc.z += w * (s.z + dl[u].z); acc.w += w * (s.w + dl[u].w);
                }
            }
        }
        store4<DT>(a.h_out, row + i, acc);
        i += kThreads * 4;
        if (i < a.d) {
            h = load4<DT>(a.h_in, row + i);
            s = *reinterpret_cast<const float4*>(a.y_shared + row + i);
        }
    }
}

}  // namespace

hipError_t launch_spec_update(const SpecArgs& a, hipStream_t s) {
    if (a.T == 0) return hipSuccess;
    if (a.dtype == SPICE_BF16)
        hipLaunchKernelGGL(spec_update_kernel<SPICE_BF16>, dim3((unsigned)a.T), dim3(kThreads), 0, s, a);
    else
        hipLaunchKernelGGL(spec_update_kernel<SPICE_F32>, dim3((unsigned)a.T), dim3(kThreads), 0, s, a);
    return hipGetLastError();
}

}  // namespace spice
