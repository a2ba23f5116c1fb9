// Device steps of the LoRE calibration fit (Sec. 4.2, Eq. 8-10) for one expert:
//   fit_setup      a one-expert bucket of all n calibration tokens (perm = identity,
//                  HIT class only) for the grouped FFN, which computes E_e(x) and S(x);
//   fit_residual   Y = E_e(x) - S(x), the target of Eq. 8, in place;
//   fit_gram       n x n Gram matrices of the rows of X (dtype) or Y (fp32), accumulated in
//                  fp64 (one 16 x 16 output tile per block, 64-column panels through LDS);
//   fit_project    rows of A = (X^T Z)^T and of B = Y^T V from n x r host coefficients.
//   and, for more than kFitHostTokens tokens, the n x n eigen-decomposition and solve between:
//   fit_tridiag    one Householder step per launch: Y^T Y to tridiagonal form;
//   fit_rotate     the plane rotations of the host's QR iteration on that form, applied to
//                  the eigenvector rows;
//   fit_back       the leading eigenvectors carried back through the Householder steps;
//   fit_chol, fit_trail   Cholesky of X^T X, a 32-column panel and its trailing update per step;
//   fit_solve      the two triangular solves per leading eigenvector, and the coefficients.
// (Fewer tokens: Jacobi rotations and Cholesky on the host.)
#include <hip/hip_runtime.h>

#include "spice_internal.h"

namespace spice {
namespace {

constexpr int kGramTile = 16;
constexpr int kGramThreads = 256;

__global__ void fit_setup_kernel(int32_t n, int32_t* perm, int32_t* offsets, int32_t* resident) {
    const int i = blockIdx.x * blockDim.x + threadIdx.x;
    if (i < n) perm[i] = i;
    if (i == 0) {
        // classes x (N + 1) with N = 1: HIT [0, n), LORE and EXACT empty
        offsets[0] = 0; offsets[1] = n;
        offsets[2] = n; offsets[3] = n;
        offsets[4] = n; offsets[5] = n;
        resident[0] = 0;
    }
}

__global__ void fit_residual_kernel(size_t count, float* y, const float* s) {
    const size_t i = (size_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i < count) y[i] -= s[i];
}

__device__ __forceinline__ double elem(const void* p, int dtype, size_t i) {
    if (dtype == SPICE_BF16) return (double)__uint_as_float((uint32_t)static_cast<const uint16_t*>(p)[i] << 16);
    return (double)static_cast<const float*>(p)[i];
}

// G[i][j] = sum_k M[i][k] M[j][k] for the 16 x 16 tile (blockIdx.y, blockIdx.x); only tiles
// on or above the diagonal are computed and mirrored.  The two 16-row panels go through
// LDS 64 columns at a time (coalesced row reads, widened to fp64); each thread owns one
// (i, j) of the tile.
__global__ __launch_bounds__(kGramThreads) void fit_gram_kernel(int32_t n, int32_t d, int dtype, const void* M,
                                                                 double* G) {
    constexpr int kChunk = 64;
    const int ti = blockIdx.y, tj = blockIdx.x;
    if (tj < ti) return;
    __shared__ double pi[kGramTile][kChunk + 1];
    __shared__ double pj[kGramTile][kChunk + 1];
    const int tid = threadIdx.x;
    const int oi = tid / kGramTile, oj = tid % kGramTile;
    double acc = 0.0;
    for (int k0 = 0; k0 < d; k0 += kChunk) {
        for (int e = tid; e < kGramTile * kChunk; e += kGramThreads) {
            const int row = e / kChunk, col = e % kChunk, k = k0 + col;
            const int gi = ti * kGramTile + row, gj = tj * kGramTile + row;
            pi[row][col] = (gi < n && k < d) ? elem(M, dtype, (size_t)gi * d + k) : 0.0;
            pj[row][col] = (gj < n && k < d) ? elem(M, dtype, (size_t)gj * d + k) : 0.0;
        }
        __syncthreads();
        for (int c = 0; c < kChunk; ++c) acc += pi[oi][c] * pj[oj][c];
        __syncthreads();
    }
    const int i = ti * kGramTile + oi, j = tj * kGramTile + oj;
    if (i < n && j < n) {
        G[(size_t)i * n + j] = acc;
        G[(size_t)j * n + i] = acc;
    }
}

// out[k][j] (b_layout) or out[j][k] = sum_i M[i][k] C[i][j]: one thread per (feature k,
// column j); a block takes 256 consecutive features of one column, so the rows of M are
// read coalesced and C[i][j] is the same for the whole block.
__global__ __launch_bounds__(256) void fit_project_kernel(int32_t n, int32_t d, int32_t r, int dtype, const void* M,
                                                          const double* C, float* out, int b_layout) {
    const int k = blockIdx.x * blockDim.x + threadIdx.x, j = blockIdx.y;
    if (k >= d) return;
    double acc = 0.0;
    for (int i = 0; i < n; ++i) acc += elem(M, dtype, (size_t)i * d + k) * C[(size_t)i * r + j];
    if (b_layout) out[(size_t)k * r + j] = (float)acc;
    else out[(size_t)j * d + k] = (float)acc;
}

// ---- eigen-decomposition of a symmetric n x n matrix, and the SPD solve ---------------------

constexpr int kEigThreads = 256;
constexpr int kEigBlocks = 64;
constexpr int kMaxN = 1024;

// Sum over the wave, in every lane: adds within rows of 16 lanes, then across them (DPP: no
// LDS round trip, a third of the time of six shuffles of 64-bit values).
template <int kCtrl, int kRows>
__device__ __forceinline__ double dpp_add(double v) {
    const long long b = __double_as_longlong(v);
    const int lo = __builtin_amdgcn_update_dpp(0, (int)b, kCtrl, kRows, 0xF, false);
    const int hi = __builtin_amdgcn_update_dpp(0, (int)(b >> 32), kCtrl, kRows, 0xF, false);
    return v + __longlong_as_double(((long long)hi << 32) | (unsigned)lo);
}
__device__ __forceinline__ double lane_value(double v, int lane) {  // lane uniform
    const long long b = __double_as_longlong(v);
    const int lo = __builtin_amdgcn_readlane((int)b, lane), hi = __builtin_amdgcn_readlane((int)(b >> 32), lane);
    return __longlong_as_double(((long long)hi << 32) | (unsigned)lo);
}
__device__ __forceinline__ double wave_sum(double v) {
    v = dpp_add<0x111, 0xF>(v);  // row_shr 1, 2, 4, 8: lane 15 of each row holds the row's sum
    v = dpp_add<0x112, 0xF>(v);
    v = dpp_add<0x114, 0xF>(v);
    v = dpp_add<0x118, 0xF>(v);
    v = dpp_add<0x142, 0xA>(v);  // row_bcast 15 into rows 1 and 3, 31 into rows 2 and 3
    v = dpp_add<0x143, 0xC>(v);
    return lane_value(v, 63);
}

// Sum over the block; part holds one value per wave (and is free again after the next barrier).
__device__ __forceinline__ double block_sum(double v, double* part) {
    v = wave_sum(v);
    if ((threadIdx.x & 63) == 0) part[threadIdx.x >> 6] = v;
    __syncthreads();
    double s = 0.0;
    for (int k = 0; k < kEigThreads / 64; ++k) s += part[k];
    return s;
}

// Step k of the Householder tridiagonalisation of A (symmetric, full storage), one launch per
// step so that no block waits for another: every block finishes step k - 1 for itself (from its
// reflector v and p = A v), takes column k with that update, forms the reflector that clears it
// below the subdiagonal, and then, for its own rows of the trailing matrix, applies the update
// of step k - 1 and multiplies by the new reflector in one pass.
//   V[k][k+1 .. n)  reflector k (its first entry 1), tau[k] its factor: H = I - tau v v^T
//   p[k & 1][i]     (A v)[i], read by the next launch
//   dv[k], ev[k]    diagonal and subdiagonal of the tridiagonal form
// Bound by the launch and two dependent round trips to L2 per step (6 us a step at n = 512;
// the matrix, 2 MB, stays in L2): 3.1 ms of the fit, whose Jacobi rotations on one host core
// took 0.9 s (the whole fit of n = 512 tokens: 928 -> 14.1 ms).
__global__ __launch_bounds__(kEigThreads) void fit_tridiag_kernel(int n, int k, double* A, double* V, double* tau, double* p,
                                                                  double* dv, double* ev) {
    __shared__ double s_v[kMaxN], s_w[kMaxN], s_x[kMaxN];
    __shared__ double s_part[3][kEigThreads / 64];
    const int tid = threadIdx.x, lane = tid & 63;
    const double* pold = p + ((k + 1) & 1) * n;
    double* pnew = p + (k & 1) * n;
    // w of step k - 1: A <- A - v w^T - w v^T with w = t p - (t^2 / 2) (p . v) v
    if (k > 0) {
        const double t = tau[k - 1];
        double dot = 0.0;
        for (int i = k + tid; i < n; i += kEigThreads) {
            const double v = V[(size_t)(k - 1) * n + i], q = pold[i];
            s_v[i] = v;
            s_w[i] = q;
            dot += v * q;
        }
        dot = block_sum(dot, s_part[0]);
        const double h = 0.5 * t * t * dot;
        for (int i = k + tid; i < n; i += kEigThreads) s_w[i] = t * s_w[i] - h * s_v[i];
    } else {
        for (int i = tid; i < n; i += kEigThreads) s_v[i] = s_w[i] = 0.0;
    }
    __syncthreads();
    // column k of the updated matrix (row k: symmetric, and no block writes it in this launch)
    const double vk = s_v[k], wk = s_w[k];
    double sq = 0.0;
    for (int i = k + tid; i < n; i += kEigThreads) {
        const double c = A[(size_t)k * n + i] - vk * s_w[i] - wk * s_v[i];
        s_x[i] = c;
        if (i > k + 1) sq += c * c;
    }
    sq = block_sum(sq, s_part[1]);  // its barrier also publishes s_x
    const double alpha = k + 1 < n ? s_x[k + 1] : 0.0;
    double beta = alpha, t = 0.0, inv = 0.0;
    if (sq > 0.0) {
        beta = -copysign(sqrt(alpha * alpha + sq), alpha);
        t = (beta - alpha) / beta;
        inv = 1.0 / (alpha - beta);
    }
    if (blockIdx.x == 0 && tid == 0) {
        dv[k] = s_x[k];
        if (k + 1 < n) ev[k] = beta;
        tau[k] = t;
    }
    __syncthreads();
    for (int i = k + 1 + tid; i < n; i += kEigThreads) {
        const double v = i == k + 1 ? 1.0 : s_x[i] * inv;
        s_x[i] = v;
        if (blockIdx.x == 0) V[(size_t)k * n + i] = v;
    }
    __syncthreads();
    // own rows of the trailing matrix, one per wave at a time
    const int waves = gridDim.x * (kEigThreads / 64);
    for (int i = k + 1 + blockIdx.x * (kEigThreads / 64) + (tid >> 6); i < n; i += waves) {
        double* row = A + (size_t)i * n;
        const double vi = s_v[i], wi = s_w[i];
        double acc = 0.0;
        for (int j = k + 1 + lane; j < n; j += 64) {
            const double x = row[j] - vi * s_w[j] - wi * s_v[j];
            row[j] = x;
            acc += x * s_x[j];
        }
        acc = wave_sum(acc);
        if (lane == 0) pnew[i] = acc;
    }
}

// Plane rotations of the QR iteration on the eigenvector rows: Zt[k][c] is component c of
// vector k (started as the identity when first).  Sweep q covers rotations of the planes
// (lo, lo + 1), (lo + 1, lo + 2), ...: z_k' = c z_k + s z_k+1, z_k+1' = c z_k+1 - s z_k, whose
// chain over k stays in a register.  A block owns kRotCols components of every vector in LDS,
// one per lane, so no block meets another.  A sweep's rotations are loaded into registers while
// the sweep before it runs and staged in LDS, and a batch's operands are read from LDS while
// the one before it is rotated; read straight from L2 the chain took more than twice as long.
// 30 ns a rotation (263k at n = 512, 7.8 ms of the fit).
constexpr int kRotCols = 16, kRotBatch = 8;
// A batch read ahead reaches up to 3 kRotBatch entries past a sweep: of the rotations, their
// padding; of a vector's rows (kRotCols doubles each), the rotations behind them and the padding.
constexpr size_t rot_lds_bytes(int n) {
    return (size_t)n * (kRotCols + 2) * sizeof(double) + 3 * kRotBatch * kRotCols * sizeof(double);
}
__global__ __launch_bounds__(64) void fit_rotate_kernel(int n, const double2* __restrict__ rot, const int2* __restrict__ sweeps,
                                                        int nsweeps, int first, double* Zt) {
    extern __shared__ double s_z[];  // [n][kRotCols], then the sweep's rotations [n] and their padding
    double2* s_r = reinterpret_cast<double2*>(s_z + (size_t)n * kRotCols);
    constexpr int kPer = kMaxN / 64;
    const int lane = threadIdx.x;
    const int c0 = blockIdx.x * kRotCols;
    for (int i = lane; i < n * kRotCols; i += 64) {
        const int k = i / kRotCols, c = c0 + i % kRotCols;
        s_z[i] = first ? (k == c ? 1.0 : 0.0) : (c < n ? Zt[(size_t)k * n + c] : 0.0);
    }
    double* z = s_z + (lane & (kRotCols - 1));  // lanes past kRotCols repeat the first ones' work
    double2 ahead[kPer];
    auto load = [&](const double2* from, int cnt) {
#pragma unroll
        for (int u = 0; u < kPer; ++u)
            if (64 * u + lane < cnt) ahead[u] = from[64 * u + lane];
    };
    int2 sw = nsweeps > 0 ? sweeps[0] : make_int2(0, 0);
    load(rot, sw.y);
    for (int q = 0; q < nsweeps; ++q) {
        const int lo = sw.x, cnt = sw.y;
        __syncthreads();  // the sweep before has read its rotations
#pragma unroll
        for (int u = 0; u < kPer; ++u)
            if (64 * u + lane < cnt) s_r[64 * u + lane] = ahead[u];
        rot += cnt;
        if (q + 1 < nsweeps) {
            sw = sweeps[q + 1];
            load(rot, sw.y);
        }
        __syncthreads();
        // whole batches at immediate offsets from two running addresses (a wave alone on its SIMD
        // is bound by the instructions it issues); reads past the sweep land in the rotations'
        // padding and are not used
        double* zp = z + lo * kRotCols;
        const double2* rp = s_r;
        double f = zp[0];
        double2 r0[kRotBatch], r1[kRotBatch];
        double y0[kRotBatch], y1[kRotBatch];
        auto fetch = [&](int at, double2 (&r)[kRotBatch], double (&y)[kRotBatch]) {
#pragma unroll
            for (int u = 0; u < kRotBatch; ++u) {
                r[u] = rp[at + u];
                y[u] = zp[(at + u + 1) * kRotCols];
            }
        };
        auto turn = [&](int at, int m, const double2 (&r)[kRotBatch], const double (&y)[kRotBatch]) {
#pragma unroll
            for (int u = 0; u < kRotBatch; ++u) {
                if (u < m) {
                    zp[(at + u) * kRotCols] = r[u].x * f + r[u].y * y[u];
                    f = r[u].x * y[u] - r[u].y * f;
                }
            }
        };
        fetch(0, r0, y0);
        int left = cnt;
        for (; left >= 2 * kRotBatch; left -= 2 * kRotBatch) {
            fetch(kRotBatch, r1, y1);
            turn(0, kRotBatch, r0, y0);
            fetch(2 * kRotBatch, r0, y0);
            turn(kRotBatch, kRotBatch, r1, y1);
            zp += 2 * kRotBatch * kRotCols;
            rp += 2 * kRotBatch;
        }
        fetch(kRotBatch, r1, y1);
        turn(0, left, r0, y0);
        turn(kRotBatch, left - kRotBatch, r1, y1);
        z[(lo + cnt) * kRotCols] = f;
    }
    __syncthreads();
    for (int i = lane; i < n * kRotCols; i += 64) {
        const int k = i / kRotCols, c = c0 + i % kRotCols;
        if (c < n) Zt[(size_t)k * n + c] = s_z[i];
    }
}

// Eigenvector ord[j] of the tridiagonal form carried back to A's: z <- H_0 H_1 ... H_{n-2} z, one
// wave per vector, its components in registers.
__global__ __launch_bounds__(64) void fit_back_kernel(int n, const double* Zt, const int32_t* ord, const double* V,
                                                      const double* tau, double* vec) {
    constexpr int kPer = kMaxN / 64;
    const int lane = threadIdx.x, j = blockIdx.x;
    double z[kPer], cur[kPer];
#pragma unroll
    for (int u = 0; u < kPer; ++u) z[u] = 64 * u + lane < n ? Zt[(size_t)ord[j] * n + 64 * u + lane] : 0.0;
    auto fetch = [&](int k, double (&v)[kPer]) {
#pragma unroll
        for (int u = 0; u < kPer; ++u) {
            const int i = 64 * u + lane;
            v[u] = k >= 0 && i > k && i < n ? V[(size_t)k * n + i] : 0.0;
        }
    };
    fetch(n - 2, cur);
    for (int k = n - 2; k >= 0; --k) {
        double nxt[kPer];
        fetch(k - 1, nxt);
        double dot = 0.0;
#pragma unroll
        for (int u = 0; u < kPer; ++u) dot += cur[u] * z[u];
        dot = wave_sum(dot) * tau[k];
#pragma unroll
        for (int u = 0; u < kPer; ++u) {
            z[u] -= dot * cur[u];
            cur[u] = nxt[u];
        }
    }
#pragma unroll
    for (int u = 0; u < kPer; ++u)
        if (64 * u + lane < n) vec[(size_t)j * n + 64 * u + lane] = z[u];
}

// Cholesky of the SPD matrix G, lower factor in place and mirrored above the diagonal, in the
// host's order of operations (each element subtracts its products one by one in column order,
// no fused multiply-add), so that the two take the same matrices for singular.
constexpr int kPanel = 32;

// Panel k0: every block factors the kPanel x kPanel diagonal tile for itself, then finishes
// kPanel rows below it.  *bad is set when a pivot is not positive.
__global__ __launch_bounds__(kEigThreads) void fit_chol_kernel(int n, int k0, const double* G, double* L, uint32_t* bad) {
#pragma clang fp contract(off)
    __shared__ double s_d[kPanel][kPanel + 1], s_r[kPanel][kPanel + 1];
    const int tid = threadIdx.x, nb = min(kPanel, n - k0);
    const int r0 = k0 + kPanel * blockIdx.x;  // block 0: the diagonal tile itself
    const int nr = min(kPanel, n - r0);
    for (int i = tid; i < kPanel * kPanel; i += kEigThreads) {
        const int r = i / kPanel, c = i % kPanel;
        s_d[r][c] = r < nb && c < nb ? G[(size_t)(k0 + r) * n + k0 + c] : (r == c ? 1.0 : 0.0);
        s_r[r][c] = r < nr && c < nb ? G[(size_t)(r0 + r) * n + k0 + c] : 0.0;
    }
    __syncthreads();
    // column j of the tile and of the rows: thread (r, which) takes one element per column
    const int r = tid & (kPanel - 1), part = tid / kPanel;
    for (int j = 0; j < nb; ++j) {
        if (part == 0 && r >= j) {
            double v = s_d[r][j];
            for (int c = 0; c < j; ++c) v -= s_d[r][c] * s_d[j][c];
            s_d[r][j] = v;
        } else if (part == 2) {
            double v = s_r[r][j];
            for (int c = 0; c < j; ++c) v -= s_r[r][c] * s_d[j][c];
            s_r[r][j] = v;
        }
        __syncthreads();
        const double piv = s_d[j][j];
        const double l = sqrt(piv);
        __syncthreads();
        if (part == 0 && r >= j) s_d[r][j] = r == j ? l : s_d[r][j] / l;
        else if (part == 2) s_r[r][j] = s_r[r][j] / l;
        if (blockIdx.x == 0 && tid == 0 && !(piv > 0.0)) *bad = 1u;
        __syncthreads();
    }
    for (int i = tid; i < kPanel * kPanel; i += kEigThreads) {
        const int rr = i / kPanel, c = i % kPanel;
        if (rr >= nr || c >= nb) continue;
        if (blockIdx.x == 0) {
            if (c <= rr) {
                L[(size_t)(k0 + rr) * n + k0 + c] = s_d[rr][c];
                L[(size_t)(k0 + c) * n + k0 + rr] = s_d[rr][c];
            }
        } else {
            L[(size_t)(r0 + rr) * n + k0 + c] = s_r[rr][c];
            L[(size_t)(k0 + c) * n + r0 + rr] = s_r[rr][c];
        }
    }
}

// Trailing update after panel k0: G[i][j] -= sum_c L[i][k0 + c] L[j][k0 + c] for i >= j past the
// panel, 32 x 32 tiles.
__global__ __launch_bounds__(kEigThreads) void fit_trail_kernel(int n, int k0, double* G, const double* L) {
#pragma clang fp contract(off)
    const int bi = blockIdx.y, bj = blockIdx.x;
    if (bj > bi) return;
    __shared__ double s_a[kPanel][kPanel + 1], s_b[kPanel][kPanel + 1];
    const int tid = threadIdx.x;
    const int i0 = k0 + kPanel * (1 + bi), j0 = k0 + kPanel * (1 + bj);
    for (int i = tid; i < kPanel * kPanel; i += kEigThreads) {
        const int r = i / kPanel, c = i % kPanel;
        s_a[r][c] = i0 + r < n ? L[(size_t)(i0 + r) * n + k0 + c] : 0.0;
        s_b[r][c] = j0 + r < n ? L[(size_t)(j0 + r) * n + k0 + c] : 0.0;
    }
    __syncthreads();
    for (int i = tid; i < kPanel * kPanel; i += kEigThreads) {
        const int r = i / kPanel, c = i % kPanel;
        if (i0 + r >= n || j0 + c >= n || j0 + c > i0 + r) continue;
        double v = G[(size_t)(i0 + r) * n + j0 + c];
        for (int q = 0; q < kPanel; ++q) v -= s_a[r][q] * s_b[c][q];
        G[(size_t)(i0 + r) * n + j0 + c] = v;
    }
}

// Coefficients of leading direction j (singular value sv[j], 0: none): cb = v / s and
// ca = (X^T X)^-1 v s from the factor L (mirrored, so both triangular solves read rows), one
// wave per direction, its right-hand side in registers and the next row of L in flight.
__global__ __launch_bounds__(64) void fit_solve_kernel(int n, int r, const double* L, const double* vec, const double* sv,
                                                       double* ca, double* cb) {
    constexpr int kPer = kMaxN / 64;
    const int lane = threadIdx.x, j = blockIdx.x;
    const double s = sv[j];
    if (!(s > 0.0)) {
        for (int i = lane; i < n; i += 64) ca[(size_t)i * r + j] = cb[(size_t)i * r + j] = 0.0;
        return;
    }
    double b[kPer], cur[kPer], nxt[kPer];
#pragma unroll
    for (int u = 0; u < kPer; ++u) {
        const int i = 64 * u + lane;
        const double v = i < n ? vec[(size_t)j * n + i] : 0.0;
        b[u] = v * s;
        if (i < n) cb[(size_t)i * r + j] = v / s;
    }
    auto fetch = [&](int i, double (&row)[kPer]) {
#pragma unroll
        for (int u = 0; u < kPer; ++u) {
            const int q = 64 * u + lane;
            row[u] = i >= 0 && i < n && q < n ? L[(size_t)i * n + q] : 0.0;
        }
    };
    // L y = b, by columns of L (rows of its mirror)
    fetch(0, cur);
#pragma unroll
    for (int U = 0; U < kPer; ++U) {
        const int last = min(64, n - 64 * U);
        for (int l = 0; l < last; ++l) {
            const int i = 64 * U + l;
            fetch(i + 1, nxt);
            const double z = lane_value(b[U], l) / lane_value(cur[U], l);
            if (lane == l) b[U] = z;
            if (lane > l) b[U] -= cur[U] * z;
#pragma unroll
            for (int u = U + 1; u < kPer; ++u) b[u] -= cur[u] * z;
#pragma unroll
            for (int u = 0; u < kPer; ++u) cur[u] = nxt[u];
        }
    }
    // L^T z = y, by rows of L
    fetch(n - 1, cur);
#pragma unroll
    for (int U = kPer - 1; U >= 0; --U) {
        for (int l = min(64, n - 64 * U) - 1; l >= 0; --l) {
            const int i = 64 * U + l;
            fetch(i - 1, nxt);
            const double z = lane_value(b[U], l) / lane_value(cur[U], l);
            if (lane == l) b[U] = z;
            if (lane < l) b[U] -= cur[U] * z;
#pragma unroll
            for (int u = 0; u < U; ++u) b[u] -= cur[u] * z;
#pragma unroll
            for (int u = 0; u < kPer; ++u) cur[u] = nxt[u];
        }
    }
#pragma unroll
    for (int u = 0; u < kPer; ++u)
        if (64 * u + lane < n) ca[(size_t)(64 * u + lane) * r + j] = b[u];
}

}  // namespace

hipError_t launch_fit_tridiag(int32_t n, double* A, double* V, double* tau, double* p, double* dv, double* ev, hipStream_t s) {
    if (n > kMaxN) return hipErrorInvalidValue;
    for (int k = 0; k < n; ++k) {
        const int blocks = (n - k + 3) / 4 < kEigBlocks ? (n - k + 3) / 4 : kEigBlocks;
        hipLaunchKernelGGL(fit_tridiag_kernel, dim3((unsigned)blocks), dim3(kEigThreads), 0, s, n, k, A, V, tau, p, dv, ev);
    }
    return hipGetLastError();
}

hipError_t launch_fit_rotate(int32_t n, const double* rot, const int32_t* sweeps, int32_t nsweeps, bool first, double* Zt,
                             hipStream_t s) {
    if (n > kMaxN) return hipErrorInvalidValue;
    hipLaunchKernelGGL(fit_rotate_kernel, dim3((unsigned)((n + kRotCols - 1) / kRotCols)), dim3(64),
                       rot_lds_bytes(n), s, n, reinterpret_cast<const double2*>(rot),
                       reinterpret_cast<const int2*>(sweeps), nsweeps, first ? 1 : 0, Zt);
    return hipGetLastError();
}

hipError_t launch_fit_back(int32_t n, int32_t m, const double* Zt, const int32_t* ord, const double* V, const double* tau,
                           double* vec, hipStream_t s) {
    if (n > kMaxN) return hipErrorInvalidValue;
    hipLaunchKernelGGL(fit_back_kernel, dim3((unsigned)m), dim3(64), 0, s, n, Zt, ord, V, tau, vec);
    return hipGetLastError();
}

hipError_t launch_fit_chol(int32_t n, double* G, double* L, uint32_t* bad, hipStream_t s) {
    for (int k0 = 0; k0 < n; k0 += kPanel) {
        const unsigned rows = (unsigned)((n - k0 + kPanel - 1) / kPanel);
        hipLaunchKernelGGL(fit_chol_kernel, dim3(rows), dim3(kEigThreads), 0, s, n, k0, G, L, bad);
        if (rows > 1) hipLaunchKernelGGL(fit_trail_kernel, dim3(rows - 1, rows - 1), dim3(kEigThreads), 0, s, n, k0, G, L);
    }
    return hipGetLastError();
}

hipError_t launch_fit_solve(int32_t n, int32_t r, const double* L, const double* vec, const double* sv, double* ca,
                            double* cb, hipStream_t s) {
    if (n > kMaxN) return hipErrorInvalidValue;
    hipLaunchKernelGGL(fit_solve_kernel, dim3((unsigned)r), dim3(64), 0, s, n, r, L, vec, sv, ca, cb);
    return hipGetLastError();
}

hipError_t launch_fit_setup(int32_t n, int32_t* perm, int32_t* offsets, int32_t* resident, hipStream_t s) {
    hipLaunchKernelGGL(fit_setup_kernel, dim3((unsigned)((n + 255) / 256)), dim3(256), 0, s, n, perm, offsets,
                       resident);
    return hipGetLastError();
}

hipError_t launch_fit_residual(size_t count, float* y, const float* shared, hipStream_t s) {
    if (count == 0) return hipSuccess;
    hipLaunchKernelGGL(fit_residual_kernel, dim3((unsigned)((count + 255) / 256)), dim3(256), 0, s, count, y,
                       shared);
    return hipGetLastError();
}

hipError_t launch_fit_gram(int32_t n, int32_t d, int dtype, const void* M, double* G, hipStream_t s) {
    const unsigned t = (unsigned)((n + kGramTile - 1) / kGramTile);
    hipLaunchKernelGGL(fit_gram_kernel, dim3(t, t), dim3(kGramThreads), 0, s, n, d, dtype, M, G);
    return hipGetLastError();
}

hipError_t launch_fit_project(int32_t n, int32_t d, int32_t r, int dtype, const void* M, const double* C, float* out,
                              bool b_layout, hipStream_t s) {
    hipLaunchKernelGGL(fit_project_kernel, dim3((unsigned)((d + 255) / 256), (unsigned)r), dim3(256), 0, s, n, d, r,
                       dtype, M, C, out, b_layout ? 1 : 0);
    return hipGetLastError();
}

}  // namespace spice
