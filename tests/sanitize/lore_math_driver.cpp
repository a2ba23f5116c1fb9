// Sanitizer driver for the host linear algebra of the LoRE fit (lore_fit.cpp's Jacobi
// eigensolver, QR iteration and Cholesky solve), included here so its internal functions are
// reachable; built with -fsanitize=address,undefined together with device_stubs.cpp.  Checks on seeded
// symmetric / SPD matrices of sizes 1..40 (odd and even, for the round-robin bye):
// A = V diag(w) V^T and V V^T = I to 1e-10, and (L L^T) z = b to 1e-10; and the same of
// tridiagonal matrices up to 300 (random, graded, clustered, split, zero, with entries that are
// not finite) under the rotations that tridiag_qr hands out.  Prints "ok".
//
// Then the whole fit against a device of host memory that performs queued copies only when its
// stream is waited for, with every single allocation of the fit made to fail in turn: no copy may
// be left that reads or writes the memory of a call that has returned.
#include <hip/hip_runtime_api.h>

#include <cstdio>
#include <cstdlib>
#include <cstring>
#include <new>

#include "spice_internal.h"

namespace fake {
struct Copy {
    void* to;
    const void* from;
    size_t bytes;
};
Copy queue[256];
int queued = 0;
long fail_after = -1;  // allocations until one fails, or -1
hipError_t memcpy_async(void* to, const void* from, size_t bytes, hipMemcpyKind, hipStream_t) {
    if (queued == 256) std::abort();
    queue[queued++] = Copy{to, from, bytes};
    return hipSuccess;
}
hipError_t synchronize(hipStream_t) {
    for (int i = 0; i < queued; ++i) std::memcpy(queue[i].to, queue[i].from, queue[i].bytes);
    queued = 0;
    return hipSuccess;
}
}  // namespace fake
void* operator new(size_t n) {
    if (fake::fail_after >= 0 && fake::fail_after-- == 0) throw std::bad_alloc();
    void* p = std::malloc(n ? n : 1);
    if (!p) throw std::bad_alloc();
    return p;
}
void* operator new(size_t n, const std::nothrow_t&) noexcept { return std::malloc(n ? n : 1); }
void operator delete(void* p) noexcept { std::free(p); }
void operator delete(void* p, size_t) noexcept { std::free(p); }
namespace spice {
template <class... A>
hipError_t launched(A...) { return hipSuccess; }
}  // namespace spice
#define hipMemcpyAsync fake::memcpy_async
#define hipStreamSynchronize fake::synchronize
#define launch_fill_u32 launched
#define launch_expert_ffn launched
#define launch_fit_setup launched
#define launch_fit_residual launched
#define launch_fit_gram launched
#define launch_fit_project launched
#define launch_fit_tridiag launched
#define launch_fit_rotate launched
#define launch_fit_back launched
#define launch_fit_chol launched
#define launch_fit_solve launched
#include "lore_fit.cpp"

namespace {
uint64_t g_rng = 0x13198A2E03707344ull;
double urand() {
    g_rng ^= g_rng >> 12; g_rng ^= g_rng << 25; g_rng ^= g_rng >> 27;
    return (double)((g_rng * 0x2545F4914F6CDD1Dull) >> 11) * (1.0 / 9007199254740992.0) * 2.0 - 1.0;
}
}  // namespace

// The fit of n tokens with its k-th allocation failing, for every k until none is left.
int failing_allocations(int n) {
    spice_moe_cfg_t c{};
    c.d = 512; c.n_experts = 4; c.top_k = 2; c.inter = 8; c.n_slots = 1; c.dtype = SPICE_BF16;
    const int r = 8;
    const FitLayout L = fit_layout(c, n, r);
    std::vector<char> ws(L.total, 0);
    auto at = [&](size_t off) { return reinterpret_cast<double*>(ws.data() + off); };
    for (int i = 0; i < n; ++i) {  // Gram matrices, and the tridiagonal form the GPU would leave
        at(L.gx)[(size_t)i * n + i] = 2.0 + urand();
        at(L.gy)[(size_t)i * n + i] = 2.0 + urand();
        if (n > kFitHostTokens) {
            at(L.small)[3 * n + i] = 2.0 + urand();
            at(L.small)[4 * n + i] = urand();
        }
    }
    float out = 0.f;
    double loss = 0.0;
    for (long k = 0;; ++k) {
        fake::fail_after = k;
        const spice_status_t st = moe_lore_fit(&c, n, r, &out, &out, &out, nullptr, nullptr, &out, &out, nullptr, &loss,
                                               ws.data(), L.total, nullptr);
        const bool all = fake::fail_after >= 0;
        fake::fail_after = -1;
        if (fake::queued != 0 || st != (all ? SPICE_OK : SPICE_ERR_INTERNAL)) {
            std::fprintf(stderr, "fit of %d tokens, allocation %ld failing: status %d, %d copies left\n", n, k, (int)st,
                         fake::queued);
            return 1;
        }
        if (all) return k < 5;  // the fit does allocate
    }
}

// T = Z^T diag(w) Z with the rows z_k of Z turned by the rotations handed out, for the tridiagonal
// matrix with diagonal d and subdiagonal e; rounding of n rotations per sweep and about two sweeps
// per eigenvalue: 4 n^1.5 units of 2^-53 of the largest entry bound both residuals.
int tridiag_case(const char* name, int n, std::vector<double> d, std::vector<double> e) {
    const std::vector<double> d0 = d, e0 = e;
    std::vector<double> z((size_t)n * n, 0.0);
    for (int i = 0; i < n; ++i) z[(size_t)i * n + i] = 1.0;
    long planes = 0;
    const bool ok = tridiag_qr(n, d, e, [&](int lo, int cnt, const std::vector<double>& cs) {
        if (lo < 0 || cnt < 1 || lo + cnt >= n || cs.size() != 2 * (size_t)cnt) std::abort();
        planes += cnt;
        for (int k = 0; k < cnt; ++k)
            for (int i = 0; i < n; ++i) {
                double &a = z[(size_t)(lo + k) * n + i], &b = z[(size_t)(lo + k + 1) * n + i];
                const double x = a, y = b, c = cs[2 * k], s = cs[2 * k + 1];
                a = c * x + s * y;
                b = c * y - s * x;
            }
    });
    double scale = 1e-300, res = 0.0, orth = 0.0;
    for (int i = 0; i < n; ++i) scale = std::fmax(scale, std::fmax(std::fabs(d0[i]), i + 1 < n ? std::fabs(e0[i]) : 0.0));
    for (int i = 0; ok && i < n; ++i)
        for (int j = 0; j <= i; ++j) {
            double t = 0.0, o = 0.0;
            for (int k = 0; k < n; ++k) {
                t += z[(size_t)k * n + i] * d[k] * z[(size_t)k * n + j];
                o += z[(size_t)i * n + k] * z[(size_t)j * n + k];
            }
            const double want = i == j ? d0[i] : i == j + 1 ? e0[j] : 0.0;
            res = std::fmax(res, std::fabs(t - want) / scale);
            orth = std::fmax(orth, std::fabs(o - (i == j ? 1.0 : 0.0)));
        }
    const double bound = 4.0 * n * std::sqrt((double)n) * 1.2e-16 + 1e-15;
    if (ok && res <= bound && orth <= bound) return 0;
    std::fprintf(stderr, "tridiag %s n=%d: %s, residual %.2e, orthogonality %.2e, %ld rotations\n", name, n,
                 ok ? "converged" : "no convergence", res, orth, planes);
    return 1;
}

int tridiagonal() {
    int fail = 0;
    for (int n : {1, 2, 3, 49, 64, 150, 300}) {
        std::vector<double> d(n), e(n > 1 ? n - 1 : 0);
        auto fill = [&](auto f, auto g) {
            for (int i = 0; i < n; ++i) d[i] = f(i);
            for (int i = 0; i + 1 < n; ++i) e[i] = g(i);
        };
        fill([&](int) { return urand(); }, [&](int) { return urand(); });
        fail |= tridiag_case("random", n, d, e);
        fill([&](int i) { return std::pow(0.8, i); }, [&](int i) { return 0.3 * std::pow(0.8, i); });
        fail |= tridiag_case("graded", n, d, e);
        fill([&](int i) { return std::pow(0.8, n - i); }, [&](int i) { return 0.3 * std::pow(0.8, n - i); });
        fail |= tridiag_case("graded upwards", n, d, e);
        fill([&](int i) { return 1.0 + (i % 3); }, [&](int) { return 1e-9 * urand(); });
        fail |= tridiag_case("clustered", n, d, e);
        fill([&](int) { return 1e30 * urand(); }, [&](int i) { return i % 5 == 4 ? 0.0 : 1e30 * urand(); });
        fail |= tridiag_case("split", n, d, e);
        fill([&](int i) { return std::fabs(n / 2 - i); }, [&](int) { return 1.0; });
        fail |= tridiag_case("Wilkinson", n, d, e);
        fill([&](int) { return 0.0; }, [&](int) { return 0.0; });
        fail |= tridiag_case("zero", n, d, e);
        fill([&](int) { return 0.0; }, [&](int) { return 1.0; });
        fail |= tridiag_case("zero diagonal", n, d, e);
        for (double bad : {std::nan(""), HUGE_VAL}) {
            d[n / 2] = bad;
            std::vector<double> dd = d, ee = e;
            if (tridiag_qr(n, dd, ee, [](int, int, const std::vector<double>&) {})) fail = 1;
        }
    }
    return fail;
}

int main() {
    int fail = tridiagonal() | failing_allocations(40) | failing_allocations(64) | failing_allocations(300);
    for (int n : {1, 2, 3, 4, 7, 8, 15, 16, 31, 40}) {
        std::vector<double> a((size_t)n * n);
        for (int i = 0; i < n; ++i)
            for (int j = 0; j <= i; ++j) a[(size_t)i * n + j] = a[(size_t)j * n + i] = urand();
        if (n > 3) a[1] = a[(size_t)n] = 0.0;  // an entry that starts at zero
        std::vector<double> a0 = a, w, vt;
        jacobi_eigen(n, a, w, vt);
        double err = 0.0, orth = 0.0, scale = 1e-300;
        for (double v : a0) scale = std::fmax(scale, std::fabs(v));
        for (int i = 0; i < n; ++i)
            for (int j = 0; j < n; ++j) {
                double s = 0.0, o = 0.0;
                for (int k = 0; k < n; ++k) {
                    s += vt[(size_t)k * n + i] * w[k] * vt[(size_t)k * n + j];
                    o += vt[(size_t)i * n + k] * vt[(size_t)j * n + k];
                }
                err = std::fmax(err, std::fabs(s - a0[(size_t)i * n + j]));
                orth = std::fmax(orth, std::fabs(o - (i == j ? 1.0 : 0.0)));
            }
        if (err > 1e-10 * scale * n || orth > 1e-10 * n) {
            std::fprintf(stderr, "jacobi n=%d: reconstruction %.3e, orthogonality %.3e\n", n, err, orth);
            fail = 1;
        }
        // SPD: G = M M^T + n I
        std::vector<double> m((size_t)n * n), g((size_t)n * n);
        for (double& v : m) v = urand();
        for (int i = 0; i < n; ++i)
            for (int j = 0; j < n; ++j) {
                double s = i == j ? n : 0.0;
                for (int k = 0; k < n; ++k) s += m[(size_t)i * n + k] * m[(size_t)j * n + k];
                g[(size_t)i * n + j] = s;
            }
        std::vector<double> g0 = g, b(n), z(n);
        for (double& v : b) v = urand();
        z = b;
        if (!cholesky(n, g)) {
            std::fprintf(stderr, "cholesky n=%d: not positive definite\n", n);
            fail = 1;
            continue;
        }
        cholesky_solve(n, g, z.data());
        double res = 0.0;
        for (int i = 0; i < n; ++i) {
            double s = 0.0;
            for (int k = 0; k < n; ++k) s += g0[(size_t)i * n + k] * z[k];
            res = std::fmax(res, std::fabs(s - b[i]));
        }
        if (res > 1e-10 * n) {
            std::fprintf(stderr, "cholesky n=%d: residual %.3e\n", n, res);
            fail = 1;
        }
        // an indefinite matrix is refused
        std::vector<double> neg = g0;
        neg[0] = -1.0;
        if (cholesky(n, neg)) {
            std::fprintf(stderr, "cholesky n=%d accepted an indefinite matrix\n", n);
            fail = 1;
        }
    }
    std::printf(fail ? "FAILED\n" : "ok\n");
    return fail;
}
