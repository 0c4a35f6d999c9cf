// Principal axes for the improved k-means (Sec. 3.2, step 1: "PCA space of {x'}"): eigen-decomposition of the
// D x D covariance matrix.  Host code, fp64: the matrix is tiny next to the data (D <= 4096) and the work is
// serial by nature -- Householder reduction to tridiagonal form, then implicit-shift QR sweeps (Wilkinson shift)
// on the tridiagonal matrix with every plane rotation applied to the accumulated transformation.  The
// transformation is kept TRANSPOSED (row i = i-th basis vector), so a rotation works on two contiguous rows and
// the result already has the axes as rows, which is how the rotation kernels take R.
//
// What bounds it is arithmetic, 6 operations per element of Vt and rotation (about 14,000 rotations at D = 128), so the four
// loops over rows run in blocks of columns that stay in registers and are compiled for each width of the host's vector unit.
// The rotations of several QR sweeps are queued and applied one block of columns after the other, which keeps the block in
// the first-level cache.  Every element sees the operations of the plain loops in their order, without contraction to fused
// multiply-adds: the same bits.  (The pragma for that stands in each function: at file scope it would hold for the rest of the
// translation unit, device kernels included.)  D = 128 (covariance of SIFT-like rows, one core of an EPYC): 1969 us as plain loops,
// 854 us (1020 with 256-bit vectors).
#pragma once
#include <math.h>
#include <stddef.h>
#include <string.h>
#include <algorithm>
#include <numeric>
#include <vector>

namespace hclae {

// One QR sweep: plane rotations (k, k+1) for k = lo..hi-1, in this order; their (c, s) start at pair `at` of the queue.
struct EigenSweep {
    int lo, hi;
    size_t at;
};

// W columns of a row-major matrix in registers.
template <int W>
struct EigenCols {
    typedef double vec __attribute__((vector_size(8 * W), aligned(8)));
    static __attribute__((always_inline)) inline vec get(const double *p) { return *reinterpret_cast<const vec *>(p); }
    static __attribute__((always_inline)) inline void put(double *p, const vec &v) { *reinterpret_cast<vec *>(p) = v; }
};

// y[j] = sum_i v[i] B[i][j] for i in ascending order, from zero; columns [j, j + W).
template <int W>
__attribute__((always_inline)) inline int eigen_mul(const double *B, int n, int len, const double *v, double *y, int j)
{
#pragma clang fp contract(off)
    using C = EigenCols<W>;
    for (; j + W <= len; j += W) {
        typename C::vec s = {};
        for (int i = 0; i < len; ++i) s += C::get(B + (size_t)i * n + j) * v[i];
        C::put(y + j, s);
    }
    return j;
}

// B[i][j] -= v[i] p[j] + q[i] x[j]
__attribute__((always_inline)) inline void eigen_rank2(double *B, int n, int len, const double *x, const double *p)
{
#pragma clang fp contract(off)
    for (int i = 0; i < len; ++i) {
        double *bi = B + (size_t)i * n;
        const double vi = x[i], qi = p[i];
#pragma clang loop vectorize(assume_safety)
        for (int j = 0; j < len; ++j) bi[j] -= vi * p[j] + qi * x[j];
    }
}

// Q[i][j] -= (b v[i]) u[j]
__attribute__((always_inline)) inline void eigen_rank1(double *Q, int n, int len, double b, const double *v, const double *u)
{
#pragma clang fp contract(off)
    for (int i = 0; i < len; ++i) {
        double *qi = Q + (size_t)i * n;
        const double bv = b * v[i];
#pragma clang loop vectorize(assume_safety)
        for (int j = 0; j < len; ++j) qi[j] -= bv * u[j];
    }
}

// The queued sweeps on columns [j, j + W) of V: row k is finished and row k+1 carried to the next rotation in registers.
template <int W>
__attribute__((always_inline)) inline int eigen_rotate(double *V, int n, const EigenSweep *sw, size_t nsw, const double *cs, int j)
{
#pragma clang fp contract(off)
    using C = EigenCols<W>;
    for (; j + W <= n; j += W)
        for (size_t q = 0; q < nsw; ++q) {
            const double *r = cs + 2 * sw[q].at;
            double *row = V + (size_t)sw[q].lo * n + j;
            typename C::vec t0 = C::get(row);
            for (int k = sw[q].lo; k < sw[q].hi; ++k, r += 2, row += n) {
                const typename C::vec t1 = C::get(row + n);
                C::put(row, t0 * r[0] - t1 * r[1]);
                t0 = t0 * r[1] + t1 * r[0];
            }
            C::put(row, t0);
        }
    return j;
}

// The four loops for one vector unit.
#define HCLAE_EIGEN_LOOPS(name, target_)                                                                                  \
    struct name {                                                                                                         \
        target_ static void mul(const double *B, int n, int len, const double *v, double *y)                              \
        {                                                                                                                 \
            eigen_mul<1>(B, n, len, v, y, eigen_mul<8>(B, n, len, v, y, eigen_mul<32>(B, n, len, v, y, 0)));              \
        }                                                                                                                 \
        target_ static void rank2(double *B, int n, int len, const double *x, const double *p)                            \
        {                                                                                                                 \
            eigen_rank2(B, n, len, x, p);                                                                                 \
        }                                                                                                                 \
        target_ static void rank1(double *Q, int n, int len, double b, const double *v, const double *u)                  \
        {                                                                                                                 \
            eigen_rank1(Q, n, len, b, v, u);                                                                              \
        }                                                                                                                 \
        target_ static void rotate(double *V, int n, const EigenSweep *sw, size_t nsw, const double *cs)                  \
        {                                                                                                                 \
            eigen_rotate<1>(V, n, sw, nsw, cs,                                                                            \
                            eigen_rotate<8>(V, n, sw, nsw, cs, eigen_rotate<32>(V, n, sw, nsw, cs, 0)));                  \
        }                                                                                                                 \
    };
HCLAE_EIGEN_LOOPS(EigenBase, )
#if defined(__x86_64__) && !defined(__HIP_DEVICE_COMPILE__)
HCLAE_EIGEN_LOOPS(EigenAvx2, __attribute__((target("avx2"))))
HCLAE_EIGEN_LOOPS(EigenAvx512, __attribute__((target("avx512f"))))
#endif
#undef HCLAE_EIGEN_LOOPS

// A: n x n symmetric, row-major; destroyed.  On return w[0] >= ... >= w[n-1] are the eigenvalues and row i of
// Vt (n x n, row-major) is a unit eigenvector of w[i], signed so that its entry of largest magnitude (the
// first one among equals) is positive.  Returns 0, or -1 when the iteration did not converge (never seen).
template <typename Loops>
inline int symmetric_eigen_with(double *A, int n, double *w, double *Vt)
{
#pragma clang fp contract(off)
    if (n <= 0) return 0;
    std::vector<double> d(n), e(n > 1 ? n - 1 : 1, 0.0), beta(n, 0.0), p(n), u(n);
    auto row = [&](int i) { return A + (size_t)i * n; };

    // a matrix that is symmetric to the last bit stays so (both triangles get the same two products), and then a product with
    // a column is the product with a row: the sums of several rows at once
    bool exact = true;
    for (int i = 0; i < n && exact; ++i)
        for (int j = 0; j < i; ++j) exact = exact && memcmp(row(i) + j, row(j) + i, sizeof(double)) == 0;

    // ---- Householder reduction: H_k = I - beta_k v_k v_k^T acts on coordinates k+1..n-1 and clears column k
    // below the sub-diagonal.  v_k is kept in row k of A (columns k+1..), which is no longer needed then.
    for (int k = 0; k + 2 < n; ++k) {
        double *x = row(k) + k + 1;                                 // = column k below the diagonal, by symmetry
        const int len = n - k - 1;
        double tail = 0.0;
        for (int i = 1; i < len; ++i) tail += x[i] * x[i];
        d[k] = row(k)[k];
        if (tail == 0.0) {                                          // already tridiagonal here
            e[k] = x[0];
            beta[k] = 0.0;
            continue;
        }
        const double norm = sqrt(x[0] * x[0] + tail);
        const double alpha = x[0] > 0.0 ? -norm : norm;
        e[k] = alpha;
        x[0] -= alpha;                                              // x is v from here on
        const double vv = x[0] * x[0] + tail;
        const double b = 2.0 / vv;
        beta[k] = b;
        // trailing block B = A[k+1.., k+1..]:  B <- B - v q^T - q v^T  with  pv = b B v,  q = pv - (b/2)(v.pv) v
        double vp = 0.0;
        if (exact) {
            Loops::mul(row(k + 1) + k + 1, n, len, x, u.data());
        } else {
            for (int i = 0; i < len; ++i) {
                const double *bi = row(k + 1 + i) + k + 1;
                double s = 0.0;
                for (int j = 0; j < len; ++j) s += bi[j] * x[j];
                u[i] = s;
            }
        }
        for (int i = 0; i < len; ++i) {
            p[i] = b * u[i];
            vp += x[i] * p[i];
        }
        const double kc = 0.5 * b * vp;
        for (int i = 0; i < len; ++i) p[i] -= kc * x[i];
        Loops::rank2(row(k + 1) + k + 1, n, len, x, p.data());
    }
    if (n >= 2) {
        d[n - 2] = row(n - 2)[n - 2];
        e[n - 2] = row(n - 2)[n - 1];
    }
    d[n - 1] = row(n - 1)[n - 1];

    // ---- Q = H_0 H_1 ... H_{n-3}, accumulated from the last reflector backwards into Vt (the part of Q that
    // is not yet the identity is the trailing block, so each step touches only that block); then transposed.
    for (int i = 0; i < n; ++i)
        for (int j = 0; j < n; ++j) Vt[(size_t)i * n + j] = (i == j) ? 1.0 : 0.0;
    for (int k = n - 3; k >= 0; --k) {
        if (beta[k] == 0.0) continue;
        const double *v = row(k) + k + 1;
        const int len = n - k - 1;
        double *Q = Vt + (size_t)(k + 1) * n + k + 1;
        Loops::mul(Q, n, len, v, u.data());
        Loops::rank1(Q, n, len, beta[k], v, u.data());
    }
    for (int i = 0; i < n; ++i)
        for (int j = i + 1; j < n; ++j) std::swap(Vt[(size_t)i * n + j], Vt[(size_t)j * n + i]);

    // ---- implicit-shift QR on the tridiagonal matrix (d, e); rotation of the plane (k, k+1) turns rows k, k+1 of Vt
    const double eps = 2.220446049250313e-16;
    int budget = 64 * n;
    constexpr size_t kQueue = 4096;                                 // rotations applied to Vt in one go, and one sweep more
    std::vector<EigenSweep> sweeps;
    std::vector<double> cs(2 * (kQueue + n));
    size_t queued = 0;
    auto apply = [&]() {
        Loops::rotate(Vt, n, sweeps.data(), sweeps.size(), cs.data());
        sweeps.clear();
        queued = 0;
    };
    for (;;) {
        for (int i = 0; i + 1 < n; ++i)
            if (fabs(e[i]) <= eps * (fabs(d[i]) + fabs(d[i + 1]))) e[i] = 0.0;
        int hi = n - 1;
        while (hi > 0 && e[hi - 1] == 0.0) --hi;
        if (hi == 0) break;
        int lo = hi - 1;
        while (lo > 0 && e[lo - 1] != 0.0) --lo;
        if (--budget < 0) return -1;
        // Wilkinson shift: the eigenvalue of the trailing 2 x 2 block nearer to d[hi]
        const double dd = 0.5 * (d[hi - 1] - d[hi]), off = e[hi - 1];
        const double den = dd + (dd >= 0.0 ? 1.0 : -1.0) * hypot(dd, off);
        const double mu = d[hi] - (den != 0.0 ? off * off / den : 0.0);
        double x = d[lo] - mu, z = e[lo];
        sweeps.push_back({lo, hi, queued});
        for (int k = lo; k < hi; ++k) {
            // c, s with [c s; -s c]^T [x; z] = [r; 0]
            const double r = hypot(x, z);
            const double c = r != 0.0 ? x / r : 1.0, s = r != 0.0 ? -z / r : 0.0;
            if (k > lo) e[k - 1] = r;
            const double a = d[k], b = e[k], g = d[k + 1];
            d[k] = c * c * a - 2.0 * c * s * b + s * s * g;
            d[k + 1] = s * s * a + 2.0 * c * s * b + c * c * g;
            e[k] = c * s * (a - g) + (c * c - s * s) * b;
            if (k + 1 < hi) {
                x = e[k];
                z = -s * e[k + 1];                                  // the bulge at (k, k+2)
                e[k + 1] = c * e[k + 1];
            }
            cs[2 * queued] = c;
            cs[2 * queued + 1] = s;
            ++queued;
        }
        if (queued >= kQueue) apply();
    }
    apply();

    // ---- descending order (equal values keep their order), sign convention
    std::vector<int> order(n);
    std::iota(order.begin(), order.end(), 0);
    std::stable_sort(order.begin(), order.end(), [&](int a, int b) { return d[a] > d[b]; });
    std::vector<double> tmp((size_t)n * n);
    for (int i = 0; i < n; ++i) {
        w[i] = d[order[i]];
        const double *src = Vt + (size_t)order[i] * n;
        double big = 0.0;
        int at = 0;
        for (int j = 0; j < n; ++j)
            if (fabs(src[j]) > big) { big = fabs(src[j]); at = j; }
        const double sg = src[at] < 0.0 ? -1.0 : 1.0;
        for (int j = 0; j < n; ++j) tmp[(size_t)i * n + j] = sg * src[j];
    }
    std::copy(tmp.begin(), tmp.end(), Vt);
    return 0;
}

inline int symmetric_eigen(double *A, int n, double *w, double *Vt)
{
#if defined(__x86_64__) && !defined(__HIP_DEVICE_COMPILE__)
    if (__builtin_cpu_supports("avx512f")) return symmetric_eigen_with<EigenAvx512>(A, n, w, Vt);
    if (__builtin_cpu_supports("avx2")) return symmetric_eigen_with<EigenAvx2>(A, n, w, Vt);
#endif
    return symmetric_eigen_with<EigenBase>(A, n, w, Vt);
}

}  // namespace hclae
