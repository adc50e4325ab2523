// bed_small.hip -- uniform batches of matrices of order n <= 4, one lane per
// matrix: cyclic Jacobi in binary64 (Golub-Van Loan 8.5; the divide step of the
// note hands nodes of this size to it as well, Sec. 2.2), the whole matrix and
// its rotations in registers.  A 64-thread team per matrix, as for larger n,
// leaves almost every lane idle: 65536 matrices of order 4 took it 214 us, and
// take 64 per wave here (about 300 issue cycles a rotation, six rotations a
// sweep, four to five sweeps: 4 us of one wave per SIMD, against 1.7 us for the
// 8.6 MB moved).
#include <hip/hip_runtime.h>

#include "bed_device.hpp"
#include "bed_internal.hpp"

namespace bed {
namespace small {

constexpr int THREADS = 64;
constexpr int SWEEPS = 16;  // cap; four or five suffice

// n x n values of one matrix: 16-byte accesses when its rows allow them.
template <typename T, int N> struct Vec {
    static constexpr int W = (N % (16 / sizeof(T)) == 0) ? 16 / sizeof(T) : 1;
    typedef T type __attribute__((ext_vector_type(W > 1 ? W : 2)));
};

template <typename T, int N>
__device__ __forceinline__ void load(const T *__restrict__ A, const bool wide, T (&a)[N * N])
{
    if constexpr (Vec<T, N>::W > 1) {
        if (wide) {
            constexpr int W = Vec<T, N>::W;
            const auto *p = reinterpret_cast<const typename Vec<T, N>::type *>(A);
#pragma unroll
            for (int q = 0; q < N * N / W; ++q) {
                const typename Vec<T, N>::type v = p[q];
#pragma unroll
                for (int e = 0; e < W; ++e) a[q * W + e] = v[e];
            }
            return;
        }
    }
#pragma unroll
    for (int i = 0; i < N; ++i)
#pragma unroll
        for (int j = 0; j < N; ++j) a[i * N + j] = j <= i ? A[i * N + j] : T(0);
}
template <typename T, int N>
__device__ __forceinline__ void store(T *__restrict__ Q, const bool wide, const T (&q)[N * N])
{
    if constexpr (Vec<T, N>::W > 1) {
        if (wide) {
            constexpr int W = Vec<T, N>::W;
            auto *p = reinterpret_cast<typename Vec<T, N>::type *>(Q);
#pragma unroll
            for (int k = 0; k < N * N / W; ++k) {
                typename Vec<T, N>::type v;
#pragma unroll
                for (int e = 0; e < W; ++e) v[e] = q[k * W + e];
                p[k] = v;
            }
            return;
        }
    }
#pragma unroll
    for (int k = 0; k < N * N; ++k) Q[k] = q[k];
}

// Reciprocal and reciprocal square root to about one ulp of binary64.
__device__ __forceinline__ double rcp2(const double x)
{
    const double r = d_rcp_nr(x);
    return fma(r, fma(-x, r, 1.0), r);
}
__device__ __forceinline__ double rsqrt2(const double x)
{
    const double y = d_rsqrt_nr(x);
    return fma(y, 0.5 * fma(-x * y, y, 1.0), y);
}

template <typename T, int N>
__global__ void __launch_bounds__(THREADS)
k_small(const T *__restrict__ A, int64_t batch, T *__restrict__ lam, T *__restrict__ Q,
        int32_t *__restrict__ info)
{
    const int64_t b = (int64_t)blockIdx.x * THREADS + threadIdx.x;
    if (b >= batch) return;  // (reads no other matrix: with Q == A one may be written by now)
    const T *Ab = A + b * (N * N);
    const bool wide_in = (reinterpret_cast<uintptr_t>(A) & 15) == 0;
    T in[N * N];
    load<T, N>(Ab, wide_in, in);
    // lower triangle; exact scaling to magnitude one (binary64 storage: the
    // squares of binary32 values are in range as they are)
    bool bad = false;
    T amax = T(0);
#pragma unroll
    for (int i = 0; i < N; ++i)
#pragma unroll
        for (int j = 0; j <= i; ++j) {
            bad = bad || !f_finite(in[i * N + j]);
            amax = f_max(amax, f_abs(in[i * N + j]));
        }
    int sh = 0;
    if constexpr (sizeof(T) == 8) {
        const int ex = exp_field(amax);
        sh = ex == 0 ? 0 : fexp<T>::BIAS - 1 - ex;
        sh = min(max(sh, -fexp<T>::SMAX), fexp<T>::SMAX);
    }
    const double sc = sizeof(T) == 8 ? fexp<double>::pow2(sh) : 1.0;
    double a[N][N], v[N][N];
    double f2 = 0.0;
#pragma unroll
    for (int i = 0; i < N; ++i)
#pragma unroll
        for (int j = 0; j < N; ++j) {
            v[i][j] = i == j ? 1.0 : 0.0;
            if (j > i) continue;
            a[i][j] = bad ? 0.0 : sc * double(in[i * N + j]);
            f2 = fma(j < i ? 2.0 * a[i][j] : a[i][j], a[i][j], f2);
        }
    // Sweeps until every off-diagonal entry is below rounding (binary32 storage:
    // 2^-44 of the norm, which the eigenvectors of eigenvalues 2^-20 apart turn
    // into 2^-24).  Each lane stops by itself, so that a matrix's result does not
    // depend on its neighbours; the wave goes on until its last lane has stopped.
    const double thr2 = f2 * (sizeof(T) == 8 ? 0x1p-108 : 0x1p-88);
    for (int sweep = 0; sweep < SWEEPS; ++sweep) {
        double off = 0.0;
#pragma unroll
        for (int p = 0; p < N; ++p)
#pragma unroll
            for (int q = p + 1; q < N; ++q) off = f_max(off, a[q][p] * a[q][p]);
        if (!(off > thr2)) break;
#pragma unroll
        for (int p = 0; p < N; ++p)
#pragma unroll
            for (int q = p + 1; q < N; ++q) {
                // Rutishauser's rotation: t = sgn(d) 2 a_pq / (|d| + sqrt(d^2 +
                // 4 a_pq^2)), d = a_qq - a_pp
                const double apq = a[q][p], d = a[q][q] - a[p][p], w = 2.0 * apq;
                const double h2 = fma(d, d, w * w);
                const bool rot = h2 > 1e-290 && apq != 0.0;
                const double h = h2 * rsqrt2(rot ? h2 : 1.0);
                const double tt = f_copysign(w, d < 0.0 ? -w : w) * rcp2(rot ? f_abs(d) + h : 1.0);
                const double t = rot ? tt : 0.0;
                const double c = rsqrt2(fma(t, t, 1.0)), s = t * c;
                a[p][p] = fma(-t, apq, a[p][p]);
                a[q][q] = fma(t, apq, a[q][q]);
                a[q][p] = rot ? 0.0 : apq;
#pragma unroll
                for (int k = 0; k < N; ++k) {
                    if (k != p && k != q) {
                        double &x = k > p ? a[k][p] : a[p][k];
                        double &y = k > q ? a[k][q] : a[q][k];
                        const double x0 = x, y0 = y;
                        x = fma(c, x0, -s * y0);
                        y = fma(s, x0, c * y0);
                    }
                    const double x0 = v[k][p], y0 = v[k][q];
                    v[k][p] = fma(c, x0, -s * y0);
                    v[k][q] = fma(s, x0, c * y0);
                }
            }
    }
    // ascending order: exchange network over the columns
#pragma unroll
    for (int e = 0; e < N - 1; ++e)
#pragma unroll
        for (int p = 0; p < N - 1 - e; ++p) {
            const bool sw = a[p + 1][p + 1] < a[p][p];
            const double l0 = a[p][p], l1 = a[p + 1][p + 1];
            a[p][p] = sw ? l1 : l0;
            a[p + 1][p + 1] = sw ? l0 : l1;
#pragma unroll
            for (int k = 0; k < N; ++k) {
                const double x0 = v[k][p], x1 = v[k][p + 1];
                v[k][p] = sw ? x1 : x0;
                v[k][p + 1] = sw ? x0 : x1;
            }
        }
    const double us = sizeof(T) == 8 ? fexp<double>::pow2(-sh) : 1.0;
#pragma unroll
    for (int i = 0; i < N; ++i) lam[b * N + i] = bad ? f_nan<T>() : T(us * a[i][i]);
    if (Q) {
        T out[N * N];
#pragma unroll
        for (int j = 0; j < N; ++j) {
            // canonical sign: the largest stored entry (lowest row on ties) positive
            T best = T(-1), val = T(0);
#pragma unroll
            for (int i = 0; i < N; ++i) {
                const T x = T(v[i][j]);
                const bool take = f_abs(x) > best;
                best = take ? f_abs(x) : best;
                val = take ? x : val;
            }
#pragma unroll
            for (int i = 0; i < N; ++i) {
                const T x = T(v[i][j]);
                out[i * N + j] = bad ? f_nan<T>() : (val < T(0) ? -x : x);
            }
        }
        store<T, N>(Q + b * (N * N), (reinterpret_cast<uintptr_t>(Q) & 15) == 0, out);
    }
    if (info) info[b] = bad ? -1 : 0;
}

template <typename T>
hipError_t launch(const void *A, int n, int64_t batch, void *lam, void *Q, int32_t *info,
                  hipStream_t s)
{
    const dim3 grid((unsigned)((batch + THREADS - 1) / THREADS)), block(THREADS);
    switch (n) {
#define X(NN)                                                                                  \
    case NN:                                                                                   \
        hipLaunchKernelGGL((k_small<T, NN>), grid, block, 0, s, (const T *)A, batch, (T *)lam, \
                           (T *)Q, info);                                                      \
        break;
        X(1)
        X(2)
        X(3)
        X(4)
#undef X
    default: return hipErrorInvalidValue;
    }
    return hipGetLastError();
}

}  // namespace small

hipError_t launch_small(bed_dtype dt, const void *A, int n, int64_t batch, void *lam, void *Q,
                        int32_t *info, hipStream_t s)
{
    return dt == BED_F32 ? small::launch<float>(A, n, batch, lam, Q, info, s)
                         : small::launch<double>(A, n, batch, lam, Q, info, s);
}

}  // namespace bed
