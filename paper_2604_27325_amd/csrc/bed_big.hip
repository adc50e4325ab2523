// bed_big.hip -- symmetric matrices of order 64 < n <= 128 in binary32: the
// reduction and the direct solver of n <= 64 laid out for 128 elements.  For
// a spectrum that the direct solver does not take, the divide step of the note
// applies at any size (Sec. 2.1): one tearing step above the n <= 64 solver, whose
// halves then fit a single team, and the top merge (Sec. 2.3) on one 512-thread
// team per matrix.
//
//   k_big_reduce  Householder tridiagonalization T = Q_H^T A Q_H with binary64
//                 arithmetic; with eigenvectors the reflectors go to the workspace
//   k_big_direct  eigenvalues and eigenvectors of T and the back-transform; or
//                 T torn at s = floor(n/2) (Eq. (3)) into T1 (s x s) and T2
//                 ((n-s) x (n-s)), written as their diagonals
//
// and, where a matrix of the batch was torn (the others are passed over; both
// launches are always there, about 4 us each, as the host does not wait to know):
//
//   children      the n <= 64 solver on tridiagonal input (no reduction, no
//                 back-transform) solves T1 and T2; for eigenvalues alone it
//                 returns only the end rows of their eigenvector matrices
//   k_big_merge   z = [sgn(beta) Q1(s-1, :), Q2(0, :)] (Eq. (5)), deflation,
//                 secular roots, Loewner vectors and the merge matrix M;
//                 E = diag(Q1, Q2) M on 16x16x4 MFMA tiles, back-transform of E
// Every kernel fits two teams per CU (at most 80 KB of LDS each).
#include <hip/hip_runtime.h>

#include <algorithm>
#include <cstddef>
#include <mutex>
#include <type_traits>

#include "bed_host.hpp"
#include "bed_internal.hpp"
#include "bed_lru.hpp"
#include "bed_syevd.hpp"

namespace bed {
namespace big {

constexpr int BN = NMAX_BIG;  // largest order
constexpr int BT = 512;       // threads per matrix (8 waves)

struct Meta {
    float beta;  // coupling b_{s-1} of the torn tridiagonal matrix (scaled)
    int shift;   // the matrix was solved as 2^shift A
    int bad;     // non-finite input
    int pad;
};

// Workspace of one batch: children (tridiagonal input, eigenvectors,
// eigenvalues, info), per-matrix meta data and, with eigenvectors, the
// reflectors.  For even n the two children's arrays are
// contiguous (child 2 of matrix b follows all children 1), so one uniform
// launch solves both.
struct Ws {
    float *c1, *c2;  // children (diagonal, then off-diagonal), 2 n1 and 2 n2 values apart
    float *q1, *q2;  // their eigenvectors
    float *l1, *l2;  // their eigenvalues
    int32_t *i1, *i2;
    Meta *meta;
    float *v;    // with eigenvectors: reflectors v_0 .. v_{n-3} (binary32 rows of n)
    float *tau;  // their tau (zero for a skipped step), n per matrix
    double *t;       // T: diagonal, off-diagonal (BN values each)
    int32_t *done;   // per matrix: no divide step (solved by k_big_direct, or non-finite)
    float *e1, *e2;  // eigenvalues only: the children's first and last eigenvector
                     // rows (2 n1 and 2 n2 values apart), in the q1 space
};

// ------------------------------------------------------------------ reduction
constexpr int RT_ = 256;  // threads of a reducing team
constexpr int RHW = RT_ / 64;

// 66 KB, so that two teams share a CU: the load staging and the buffers of the
// steps (a copy of x, by parity, and -w per wave; by parity A x, A e and the
// waves' parts of x^T A x) share the space.
struct RedSmem {
    static constexpr int SLD = BN + 1;  // odd stride
    static constexpr int SZ = HhLds<BN>::SZ;
    union {
        float st[BN * SLD];  // load staging (binary32)
        struct {
            alignas(16) double x[2][RHW][SZ];
            alignas(16) double w[RHW][SZ];
            alignas(16) double y[2][SZ];
            alignas(16) double c[2][SZ];
            alignas(16) double q[2][RHW];
        } s;
    } u;
    int badw[RHW];
    int expw[RHW];
};

// Two rows per lane, 64 positions apart (HhRow for 128 positions).
struct RedRow {
    int p0, p1, s0;
    __device__ __forceinline__ explicit RedRow(const int lane)
    {
        p0 = hh_out_row(lane) + 8 * hh_own<8>(lane);
        p1 = p0 + 64;
        s0 = hh_out_row(lane) * HhLds<BN>::ST + hh_own<8>(lane);  // p1 at s0 + 8
    }
};

struct RedState {
    HhBlock<BN, RHW> H;
    double x0, x1;          // the pivot column at this lane's rows (zero up to the pivot)
    double xl, nwl;         // x and -w of the last step at row p1
};

// Steps whose pivot row lies in chunk B0, then the later chunks.
template <int B0>
__device__ __forceinline__ void red_steps(RedSmem &S, const int n, const int lane, const int wave,
                                          const HhSelect<HhBlock<BN, RHW>::NA> &sel, RedState &R,
                                          float *__restrict__ V, float *__restrict__ tau,
                                          double *__restrict__ T)
{
    using B = HhBlock<BN, RHW>;
    constexpr int A0 = 8 * B0 / B::GI;
    constexpr int ST = HhLds<BN>::ST;
    const int pad = BN - n;
    const RedRow row(lane);
    const int i = 8 * wave + hh_row_of(lane), j = hh_col_of(lane);
    double *W = S.u.s.w[wave];
    const int yslot = hh_out_row(lane) * ST + wave + RHW * hh_own<B::NA>(lane);
    hh_chunk<BN>(B0, pad, [&](const int kp, const int i0) {
        const int k = kp - pad, par = kp & 1;
        const int sp = i0 * ST + B0;
        const double *X = S.u.s.x[par][wave];
        double *Xn = S.u.s.x[par ^ 1][wave];  // the last step's x, then the next one's
        wave_sync();
        const double x0 = X[sp];
        const bool l0 = row.p0 > kp + 1, l1 = row.p1 > kp + 1;
        const double sig = wave_sum_all(fma(l0 ? R.x0 : 0.0, R.x0, l1 ? R.x1 * R.x1 : 0.0));
        double y[B::NA];
        double q = R.H.template step<A0, B0>(X, W, Xn, S.u.s.c[par], i, j, i0, y);
        const double yo = hh_reduce_scatter<B::NA, A0>(y, sel, lane);
        q = wave_sum_all(q);
        S.u.s.y[par][yslot] = yo;
        S.u.s.q[par][wave] = q;
        const HhRefl<float> h = hh_reflector<float>(x0, sig);
        const double xt0 = x0 - h.alpha, hb = 0.5 * h.beta * h.beta;
        __syncthreads();
        const double *Y = S.u.s.y[par], *C = S.u.s.c[par];
        const double y0 = Y[row.s0], y1 = Y[row.s0 + 8], c0 = C[row.s0], c1 = C[row.s0 + 8];
        const double s1 = Y[sp], a00 = C[sp];
        double qs = S.u.s.q[par][0];
#pragma unroll
        for (int w2 = 1; w2 < RHW; ++w2) qs += S.u.s.q[par][w2];
        const HhStep o0 = hh_step(R.x0, y0, c0, s1, a00, qs, h.alpha, h.beta, hb, xt0);
        const HhStep o1 = hh_step(R.x1, y1, c1, s1, a00, qs, h.alpha, h.beta, hb, xt0);
        if (wave == (kp & (RHW - 1))) {  // the waves take the steps' outputs in turn
            if (V) {
                // reflector k, normalized to v_{k+1} = 1
                const float v0 = float(row.p0 == kp + 1 ? 1.0 : R.x0 * h.rx0);
                const float v1 = float(row.p1 == kp + 1 ? 1.0 : R.x1 * h.rx0);
                if (row.p0 >= pad) V[(int64_t)k * n + row.p0 - pad] = v0;
                V[(int64_t)k * n + row.p1 - pad] = v1;
                if (lane == 0) tau[k] = float(h.tau);
            }
            if (lane == 0) {
                T[BN + k] = h.alpha;
                T[k + 1] = fma(-2.0 * xt0, o0.w0, a00);
            }
        }
        R.xl = R.x1;
        R.nwl = o1.nw;
        R.x0 = l0 ? o0.xn : 0.0;
        R.x1 = l1 ? o1.xn : 0.0;
        W[row.s0] = o0.nw;
        W[row.s0 + 8] = o1.nw;
        Xn[row.s0] = R.x0;
        Xn[row.s0 + 8] = R.x1;
    });
    if constexpr (B0 + 1 < BN / 8) red_steps<B0 + 1>(S, n, lane, wave, sel, R, V, tau, T);
}

// Householder tridiagonalization in binary64 as for n <= 64 (hh_product), on
// four waves that all form the norm and the reflector: a control wave would
// share a SIMD with a product wave, whose issue bounds the step (about 270
// instructions a wave and step at the start, two waves per SIMD with two teams
// per CU).  One barrier per step instead of three, and each lane's 4 x 16 block
// shrinks in both directions.  With eigenvectors the reflectors (rounded to
// binary32) and their tau go to the workspace for the back-transform.
__global__ void __launch_bounds__(RT_, 2)
k_big_reduce(const float *__restrict__ A, int n, int64_t batch, Ws ws)
{
    __shared__ RedSmem S;
    const int64_t bi = blockIdx.x;
    if (bi >= batch) return;
    const int t = threadIdx.x, lane = t & 63, wave = __builtin_amdgcn_readfirstlane(t >> 6);
    const float *Ab = A + bi * n * n;
    constexpr int SLD = RedSmem::SLD;
    bool bad = false;
    float amax = 0.f;
    {
        // lane (j, i0) = (t % BN, t / BN) stages rows i0, i0 + 2, ... at column j,
        // sixteen loads issued before the first LDS write
        constexpr int RS = RT_ / BN, RPL = BN / RS, LB = 16;
        const int j = t & (BN - 1), i0 = t / BN;
#pragma unroll 1
        for (int q0 = 0; q0 < RPL; q0 += LB) {
            float ld[LB];
#pragma unroll
            for (int q = 0; q < LB; ++q) {
                const int i = i0 + RS * (q0 + q);
                ld[q] = Ab[(i < n && j <= i) ? i * n + j : 0];  // lower triangle, clamped
            }
#pragma unroll
            for (int q = 0; q < LB; ++q) {
                const int i = i0 + RS * (q0 + q);
                const bool in = i < n && j <= i;
                bad = bad || (in && !f_finite(ld[q]));
                amax = in ? f_max(amax, f_abs(ld[q])) : amax;
                S.u.st[i * SLD + j] = ld[q];
            }
        }
        const bool wb = __ballot(bad) != 0;
        const int we = group_max<64>(exp_field(amax), lane);
        if (lane == 0) {
            S.badw[wave] = wb ? 1 : 0;
            S.expw[wave] = we;
        }
    }
    __syncthreads();
    int anybad = 0, emax = 0;
#pragma unroll
    for (int w = 0; w < RHW; ++w) {
        anybad |= S.badw[w];
        emax = max(emax, S.expw[w]);
    }
    // exact power-of-two scaling to max |a_ij| in [1/2, 1), as for n <= 64
    int sh = (emax == 0) ? 0 : fexp<float>::BIAS - 1 - emax;
    sh = min(max(sh, -fexp<float>::SMAX), fexp<float>::SMAX);
    if (anybad) {
        if (t == 0) {
            ws.meta[bi] = Meta{0.f, 0, 1, 0};
            ws.done[bi] = 1;
        }
        return;
    }
    const double hs = double(fexp<float>::pow2(sh));
    const int pad = BN - n;
    using B = HhBlock<BN, RHW>;
    RedState R;
    const RedRow row(lane);
    {
        auto entry = [&](const int pr, const int pc) {  // lower triangle, zero in the padding
            const int hi = max(pr, pc) - pad, lo = min(pr, pc) - pad;
            const float v = S.u.st[lo >= 0 ? hi * SLD + lo : 0];
            return lo >= 0 ? hs * double(v) : 0.0;
        };
        const int i = 8 * wave + hh_row_of(lane), j = hh_col_of(lane);
#pragma unroll
        for (int a = 0; a < B::NA; ++a) {
#pragma unroll
            for (int b = 0; b < B::NB; ++b) R.H.a[a][b] = entry(i + B::GI * a, j + 8 * b);
        }
        const double e0 = entry(row.p0, pad), e1 = entry(row.p1, pad);
        R.x0 = row.p0 > pad ? e0 : 0.0;
        R.x1 = e1;  // p1 >= 64 > pad
        if (t == 0) ws.t[bi * 2 * BN] = hs * double(S.u.st[0]);
    }
    R.xl = R.nwl = 0.0;
    __syncthreads();  // the staging buffer becomes the step buffers
    S.u.s.w[wave][row.s0] = S.u.s.w[wave][row.s0 + 8] = 0.0;
    {
        const int par = pad & 1;
        S.u.s.x[par][wave][row.s0] = R.x0;
        S.u.s.x[par][wave][row.s0 + 8] = R.x1;
        S.u.s.x[par ^ 1][wave][row.s0] = S.u.s.x[par ^ 1][wave][row.s0 + 8] = 0.0;
    }
    const HhSelect<B::NA> sel(lane);
    red_steps<0>(S, n, lane, wave, sel, R, ws.v ? ws.v + bi * (n - 2) * n : nullptr,
                 ws.tau ? ws.tau + bi * n : nullptr, ws.t + bi * 2 * BN);
    // b_{n-2} is the pivot column's last value, a_{n-1} the last diagonal entry
    // after the last update (position BN - 1: lane 63 of the last wave)
    if (wave == RHW - 1 && lane == 63) {
        double *T = ws.t + bi * 2 * BN;
        T[BN + n - 2] = R.x1;
        T[n - 1] = fma(2.0 * R.xl, R.nwl, R.H.a[B::NA - 1][B::NB - 1]);
        ws.meta[bi] = Meta{0.f, sh, 0, 0};
    }
}

// ------------------------------------------------------------------ back-transform
// Q = H_0 H_1 ... H_{n-3} V in compact-WY blocks of 16 reflectors,
// H_{16b} ... H_{16b+15} = I - V_b T_b V_b^T (T_b upper triangular), applied
// for b = last .. 0 on 16x16x4 binary64 MFMA tiles; Q_H is never formed.  The
// reflectors come rounded to binary32 (exact to convert back) and are staged
// in LDS at odd stride; the binary64 Gram matrices G_b = V_b^T V_b of the
// rounded reflectors and then the T factors sit in packed upper triangles
// (element (i, j) at j (j + 1) / 2 + i).  T is formed with tau_j = 2 / G(j, j),
// so each block is exactly orthogonal for the reflectors as stored, up to
// binary64 rounding; only the final binary32 rounding of Q remains
// (binary32 products here would add a few 1e-6 to ||Q^T Q - I||_F at n = 128).
// One wave per block forms G_b and T_b; after one barrier each wave keeps its
// 16 columns in accumulators through all blocks, so the sign rule needs no
// other wave.  Bound by the binary64 matrix rate: 320 products of 16x16x4 a
// wave at n = 128, 20 us a team.  (Q_H formed first and multiplied in binary32 took
// the same matrix time, 53 us more for Q_H's kernel, and twice the error.)
struct BackSmem {
    static constexpr int VLD = BN + 1;
    static constexpr int TP = 136;  // packed 16 x 16 upper triangle
    static constexpr int TF = (BN / 16) * TP;
    float V[BN * VLD];
    double tf[TF];  // G_b, then T_b
};

// This wave's 16 columns of the eigenvectors of T; at(i, j) is entry i of vector j.
template <typename At>
__device__ __forceinline__ void back_load(Mf<double>::acc (&qa)[BN / 16], const int n, const int t,
                                          const At &at)
{
    const int lane = t & 63, c = 16 * (t >> 6) + (lane & 15);
#pragma unroll
    for (int rt = 0; rt < BN / 16; ++rt)
#pragma unroll
        for (int v = 0; v < 4; ++v) {
            const int r = 16 * rt + Mf<double>::crow(lane, v);
            const bool in = r < n && c < n;
            const double q = at(in ? r : 0, in ? c : 0);
            qa[rt][v] = in ? q : 0.0;
        }
}

// The nb x n reflector block, loaded ahead of the space that it is staged in: lane
// (j, i0) = (t % BN, t / BN) takes rows i0, i0 + 4, ... at column j.
constexpr int BACK_RPL = BN * BN / BT, BACK_RS = BT / BN;
__device__ __forceinline__ void back_fetch(float (&ld)[BACK_RPL], const float *__restrict__ Vb,
                                           const int n, const int t)
{
    const int j = t & (BN - 1), i0 = t / BN;
#pragma unroll
    for (int q = 0; q < BACK_RPL; ++q) {
        const int i = i0 + BACK_RS * q;
        ld[q] = Vb[(i < n - 2 && j < n) ? i * n + j : 0];
    }
}
__device__ __forceinline__ void back_stage(float *V, const float (&ld)[BACK_RPL], const int n,
                                           const int t)
{
    const int j = t & (BN - 1), i0 = t / BN;
#pragma unroll
    for (int q = 0; q < BACK_RPL; ++q) {
        const int i = i0 + BACK_RS * q;
        V[i * BackSmem::VLD + j] = (i < n - 2 && j < n) ? ld[q] : 0.f;
    }
}

// V, tf: as in BackSmem (the caller has put a barrier behind the last use of the
// space); ld, tau: the matrix's reflectors.
__device__ __forceinline__ void back_transform(float *V, double *tf, Mf<double>::acc (&qa)[BN / 16],
                                               const float (&ld)[BACK_RPL],
                                               const float *__restrict__ tau, const int n,
                                               const int t, float *__restrict__ Qb)
{
    using MF = Mf<double>;
    constexpr int VLD = BackSmem::VLD;
    constexpr int TP = BackSmem::TP;
    const int lane = t & 63, wave = t >> 6;
    const int nb = n - 2;  // reflectors
    const int NB = (nb + 15) / 16;
    back_stage(V, ld, n, t);
    __syncthreads();
    auto tix = [](int i, int j) { return ((j * (j + 1)) >> 1) + i; };  // i <= j
    const int i16 = lane & 15;
    for (int bk = wave; bk < NB; bk += BT / 64) {
        const int k0 = 16 * bk;
        double *tb = tf + bk * TP;
        // G_b: one MFMA chain per row tile at or below the block (rows <= k0 of
        // its reflectors are zero), summed
        MF::acc g = MF::zero();
#pragma unroll
        for (int rt = 0; rt < BN / 16; ++rt) {
            if (rt < bk || 16 * rt >= n) continue;
            MF::acc gt = MF::zero();
#pragma unroll
            for (int s4 = 0; s4 < 4; ++s4) {
                const double vv = V[(k0 + i16) * VLD + 16 * rt + MF::crow(lane, s4)];
                gt = MF::mma(vv, vv, gt);
            }
            g += gt;
        }
#pragma unroll
        for (int v = 0; v < 4; ++v) {
            const int gr = MF::crow(lane, v);
            if (gr <= i16) tb[tix(gr, i16)] = g[v];
        }
        wave_sync();
        // T_b: T(j, j) = tau_j, T(0:j, j) = -tau_j T(0:j, 0:j) G(0:j, j); lane i <
        // 16 forms row i, then (all reads of G_b done) writes it over G_b
        // tau_j = 2 / G(j, j) on lane j (zero marks a skipped step: v = e_{k+1}
        // stored, no reflection), then broadcast
        double tl = 0.0;
        if (lane < 16 && k0 + lane < nb && tau[k0 + lane] != 0.f)
            tl = 2.0 / tb[tix(lane, lane)];
        if (lane < 16) {
            double trow[16];
#pragma unroll
            for (int j = 0; j < 16; ++j) {
                const double tj = __shfl(tl, j);
                // column j's loads are made to wait for T(i, j - 1) through an
                // empty asm (hoisting all 120 would exhaust the registers)
                int cb = tix(0, j);
                if (j > 0) asm volatile("" : "+v"(cb) : "v"(trow[j - 1]));
                double acc = 0.0;
#pragma unroll
                for (int kk = 0; kk < j; ++kk) acc = fma(trow[kk], tb[cb + kk], acc);
                trow[j] = (lane < j) ? -tj * acc : (lane == j ? tj : 0.0);
            }
            wave_sync();
#pragma unroll
            for (int j = 0; j < 16; ++j)
                if (lane <= j) tb[tix(lane, j)] = trow[j];
        }
    }
    __syncthreads();
    if (16 * wave >= n) return;
    for (int bk = NB - 1; bk >= 0; --bk) {
        const int k0 = 16 * bk;
        // X = V_b^T Q (16 x 16 tile of this column block); staged rows past the
        // last reflector are zero
        MF::acc xp[2] = {MF::zero(), MF::zero()};  // two chains (MFMA latency)
#pragma unroll
        for (int rt = 0; rt < BN / 16; ++rt) {
            if (rt < bk || 16 * rt >= n) continue;
#pragma unroll
            for (int s4 = 0; s4 < 4; ++s4) {
                const double va = V[(k0 + i16) * VLD + 16 * rt + MF::crow(lane, s4)];
                xp[rt & 1] = MF::mma(va, qa[rt][s4], xp[rt & 1]);
            }
        }
        MF::acc x;
#pragma unroll
        for (int v = 0; v < 4; ++v) x[v] = xp[0][v] + xp[1][v];
        // Y = T_b X
        MF::acc y = MF::zero();
#pragma unroll
        for (int s4 = 0; s4 < 4; ++s4) {
            const int kk = MF::crow(lane, s4);
            const double ta = (kk >= i16) ? tf[bk * TP + tix(i16, kk)] : 0.0;
            y = MF::mma(ta, x[s4], y);
        }
        // Q -= V_b Y (its operand loads are not hoisted above X: the register
        // budget holds one product's operands at a time)
        __builtin_amdgcn_sched_barrier(0);
#pragma unroll
        for (int rt = 0; rt < BN / 16; ++rt) {
            if (rt < bk || 16 * rt >= n) continue;
#pragma unroll
            for (int s4 = 0; s4 < 4; ++s4) {
                const double vb = -double(V[(k0 + MF::crow(lane, s4)) * VLD + 16 * rt + i16]);
                qa[rt] = MF::mma(vb, y[s4], qa[rt]);
            }
        }
    }
    // sign rule: the entry of largest magnitude (lowest row on ties) is positive
    const int c = 16 * wave + i16;
    float best = -1.f, bval = 0.f;
    int brow = 1 << 20;
#pragma unroll
    for (int rt = 0; rt < BN / 16; ++rt)
#pragma unroll
        for (int v = 0; v < 4; ++v) {
            const int row = 16 * rt + MF::crow(lane, v);
            const float q = float(qa[rt][v]), av = f_abs(q);
            const bool take = row < n && av > best;
            best = take ? av : best;
            brow = take ? row : brow;
            bval = take ? q : bval;
        }
    auto least = [&](const float ob, const int orow, const float oval) {
        const bool take = ob > best || (ob == best && orow < brow);
        best = take ? ob : best;
        brow = take ? orow : brow;
        bval = take ? oval : bval;
    };
    least(xmove<16>(best, lane), xmove<16>(brow, lane), xmove<16>(bval, lane));
    least(xmove<32>(best, lane), xmove<32>(brow, lane), xmove<32>(bval, lane));
    const float sgn = bval < 0.f ? -1.f : 1.f;
#pragma unroll
    for (int rt = 0; rt < BN / 16; ++rt)
#pragma unroll
        for (int v = 0; v < 4; ++v) {
            const int row = 16 * rt + MF::crow(lane, v);
            if (row < n && c < n) Qb[row * n + c] = sgn * float(qa[rt][v]);
        }
}

// ------------------------------------------------------------------ direct solve
struct DirSmem {
    static constexpr int LD = BN / 2 + 1;
    union {
        struct {
            union {
                // factors from the top and from the bottom of half the
                // eigenvectors, then the eigenvectors of T, a half each
                float L[2][BN * LD];
                struct {
                    double a[BN], b[BN];
                } t;               // T, until it is set up
                DirectGrid<BT> g;  // during the first grid
            } u;
            DirectArrays<BN> t;
        } d;
        BackSmem q;
    } u;
    float lout[BN];
};

// The spectrum of T directly, as for n <= 64 (direct_solve), and the back-transform;
// a matrix that it does not take is torn at s = floor(n/2) (Eq. (3)) for
// the children and the top merge.  The eigenvectors are formed in two halves of
// 64 columns, whose factors leave room (76 KB) for two teams per CU: one team's
// serial factorizations run beside the other's matrix products and sections.
// Batch 512, n = 128: 140 us for the 241 that forming Q_H, the children and the top
// merge took; 38 without eigenvectors, for 186.  No unit is full: counted with 10%
// planted pairs (159 us), each SIMD issues vector instructions for 64 us (a third of
// them binary64) and its matrix core is busy for 36; the waves wait for half of their
// cycles, in the sections' and the factors' dependent chains.
__global__ void __launch_bounds__(BT, 4)  // two teams per CU
k_big_direct(int n, int64_t batch, float *__restrict__ lam, float *__restrict__ Q,
             int32_t *__restrict__ info, Ws ws)
{
    __shared__ DirSmem S;
    const int64_t bi = blockIdx.x;
    if (bi >= batch) return;
    if (ws.meta[bi].bad) return;  // the merge writes NaN
    const int t = threadIdx.x, lane = t & 63, wave = __builtin_amdgcn_readfirstlane(t >> 6);
    constexpr int LD = DirSmem::LD;
    auto &L = S.u.d.u.L;
    DirectArrays<BN> &D = S.u.d.t;
    const double *T = ws.t + bi * 2 * BN;
    if (t < n) {
        S.u.d.u.t.a[t] = T[t];
        S.u.d.u.t.b[t] = t + 1 < n ? T[BN + t] : 0.0;
    }
    __syncthreads();
    if (wave == 0) direct_setup<BN, BT / BN>(D, S.u.d.u.t.a, S.u.d.u.t.b, n, lane, Q != nullptr);
    __syncthreads();
    if (!direct_eigenvalues<BN, BT>(D, S.u.d.u.g, n, t, Q != nullptr, S.lout)) {
        const int n1 = n / 2, n2 = n - n1;
        const float beta = float(T[BN + n1 - 1]);
        const float rho = f_abs(beta);
        float *C1 = ws.c1 + bi * 2 * n1;
        float *C2 = ws.c2 + bi * 2 * n2;
        for (int e = t; e < 2 * n1 - 1; e += BT)
            C1[e] = (e < n1) ? float(T[e]) - (e == n1 - 1 ? rho : 0.f) : float(T[BN + e - n1]);
        for (int e = t; e < 2 * n2 - 1; e += BT)
            C2[e] = (e < n2) ? float(T[n1 + e]) - (e == 0 ? rho : 0.f)
                             : float(T[BN + n1 + e - n2]);
        if (t == 0) {
            ws.meta[bi].beta = beta;
            ws.done[bi] = 0;
        }
        return;
    }
    const float unscale = fexp<float>::pow2(-ws.meta[bi].shift);
    if (t < n) lam[bi * n + t] = unscale * S.lout[t];
    if (t == 0) {
        ws.done[bi] = 1;
        if (info) info[bi] = 0;
    }
    if (!Q) return;
    constexpr int HC = BN / 2, LPR = BT / HC, SG = BN / LPR;
    const int j = t / LPR, i0 = (t % LPR) * SG;
    float z0[SG], z[SG] = {};  // the first and the second half's entries
#pragma unroll 1
    for (int h = 0; h < 2; ++h) {
#pragma unroll
        for (int s = 0; s < SG; ++s) z0[s] = z[s];
        // a serial chain: ahead of the other team's matrix products (25 us behind
        // them, 10 so)
        __builtin_amdgcn_s_setprio(3);
        direct_factors<BN, BT, HC, BT / BN, LD>(D, L[0], L[1], n, t, HC * h);
        __builtin_amdgcn_s_setprio(0);
        __syncthreads();
        // opaque: rows and bounds are formed here, not kept through the factors
        int th = t, nh = n;
        asm volatile("" : "+v"(th), "+s"(nh));
        const bool act = HC * h + th / LPR < nh;
        const int e = act ? th / LPR : 0;
        direct_vector<BN, LPR, LD>(D, L[0] + e, L[1] + e, HC * h + e, act, nh, th, z);
        __syncthreads();
    }
#pragma unroll
    for (int s = 0; s < SG; ++s) {
        L[0][(i0 + s) * LD + j] = z0[s];
        L[1][(i0 + s) * LD + j] = z[s];
    }
    __syncthreads();
    auto at = [&](const int i, const int j) -> float & { return L[j >= HC][i * LD + (j & (HC - 1))]; };
    if (direct_close(D)) {
        if (wave == 0) direct_orthogonal(D, n, lane, at);
        __syncthreads();
    }
    float ld[BACK_RPL];
    back_fetch(ld, ws.v + bi * (n - 2) * n, n, t);
    Mf<double>::acc qa[BN / 16];
    back_load(qa, n, t, at);
    __syncthreads();
    back_transform(S.u.q.V, S.u.q.tf, qa, ld, ws.tau + bi * n, n, t, Q + bi * n * n);
}

// ------------------------------------------------------------------ top merge
struct MrgSmem {
    static constexpr int LD = BN + 1;  // odd stride; column BN is the padding column of M
    // rows 0 and 1 first hold the children's eigenvalues and z; then the
    // merge matrix M; then E = diag(Q1, Q2) M; then the reflectors
    float M[BN * LD];
    union {
        MergeArrays<float, BN> m;
        double tf[BackSmem::TF];
    } u;
    float lout[BN];  // eigenvalues, ascending
    float red[4][2];
    uint64_t live[2], dead[2], cmask[2];
    int capped, anyrot;
};

__global__ void __launch_bounds__(BT, 4)  // two teams per CU
k_big_merge(int n, int64_t batch, float *__restrict__ lam, float *__restrict__ Q,
            int32_t *__restrict__ info, Ws ws)
{
    __shared__ MrgSmem S;
    constexpr int LD = MrgSmem::LD;
    const int64_t bi = blockIdx.x;
    if (bi >= batch) return;
    const int t = threadIdx.x, lane = t & 63, wave = t >> 6;
    const int s = n / 2, n1 = s, n2 = n - s;
    const Meta md = ws.meta[bi];
    float *Qb = Q ? Q + bi * n * n : nullptr;
    if (md.bad) {
        if (Qb)
            for (int e = t; e < n * n; e += BT) Qb[e] = f_nan<float>();
        for (int e = t; e < n; e += BT) lam[bi * n + e] = f_nan<float>();
        if (t == 0 && info) info[bi] = -1;
        return;
    }
    if (ws.done[bi]) return;
    const float *Q1 = ws.q1 + bi * n1 * n1;
    const float *Q2 = ws.q2 + bi * n2 * n2;
    const float rho = f_abs(md.beta);
    const float sgm = (md.beta < 0.f) ? -1.f : 1.f;
    // the children's eigenvalues, and z (Eq. (5)): sgn(beta) times the last
    // row of Q1 over the first row of Q2, into rows 0 and 1 of M
    float *lamc = S.M, *zin = S.M + LD;
    if (t < n) {
        lamc[t] = (t < n1) ? ws.l1[bi * n1 + t] : ws.l2[bi * n2 + t - n1];
        if (Qb)
            zin[t] = (t < n1) ? sgm * Q1[(n1 - 1) * n1 + t] : Q2[t - n1];
        else  // the children's end rows (last row of Q1 second, first row of Q2 first)
            zin[t] = (t < n1) ? sgm * ws.e1[bi * 2 * n1 + n1 + t] : ws.e2[bi * 2 * n2 + t - n1];
    }
    if (t == 0) {
        S.capped = 0;
        S.anyrot = 0;
    }
    __syncthreads();
    // stable merge of the two ascending child lists
    if (t < n) {
        const float de = lamc[t], ze = zin[t];
        const bool left = t < n1;
        const int pos = (left ? t : t - n1) +
                        count_below(lamc + (left ? n1 : 0), left ? n2 : n1, de, !left);
        S.u.m.sd[pos] = de;
        S.u.m.sz[pos] = ze;
        S.u.m.sperm[pos] = t;
    }
    __syncthreads();
    for (int e = t; e < BN * LD; e += BT) S.M[e] = 0.f;  // the merge matrix, zero padded
    __syncthreads();

    // ---- deflation (type 1: rho |z_i| <= tol; type 2: Givens rotation of a
    // close pair), tol = 8u max(max |d|, rho z^T z), as for n <= 64 ----------
    const bool act = t < n;
    float dp = act ? S.u.m.sd[t] : 0.f, zp = act ? S.u.m.sz[t] : 0.f;
    if (wave < 2) {
        const float v0 = wave_total(zp * zp), v1 = wave_total(dp * zp * zp), v2 = wave_total(dp * dp);
        if (lane == 0) {
            S.red[0][wave] = v0;
            S.red[1][wave] = v1;
            S.red[2][wave] = v2;
        }
    }
    __syncthreads();
    const float zz0 = S.red[0][0] + S.red[0][1];
    const float dz = S.red[1][0] + S.red[1][1];
    const float d2 = S.red[2][0] + S.red[2][1];
    const float dmax = f_max(f_abs(S.u.m.sd[0]), f_abs(S.u.m.sd[n - 1]));
    const float u = fp<float>::u;
    const float tol = 8.f * u * f_max(dmax, rho * zz0);
    const float fro2 = d2 + 2.f * rho * dz + rho * rho * zz0 * zz0;  // ||node||_F^2 (Eq. (10))
    bool defl = act && (rho * f_abs(zp) <= tol);
    if (defl) zp = 0.f;
    if (act) {
        S.u.m.sdefl[t] = defl ? 1 : 0;
        S.u.m.sz[t] = zp;
        S.u.m.rpart[t] = -1;
    }
    {
        const uint64_t lv = __ballot(act && !defl);
        if (wave < 2 && lane == 0) S.live[wave] = lv;
    }
    __syncthreads();
    // Pairs of consecutive live elements that may pass the type-2 test (with
    // a factor 2 of slack for the different rounding of this test) mark their
    // second element as a candidate.
    bool cand = false;
    if (act && !defl) {
        const uint64_t l0 = S.live[0], l1 = S.live[1];
        int prev = -1;
        if (t >= 64) {
            const uint64_t bl = l1 & lane_range(0, t - 64);
            prev = bl ? 64 + 63 - __clzll(bl) : (l0 ? 63 - __clzll(l0) : -1);
        } else {
            const uint64_t bl = l0 & lane_range(0, t);
            prev = bl ? 63 - __clzll(bl) : -1;
        }
        if (prev >= 0) {
            const float zpr = S.u.m.sz[prev], dpr = S.u.m.sd[prev];
            const float rr = f_hypot(zpr, zp);
            cand = f_abs((dp - dpr) * (zp / rr) * (zpr / rr)) <= 2.f * tol;
        }
    }
    {
        const uint64_t cm = __ballot(cand);
        if (wave < 2 && lane == 0) S.cmask[wave] = cm;
    }
    __syncthreads();
    if (t == 0) {
        // The exact sequential scan over consecutive live pairs (last, p) in
        // ascending order changes something only at a pair that passes the
        // test.  A pair whose `last` no rotation has touched and that is not
        // a candidate fails it, so only candidates and the successor of each
        // rotated element are visited (as for n <= 64), each decided by the
        // exact test.  Element masks are two 64-bit words.
        uint64_t lv0 = S.live[0], lv1 = S.live[1];
        uint64_t cm0 = S.cmask[0], cm1 = S.cmask[1];
        auto lowest = [](uint64_t a0, uint64_t a1) {
            return a0 ? __builtin_ctzll(a0) : (a1 ? 64 + __builtin_ctzll(a1) : 128);
        };
        int nr = 0, mod = -1;  // mod: element changed by the latest rotation
        for (;;) {
            int succ = 128;
            if (mod >= 0) {  // first live element after mod
                const uint64_t a0 = (mod < 63) ? (lv0 & ~lane_range(0, mod + 1)) : 0ull;
                const uint64_t a1 = (mod < 63) ? lv1 : (lv1 & ~lane_range(0, mod - 63));
                succ = lowest(a0, a1);
            }
            const int p = min(succ, lowest(cm0, cm1));
            if (p >= n) break;
            if (p < 64) cm0 &= ~(1ull << p);
            else cm1 &= ~(1ull << (p - 64));
            // last live element before p
            int last = -1;
            if (p > 64) {
                const uint64_t b1 = lv1 & lane_range(0, p - 64);
                last = b1 ? 64 + 63 - __builtin_clzll(b1) : (lv0 ? 63 - __builtin_clzll(lv0) : -1);
            } else {
                const uint64_t b0 = lv0 & lane_range(0, p);
                last = b0 ? 63 - __builtin_clzll(b0) : -1;
            }
            if (last < 0) {
                mod = -1;
                continue;
            }
            const float zl = S.u.m.sz[last], zi = S.u.m.sz[p];
            const float dl = S.u.m.sd[last], di = S.u.m.sd[p];
            const float rr = f_hypot(zl, zi);
            const float c = zi / rr, sn = zl / rr;
            if (f_abs((di - dl) * c * sn) <= tol) {
                S.u.m.sd[last] = dl * c * c + di * sn * sn;
                S.u.m.sd[p] = dl * sn * sn + di * c * c;
                S.u.m.sz[last] = 0.f;
                S.u.m.sz[p] = rr;
                S.u.m.sdefl[last] = 1;
                S.u.m.rc[last] = c;
                S.u.m.rs[last] = sn;
                S.u.m.rpart[last] = p;
                S.u.m.rlist[nr++] = last;
                if (last < 64) lv0 &= ~(1ull << last);
                else lv1 &= ~(1ull << (last - 64));
                mod = p;
            } else {
                mod = -1;
            }
        }
        S.u.m.nrot[0] = nr;
        S.anyrot = nr > 0 ? 1 : 0;
    }
    __syncthreads();
    // compaction: non-deflated (poles, weights, child-order rows) first, then
    // the deflated items
    if (act) {
        dp = S.u.m.sd[t];
        zp = S.u.m.sz[t];
        defl = S.u.m.sdefl[t] != 0;
    }
    {
        const uint64_t lv = __ballot(act && !defl), dv = __ballot(act && defl);
        if (wave < 2 && lane == 0) {
            S.live[wave] = lv;
            S.dead[wave] = dv;
        }
        if (wave < 2) {
            const float zz = wave_total((act && !defl) ? zp * zp : 0.f);
            if (lane == 0) S.red[3][wave] = zz;
        }
    }
    __syncthreads();
    const uint64_t L0 = S.live[0], L1 = S.live[1], D0 = S.dead[0], D1 = S.dead[1];
    const int k = __popcll(L0) + __popcll(L1);
    if (act) {
        const int row = S.u.m.sperm[t];
        if (!defl) {
            const int idx = (t < 64) ? __popcll(L0 & lane_range(0, t))
                                     : __popcll(L0) + __popcll(L1 & lane_range(0, t - 64));
            S.u.m.dk[idx] = dp;
            S.u.m.zk[idx] = zp;
            S.u.m.ndrow[idx] = row;
        } else {
            const int idx = k + ((t < 64) ? __popcll(D0 & lane_range(0, t))
                                          : __popcll(D0) + __popcll(D1 & lane_range(0, t - 64)));
            S.u.m.itv[idx] = dp;
            S.u.m.itrow[idx] = row;
        }
    }
    __syncthreads();
    if (t == 0) {
        S.u.m.nk[0] = k;
        S.u.m.nrho[0] = rho;
        S.u.m.nzz[0] = S.red[3][0] + S.red[3][1];
        S.u.m.nfro[0] = f_sqrt(f_max(fro2, 0.f));
        S.u.m.nback[0] = 1.f;
    }
    __syncthreads();

    // ---- secular roots, Loewner vectors, merge matrix (one node, depth 0) --
    roots_vectors<float, BN, BT, BN / (BT / BN)>(S, n, 0, t, S.lout, BN / 2);

    // ---- Q = Q_H (diag(Q1, Q2) M) with the sign rule ------------------------
    const float unscale = fexp<float>::pow2(-md.shift);
    for (int e = t; e < n; e += BT) lam[bi * n + e] = unscale * S.lout[e];
    if (t == 0 && info) info[bi] = S.capped + ws.i1[bi] + ws.i2[bi];
    // Wave w takes row tile w of E = diag(Q1, Q2) M on 16x16x4 MFMA tiles, its A
    // rows loaded from HBM into registers, B from LDS; E replaces M.
    if (Qb) {
        using MF = Mf<float>;
        constexpr int KS = BN / 4;  // k steps
        const int i16 = lane & 15, kk = lane >> 4;
        const int r = 16 * wave + i16;  // this lane's A row
        const bool rows = 16 * wave < n;
        f32x4 acc[BN / 16];
        float a[KS];
        if (rows) {
            // loads from clamped addresses (Q1[0] outside both blocks), the
            // zeros selected afterwards
#pragma unroll
            for (int s4 = 0; s4 < KS; ++s4) {
                const int k = 4 * s4 + kk;
                const bool b1 = r < n1 && k < n1;
                const bool b2 = r >= n1 && r < n && k >= n1 && k < n;
                a[s4] = *(b1 ? Q1 + r * n1 + k : (b2 ? Q2 + (r - n1) * n2 + (k - n1) : Q1));
            }
#pragma unroll
            for (int s4 = 0; s4 < KS; ++s4) {
                const int k = 4 * s4 + kk;
                const bool b1 = r < n1 && k < n1;
                const bool b2 = r >= n1 && r < n && k >= n1 && k < n;
                a[s4] = (b1 || b2) ? a[s4] : 0.f;
            }
#pragma unroll
            for (int ct = 0; ct < BN / 16; ++ct) acc[ct] = MF::zero();
#pragma unroll
            for (int s4 = 0; s4 < KS; ++s4) {
                const float *mrow = S.M + (4 * s4 + kk) * LD + i16;
#pragma unroll
                for (int ct = 0; ct < BN / 16; ++ct) acc[ct] = MF::mma(a[s4], mrow[16 * ct], acc[ct]);
            }
        }
        __syncthreads();  // every read of M is done
        if (rows) {
#pragma unroll
            for (int ct = 0; ct < BN / 16; ++ct)
#pragma unroll
                for (int v = 0; v < 4; ++v)
                    S.M[(16 * wave + MF::crow(lane, v)) * LD + 16 * ct + i16] = acc[ct][v];
        }
        __syncthreads();  // E complete
        float ld[BACK_RPL];
        back_fetch(ld, ws.v + bi * (n - 2) * n, n, t);
        Mf<double>::acc qa[BN / 16];
        back_load(qa, n, t, [&](const int i, const int j) { return S.M[i * LD + j]; });
        __syncthreads();
        back_transform(S.M, S.u.tf, qa, ld, ws.tau + bi * n, n, t, Qb);
    }
}

// ------------------------------------------------------------------ host
// One workspace per stream, grown on demand.  A buffer that a captured graph
// uses is pinned: it is never freed, and a stream whose pinned buffer is too
// small for a later call gets a new one while the old one stays, retired,
// until the process ends.
struct Buf {
    void *ptr = nullptr;
    size_t bytes = 0;
    bool pinned = false;
};
std::mutex g_mu;
Lru<void *, Buf> g_bufs(8);
std::vector<void *> g_retired;

size_t align_up(size_t x) { return (x + 255) & ~size_t(255); }

}  // namespace big

bed_status big_solve(bed_dtype dt, int64_t batch, int n, const void *A, void *lam, void *Q,
                     int32_t *info, hipStream_t s)
{
    using namespace big;
    if (dt != BED_F32)
        return fail(BED_ERR_UNSUPPORTED, "n = %d > 64 is supported in binary32 only", n);
    if (n <= 64 || n > BN) return fail(BED_ERR_INVALID_ARG, "big_solve: n = %d", n);
    const int n1 = n / 2, n2 = n - n1;
    const size_t B = (size_t)batch;
    // children contiguous per kind: c1 then c2, q1 then q2, l1 then l2, i1 then i2
    const size_t c_bytes = align_up(B * 2 * (n1 + n2) * sizeof(float));
    const size_t q_bytes = align_up(B * (n1 * n1 + n2 * n2) * sizeof(float));
    const size_t l_bytes = align_up(B * n * sizeof(float));
    const size_t i_bytes = align_up(2 * B * sizeof(int32_t));
    const size_t m_bytes = align_up(B * sizeof(Meta));
    const size_t v_bytes = Q ? align_up(B * (n - 2) * n * sizeof(float)) : 0;
    const size_t t_bytes = Q ? align_up(B * n * sizeof(float)) : 0;
    const size_t d_bytes = align_up(B * 2 * BN * sizeof(double));
    const size_t f_bytes = align_up(B * sizeof(int32_t));
    const size_t need =
        c_bytes + q_bytes + l_bytes + i_bytes + m_bytes + d_bytes + f_bytes + v_bytes + t_bytes;
    const bool capturing = stream_capturing(s);
    char *base = nullptr;
    {
        std::lock_guard<std::mutex> lk(g_mu);
        Buf *b = g_bufs.find((void *)s);
        if (!b || b->bytes < need) {
            if (capturing)
                return fail(BED_ERR_CAPTURE, "workspace for n > 64 would be allocated during capture");
            if (b) {
                if (b->pinned) {
                    g_retired.push_back(b->ptr);  // a graph still reads and writes it
                } else {
                    hipError_t e = hipStreamSynchronize(s);
                    if (e != hipSuccess) return hip_fail(e, "hipStreamSynchronize");
                    (void)hipFree(b->ptr);
                }
                b->ptr = nullptr;
                b->bytes = 0;
                b->pinned = false;
                hipError_t e = hipMalloc(&b->ptr, need);
                if (e != hipSuccess) return hip_fail(e, "hipMalloc(workspace)");
                b->bytes = need;
            } else {
                Buf nb;
                hipError_t e = hipMalloc(&nb.ptr, need);
                if (e != hipSuccess) return hip_fail(e, "hipMalloc(workspace)");
                nb.bytes = need;
                std::vector<Buf> old = g_bufs.insert((void *)s, nb);
                if (!old.empty()) {
                    (void)hipDeviceSynchronize();  // their last uses were on other streams
                    for (Buf &o : old) (void)hipFree(o.ptr);
                }
                b = g_bufs.find((void *)s);
            }
        }
        if (capturing) {
            g_bufs.pin((void *)s);
            b->pinned = true;
        }
        base = (char *)b->ptr;
    }
    Ws ws;
    auto take = [&](const size_t bytes) {
        char *p = base;
        base += bytes;
        return p;
    };
    ws.c1 = (float *)take(c_bytes);
    ws.c2 = ws.c1 + B * 2 * n1;
    ws.q1 = (float *)take(q_bytes);
    ws.q2 = ws.q1 + B * n1 * n1;
    ws.l1 = (float *)take(l_bytes);
    ws.l2 = ws.l1 + B * n1;
    ws.i1 = (int32_t *)take(i_bytes);
    ws.i2 = ws.i1 + B;
    ws.meta = (Meta *)take(m_bytes);
    ws.t = (double *)take(d_bytes);
    ws.done = (int32_t *)take(f_bytes);
    ws.v = Q ? (float *)take(v_bytes) : nullptr;
    ws.tau = Q ? (float *)take(t_bytes) : nullptr;
    ws.e1 = Q ? nullptr : ws.q1;
    ws.e2 = Q ? nullptr : ws.q1 + B * 2 * n1;

    hipLaunchKernelGGL(k_big_reduce, dim3((unsigned)batch), dim3(RT_), 0, s, (const float *)A, n,
                       (int64_t)batch, ws);
    hipError_t e = hipGetLastError();
    if (e != hipSuccess) return hip_fail(e, "k_big_reduce launch");
    hipLaunchKernelGGL(k_big_direct, dim3((unsigned)batch), dim3(BT), 0, s, n, (int64_t)batch,
                       (float *)lam, (float *)Q, info, ws);
    e = hipGetLastError();
    if (e != hipSuccess) return hip_fail(e, "k_big_direct launch");
    const bed_tune dflt = default_tune(dt);
    // the halves of what is left: eigenvectors, or (eigenvalues only) just the end rows z needs
    float *q1 = Q ? ws.q1 : nullptr, *q2 = Q ? ws.q2 : nullptr;
    if (n1 == n2) {
        e = launch_tri(class_shape(size_class(n1), dflt), ws.c1, n1, 2 * batch, ws.l1, q1,
                       ws.i1, ws.e1, ws.done, batch, s);
    } else {
        e = launch_tri(class_shape(size_class(n1), dflt), ws.c1, n1, batch, ws.l1, q1, ws.i1,
                       ws.e1, ws.done, batch, s);
        if (e == hipSuccess)
            e = launch_tri(class_shape(size_class(n2), dflt), ws.c2, n2, batch, ws.l2, q2,
                           ws.i2, ws.e2, ws.done, batch, s);
    }
    if (e != hipSuccess) return hip_fail(e, "child solve launch");
    hipLaunchKernelGGL(k_big_merge, dim3((unsigned)batch), dim3(BT), 0, s, n, (int64_t)batch,
                       (float *)lam, (float *)Q, info, ws);
    e = hipGetLastError();
    if (e != hipSuccess) return hip_fail(e, "k_big_merge launch");
    return BED_OK;
}

}  // namespace bed
