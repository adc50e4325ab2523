// bed_syevd.hpp -- one team (a workgroup or a single wave) computes the full
// eigendecomposition of one symmetric n x n matrix (n <= NMAX <= 64) held in
// LDS/VGPRs:
//
//   load -> Householder tridiagonalization (binary64 arithmetic) -> spectrum of
//   T -> Householder back-transform -> sign canonicalization -> store.
//
// The spectrum of T, by the divide step of the note: rank-one tearing (Sec.
// 2.1, Eq. (1)-(3)) -> leaves of at most 2, 4 or 8 elements by cyclic Jacobi
// (Sec. 2.2) -> bottom-up merges (Sec. 2.3): z/sort (Eq. (4)-(5)), deflation,
// secular roots by hybrid-section + Halley under bounded interlacing (Eq.
// (8)-(21)), progressive removal of converged roots (Eq. (22)), Loewner
// eigenvectors (Eq. (23)-(25)), back-multiplication (Eq. (4)); without
// eigenvectors the merges carry only the end rows of each node's block.  By
// default binary32 spectra without nearly equal eigenvalues are solved directly
// instead (direct_solve below).
//
// Team geometry (NT threads, thread t):
//   Householder: wave 0 reduces, lane (i, j) of an 8 x 8 grid holding the
//     entries (i + 8a, j + 8b); other waves form Q_H.
//   Per-element phases: wave 0, lane e = element e (n <= 64 fits one wave).
//   Per-root phases: root q = t / LPR, LPR = NT / NMAX lanes share one root's
//     pole sums (aligned lane groups, butterfly reductions).
//   Back-transform: each wave owns NMAX/NW whole columns (no team barrier).
#pragma once

#include <type_traits>

#include "bed_device.hpp"
#include "bed_mfma.hpp"

// Phase markers: no-ops in the library; a profiling build may define
// BED_PHASE(id) to timestamp the phases of one team.
#ifndef BED_PHASE
#define BED_PHASE(id) ((void)0)
#endif
#ifndef BED_COUNT
#define BED_COUNT(id, value) ((void)0)
#endif
#ifndef BED_MARK
#define BED_MARK(depth, id) ((void)0)
#endif
#ifndef BED_ROOT
#define BED_ROOT(depth, root, evals, reason) ((void)0)
#endif
// Householder step markers (a profiling build may timestamp the sub-steps of
// one chosen step k; `wave` and `lane` are in scope where they are used).
#ifndef BED_HSTEP
#define BED_HSTEP(k, id) ((void)0)
#endif
// Deflation counts of one merge depth (type 1: rho |z_i| <= tol; type 2:
// Givens rotations), reported by lane 0 of wave 0 in a profiling build.
#ifndef BED_DEFL
#define BED_DEFL(type1, type2) ((void)0)
#endif

namespace bed {

// Waves per SIMD that the resident teams of a shape need (four SIMDs per CU);
// register allocation is capped accordingly (n > 32: two teams, 256 registers
// at 256 threads, 128 at 512).
template <int NMAX, int NT> struct Occ {
    static constexpr int teams_per_cu = NMAX >= 64 ? 2 : (NMAX >= 32 ? 4 : 8);
    static constexpr int v = (teams_per_cu * NT / 64 + 3) / 4;
    static constexpr int wpe = v < 1 ? 1 : (v > 8 ? 8 : v);
};
#define BED_OCC(NMAX, NT) __attribute__((amdgpu_waves_per_eu(Occ<NMAX, NT>::wpe)))

// Waves of a team during the Householder reduction.  Teams of four or more
// waves: HW product waves hold the matrix, one control wave forms the norms
// and reflectors beside them, AW waves accumulate Q_H; smaller teams reduce on
// one wave (HW = 1, no control wave), a second one accumulating Q_H.
template <typename T, int NMAX, int NT> struct HhWaves {
    static constexpr int NW = NT / 64;
    static constexpr bool team = NW >= 4;
    static constexpr int HW = NW >= 8 ? 4 : ((NW >= 4 && NMAX >= 64) ? 2 : 1);
    static constexpr int first_qh = team ? HW + 1 : 1;
};
// Waves that form Q_H = H_0 H_1 ... H_{n-3} explicitly beside the reduction
// (0: the back-transform applies the reflectors in compact-WY form instead).
// Each holds NMAX/AW >= 16 rows of Q_H, at most 256 bytes of values per lane;
// the product with Q_H that follows takes a wave per column tile.
template <typename T, int NMAX, int NT> struct QH_WAVES {
    static constexpr int spare = NT / 64 - HhWaves<T, NMAX, NT>::first_qh;
    static constexpr int p = (spare >= 4 && NMAX >= 64) ? 4 : ((spare >= 2 && NMAX >= 32) ? 2 : (spare >= 1 ? 1 : 0));
    static constexpr int value =
        (p > 0 && NT / 64 >= NMAX / 16 && NMAX * NMAX / (64 * p) * int(sizeof(T)) <= 256) ? p : 0;
};
// A wave that reduces alone needs no barrier; its team meets after every
// QH_SYNC steps so that the accumulating wave can follow.
constexpr int QH_SYNC = 4;

// Cutoff of the divide step when none is given (measured on the batch-512
// workloads): 8 for the n > 32 class, whose one fewer merge depth outweighs the
// longer Jacobi sweeps, 4 below.
__host__ __device__ constexpr int leaf_default(int nmax) { return nmax >= 64 ? 8 : 4; }

constexpr int SEC_CAP = 100;  // Halley-phase evaluations per root before "capped"

// The Householder reduction runs in binary64 for both storage types.  Its
// rounding errors are a backward error of A, which the eigenvalue differences
// and the eigenvectors of close pairs amplify by 1/gap (the backward of the
// decomposition divides by those differences).  In binary64 -- whose FMA
// issues at the rate of unpacked binary32 on gfx950 -- they stay far below
// binary32's unit roundoff; T, the reflectors and tau are then rounded once to
// the storage type.
//
// Vectors in LDS are laid out for the reduction's 8 x 8 lane grid: position
// i + 8a at i * HhLds<NMAX>::ST + a, so that a lane reads its NL = NMAX / 8
// row (or column) values as 16-byte vectors; the stride keeps the eight groups
// on distinct banks.
template <int NMAX> struct HhLds {
    static constexpr int NL = NMAX / 8;
    static constexpr int ST = NL > 2 ? NL + 2 : 2;
    static constexpr int SZ = 8 * ST;
};

// Per-element state of the merges of one depth; arrays indexed by global
// position (node-local at [lo, hi)).
template <typename T, int NMAX>
struct MergeArrays {
    T sd[NMAX], sz[NMAX];     // sorted poles / weights (deflation in place)
    int sperm[NMAX], sdefl[NMAX];
    T dk[NMAX], zk[NMAX];     // non-deflated poles / weights at [lo, lo + k)
    int ndrow[NMAX];          // child-order row of non-deflated component
    int itrow[NMAX];          // child-order row of deflated item at [lo + k, hi)
    T itv[NMAX];              // item values: roots at [lo, lo+k), deflated after
    T rtau[NMAX], rdo[NMAX];  // root offset and its origin pole value
    T zh[NMAX];
    T rc[NMAX], rs[NMAX];
    int rpart[NMAX];
    int rlist[NMAX], nrot[NMAX];  // per node: deflated index of each rotation, in scan order
    int nlo[NMAX], nhi[NMAX];  // node of each element at this depth
    int ckl[NMAX], ckh[NMAX];  // child block of each row (its own block for an unmerged leaf)
    int tklo[NMAX / 16], tkhi[NMAX / 16];  // per 16-row tile: K range of the product
    int tnlo[NMAX / 16], tnhi[NMAX / 16];  // per 16-row tile: span of its nodes
    int nk[NMAX];
    T nrho[NMAX], nzz[NMAX], nfro[NMAX];
    T nback[NMAX];  // from the node's scale (of dk, nrho, nfro) back to T's
};

// Direct solver: det and counts on the first grid.
template <int NT>
struct DirectGrid {
    double f[NT];
    int c[NT];
};
// Rows {a_i, b_{i-1}^2} from the top and {a_i, b_i^2} from the bottom, b_i in
// both orders, eigenvalues.
template <int NMAX>
struct DirectArrays {
    alignas(16) double ab[2][NMAX][2];
    double b[2][NMAX];
    double lam[NMAX];
    double lo, hi, unscale;
    int cell[NMAX];
    uint32_t twist[2][NMAX];  // per half of the rows: float bits of gamma (upper 25), row
    uint64_t close[(NMAX + 63) / 64];  // bit j: eigenvalues j and j + 1 are close
    int ok;
    int single;  // eigenvalues that the first grid shows apart from the others
};

// Its factors: of the default teams for n <= 32 in binary64, one set of them beside its
// other arrays, the other in Q1 and M; else in binary32 in Q0 and Q1.
template <typename T, int NMAX, int NT> struct DirectWide {
    static constexpr bool value = sizeof(T) == 4 && (NMAX == 16 || (NMAX == 32 && NT == 256));
};
template <int NMAX, bool WIDE> struct DirectFactors {
    double l[NMAX * (NMAX + 1)];
};
template <int NMAX> struct DirectFactors<NMAX, false> {};

template <typename T, int NMAX, int NT>
struct Smem {
    static constexpr int LD = NMAX + 1;  // odd row stride: column walks hit distinct banks
    static constexpr int NW = NT / 64;
    static constexpr int G = NT / NMAX;
    T Q0[NMAX * LD];  // eigenvector blocks (ping)
    union {
        struct {
            T Q1[NMAX * LD];  // eigenvector blocks (pong)
            T M[NMAX * LD];   // load staging, merge matrix, output staging
        };
        DirectFactors<NMAX, DirectWide<T, NMAX, NT>::value> fm;
    };
    // reflector k in row k: Vt[k*VLD + r] = v_k[r].  Compact WY: the odd row
    // stride keeps the MFMA operand reads (16 reflectors x 4 rows per
    // instruction) on distinct banks.  Explicit Q_H: 16-byte aligned rows for
    // vector reads; the buffer holds Q_H (row-major) once the reduction ends.
    static constexpr int VLD = QH_WAVES<T, NMAX, NT>::value ? NMAX + 4 : NMAX + 1;
    alignas(16) T Vt[NMAX * VLD];
    double ta[NMAX], tb[NMAX];  // T as the reduction leaves it
    T a[NMAX], b[NMAX], tau[NMAX];
    T lam0[NMAX], lam1[NMAX];
    union {
        struct {  // Householder: pivot column x and -w (a copy per product wave);
                  // by step parity: A x, the next pivot column A e, the waves'
                  // parts of x^T A x, the reflector's scalars
            alignas(16) double x[HhWaves<T, NMAX, NT>::HW][HhLds<NMAX>::SZ];
            alignas(16) double w[HhWaves<T, NMAX, NT>::HW][HhLds<NMAX>::SZ];
            alignas(16) double y[2][HhLds<NMAX>::SZ];
            alignas(16) double c[2][HhLds<NMAX>::SZ];
            alignas(16) double q[2][HhWaves<T, NMAX, NT>::HW < 2 ? 2 : HhWaves<T, NMAX, NT>::HW];
            alignas(16) double sc[2][4];
        } h;
        MergeArrays<T, NMAX> m;
        struct {  // direct solver
            DirectArrays<NMAX> t;
            union {
                DirectGrid<NT> g;  // during the first grid
                DirectFactors<NMAX, DirectWide<T, NMAX, NT>::value> f;
            };
        } d;
        struct {  // back-transform: per block of 16 reflectors, Gram matrix and T factor
            // 16 x 16 tiles with row stride 17 (bank-conflict free column reads)
            T gram[((NMAX + 13) / 16) * 272];
            T tf[((NMAX + 13) / 16) * 272];
        } b;
    } u;
    int badw[NW];
    int expw[NW];  // per wave: largest exponent field of the lower triangle
    int capped;
    int anyrot;
};

// The solver runs on 2^s A with max |a_ij| in [1/2, 1) (s clamped, 0 for a
// zero matrix): the scaling is exact, and keeps the secular offsets of roots
// next to their poles out of the subnormal range, where the hardware
// reciprocal flushes.  Eigenvalues are scaled back on output; eigenvectors do
// not change.  s comes from the per-wave exponents the load leaves in LDS
// (formed where it is needed, so that it holds no registers in between).
template <typename T, int NMAX, int NT>
__device__ __forceinline__ int input_shift(const Smem<T, NMAX, NT>& S)
{
    int emax = 0;
#pragma unroll
    for (int w = 0; w < NT / 64; ++w) emax = max(emax, S.expw[w]);
    emax = __builtin_amdgcn_readfirstlane(emax);
    const int sh = (emax == 0) ? 0 : fexp<T>::BIAS - 1 - emax;
    return min(max(sh, -fexp<T>::SMAX), fexp<T>::SMAX);
}

// Couplings of T below 2^-64 of the matrix's scale count as zero in binary32: the
// reduction of a null block leaves its rounding there, and that one's rounding, 1e-17,
// 1e-34, ... down to where binary32 has no reciprocals.
__device__ __forceinline__ float coupling(const float b) { return f_abs(b) < 0x1p-64f ? 0.f : b; }
__device__ __forceinline__ double coupling(const double b) { return b; }

// Node of a dyadic tearing tree over [0, n): node j at depth d covers
// [floor(j n / 2^d), floor((j+1) n / 2^d)); nodes of more than `leaf`
// elements (the cutoff: 2, 4 or 8) split at the floor of their dyadic
// midpoint, the others are leaves.
struct Node {
    int lo, hi, s;
};
__device__ __forceinline__ Node node_of(int e, int d, int n)
{
    int j = (((e + 1) << d) - 1) / n;
    Node nd;
    nd.lo = (j * n) >> d;
    nd.hi = ((j + 1) * n) >> d;
    nd.s = ((2 * j + 1) * n) >> (d + 1);
    return nd;
}

__device__ __forceinline__ int node_index(int e, int d, int n) { return (((e + 1) << d) - 1) / n; }

// Jacobi rotation that annihilates a_pq of the symmetric 2x2 block
// [a_pp a_pq; a_pq a_qq] (Rutishauser's form): t = tan(phi) with
// th = (a_qq - a_pp) / (2 a_pq), t = sgn(th) / (|th| + sqrt(th^2 + 1)),
// c = 1/sqrt(1 + t^2), s = t c.  Then a_pp' = a_pp - t a_pq, a_qq' = a_qq + t a_pq.
// Written without the quotient th: with d = a_qq - a_pp (sgn 0 = +1),
// t = sgn(d) 2 a_pq / (|d| + sqrt(d^2 + 4 a_pq^2)), whose denominator is at
// least 2|a_pq|.  The reciprocal and 1/sqrt are refined to about one ulp, so
// that c^2 + s^2 = 1 and the rotation is orthogonal to the working precision.
template <typename T>
__device__ __forceinline__ void jacobi_rot(const T app, const T aqq, const T apq, T& c, T& s, T& t)
{
    const T d = aqq - app;
    const T ap2 = T(2) * apq;
    const T den = f_abs(d) + f_sqrt(fma(d, d, ap2 * ap2));
    // no rotation for a zero (or vanishing) a_pq: the block is already diagonal
    const bool rot = apq != T(0) && den > T(sizeof(T) == 4 ? 1e-30f : 1e-290);
    const T tt = (d < T(0) ? -ap2 : ap2) * f_rcp(rot ? den : T(1));
    const T cc = f_rsqrt(fma(tt, tt, T(1)));
    t = rot ? tt : T(0);
    c = rot ? cc : T(1);
    s = rot ? tt * cc : T(0);
}

// Value of lane ^ K inside aligned groups of 8 lanes, by DPP: a quad permute
// for K < 4; for K >= 4 the half-row mirror (lane ^ 7 within 8), followed by
// the quad permute of K ^ 7 when K < 7 -- lane i then reads lane (i ^ (K ^ 7))
// ^ 7 = i ^ K.
template <int K, typename T> __device__ __forceinline__ T lxor(T x)
{
    if constexpr (K < 4) return qxor<K>(x);
    else if constexpr (K == 7) return xmove<4>(x, 0);
    else return qxor<K ^ 7>(xmove<4>(x, 0));
}

// f(integral_constant<int, K>) for K = B, ..., E - 1 (compile-time indices).
template <int B, int E, typename F> __device__ __forceinline__ void static_for(F&& f)
{
    if constexpr (B < E) {
        f(std::integral_constant<int, B>{});
        static_for<B + 1, E>(f);
    }
}

// One simultaneous round of the leaf Jacobi sweep: the pairs (i, i ^ M) of
// every leaf (GS lanes per leaf).  Lane i keeps row i of A and of V = J_1 J_2
// ... in XOR-relative order, a[k] = A(i, i ^ k), v[k] = V(i, i ^ k).  With J
// the product of the round's disjoint rotations, A <- J^T A J and V <- V J:
// each lane rotates its row's column pairs (j, j ^ M) with the parameters held
// by lane j, then combines its row with the partner row i ^ M.  The pair's own
// 2x2 block takes the exact form (a_pq' = 0, a_pp' = a_pp - t a_pq, a_qq' =
// a_qq + t a_pq).  The rounds M = 1, ..., GS - 1 of a sweep pair every two
// rows of the leaf exactly once (M = i ^ j).
template <int GS, int M, typename T>
__device__ __forceinline__ void jacobi_round(T (&a)[GS], T (&v)[GS], const int i, const int msz)
{
    const int ip = i ^ M;
    const T pd = lxor<M>(a[0]);  // A(ip, ip)
    const T po = lxor<M>(a[M]);  // A(ip, i)
    const bool low = i < ip;     // this row is p of the pair (p, q), p < q
    // both lanes of the pair form the same a_pq (the rounded rows need not be
    // exactly symmetric)
    const T apq = T(0.5) * (a[M] + po);
    T c, s, t;
    jacobi_rot(low ? a[0] : pd, low ? pd : a[0], apq, c, s, t);
    const bool rot = i < msz && ip < msz && apq != T(0);  // pairs with a padding row stay fixed
    c = rot ? c : T(1);
    s = rot ? s : T(0);
    t = rot ? t : T(0);
    const T sg = low ? T(-1) : T(1);  // A'(p, :) = c A(p, :) - s A(q, :), A'(q, :) = c A(q, :) + s A(p, :)
    const T ss = sg * s;
    // column parameters (c_j, sigma_j s_j) of column j = i ^ k
    T cj[GS], sj[GS];
    cj[0] = c;
    sj[0] = ss;
    cj[M] = c;
    sj[M] = -ss;
    static_for<1, GS>([&](auto K) {
        constexpr int k = decltype(K)::value;
        if constexpr (k != M) {
            cj[k] = lxor<k>(c);
            sj[k] = lxor<k>(ss);
        }
    });
    T b[GS], w[GS];
#pragma unroll
    for (int k = 0; k < GS; ++k) {
        b[k] = fma(sj[k], a[k ^ M], cj[k] * a[k]);
        w[k] = fma(sj[k], v[k ^ M], cj[k] * v[k]);
    }
    // partner row after its column rotation: B(ip, i ^ k) sits in its slot k ^ M
    T pb[GS];
#pragma unroll
    for (int k = 0; k < GS; ++k) pb[k] = lxor<M>(b[k ^ M]);
    const T dnew = fma(sg * t, apq, a[0]);
#pragma unroll
    for (int k = 0; k < GS; ++k) {
        a[k] = fma(ss, pb[k], c * b[k]);
        v[k] = w[k];
    }
    a[0] = rot ? dnew : a[0];
    a[M] = rot ? T(0) : a[M];
}

// Leaves of at most GS elements (the cutoff of the divide step, 2, 4 or 8) are
// solved by cyclic Jacobi -- the divide step may stop at small blocks and hand
// them to another eigensolver (Sec. 2.2).  Wave 0: lane (g, i) = (lane / GS,
// lane % GS) holds row i of the leaf of group g, group g standing for node g
// of depth D (the first such node of a leaf owns it; 2^D <= 64 / GS for n <=
// 64).  Sweeps of the rounds M = 1, ..., GS - 1 run until every off-diagonal
// entry is at most 8u ||T_leaf||_F (the wave's largest); the eigenvalues are
// then ranked ascending and the leaf's block of Q written.
template <int GS, typename T, int NMAX, int NT>
__device__ __forceinline__ void jacobi_leaves(Smem<T, NMAX, NT>& S, const int n, const int D,
                                              const int lane, T* __restrict__ Qc,
                                              T* __restrict__ Lc)
{
    static_assert((GS == 2 || GS == 4 || GS == 8) && NMAX <= 64, "leaf groups of 2, 4 or 8 lanes");
    constexpr int LD = Smem<T, NMAX, NT>::LD;
    constexpr int CAP = 16;  // sweeps (three to five suffice in binary32 and binary64 alike)
    const int g = lane / GS, i = lane % GS;
    const int e0 = (g * n) >> D;  // first element of node g at depth D
    int lo = 0, hi = 0;
    bool found = false;
    for (int d = 0; d <= D; ++d) {
        const Node nd = node_of(e0 < n ? e0 : 0, d, n);
        const bool hit = !found && nd.hi - nd.lo <= GS;
        lo = hit ? nd.lo : lo;
        hi = hit ? nd.hi : hi;
        found = found || hit;
    }
    const bool own = g < (1 << D) && found && lo == e0;
    const int msz = own ? hi - lo : 0;
    const bool row = i < msz;
    T a[GS], v[GS];
#pragma unroll
    for (int k = 0; k < GS; ++k) {
        const int j = i ^ k;
        const bool ok = row && j < msz;
        const bool adj = j == i + 1 || j == i - 1;
        const int bi = lo + (i < j ? i : j);
        T x = T(0);
        if (k == 0) x = S.a[ok ? lo + i : 0];
        else if (adj) x = S.b[ok ? bi : 0];
        a[k] = ok ? x : T(0);
        v[k] = (k == 0) ? T(1) : T(0);
    }
    T f2 = T(0);
#pragma unroll
    for (int k = 0; k < GS; ++k) f2 = fma(a[k], a[k], f2);
    f2 = group_sum<GS>(f2, lane);
    const T thr = T(8) * fp<T>::u * f_sqrt(f2);
    for (int sw = 0; sw < CAP; ++sw) {
        T off = T(0);
#pragma unroll
        for (int k = 1; k < GS; ++k) off = f_max(off, f_abs(a[k]));
        if (!__ballot(off > thr)) break;
        static_for<1, GS>([&](auto K) { jacobi_round<GS, decltype(K)::value>(a, v, i, msz); });
    }
    // ascending rank of this row's eigenvalue among the leaf's (ties by index)
    int rk = 0;
    static_for<1, GS>([&](auto K) {
        constexpr int k = decltype(K)::value;
        const T o = lxor<k>(a[0]);
        rk += ((i ^ k) < msz && (o < a[0] || (o == a[0] && (i ^ k) < i))) ? 1 : 0;
    });
    int rj[GS];
    rj[0] = rk;
    static_for<1, GS>([&](auto K) { rj[decltype(K)::value] = lxor<decltype(K)::value>(rk); });
    if (row) {
        Lc[lo + rk] = a[0];
        // V(i, j) is entry i of the eigenvector of eigenvalue j
#pragma unroll
        for (int k = 0; k < GS; ++k)
            if ((i ^ k) < msz) Qc[(lo + i) * LD + lo + rj[k]] = v[k];
    }
}

// Number of entries of the ascending list x[0..len) that are < v (strict) or
// <= v (inclusive).
template <typename T>
__device__ __forceinline__ int count_below(const T* x, int len, T v, bool inclusive)
{
    int lo = 0, hi = len;
    while (lo < hi) {
        int mid = (lo + hi) >> 1;
        bool below = inclusive ? (x[mid] <= v) : (x[mid] < v);
        if (below) lo = mid + 1;
        else hi = mid;
    }
    return lo;
}

// The same count by binary lifting with power-of-two steps STEP, STEP/2, ..., 1
// (STEP a compile-time bound >= half of the longest list): a fixed chain of
// loads from clamped addresses and selects, with no branch.
template <int STEP, typename T>
__device__ __forceinline__ int count_lift(const T* x, int len, T v, bool inclusive, int base)
{
    const int probe = base + STEP;
    const int idx = (probe <= len ? probe : len) - 1;
    const T xv = x[idx > 0 ? idx : 0];
    const bool below = inclusive ? (xv <= v) : (xv < v);
    base = (probe <= len && below) ? probe : base;
    if constexpr (STEP > 1) return count_lift<STEP / 2>(x, len, v, inclusive, base);
    else return base;
}
template <int NMAX, typename T>
__device__ __forceinline__ int count_below_steps(const T* x, int len, T v, bool inclusive,
                                                 int step)
{
    // step is wave-uniform: one branch selects the unrolled chain
    if (step >= 32 && NMAX >= 64) return count_lift<32>(x, len, v, inclusive, 0);
    if (step >= 16 && NMAX >= 32) return count_lift<16>(x, len, v, inclusive, 0);
    if (step >= 8) return count_lift<8>(x, len, v, inclusive, 0);
    if (step >= 4) return count_lift<4>(x, len, v, inclusive, 0);
    if (step >= 2) return count_lift<2>(x, len, v, inclusive, 0);
    return count_lift<1>(x, len, v, inclusive, 0);
}

// Uniform index into a register array without dynamic VGPR indexing: a
// log-depth chain of selects (idx is wave-uniform in every caller).
template <int N, typename T>
__device__ __forceinline__ T pick(const T* a, int idx)
{
    if constexpr (N == 1) {
        return a[0];
    } else {
        const T lo = pick<N / 2>(a, idx);
        const T hi = pick<N / 2>(a + N / 2, idx);
        return (idx & (N / 2)) ? hi : lo;
    }
}

// M2 of one depth: secular roots (Sec. 2.3.1-2.3.4) with SL lanes per root and
// KPL poles per lane in registers.  Threads [0, NMAX SL) take part (whole
// waves); the per-root bracket and Halley logic runs on every lane of a root,
// so fewer lanes per root cost less issue time than they add in sums.
template <typename T, int NMAX, int NT, int SL, int KPL, typename SM>
__device__ __forceinline__ void secular_roots(SM& S, const int n, const int d, const int t,
                                              const int leaf)
{
    constexpr int LPR = SL;
    const int lane = t & 63;
    const T u = fp<T>::u;
    // absent poles: a far, finite pole with zero weight (its terms vanish and
    // its reciprocal stays a normal number)
    const T FAR = sizeof(T) == 4 ? T(1e30f) : T(1e300);
    const int q = t / LPR, sub = t % LPR;
    const Node qn = node_of(q < n ? q : 0, d, n);
    const bool qact = (q < n) && (qn.hi - qn.lo > leaf);
    const int qlo = qn.lo;
    const int kq = qact ? S.u.m.nk[qlo] : 0;
    const int jr = q - qlo;
    const T* dk = S.u.m.dk + qlo;
    const T* zk = S.u.m.zk + qlo;
    const T rho = qact ? S.u.m.nrho[qlo] : T(0);
    {
        const bool live = qact && jr < kq;
        // this lane's share of the poles: i = sub + LPR*j
        // df = pole - origin pole; the poles themselves are read again from
        // LDS if the origin moves
        T z2[KPL], df[KPL];
#pragma unroll
        for (int j = 0; j < KPL; ++j) {
            const int i = sub + LPR * j;
            const bool ok = live && i < kq;
            const T dv = dk[ok ? i : 0], zv = zk[ok ? i : 0];
            df[j] = ok ? dv : FAR;
            z2[j] = ok ? zv * zv : T(0);
        }
        T ao = live ? rho * zk[jr] * zk[jr] : T(0);  // rho z_o^2 of the origin pole
        bool done = !live, capped = false;
        T L = T(0), U = T(0), h = T(0), w0 = T(1), gap = T(0), top = T(0);
        const T dj = live ? dk[jr] : T(0);
        const bool topr = live && jr == kq - 1;  // the unbounded-above root
        T dorg = dj;
        if (live) {
            if (!topr) {
                gap = dk[jr + 1] - dj;
                h = T(0.5) * gap;  // Eq. (13): midpoint of the root's own bracket
                w0 = gap;
            } else {
                // bracket (0, rho z^T z]; first probe at the Frobenius bound of
                // Eq. (10)-(11) when it is tighter, else at the midpoint
                top = rho * S.u.m.nzz[qlo];
                const T ubf = S.u.m.nfro[qlo] - dj;
                w0 = top;
                h = (ubf > T(0) && ubf < top) ? ubf : T(0.5) * top;
            }
        }
#pragma unroll
        for (int j = 0; j < KPL; ++j) df[j] = df[j] - dorg;
        int rounds = 0, nev = 0, why = 0, nhal = 0;
        // Eq. (8), (18), (21) at h: delta_i = (d_i - d_o) - h; returns f, f',
        // f'' and the stopping bound 8u(1 + rho sum |z_i^2 / delta_i|)
        auto secular = [&](const T hh, T& f, T& f1, T& f2, T& eb) {
            T s0 = 0, s1 = 0, s2 = 0, e = 0;
#pragma unroll
            for (int j = 0; j < KPL; ++j) {
                const T rinv = f_rcp(df[j] - hh);
                const T t0 = z2[j] * rinv;
                const T t1 = t0 * rinv;
                s0 += t0;
                s1 += t1;
                s2 = fma(t1, rinv, s2);
                e += f_abs(t0);
            }
            s0 = group_sum<LPR>(s0, lane);
            s1 = group_sum<LPR>(s1, lane);
            s2 = group_sum<LPR>(s2, lane);
            e = group_sum<LPR>(e, lane);
            f = T(1) + rho * s0;
            f1 = rho * s1;
            f2 = T(2) * rho * s2;
            eb = T(8) * u * (T(1) + rho * e);
        };
        // Round 1, bisection (Eq. (14)-(15)): the sign of f at the midpoint
        // picks the nearer pole as origin of tau = lambda - d_origin; the top
        // root keeps d_k and takes the bracket side by the same sign.
        {
            T f, f1, f2, eb;
            secular(h, f, f1, f2, eb);
            rounds = 1;
            nev = live ? 1 : 0;
            const bool up = f > T(0);
            const bool shift = live && !topr && !up && f != T(0);
            if (__ballot(shift)) {
                const T dnew = shift ? dk[jr + 1] : dorg;
                const T znew = shift ? zk[jr + 1] : T(0);
                if (shift) {
                    ao = rho * znew * znew;
#pragma unroll
                    for (int j = 0; j < KPL; ++j) {
                        const int i = sub + LPR * j;
                        const bool ok = i < kq;  // shift implies live
                        df[j] = (ok ? dk[ok ? i : 0] : FAR) - dnew;
                    }
                    dorg = dnew;
                }
            }
            L = up ? T(0) : (topr ? h : h - gap);
            U = up ? h : (topr ? top : T(0));
            // The next point is Halley's from the midpoint (in the shifted
            // variable when the origin moved) when that step is short (within
            // a quarter of the bracket: the root lies near the midpoint), else
            // (Eq. (16)) one multi-section probe toward the origin pole while
            // the bracket is wide, else the one-pole model's point, else the
            // midpoint.
            const T hs = shift ? h - gap : h;  // the evaluated point, from the new origin
            const T den = T(2) * f1 * f1 - f * f2;
            const T hh = hs - T(2) * f * f1 * f_rcp_fast(den);
            const T hm = ao * hs * f_rcp_fast(fma(f, hs, ao));
            const bool okh = den > T(0) && hh > L && hh < U && f_abs(hh - hs) <= T(0.25) * (U - L);
            const bool okm = hm > L && hm < U;
            const bool probe = (U - L) > T(1e-2) * w0;
            const T hp = shift ? U - T(0.25) * (U - L) : L + T(0.25) * (U - L);
            const bool stop = live && f == T(0);
            why = stop ? 1 : 0;
            done = done || stop;
            h = stop ? h : (okh ? hh : (probe ? hp : (okm ? hm : T(0.5) * (L + U))));
            nhal = 0;
        }
        // Progressive removal (Eq. (22)): a converged root's lanes idle; the
        // wave leaves the loop once all of its roots have stopped.  The body
        // is select-based: every live root updates its bracket by the sign of
        // f (Eq. (14)); the next point is Halley's from the evaluated point
        // (the probe's included) if inside the bracket, else the root of the
        // one-pole model f ~ c - ao/tau through (h, f) (exact next to a light
        // origin pole), else the midpoint.  A root stops at
        // f = 0 or |f| <= eb, at a bracket with no interior float, when the
        // step does not move h, or at the cap.
        while (__ballot(!done)) {
            ++rounds;
            nev += done ? 0 : 1;
            T f, f1, f2, eb;
            secular(h, f, f1, f2, eb);
            const bool conv = f == T(0) || f_abs(f) <= eb;
            const bool up = f > T(0);
            const T U2 = up ? h : U;
            const T L2 = up ? L : h;
            const bool tight = (U2 - L2) <= T(2) * u * (f_abs(L2) + f_abs(U2));
            const T den = T(2) * f1 * f1 - f * f2;
            const T hh = h - T(2) * f * f1 * f_rcp_fast(den);
            const T hm = ao * h * f_rcp_fast(fma(f, h, ao));
            const bool okh = den > T(0) && hh > L2 && hh < U2;
            const bool okm = hm > L2 && hm < U2;
            const T mid = T(0.5) * (L2 + U2);
            const T hn = okh ? hh : (okm ? hm : mid);
            const bool step = !(conv || tight) && hn != h;
            // A root that meets the stopping bound still takes the Halley
            // step from its last evaluation when that step stays in the
            // bracket: the bound allows |f| up to 8u(1 + rho sum|z^2/delta|),
            // and the step (third order from there) brings the root to the
            // rounding level of f at no further evaluation.
            const bool fin = conv && okh;
            const int nh = nhal + 1;
            const bool cap = step && nh >= SEC_CAP;
            const bool act = !done;
            U = act ? U2 : U;
            L = act ? L2 : L;
            why = act ? (f == T(0) ? 1 : (conv ? 2 : (tight ? 3 : (!step ? 4 : (cap ? 5 : 0))))) : why;
            h = (act && (step || fin)) ? hn : h;
            nhal = act ? nh : nhal;
            capped = act ? cap : capped;
            done = done || !step || cap;
        }
        BED_COUNT(d, rounds);
        if (live && sub == 0) BED_ROOT(d, q, nev, why);
        if (live && sub == 0) {
            S.u.m.rdo[q] = dorg;
            S.u.m.rtau[q] = h;
            S.u.m.itv[q] = S.u.m.nback[qlo] * (dorg + h);
            if (capped) atomicAdd(&S.capped, 1);
        }
    }
}

// Merge phases M2-M5 of one depth with KPL poles (or items) per lane held in
// registers: secular roots, Loewner zhat, eigenvector norms and output order,
// merge-matrix assembly (incl. type-2 rotations).  All team threads call it.
template <typename T, int NMAX, int NT, int KPL, typename SM>
__device__ __forceinline__ void roots_vectors(SM& S, const int n, const int d, const int t0,
                                              T* __restrict__ Ln, const int leaf)
{
    constexpr int LD = SM::LD;
    constexpr int LPR = NT / NMAX;
    // opaque copy of the thread index: the lane addresses derived from it are
    // formed again at every depth rather than hoisted out of the depth loop
    // (where they would be spilled)
    int t = t0;
    asm volatile("" : "+v"(t));
    const int lane = t & 63;
    (void)lane;
    const int q = t / LPR, sub = t % LPR;
    const Node qn = node_of(q < n ? q : 0, d, n);
    const bool qact = (q < n) && (qn.hi - qn.lo > leaf);
    const int qlo = qn.lo;
    const int mq = qn.hi - qn.lo;
    const int kq = qact ? S.u.m.nk[qlo] : 0;
    const int jr = q - qlo;
    const T* dk = S.u.m.dk + qlo;
    const T* zk = S.u.m.zk + qlo;
    const T rho = qact ? S.u.m.nrho[qlo] : T(0);

    // ---- M2: secular roots --------------------------------------------------
    {
        constexpr int SL = LPR < 4 ? LPR : 4;
        if (t < NMAX * SL) secular_roots<T, NMAX, NT, SL, KPL * LPR / SL>(S, n, d, t, leaf);
    }
    team_sync<NT>();
    BED_PHASE(10 + 8 * d + 1);

    // ---- M3: Loewner zhat (Eq. (25)) as a product of positive ratios ---------
    if (qact && jr < kq) {
        const T di = dk[jr];
        T p = T(1);
#pragma unroll
        for (int j = 0; j < KPL; ++j) {
            const int jj = sub + LPR * j;
            const bool ok = jj < kq;
            const int js = ok ? jj : 0;
            const T del = (di - S.u.m.rdo[qlo + js]) - S.u.m.rtau[qlo + js];  // d_i - lam_j
            const T fac = -del * f_rcp((jj == jr) ? rho : (dk[js] - di));
            p *= ok ? fac : T(1);
        }
        p = group_prod<LPR>(p, lane);
        if (sub == 0) S.u.m.zh[q] = f_copysign(f_sqrt(p), zk[jr]);
    }
    team_sync<NT>();
    BED_PHASE(10 + 8 * d + 2);

    // ---- M4: output order, eigenvector norms (Eq. (24)) and the merge matrix
    // M = P G (U (+) I) with rows in child order, in one pass per root: the
    // lanes of root j form w_i = zhat_i / (d_i - lambda_j), reduce |w|^2, and
    // write -w_i / ||w|| into column rank(j).  Slots outside the node go to
    // the padding column NMAX of M, which no product reads (no branches).
    if (qact) {
        // rank of item jr among the node's m items (roots, then deflated)
        const T my = S.u.m.itv[q];
        int cnt = 0;
#pragma unroll
        for (int j = 0; j < KPL; ++j) {
            const int vv = sub + LPR * j;
            const bool ok = vv < mq;
            const T ov = S.u.m.itv[qlo + (ok ? vv : 0)];
            cnt += (ok && (ov < my || (ov == my && vv < jr))) ? 1 : 0;
        }
        cnt = group_sum<LPR>(cnt, lane);
        const int c = qlo + cnt;
        if (sub == 0) Ln[c] = my;
        if (jr < kq) {
            const T dorg = S.u.m.rdo[q];
            const T tj = S.u.m.rtau[q];
            T wv[KPL];
            T s2 = T(0);
#pragma unroll
            for (int j = 0; j < KPL; ++j) {
                const int ii = sub + LPR * j;
                const bool ok = ii < kq;
                const int is = ok ? ii : 0;
                const T w = S.u.m.zh[qlo + is] * f_rcp((dk[is] - dorg) - tj);
                wv[j] = w;
                s2 += ok ? w * w : T(0);
            }
            s2 = group_sum<LPR>(s2, lane);
            const T nr = f_rcp(f_sqrt(s2));
#pragma unroll
            for (int j = 0; j < KPL; ++j) {
                const int ii = sub + LPR * j;
                const bool nd = ii < kq, df = !nd && ii < mq;
                const int is = (nd || df) ? ii : 0;
                const int rn = S.u.m.ndrow[qlo + is], rd = S.u.m.itrow[qlo + is];
                const int row = nd ? rn : (df ? rd : 0);  // row 0 for unused slots
                S.M[row * LD + ((nd || df) ? c : NMAX)] = nd ? -wv[j] * nr : T(0);
            }
        } else {
            const int myrow = S.u.m.itrow[q];
#pragma unroll
            for (int j = 0; j < KPL; ++j) {
                const int row = qlo + sub + LPR * j;
                const bool in = row < qlo + mq;
                S.M[(in ? row : qlo) * LD + (in ? c : NMAX)] = (row == myrow) ? T(1) : T(0);
            }
        }
    }
    team_sync<NT>();
    BED_PHASE(10 + 8 * d + 3);
    if (S.anyrot) {
        // Type-2 rotations act on the rows of M in reverse scan order.
        if (qact && sub == 0) {
            const int c = qlo + jr;
            for (int i = S.u.m.nrot[qlo] - 1; i >= 0; --i) {
                const int p = S.u.m.rlist[qlo + i];
                const int part = S.u.m.rpart[p];
                const int rp = S.u.m.sperm[p], ri = S.u.m.sperm[part];
                const T cc = S.u.m.rc[p], ss = S.u.m.rs[p];
                const T mp = S.M[rp * LD + c], mi = S.M[ri * LD + c];
                S.M[rp * LD + c] = cc * mp + ss * mi;
                S.M[ri * LD + c] = -ss * mp + cc * mi;
            }
        }
        team_sync<NT>();
    }
}

// Calls roots_vectors with the smallest power-of-two KPL >= need.
template <typename T, int NMAX, int NT, int KPL, typename SM>
__device__ __forceinline__ void roots_vectors_dispatch(SM& S, const int n,
                                                       const int d, const int t, T* Ln, int need,
                                                       const int leaf)
{
    if constexpr (KPL >= NMAX / (NT / NMAX)) {
        roots_vectors<T, NMAX, NT, KPL>(S, n, d, t, Ln, leaf);
    } else {
        if (need <= KPL)
            roots_vectors<T, NMAX, NT, KPL>(S, n, d, t, Ln, leaf);
        else
            roots_vectors_dispatch<T, NMAX, NT, KPL * 2>(S, n, d, t, Ln, need, leaf);
    }
}

// One 16-row tile of the back-multiplication with a K loop of exactly KS
// steps of four (the caller picks KS >= the tile's K range).  Lane l supplies
// A[r0 + l%16][k] and B[k][c0 + l%16] for k = kb0 + 4 st + l/16; A entries
// outside the row's child block are zero and out-of-range rows of B are read
// at row 0 (finite) against a zero A entry.
template <typename T, int NMAX, int NT, int KS>
__device__ __forceinline__ void backmul_rowtile(Smem<T, NMAX, NT>& S, const T* __restrict__ Qc,
                                                T* __restrict__ Qn, const int n, const int lane,
                                                const int r0, const int cg, const int CG,
                                                const int kb0, const int nlo, const int nhi)
{
    using MF = Mf<T>;
    constexpr int LD = Smem<T, NMAX, NT>::LD;
    constexpr int RT = NMAX / 16;
    const int i16 = lane & 15;
    const int r = r0 + i16;
    const int ckl = S.u.m.ckl[r], ckh = S.u.m.ckh[r];
    T av[KS];
#pragma unroll
    for (int st = 0; st < KS; ++st) {
        const int k = kb0 + 4 * st + (lane >> 4);
        const bool ok = k >= ckl && k < ckh;
        const T a = Qc[r * LD + (ok ? k : 0)];
        av[st] = ok ? a : T(0);
    }
    for (int ct = cg; ct < RT; ct += CG) {
        const int c0 = 16 * ct;
        if (c0 >= n || c0 >= nhi || c0 + 16 <= nlo) continue;
        const int c = c0 + i16;
        T bv[KS];
#pragma unroll
        for (int st = 0; st < KS; ++st) {
            const int k = kb0 + 4 * st + (lane >> 4);
            bv[st] = S.M[(k < NMAX ? k : 0) * LD + c];
        }
        typename MF::acc acc = MF::zero();
#pragma unroll
        for (int st = 0; st < KS; ++st) acc = MF::mma(av[st], bv[st], acc);
#pragma unroll
        for (int v = 0; v < 4; ++v) Qn[(r0 + MF::crow(lane, v)) * LD + c] = acc[v];
    }
}

// Householder tridiagonalization (Sec. 2; textbook, Golub-Van Loan 8.3).  The
// product waves hold the matrix in registers: lane (i, j) = (8 wave + lane / 8,
// lane % 8) keeps the entries A(i + GI a, j + 8 b), GI = 8 HW, a < NA = NMAX /
// GI, b < NB = NMAX / 8: a two-dimensional cyclic split, so that a lane needs
// only NA row and NB column values of each vector, and chunks of finished rows
// and columns drop out of the products altogether.  Every wave holds whole
// rows: A x is complete after a reduction over the eight lanes of a group.
// The matrix sits at the high end of the NMAX positions (position = index +
// NMAX - n): the chunks that padding would fill are simply finished ones.
//
// With x the pivot column below the diagonal, alpha = -sgn(x_0)||x|| and
// xt = x - alpha e, the reflector is I - beta xt xt^T, beta = 1/(mu(mu + |x_0|)),
// mu = ||x||.  The products run on x, before its norm is known:
//   A xt = A x - alpha A e,   xt^T A xt = x^T A x - 2 alpha (A x)_0 + alpha^2 A_00
// (A e is the next pivot column, which the step needs anyway), so the norm's
// wave sum and the reflector's scalar chain run beside the rank-2 update of
// the step before and the product, on a wave of their own in the larger teams.
// xt is x except at its first entry, where both terms have one sign: no
// cancellation enters.  With p = beta A xt, K = (beta/2) xt^T p, w = p - K xt
// the update is A - xt w^T - w xt^T; rows and columns up to the pivot row are
// finished after it, so the update of the others needs x itself, not xt, and
// the next pivot column is A e - w xt_0 - x w_0 per row.
//
// A step of a team has one barrier: before it the product waves apply the
// previous update, form A x, their parts of x^T A x and A e; after it every
// product wave (and the control wave) forms w and the next x for all rows, one
// row per lane, and hands them to its own lanes through its own LDS copies.
template <typename T> struct HhRefl {
    double alpha, beta, rx0;  // rx0 = 1 / (x_0 - alpha)
    double tau;               // beta (x_0 - alpha)^2 = 1 + |x_0| / mu
};
template <typename T>
__device__ __forceinline__ HhRefl<T> hh_reflector(const double x0, const double sig)
{
    // sig = ||x||^2 - x_0^2.  A sub-column below 1e-75 (of a matrix scaled to
    // magnitude one) counts as zero: beta = 0, alpha = x_0; beta^2 stays finite.
    // 1/mu and 1/(|x_0| + mu) are hardware estimates refined by Newton steps:
    // one for binary32 storage (below 1e-12); two for binary64, where mu, beta and
    // tau are also formed to about their rounding: H is as orthogonal as they are.
    const bool z = sig < 1e-150;
    const double s2 = fma(x0, x0, sig);
    double rmu = d_rsqrt_nr(s2);
    if constexpr (sizeof(T) == 8) rmu = fma(rmu, 0.5 * fma(-s2 * rmu, rmu, 1.0), rmu);
    double mu = s2 * rmu;
    if constexpr (sizeof(T) == 8) mu = fma(0.5 * fma(-mu, mu, s2), rmu, mu);
    const double ax = f_abs(x0);
    double rs = d_rcp_nr(ax + mu);
    if constexpr (sizeof(T) == 8) rs = fma(rs, fma(-(ax + mu), rs, 1.0), rs);
    HhRefl<T> h;
    h.alpha = z ? x0 : -f_copysign(mu, x0);
    h.beta = z ? 0.0 : rmu * rs;
    h.tau = z ? 0.0 : fma(ax, rmu, 1.0);
    if constexpr (sizeof(T) == 8) {
        const double d = mu * (ax + mu);
        h.beta = z ? 0.0 : fma(h.beta, fma(-d, h.beta, 1.0), h.beta);
    }
    h.rx0 = z ? 0.0 : f_copysign(rs, x0);
    return h;
}

// Lanes of a product wave: lane l holds rows i = l % 8 (+ 8 wave) and columns
// j = l / 16 + 4 (l / 8 % 2).  A binary64 4x4x4 MFMA (four blocks, block l / 4
// % 4: A row l % 4, k = l / 16; D row l / 16, column l % 4) against a B of ones
// in some columns sums a value over the four lanes l / 16 of a row and leaves
// the sum in lanes l / 16 = row, at those columns: NA such products reduce NA
// values and place them in different lanes, in one instruction each instead of
// the moves and selects of a butterfly (7 for a pair of values and stage).
__device__ __forceinline__ int hh_row_of(const int l) { return l & 7; }
__device__ __forceinline__ int hh_col_of(const int l) { return (l >> 4) | ((l >> 1) & 4); }
// Lane l ends with the row hh_out_row(l) and the value a = hh_own<NA>(l).
__device__ __forceinline__ int hh_out_row(const int l) { return (l >> 4) | (l & 4); }
template <int NA> __device__ __forceinline__ int hh_own(const int l)
{
    if constexpr (NA == 8) return (l & 3) | ((l >> 1) & 4);
    else if constexpr (NA == 4) return l & 3;
    else return NA == 2 ? (l >> 1) & 1 : 0;
}
// A lane that ends with row i (0..7) and value a.
template <int NA> __device__ __forceinline__ int hh_lane_of(const int i, const int a)
{
    const int o = NA == 8 ? (a & 3) | ((a & 4) << 1) : (NA == 4 ? a : (NA == 2 ? 2 * a : 0));
    return ((i & 3) << 4) | (i & 4) | o;
}
constexpr int DPP_ROR8 = 0x128;  // lane ^ 8 within 16

// The B operands: sel[a] is one in the columns that value a is left in.
template <int NA> struct HhSelect {
    static constexpr int NS = NA < 4 ? NA : 4;
    double sel[NS];
    __device__ __forceinline__ explicit HhSelect(const int l)
    {
#pragma unroll
        for (int a = 0; a < NS; ++a) sel[a] = (NS == 1 || hh_own<NS>(l) == a) ? 1.0 : 0.0;
    }
};
// y[a] summed over the eight columns' lanes; values of finished chunks (a <
// A0) are left out.
template <int NA, int A0>
__device__ __forceinline__ double hh_reduce_scatter(const double (&y)[NA], const HhSelect<NA>& B,
                                                    const int l)
{
    constexpr int NS = HhSelect<NA>::NS;
    double u = 0.0, v = 0.0;
#pragma unroll
    for (int a = 0; a < NS; ++a) {
        if (a >= A0) u = __builtin_amdgcn_mfma_f64_4x4x4f64(y[a], B.sel[a], u, 0, 0, 0);
        if constexpr (NA == 8)
            if (a + 4 >= A0) v = __builtin_amdgcn_mfma_f64_4x4x4f64(y[a + 4], B.sel[a], v, 0, 0, 0);
    }
    if constexpr (NA == 8) {
        if (A0 >= 4) return v + dpp_move64<DPP_ROR8>(v);
        const bool up = (l & 8) != 0;
        const double keep = up ? v : u, send = up ? u : v;
        return keep + dpp_move64<DPP_ROR8>(send);
    }
    return u + dpp_move64<DPP_ROR8>(u);
}

// One row per lane, in the same places: lane l stands for position
// hh_out_row(l) + 8 own(l) (duplicates for NMAX < 64).
template <int NMAX> struct HhRow {
    static constexpr int NB = NMAX / 8;
    int pos, slot;
    __device__ __forceinline__ explicit HhRow(const int lane)
    {
        const int i = hh_out_row(lane), o = hh_own<NB>(lane);
        pos = i + 8 * o;
        slot = i * HhLds<NMAX>::ST + o;
    }
    static __device__ __forceinline__ int slot_of(const int pos)
    {
        return (pos & 7) * HhLds<NMAX>::ST + (pos >> 3);
    }
    static __device__ __forceinline__ int lane_of(const int pos)
    {
        return hh_lane_of<NB>(pos & 7, pos >> 3);
    }
    // sum over the positions of a per-row value, in every lane
    static __device__ __forceinline__ double sum(const double x)
    {
        return (NMAX / 64.0) * wave_sum_all(x);  // 64 / NMAX lanes per position
    }
};

// Step k once A x (yr), A e (ce), their values s1, a00 at the pivot row and
// q = x^T A x are known: -w and the next pivot column at this lane's row; w0 =
// w at the pivot row.  hb = beta^2 / 2.
struct HhStep {
    double nw, xn, w0;
};
__device__ __forceinline__ HhStep hh_step(const double x, const double yr, const double ce,
                                          const double s1, const double a00, const double q,
                                          const double alpha, const double beta, const double hb,
                                          const double xt0)
{
    const double kk = hb * fma(alpha, fma(alpha, a00, -2.0 * s1), q);
    HhStep o;
    o.nw = fma(kk, x, -beta * fma(-alpha, ce, yr));
    o.w0 = fma(-kk, xt0, beta * fma(-alpha, a00, s1));
    o.xn = fma(o.nw, xt0, fma(-x, o.w0, ce));
    return o;
}

// Entries of one product wave, with its update and product at the chunk level.
template <int NMAX, int HW> struct HhBlock {
    static constexpr int GI = 8 * HW;
    static constexpr int NA = NMAX / GI, NB = NMAX / 8, ST = HhLds<NMAX>::ST;
    // Large blocks leave no registers for the vectors' operands: they read the
    // last x again and take the columns one at a time.
    static constexpr bool LARGE = NMAX > 64;
    double a[NA][NB];  // A(i + GI a, j + 8 b) after the updates of all steps but the last
    double xr[LARGE ? 1 : NA], xc[LARGE ? 1 : NB];  // x of the last step at this lane's rows, columns

    // Applies the update of the last step (-w in wl; x of that step in xo, for
    // LARGE blocks) and forms the products of this step with x in xl, for rows
    // and columns from chunks A0, B0 on.  The column of position 8 B0 + j0 goes
    // to cl.  Returns this lane's part of x^T A x.
    template <int A0, int B0>
    __device__ __forceinline__ double step(const double* xl, const double* wl, const double* xo,
                                           double* cl, const int i, const int j, const int j0,
                                           double (&y)[NA])
    {
        const int ri = (i & 7) * ST + (i >> 3);
        auto column = [&] {
            if (j == j0) {
#pragma unroll
                for (int c = A0; c < NA; ++c) cl[ri + HW * c] = a[c][B0];
            }
        };
        double q = 0.0;
        if constexpr (LARGE) {
            double wr[NA], nr[NA];
#pragma unroll
            for (int c = A0; c < NA; ++c) {
                wr[c] = wl[ri + HW * c];
                nr[c] = xo[ri + HW * c];
            }
#pragma unroll
            for (int b = B0; b < NB; ++b) {
                const double wc = wl[j * ST + b], xc1 = xo[j * ST + b];
#pragma unroll
                for (int c = A0; c < NA; ++c)
                    a[c][b] = fma(wr[c], xc1, fma(nr[c], wc, a[c][b]));
            }
            __builtin_amdgcn_sched_barrier(0);
            column();
#pragma unroll
            for (int c = 0; c < NA; ++c) y[c] = 0.0;
#pragma unroll
            for (int b = B0; b < NB; ++b) {
                const double nc = xl[j * ST + b];
#pragma unroll
                for (int c = A0; c < NA; ++c) y[c] = fma(a[c][b], nc, y[c]);
            }
#pragma unroll
            for (int c = A0; c < NA; ++c) q = fma(xl[ri + HW * c], y[c], q);
        } else {
            double wr[NA], wc[NB], nr[NA], nc[NB];
#pragma unroll
            for (int c = A0; c < NA; ++c) {
                wr[c] = wl[ri + HW * c];
                nr[c] = xl[ri + HW * c];
            }
#pragma unroll
            for (int b = B0 & ~1; b < NB; ++b) {
                wc[b] = wl[j * ST + b];
                nc[b] = xl[j * ST + b];
            }
#pragma unroll
            for (int c = A0; c < NA; ++c)
#pragma unroll
                for (int b = B0; b < NB; ++b)
                    a[c][b] = fma(wr[c], xc[b], fma(xr[c], wc[b], a[c][b]));
            column();
#pragma unroll
            for (int c = 0; c < NA; ++c) {
                y[c] = 0.0;
                if (c < A0) continue;
                double y1 = a[c][B0] * nc[B0], y2 = 0.0;
#pragma unroll
                for (int b = B0 + 1; b < NB; ++b) {
                    double& acc = ((b - B0) & 1) ? y2 : y1;
                    acc = (b == B0 + 1) ? a[c][b] * nc[b] : fma(a[c][b], nc[b], acc);
                }
                y[c] = (B0 + 1 < NB) ? y1 + y2 : y1;
                q = (c == A0) ? nr[c] * y[c] : fma(nr[c], y[c], q);
            }
#pragma unroll
            for (int c = A0; c < NA; ++c) xr[c] = nr[c];
#pragma unroll
            for (int b = B0; b < NB; ++b) xc[b] = nc[b];
        }
        return q;
    }
};

// The steps kp (padded index) whose pivot row kp + 1 = 8 B0 + i0 lies in chunk
// B0: f(kp, i0).  (One copy of the body: unrolled by the parity that the
// exchange buffers alternate with, it spends more on register copies than the
// addresses cost.)
template <int NMAX, typename F>
__device__ __forceinline__ void hh_chunk(const int b0, const int pad, F&& f)
{
    const int kb = max(8 * b0 - 1, pad), ke = min(8 * b0 + 7, NMAX - 2);
#pragma unroll 1
    for (int kp = kb; kp < ke; ++kp) f(kp, (kp + 1) & 7);
}

// One wave alone, chunks B0, B0 + 1, ...  x: the pivot column at this lane's
// row (zero up to the pivot); xl, nwl: x and -w of the last step there.
template <typename T, int NMAX, int NT, int B0>
__device__ __forceinline__ void hh_solo(Smem<T, NMAX, NT>& S, const int n, const int lane,
                                        const HhSelect<NMAX / 8>& sel, HhBlock<NMAX, 1>& H,
                                        double& x, double& xl, double& nwl)
{
    constexpr int NB = NMAX / 8;
    constexpr int VLD = Smem<T, NMAX, NT>::VLD;
    constexpr int ST = HhLds<NMAX>::ST;
    const int wave = 0;
    (void)wave;
    const int pad = NMAX - n;
    const HhRow<NMAX> R(lane);
    const int vr = R.pos - pad + (R.pos < pad ? NMAX : 0);
    hh_chunk<NMAX>(B0, pad, [&](const int kp, const int i0) {
        const int k = kp - pad;
        const int s0 = i0 * ST + B0;
        wave_sync();
        BED_HSTEP(k, 0);
        const double x0 = S.u.h.x[0][s0];
        const double sig = HhRow<NMAX>::sum(R.pos > kp + 1 ? x * x : 0.0);
        double y[NB];
        double q = H.template step<B0, B0>(S.u.h.x[0], S.u.h.w[0], nullptr, S.u.h.c[0], hh_row_of(lane),
                                           hh_col_of(lane), i0, y);
        BED_HSTEP(k, 1);
        const HhRefl<T> h = hh_reflector<T>(x0, sig);
        wave_sync();
        const double ce = S.u.h.c[0][R.slot], a00 = S.u.h.c[0][s0];
        const double yr = hh_reduce_scatter<NB, B0>(y, sel, lane);
        q = wave_sum_all(q);
        const double s1 = bcast(yr, hh_lane_of<NB>(i0, B0));
        BED_HSTEP(k, 2);
        const double xt0 = x0 - h.alpha;
        const HhStep o = hh_step(x, yr, ce, s1, a00, q, h.alpha, h.beta, 0.5 * h.beta * h.beta, xt0);
        xl = x;
        nwl = o.nw;
        // reflector k, normalized to v_{k+1} = 1, at index r of the original
        // matrix (padding positions hold zeros at indices >= n)
        const double v = (R.pos == kp + 1) ? 1.0 : x * h.rx0;
        x = (R.pos > kp + 1) ? o.xn : 0.0;
        S.u.h.w[0][R.slot] = o.nw;
        S.u.h.x[0][R.slot] = x;
        BED_HSTEP(k, 3);
        S.Vt[k * VLD + vr] = T(v);
        // (every lane writes the same values)
        S.tau[k] = T(h.tau);
        S.tb[k] = h.alpha;
        S.ta[k + 1] = fma(-2.0 * xt0, o.w0, a00);
        BED_HSTEP(k, 8);
        if constexpr (QH_WAVES<T, NMAX, NT>::value > 0)
            if (k % QH_SYNC == QH_SYNC - 1) team_sync<NT>();
    });
    if constexpr (B0 + 1 < NB) hh_solo<T, NMAX, NT, B0 + 1>(S, n, lane, sel, H, x, xl, nwl);
}

// A product wave of a team (wave < HW).
template <typename T, int NMAX, int NT, int B0>
__device__ __forceinline__ void hh_product(Smem<T, NMAX, NT>& S, const int n, const int lane,
                                           const int wave,
                                           const HhSelect<HhBlock<NMAX, HhWaves<T, NMAX, NT>::HW>::NA>& sel,
                                           HhBlock<NMAX, HhWaves<T, NMAX, NT>::HW>& H, double& x,
                                           double& xl, double& nwl)
{
    constexpr int HW = HhWaves<T, NMAX, NT>::HW;
    using B = HhBlock<NMAX, HW>;
    constexpr int A0 = 8 * B0 / B::GI;
    constexpr int ST = HhLds<NMAX>::ST;
    const int pad = NMAX - n;
    const HhRow<NMAX> R(lane);
    const int i = 8 * wave + hh_row_of(lane), j = hh_col_of(lane);
    double* X = S.u.h.x[wave];
    double* W = S.u.h.w[wave];
    // this lane's row after the reduction over the columns
    const int yslot = HhRow<NMAX>::slot_of(8 * wave + hh_out_row(lane) + B::GI * hh_own<B::NA>(lane));
    hh_chunk<NMAX>(B0, pad, [&](const int kp, const int i0) {
        const int k = kp - pad, par = kp & 1;
        (void)k;
        const int s0 = i0 * ST + B0;
        wave_sync();
        BED_HSTEP(k, 0);
        double y[B::NA];
        double q = H.template step<A0, B0>(X, W, nullptr, S.u.h.c[par], i, j, i0, y);
        BED_HSTEP(k, 1);
        const double yo = hh_reduce_scatter<B::NA, A0>(y, sel, lane);
        q = wave_sum_all(q);
        S.u.h.y[par][yslot] = yo;
        S.u.h.q[par][wave] = q;  // (every lane writes the same value)
        team_sync<NT>();
        BED_HSTEP(k, 2);
        const double yr = S.u.h.y[par][R.slot], ce = S.u.h.c[par][R.slot];
        const double s1 = S.u.h.y[par][s0], a00 = S.u.h.c[par][s0];
        const double alpha = S.u.h.sc[par][0], beta = S.u.h.sc[par][1];
        const double hb = S.u.h.sc[par][2], xt0 = S.u.h.sc[par][3];
        double qs = S.u.h.q[par][0];
#pragma unroll
        for (int w2 = 1; w2 < HW; ++w2) qs += S.u.h.q[par][w2];
        const HhStep o = hh_step(x, yr, ce, s1, a00, qs, alpha, beta, hb, xt0);
        xl = x;
        nwl = o.nw;
        x = (R.pos > kp + 1) ? o.xn : 0.0;
        W[R.slot] = o.nw;
        X[R.slot] = x;
        BED_HSTEP(k, 3);
        BED_HSTEP(k, 8);
    });
    if constexpr (B0 + 1 < NMAX / 8)
        hh_product<T, NMAX, NT, B0 + 1>(S, n, lane, wave, sel, H, x, xl, nwl);
}

// The control wave of a team: norm and reflector of step k before its barrier,
// then (as the product waves) the next pivot column; writes T, the reflectors
// and tau (values that all lanes hold alike are written by all of them).
template <typename T, int NMAX, int NT>
__device__ __forceinline__ void hh_control(Smem<T, NMAX, NT>& S, const int n, const int lane, double x)
{
    constexpr int HW = HhWaves<T, NMAX, NT>::HW;
    constexpr int VLD = Smem<T, NMAX, NT>::VLD;
    constexpr int ST = HhLds<NMAX>::ST;
    const int pad = NMAX - n;
    const HhRow<NMAX> R(lane);
    const int vr = R.pos - pad + (R.pos < pad ? NMAX : 0);
#pragma unroll 1
    for (int b0 = pad / 8; b0 < NMAX / 8; ++b0)
        hh_chunk<NMAX>(b0, pad, [&](const int kp, const int i0) {
            const int k = kp - pad, par = kp & 1;
            const int s0 = i0 * ST + b0;
            const double x0 = bcast(x, hh_lane_of<NMAX / 8>(i0, b0));
            const double sig = HhRow<NMAX>::sum(R.pos > kp + 1 ? x * x : 0.0);
            const HhRefl<T> h = hh_reflector<T>(x0, sig);
            const double xt0 = x0 - h.alpha, hb = 0.5 * h.beta * h.beta;
            S.u.h.sc[par][0] = h.alpha;
            S.u.h.sc[par][1] = h.beta;
            S.u.h.sc[par][2] = hb;
            S.u.h.sc[par][3] = xt0;
            // normalized to v_{k+1} = 1, at index r of the original matrix
            // (padding positions hold zeros at indices >= n)
            S.Vt[k * VLD + vr] = T((R.pos == kp + 1) ? 1.0 : x * h.rx0);
            S.tau[k] = T(h.tau);
            S.tb[k] = h.alpha;
            team_sync<NT>();
            const double yr = S.u.h.y[par][R.slot], ce = S.u.h.c[par][R.slot];
            const double s1 = S.u.h.y[par][s0], a00 = S.u.h.c[par][s0];
            double qs = S.u.h.q[par][0];
#pragma unroll
            for (int w2 = 1; w2 < HW; ++w2) qs += S.u.h.q[par][w2];
            const HhStep o = hh_step(x, yr, ce, s1, a00, qs, h.alpha, h.beta, hb, xt0);
            x = (R.pos > kp + 1) ? o.xn : 0.0;
            S.ta[k + 1] = fma(-2.0 * xt0, o.w0, a00);
        });
}

// Explicit Q_H = H_0 H_1 ... H_{n-3} on the AW waves that do not reduce:
// Q_H <- Q_H (I - tau_k v_k v_k^T) = Q_H - tau_k (Q_H v_k) v_k^T for k = 0, 1,
// ..., once reflector k (row k of Vt, tau[k]) has passed a team barrier.
// Wave aw holds rows [aw RW, aw RW + RW) of Q_H; lane (rl, cg) holds row
// aw RW + rl, columns [cg VPL, cg VPL + VPL).
template <typename T, int NMAX, int NT>
struct QhShape {
    static constexpr int AW = QH_WAVES<T, NMAX, NT>::value;
    static constexpr int RW = AW ? NMAX / AW : NMAX;  // rows per wave
    static constexpr int VPL = AW ? NMAX * RW / 64 : 1;  // values per lane
};
template <typename T, int NMAX, int NT>
__device__ __forceinline__ void qh_apply(const Smem<T, NMAX, NT>& S, const int lane, const int k,
                                         T (&qh)[QhShape<T, NMAX, NT>::VPL])
{
    constexpr int RW = QhShape<T, NMAX, NT>::RW;
    constexpr int VPL = QhShape<T, NMAX, NT>::VPL;
    constexpr int VLD = Smem<T, NMAX, NT>::VLD;
    constexpr int VW = 16 / sizeof(T);
    static_assert(RW >= 16 && VPL % VW == 0 && VLD % VW == 0, "explicit Q_H layout");
    typedef T vec_t __attribute__((ext_vector_type(VW)));
    const int cg = lane / RW;
    const vec_t* vp = reinterpret_cast<const vec_t*>(S.Vt + k * VLD + cg * VPL);
    T v[VPL];
#pragma unroll
    for (int q = 0; q < VPL / VW; ++q) {
        const vec_t x = vp[q];
#pragma unroll
        for (int e = 0; e < VW; ++e) v[q * VW + e] = x[e];
    }
    T s0 = T(0), s1 = T(0);
#pragma unroll
    for (int i = 0; i < VPL; i += 2) {
        s0 = fma(qh[i], v[i], s0);
        s1 = fma(qh[i + 1], v[i + 1], s1);
    }
    T s = s0 + s1;  // (Q_H v_k) at this row: sum over the column groups
    if constexpr (RW <= 16) s += xmove<16>(s, lane);
    if constexpr (RW <= 32) s += xmove<32>(s, lane);
    const T ts = S.tau[k] * s;
#pragma unroll
    for (int i = 0; i < VPL; ++i) qh[i] = fma(-ts, v[i], qh[i]);
}

template <typename T, int NMAX, int NT>
__device__ __forceinline__ int householder(Smem<T, NMAX, NT>& S, const int n, const int lane,
                                           const int wave, const bool want_q, const T sc,
                                           T (&qh)[QhShape<T, NMAX, NT>::VPL])
{
    constexpr int LD = Smem<T, NMAX, NT>::LD;
    using WV = HhWaves<T, NMAX, NT>;
    constexpr int HW = WV::HW;
    constexpr int AW = QH_WAVES<T, NMAX, NT>::value;
    if (wave >= WV::first_qh) {
        // barriers of the reduction: every step of a team, else every QH_SYNC-th
        // where a wave accumulates Q_H
        constexpr int step = WV::team ? 1 : QH_SYNC;
        if constexpr (AW > 0) {
            if (wave < WV::first_qh + AW) {
                // returns the first reflector not yet applied (the rest follow
                // the barrier that closes the reduction)
                constexpr int RW = QhShape<T, NMAX, NT>::RW;
                constexpr int VPL = QhShape<T, NMAX, NT>::VPL;
                const int row = (wave - WV::first_qh) * RW + lane % RW, c0 = (lane / RW) * VPL;
#pragma unroll
                for (int i = 0; i < VPL; ++i) qh[i] = (row == c0 + i) ? T(1) : T(0);
                int j = 0;
                for (int k = step - 1; k < n - 2; k += step) {
                    team_sync<NT>();  // visible: reflectors up to k
                    for (; j <= k; ++j)
                        if (want_q) qh_apply<T, NMAX, NT>(S, lane, j, qh);
                }
                return j;
            }
        }
        // the other waves only keep the barrier count
        if constexpr (WV::team || AW > 0)
            for (int k = step - 1; k < n - 2; k += step) team_sync<NT>();
        return 0;
    }
    // The reduction is one dependent chain; its waves issue ahead of the
    // accumulating waves that share their SIMDs.
    if constexpr (AW > 0) __builtin_amdgcn_s_setprio(1);
    const double hs = double(sc);  // exact power of two
    const int pad = NMAX - n;
    // lower triangle, zero in the padding, from a clamped address (no branch)
    auto entry = [&](const int pr, const int pc) {
        const int hi = max(pr, pc) - pad, lo = min(pr, pc) - pad;
        const T v = S.M[lo >= 0 ? hi * LD + lo : 0];
        return lo >= 0 ? hs * double(v) : 0.0;
    };
    const HhRow<NMAX> R(lane);
    const double col0 = entry(R.pos, pad);
    double x = R.pos > pad ? col0 : 0.0;
    if (WV::team && wave == HW) {
        if (lane == 0) S.ta[0] = hs * double(S.M[0]);
        hh_control<T, NMAX, NT>(S, n, lane, x);
    } else {
        using B = HhBlock<NMAX, HW>;
        const int i = 8 * wave + hh_row_of(lane), j = hh_col_of(lane);
        const HhSelect<B::NA> sel(lane);
        B H;
#pragma unroll
        for (int a = 0; a < B::NA; ++a) {
            H.xr[a] = 0.0;
#pragma unroll
            for (int b = 0; b < B::NB; ++b) H.a[a][b] = entry(i + B::GI * a, j + 8 * b);
        }
#pragma unroll
        for (int b = 0; b < B::NB; ++b) H.xc[b] = 0.0;
        S.u.h.w[wave][R.slot] = 0.0;
        S.u.h.x[wave][R.slot] = x;
        double xl = 0.0, nwl = 0.0;  // x and -w of the last step at this lane's row
        if constexpr (WV::team) hh_product<T, NMAX, NT, 0>(S, n, lane, wave, sel, H, x, xl, nwl);
        else {
            if (lane == 0) S.ta[0] = hs * double(S.M[0]);
            hh_solo<T, NMAX, NT, 0>(S, n, lane, sel, H, x, xl, nwl);
        }
        // last entries: b_{n-2} is the pivot column's last value, a_{n-1} the
        // last diagonal entry after the last update (position NMAX - 1: lane 63
        // of the last product wave)
        if (wave == HW - 1 && lane == 63 && n >= 2) {
            S.tb[n - 2] = x;
            S.ta[n - 1] = fma(2.0 * xl, nwl, H.a[B::NA - 1][B::NB - 1]);
        }
    }
    if constexpr (AW > 0) __builtin_amdgcn_s_setprio(0);
    return 0;
}

// ---------------------------------------------------------------- direct solver
// Binary32 spectra whose eigenvalues are not extremely close are solved without
// the divide step: every eigenvalue by sections and secants of det(T - x I) in
// binary64, every eigenvector by the twisted factorization of T - lambda I
// (Dhillon, Parlett).  Both work on all eigenvalues at once, lanes apart from
// each other, where the divide step is three or four dependent merges of five
// to seven phases each: batch 512, n = 64: 36 -> 20 us after the reduction, n =
// 32: 21 -> 11 us.  A vector's error is about 3e-14 / gap (eigenvalue rounding
// times the vector's length over its twist entry; the twist is found in binary64,
// see direct_factors), inside the space of its close neighbours: vectors of
// eigenvalues closer than DIRECT_CLOSE are made orthogonal in order.  A matrix with a
// pair closer than DIRECT_GAP, with more than DIRECT_MOST close pairs, or whose
// determinants leave the exponent range, goes through the divide step, which does not
// depend on gaps.  (DIRECT_GAP: at 4e-12 the two vectors of a pair are still a few
// hundredths from orthogonal at most before they are made so; an eigenvalue repeated
// exactly in a dense binary32 matrix is 1e-9 apart in most and 1e-10 in some.
// DIRECT_MOST: 64 eigenvalues over four decades leave six close pairs now and then,
// beside one that is 6400 times as large ten; with them n = 64 takes 83 and 93 us, by
// the divide step after all rounds 118 and 142.)
// Distances are of the Gershgorin interval's scale (|T| in [1/2, 1)).
constexpr double DIRECT_CLOSE = 1e-6, DIRECT_GAP = 4e-12;
constexpr int DIRECT_MOST = 16;
constexpr int DIRECT_CAP = 64;       // rounds per eigenvalue
constexpr int DIRECT_LOOK = 5;       // rounds that separated spectra do with
// With vectors, a matrix that will be refused is to be known early: the divide step
// alone takes as long as it took without a direct solver, so the rounds ahead of it
// were lost.  Three looks (us a solve at n = 32 and 64, batch 512, without and with it):
//   at the couplings: DIRECT_SPLIT of them below DIRECT_CLOSE, T has low rank (half
//   rank: 60 -> 45, 114 -> 99); one below DIRECT_APART, T comes apart, and its parts
//   most often share eigenvalues (graph components, Kronecker products; one common
//   eigenvalue: 61 -> 45, 126 -> 96; none: 37 -> 41, 78 -> 88);
//   at the grid (fourfold eigenvalues: 63 -> 48, 132 -> 104; the divide step alone: 46
//   and 100);
//   after DIRECT_LOOK rounds at the brackets.
constexpr int DIRECT_SPLIT = 3;
constexpr double DIRECT_APART = 1e-13;

// Wave 0: T scaled by a power of two to |T| in [1/2, 1) (Gershgorin), as rows
// {a_i, b_{i-1}^2} from the top and, for the bottom half's minors, {a_i, b_i^2}
// from the bottom of the padded order m; padding rows are {4, 0}, whose factors
// 4 - x keep signs.  Couplings count as 2^-52 at least for the minors: with a zero
// one every minor below would be zero where x meets an eigenvalue above.
template <int LPR> __device__ __forceinline__ int direct_order(const int n)
{
    return LPR == 8 ? (n + 15) & ~15 : (n + 7) & ~7;
}
template <int NMAX, int LPR>
__device__ __forceinline__ void direct_setup(DirectArrays<NMAX>& D, const double* ta,
                                             const double* tb, const int n, const int lane,
                                             const bool want_q)
{
    constexpr int R = NMAX > 64 ? NMAX / 64 : 1;  // rows per lane
    double a[R], bl[R], br[R];
    float hi = -3e38f, nlo = -3e38f;
#pragma unroll
    for (int k = 0; k < R; ++k) {
        const int e = lane + 64 * k;
        const bool in = e < n;
        a[k] = ta[in ? e : 0];
        bl[k] = (in && e > 0) ? tb[e - 1] : 0.0;
        br[k] = (e + 1 < n) ? tb[e] : 0.0;
        const double r = f_abs(bl[k]) + f_abs(br[k]);
        hi = in ? f_max(hi, float(a[k] + r)) : hi;
        nlo = in ? f_max(nlo, float(r - a[k])) : nlo;
    }
#define BED_MAX_STAGE(ST) hi = f_max(hi, xmove<ST>(hi, lane)), nlo = f_max(nlo, xmove<ST>(nlo, lane))
    BED_MAX_STAGE(1);
    BED_MAX_STAGE(2);
    BED_MAX_STAGE(4);
    BED_MAX_STAGE(8);
    BED_MAX_STAGE(16);
    BED_MAX_STAGE(32);
#undef BED_MAX_STAGE
    const int ex = exp_field(f_max(hi, nlo));
    const int sh = min(max(fexp<float>::BIAS - 1 - ex, -fexp<float>::SMAX), fexp<float>::SMAX);
    const double sc = double(fexp<float>::pow2(sh));
    const int m = direct_order<LPR>(n);
    bool several;
    if (want_q) {
        int split = 0;
        bool apart = false;
#pragma unroll
        for (int k = 0; k < R; ++k) {
            const bool in = lane + 64 * k + 1 < n;
            split += __popcll(__ballot(in && f_abs(br[k]) * sc < DIRECT_CLOSE));
            apart = apart || (in && f_abs(br[k]) * sc < DIRECT_APART);
        }
        several = split >= DIRECT_SPLIT || __ballot(apart);
    } else {
        // Eigenvalues alone have no gap to keep, but a determinant that must not vanish:
        // near an eigenvalue of its null block each row without a coupling costs it up to
        // 51 bits (the last rounds' distance), a halves' determinant those of its lower
        // half.  More than start and end of the range hold: to the divide step at once
        // (half rank, n = 128: 284 us, 358 after all rounds).
        int lost = 0;
#pragma unroll
        for (int k = 0; k < R; ++k) {
            const int e = lane + 64 * k, bits = min(1022 - exp_field(bl[k] * sc), 51);
            lost += (e > 0 && e < n && (LPR == 4 || e >= m / 2) && bits >= 20) ? bits : 0;
        }
        several = group_sum<64>(lost, lane) > (LPR == 4 ? 1580 : 840);
    }
#pragma unroll
    for (int k = 0; k < R; ++k) {
        const int e = lane + 64 * k;
        const bool in = e < n;
        if (e < m) {
            const double as = in ? a[k] * sc : 4.0, bs = bl[k] * sc, bt = br[k] * sc;
            D.ab[0][e][0] = as;
            D.ab[0][e][1] = in && e > 0 ? fmax(bs * bs, 0x1p-104) : 0.0;
            D.ab[1][m - 1 - e][0] = as;
            D.ab[1][m - 1 - e][1] = e + 1 < n ? fmax(bt * bt, 0x1p-104) : 0.0;
            D.b[0][e] = bt;
            D.b[1][in ? n - 1 - e : e] = in ? bs : 0.0;  // coupling of row e to the row above
            D.cell[e] = -2;
        }
    }
    if (lane == 0) {
        D.lo = -double(nlo) * sc - 1e-6;
        D.hi = double(hi) * sc + 1e-6;
        D.unscale = double(fexp<float>::pow2(-sh));
        D.single = 0;
        D.ok = (n >= 2 && ex > fexp<float>::BIAS - 64 && !several) ? 1 : 0;
    }
}

// Minors of T - x I over `blocks` blocks of eight rows of a table {a, b^2}, p_i =
// (a_i - x) p_{i-1} - b^2 p_{i-2}: the last two (p1, p0) and the number of sign
// changes.  |a_i - x| <= 2, so n <= 128 minors stay within 2^192; they start at 2^800
// (halves, whose products are formed: 2^400), which leaves the small ones that much
// more room.  (Eigenvalues alone, us, without and with these two: half rank n = 64
// 122 -> 73, six-fold n = 30 63 -> 40, which is what the divide step takes.)
// `wide`: minors below 1 after half of the blocks go on 2^800 times as large (`scaled`).
template <int LPR>
__device__ __forceinline__ int direct_minors(const double* rows, const int blocks, const double x,
                                             const bool wide, double& p1, double& p0, bool& scaled)
{
    typedef double d2 __attribute__((ext_vector_type(2)));
    p0 = 0.0;
    p1 = LPR == 8 ? 0x1p400 : 0x1p800;
    scaled = false;
    uint32_t m = 0;  // signs of the minors, the latest in bit 0
    int c = 0;
    const d2* row = reinterpret_cast<const d2*>(rows);
    int left = wide ? blocks >> 1 : blocks;
#pragma unroll 1
    for (int part = 0;; ++part) {
#pragma unroll 1
        for (int b = 0; b < left; ++b) {
            d2 cur[8];
#pragma unroll
            for (int q = 0; q < 8; ++q) cur[q] = row[q];
#pragma unroll
            for (int q = 0; q < 8; ++q) {
                const double p2 = fma(cur[q].x - x, p1, -(cur[q].y * p0));
                m = __builtin_amdgcn_alignbit(m, (uint32_t)__double2hiint(p2), 31);
                p0 = p1;
                p1 = p2;
            }
            c += __popc((m ^ (m >> 1)) & 0xFFu);
            row += 8;
        }
        if (!wide || part == 1) break;
        left = blocks - left;
        const double top = f_max(f_abs(p1), f_abs(p0));
        scaled = top < 1.0 && top >= 0x1p-950;  // (below: too small to trust)
        p1 *= scaled ? 0x1p800 : 1.0;
        p0 *= scaled ? 0x1p800 : 1.0;
    }
    return c;
}

// det(T - x I) and the number of eigenvalues below x.  LPR = 8: the lane and
// lane ^ 4 share a point x, the first taking the leading minors P of the upper
// half, the other the trailing minors R of the lower half (rows h ..):
//   det = P_h R_h - b_{h-1}^2 P_{h-1} R_{h+1},
// and the count is the inertia of the factorization twisted at row h, whose last
// pivot has the sign of det / (P_h R_{h+1}).  `tiny`: too small to trust.
// `wide` (n > 64, eigenvalues alone): the minors at a point among 127 eigenvalues
// within 2e-4 of the interval fall by 1800 bits, more than one exponent range, so they
// are scaled once on the way where they need it.  Such a bulk beside an eigenvalue
// 6400 times as large, n = 128, batch 512: 484 -> 233 us, the divide step alone 389.
// With vectors its gaps are refused, the sooner the better.
template <int LPR, int NMAX>
__device__ __forceinline__ double direct_det(const double (*ab)[NMAX][2], const int m, const int sub,
                                             const double x, const bool wide, int& count, bool& tiny,
                                             bool& scaled)
{
    // both of the last minors near the end of the exponent range (for halves,
    // of their products)
    auto vanished = [](const double u, const double v) {
        const int eu = __double2hiint(u) & 0x7fffffff, ev = __double2hiint(v) & 0x7fffffff;
        return max(eu, ev) < (1023 - (LPR == 8 ? 480 : 950)) << 20;
    };
    double p1, p0;
    if constexpr (LPR == 4) {
        count = direct_minors<LPR>(&ab[0][0][0], m >> 3, x, wide, p1, p0, scaled);
        tiny = vanished(p1, p0);
        return p1;
    } else {
        const bool low = sub >= 4;
        int c = direct_minors<LPR>(&ab[low ? 1 : 0][0][0], m >> 4, x, false, p1, p0, scaled);
        const double bh = ab[0][m >> 1][1];
        const double q1 = lxor<4>(p1), q0 = lxor<4>(p0);
        const int oc = lxor<4>(c);
        const double det = fma(p1, q1, -(bh * (p0 * q0)));
        const double P = low ? q1 : p1, R = low ? p0 : q0, Rh = low ? p1 : q1;
        auto neg = [](const double v) { return __double2hiint(v) < 0; };
        count = c + oc - (neg(Rh) != neg(R) ? 1 : 0) + ((neg(det) != neg(P)) != neg(R) ? 1 : 0);
        tiny = vanished(p1, p0);
        return det;
    }
}

// Eigenvalues: the team evaluates a grid of NT points first, which brackets
// every eigenvalue; then each eigenvalue's lanes evaluate four points a round
// inside its bracket: equally spaced, or, once the bracket holds this
// eigenvalue alone, around the root of the cubic that interpolates x as a
// function of det at the last four points, at one and eight times its error.
// That is taken as its distance from the quadratic's root, or as what the
// quadratic's distance from the secant's lets expect (the distance alone can
// vanish by accident where det varies strongly).  A root stops when it is below
// 2^-44 of the interval and the points enclose this eigenvalue alone (the
// cubic's own error is then at rounding level).  About four rounds after the grid.
// With vectors: every gap at least DIRECT_GAP.  Returns whether solved.
template <int NMAX, int NT>
__device__ __forceinline__ bool direct_eigenvalues(DirectArrays<NMAX>& D, DirectGrid<NT>& G,
                                                   const int n, const int t, const bool want_q,
                                                   float* __restrict__ Lc)
{
    constexpr int LPR = NT / NMAX;
    static_assert(LPR == 4 || LPR == 8, "lanes per eigenvalue");
    const int lane = t & 63;
    const int m = direct_order<LPR>(n);
    if (!D.ok) return false;
    const int j = t / LPR, sub = t % LPR;
    const bool act = j < n;
    bool bad = false;
    const bool wide = NMAX > 64 && !want_q;
    constexpr int SCALED = 1 << 16;  // in the grid's counts
    auto number = [](const int c) { return NMAX > 64 ? c & (SCALED - 1) : c; };
    {
        const double glo = D.lo, ghi = D.hi;
        // grid points: lane pairs of LPR = 8 share one
        constexpr int NG = LPR == 8 ? NT / 2 : NT;
        const int gi = LPR == 8 ? (t >> 3) * 4 + (t & 3) : t;
        const double step = (ghi - glo) * (1.0 / (NG + 1));
        auto grid = [&](const int i) { return fma(double(i + 1), step, glo); };
        double lo = glo, hi = ghi;
        int clo = 0, chi = n;
        double X[4] = {0.0, 0.0, 0.0, 0.0}, F[4] = {0.0, 0.0, 0.0, 0.0};
        bool have = false;    // X, F hold four points
        bool strict = false;  // they enclose this eigenvalue and no other
        int near = 0;         // eigenvalues that the first four enclose
        {
            int c;
            bool tiny, scaled;
            const double f = direct_det<LPR, NMAX>(D.ab, m, sub, grid(gi), wide, c, tiny, scaled);
            bad = tiny;
            if (LPR == 4 || sub < 4) {
                G.f[gi] = f;
                G.c[gi] = scaled ? c | SCALED : c;
            }
            team_sync<NT>();
            if (LPR == 4 || sub < 4) {
                // eigenvalues between this point and the next (before the first)
                const int cn = (gi + 1 < NG) ? number(G.c[gi + 1]) : n;
                for (int q = max(c, 0); q < min(cn, n); ++q) D.cell[q] = gi;
                if (gi == 0)
                    for (int q = 0; q < min(c, n); ++q) D.cell[q] = -1;
            }
            team_sync<NT>();
            const int cell = act ? D.cell[j] : -2;
            if (cell >= 0) lo = grid(cell), clo = number(G.c[cell]);
            if (cell >= -1 && cell + 1 < NG) hi = grid(cell + 1), chi = number(G.c[cell + 1]);
            const int k0 = min(max(cell - 1, 0), NG - 4);
            have = cell >= -1;
            if (NMAX > 64) {  // (as in the rounds)
                const int c0 = G.c[k0], d = (c0 ^ G.c[k0 + 1]) | (c0 ^ G.c[k0 + 2]) | (c0 ^ G.c[k0 + 3]);
                have = have && (d & SCALED) == 0;
            }
            {
                const int ca = number(G.c[k0]), cb = number(G.c[k0 + 3]);
                strict = ca == j && cb == j + 1;
                near = cb - ca;
            }
#pragma unroll
            for (int q = 0; q < 4; ++q) {
                X[q] = grid(k0 + q);
                F[q] = G.f[k0 + q];
            }
        }
        // Most eigenvalues in cells (a quarter of the mean spacing wide) with others, the
        // cells beside them empty: they are multiple ones.  Graded and clustered spectra
        // fill neighbouring cells, or crowd one.
        if (want_q) {
            const int here = chi - clo;
            const int own = __popcll(__ballot(act && (here == 1 || near != here || 4 * here > n))) / LPR;
            if (lane == 0 && own > 0) atomicAdd(&D.single, own);
            if (__ballot(bad) && lane == 0) D.ok = 0;
            team_sync<NT>();
            if (!D.ok || 4 * D.single <= n) return false;
        }
        const int pt = sub & 3;
        const double spread = pt == 0 ? -8.0 : (pt == 1 ? -1.0 : (pt == 2 ? 1.0 : 8.0));
        const double even = double(pt + 1) * 0.2, fl = double(pt + 1) * 0x1p-9, fh = double(4 - pt) * -0x1p-9;
        double lam = 0.0;
        bool done = !act;
        int rounds = 0;
        for (;;) {
            const double w = hi - lo;
            // inverse interpolation at det = 0 (Neville), offsets from X[1]
            double est = fma(0.5, w, lo), err = w;
            {
                const double x2 = X[2] - X[1], x0 = X[0] - X[1], x3 = X[3] - X[1];
                auto comb = [](const double pa, const double pb, const double fa, const double fb) {
                    return fma(pb - pa, fa * __builtin_amdgcn_rcp(fa - fb), pa);
                };
                const double a0 = x2 * (F[1] * __builtin_amdgcn_rcp(F[1] - F[2]));
                const double a1 = comb(x2, x0, F[2], F[0]);
                const double a2 = comb(x0, x3, F[0], F[3]);
                const double b0 = comb(a0, a1, F[1], F[0]);
                const double b1 = comb(a1, a2, F[2], F[3]);
                const double c0 = comb(b0, b1, F[1], F[3]);
                const double e = X[1] + c0;
                // (comparisons are false for a NaN)
                const bool in = have && chi - clo == 1 && e >= lo && e <= hi;
                est = in ? e : est;
                const double d = b0 - a0;
                err = in ? f_max(f_max(f_abs(c0 - b0), d * d * __builtin_amdgcn_rcp(f_abs(x2))), 0x1p-53) : w;
            }
            const bool stop = !(w > 0x1p-51) || (strict && err <= 0x1p-44);
            lam = done ? lam : est;
            done = done || stop;
            if (rounds >= (want_q ? DIRECT_LOOK : DIRECT_CAP)) {
                // what the checks below will most likely refuse (seven of the wave's 16, four
                // of its 8 eigenvalues next to another): no use in finding it exactly
                const bool pair = want_q && act && j + 1 < chi;  // the next one is in here too
                bad = bad || (pair && w < DIRECT_GAP) || (rounds >= DIRECT_CAP && !done);
                if (__ballot(bad) || __popcll(__ballot(pair && w < 6.0 * DIRECT_CLOSE)) >= 28)
                    bad = done = true;
            }
            if (!__ballot(!done)) break;  // Eq. (22): converged lanes idle till here
            // points in ascending order over the lanes
            const double xn = fmin(fmax(fma(err, spread, est), fma(w, fl, lo)), fma(w, fh, hi));
            const double x = err < 0.25 * w ? xn : fma(w, even, lo);
            int c;
            bool tiny, scaled;
            const double f = direct_det<LPR, NMAX>(D.ab, m, sub, x, wide, c, tiny, scaled);
            bad = bad || (tiny && !done);
            int C[4];
            bool Bl[4];
            auto gather = [&](auto Q, const double v) {
                constexpr int q = decltype(Q)::value;
                return dpp_move64<q * 0x55>(v);  // quad_perm [q, q, q, q]
            };
            static_for<0, 4>([&](auto Q) {
                constexpr int q = decltype(Q)::value;
                X[q] = gather(Q, x);
                F[q] = gather(Q, f);
                C[q] = __builtin_amdgcn_mov_dpp(c, q * 0x55, 0xF, 0xF, false);
                Bl[q] = C[q] <= j;
            });
#pragma unroll
            for (int q = 0; q < 4; ++q) {
                lo = Bl[q] ? X[q] : lo;
                clo = Bl[q] ? C[q] : clo;
                hi = Bl[3 - q] ? hi : X[3 - q];
                chi = Bl[3 - q] ? chi : C[3 - q];
            }
            have = true;
            if (NMAX > 64) {
                // determinants of one scale only are interpolated
                const uint64_t sb = __ballot(scaled);
                if (sb != 0) {
                    const uint32_t four = uint32_t(sb >> (lane & 60)) & 15;
                    have = four == 0 || four == 15;
                }
            }
            strict = C[0] == j && C[3] == j + 1;
            ++rounds;
        }
        if (act && sub == 0) {
            D.lam[j] = lam;
            Lc[j] = float(lam * D.unscale);
        }
    }
    if (__ballot(bad) && lane == 0) D.ok = 0;
    team_sync<NT>();
    BED_PHASE(3);
    constexpr int CW = (NMAX + 63) / 64;  // words of the mask of close pairs
    if (want_q && t < 64 * CW) {
        const double gap = t + 1 < n ? D.lam[t + 1 < n ? t + 1 : 0] - D.lam[t < n ? t : 0] : 1.0;
        const uint64_t close = __ballot(!(gap >= DIRECT_CLOSE));
        if (lane == 0) D.close[t >> 6] = close;
        if (__ballot(!(gap >= DIRECT_GAP)) != 0 || __popcll(close) > DIRECT_MOST) D.ok = 0;
    }
    team_sync<NT>();
    return D.ok != 0;
}

// Factors of T - lambda I from the top (L D L^T) and from the bottom (U D U^T)
// for the NC eigenvalues from c0 on, one lane each per eigenvalue: l_i = b / D_i
// toward the next row, rounded to binary32 (a relative perturbation of the
// vector's entries).  A zero pivot becomes 1e-25, far below the rounding of T.
//
// F = float: the lanes of an eigenvalue meet in the middle, and each forms on its
// second half gamma_i = D_i - b l', its own pivot in binary64 and the other one's l' of
// the row ahead: as two binary32 parts, the low one kept where the lane itself
// will write that row.  The twist has to come from there: gamma from the rounded
// factors is known to about 5e-8 of T, and where T comes apart (a vanishing
// coupling, which no product of factors crosses) such noise chose between the
// parts' rows for eigenvalues that the parts share to less than that.  The row of
// smallest |gamma_i| + 2^-46 |D_i| (2^-46: the parts' rounding) goes to D.twist,
// one entry per lane.  F = double keeps the factors in full, where LDS has room, and
// leaves gamma to direct_vector, whose lanes share the rows.  (Batch 64, us, gamma of
// rounded factors / in halves / in full: n = 16 17.2, 18.0, 17.5, n = 32 25.8, 26.5,
// 26.3; batch 512: n = 64 72.3, 72.9, n = 128 314.8, 313.2, no room for the full ones.)
template <int NMAX, int NT, int NC, int LPR, int LD, typename F>
__device__ __forceinline__ void direct_factors(DirectArrays<NMAX>& D, F* Lp, F* Lm, const int n,
                                               const int t, const int c0)
{
    constexpr bool WIDE = sizeof(F) == 8;
    const int j = t % NC, e = c0 + j;
    const bool up = t / NC != 0;
    const bool act = t < 2 * NC && e < n;
    const double x = D.lam[act ? e : 0];
    const double* ar = &D.ab[up ? 1 : 0][up ? direct_order<LPR>(n) - n : 0][0];
    const double* bk = &D.b[up ? 1 : 0][0];
    if (act && up && n < NMAX) Lm[n * LD + j] = F(0);  // below the last row (its coupling is zero)
    const int dL = up ? -LD : LD, first = up ? (n - 1) * LD + j : j;
    F* L = (up ? Lm : Lp) + first;  // this lane's factors, at row k
    F* O = (up ? Lp : Lm) + first;  // the other lane's
    const int h = WIDE ? n : (up ? n - n / 2 : n / 2);
    double bp = 0.0, l = 0.0;
    auto pivot = [&](const int k) { return fma(-bp, l, ar[2 * k] - x); };
    auto next = [&](double d, const double bn, F* at) {
        d = f_abs(d) < 1e-25 ? 1e-25 : d;
        // b / d: one third-order step from the hardware's estimate
        const double r = __builtin_amdgcn_rcp(d), br = bn * r, er = fma(-d, r, 1.0);
        l = fma(br, fma(er, er, er), br);
        bp = bn;
        *at = F(l);
    };
    if (act) {
#pragma unroll 4
        for (int k = 0; k < h; ++k) {
            next(pivot(k), bk[k], L);
            if constexpr (!WIDE) *O = F(l - double(*L));
            L += dL;
            O += dL;
        }
    }
    if constexpr (WIDE) return;
    if constexpr (2 * NC > 64) team_sync<NT>();  // the two lanes sit in different waves
    else wave_sync();
    if (act) {
        uint32_t best = ~0u;
        F oh = F(0), ol = F(0);  // the other lane's factor of the row ahead
        auto ahead = [&] {
            oh = O[dL];
            ol = L[dL];
        };
        auto row = [&](const int k, auto another) {
            const double bn = bk[k], d = pivot(k);
            const double lx = double(oh) + double(ol);
            L += dL;
            O += dL;
            if constexpr (decltype(another)::value) ahead();
            const double g = fma(0x1p-46, f_abs(d), f_abs(fma(-bn, lx, d)));
            const uint32_t key = (__float_as_uint(float(g)) & ~127u) | (uint32_t)k;
            best = key < best ? key : best;
            next(d, bn, L - dL);
        };
        if (h < n - 1) ahead();
        int k = h;
#pragma unroll 4
        for (; k < n - 2; ++k) row(k, std::true_type{});
        for (; k < n; ++k) row(k, std::false_type{});  // (at the last row b = 0)
        if (up) best = (best & ~127u) | (uint32_t)(n - 1 - (int)(best & 127u));
        D.twist[up ? 1 : 0][e] = best;
    }
}

// Entries i0 = SG (t % LPR), i0 + 1, ... of the eigenvector of eigenvalue e (Lp, Lm:
// its columns of the factors), of norm one: z = 1 at the twist row, where
// |gamma_i| = |e_i^T (T - x)^{-1} e_i|^{-1} is smallest, and products of -l
// outward; rows of a group's lane are consecutive, its products are finished by
// a scan over the group.  act: lanes that hold an eigenvalue (the others compute
// on a valid column).  Rows past n hold anything; the products stop at n.
template <int NMAX, int LPR, int LD, typename T>
__device__ __forceinline__ void direct_vector(const DirectArrays<NMAX>& D, const T* Lp, const T* Lm,
                                              const int e, const bool act, const int n, const int t,
                                              float (&out)[NMAX / LPR])
{
    constexpr int SG = NMAX / LPR;
    const int lane = t & 63, sub = t % LPR;
    const int i0 = sub * SG;
    T lp[SG], lm[SG];
#pragma unroll
    for (int s = 0; s < SG; ++s) {
        lp[s] = Lp[(i0 + s) * LD];
        lm[s] = Lm[(i0 + s) * LD];
    }
    int r;
    if constexpr (sizeof(T) == 8) {
        const double x = D.lam[e];
        const int ia = max(i0 - 1, 0);
        double lprev = Lp[ia * LD], bprev = i0 > 0 ? D.b[0][ia] : 0.0;  // of the row before
        const double lafter = Lm[min(i0 + SG, NMAX - 1) * LD];
        int best = 0x7fffffff;
#pragma unroll
        for (int s = 0; s < SG; ++s) {
            const int i = i0 + s;
            const double bn = D.b[0][i];  // zero at the last row
            const double below = bn * (s + 1 < SG ? lm[s + 1 < SG ? s + 1 : 0] : lafter);
            const double gam = fma(-bprev, lprev, D.ab[0][i][0] - x - below);
            const int key = (__float_as_int(float(fma(0x1p-46, f_abs(below), f_abs(gam)))) & ~127) | i;
            best = i < n ? min(best, key) : best;
            lprev = lp[s];
            bprev = bn;
        }
        best = min(best, xmove<1>(best, lane));
        best = min(best, xmove<2>(best, lane));
        if constexpr (LPR == 8) best = min(best, xmove<4>(best, lane));
        r = best & 127;
    } else {
        r = min(D.twist[0][e], D.twist[1][e]) & 127u;
    }
    double z[SG];
    double n2 = 0.0;
    // second pass: from the largest entry, where the first twist row was
    // much smaller (an eigenvalue exact to rounding leaves only noise in gamma)
    for (int pass = 0; pass < 2; ++pass) {
        // opaque, or the compiler widens all of them once, ahead of the loop,
        // into registers that it has not got
#pragma unroll
        for (int s = 0; s < SG; ++s) asm volatile("" : "+v"(lp[s]), "+v"(lm[s]));
        // products within the lane, from its last row up to the twist and
        // from its first row down, one where the twist does not lie beyond
        double up = 1.0, dn = 1.0;
#pragma unroll
        for (int s = SG - 1; s >= 0; --s) {
            const bool above = i0 + s < r;
            up = above ? -up * double(lp[s]) : 1.0;
            z[s] = up;
        }
#pragma unroll
        for (int s = 0; s < SG; ++s) {
            const int i = i0 + s;
            dn = i > r ? -dn * double(i < n ? lm[s] : T(0)) : 1.0;
            z[s] = i > r ? dn : z[s];
        }
        // products of the lanes below (up) and above (dn) in the group
        double cu = 1.0, cd = 1.0;
#pragma unroll
        for (int q = 1; q < LPR; ++q) {
            const double ou = __shfl(up, lane + q), od = __shfl(dn, lane - q);
            cu *= sub + q < LPR ? ou : 1.0;
            cd *= sub - q >= 0 ? od : 1.0;
        }
        n2 = 0.0;
        double zb = 0.0;
        int ri = 0;
#pragma unroll
        for (int s = 0; s < SG; ++s) {
            const int i = i0 + s;
            z[s] *= i < r ? cu : (i > r ? cd : 1.0);
            n2 = fma(z[s], z[s], n2);
            const double az = f_abs(z[s]);
            ri = az > zb ? i : ri;
            zb = f_max(zb, az);
        }
        n2 = group_sum<LPR>(n2, lane);
        const bool far = act && zb > 8.0;
        if (!__ballot(far)) break;
        auto most = [&](const double ob, const int orr) {
            const bool take = ob > zb || (ob == zb && orr < ri);
            zb = take ? ob : zb;
            ri = take ? orr : ri;
        };
        most(xmove<1>(zb, lane), xmove<1>(ri, lane));
        most(xmove<2>(zb, lane), xmove<2>(ri, lane));
        if constexpr (LPR == 8) most(xmove<4>(zb, lane), xmove<4>(ri, lane));
        r = zb > 8.0 ? ri : r;
    }
    const double sc = d_rsqrt_nr(n2);
#pragma unroll
    for (int s = 0; s < SG; ++s) out[s] = float(z[s] * sc);
}

// One wave: Gram-Schmidt along each run of close eigenvalues, in order; at(i, j)
// is entry i of vector j.
template <int NMAX, typename At>
__device__ __forceinline__ void direct_orthogonal(const DirectArrays<NMAX>& D, const int n,
                                                  const int lane, const At& at)
{
    constexpr int R = (NMAX + 63) / 64;  // rows lane + 64 k
    int first = 0, last = -2;  // of the current run
#pragma unroll 1
    for (int w = 0; w < R; ++w) {
        uint64_t todo = D.close[w];
        while (todo) {
            const int j = 64 * w + __builtin_ctzll(todo);
            todo &= todo - 1;
            first = j == last + 1 ? first : j;
            last = j;
            double v[R];
#pragma unroll
            for (int k = 0; k < R; ++k)
                v[k] = lane + 64 * k < n ? double(at(lane + 64 * k, j + 1)) : 0.0;
            for (int q = first; q <= j; ++q) {
                double u[R], d = 0.0;
#pragma unroll
                for (int k = 0; k < R; ++k) {
                    u[k] = lane + 64 * k < n ? double(at(lane + 64 * k, q)) : 0.0;
                    d = fma(u[k], v[k], d);
                }
                d = wave_sum_all(d);
#pragma unroll
                for (int k = 0; k < R; ++k) v[k] = fma(-d, u[k], v[k]);
            }
            double d = 0.0;
#pragma unroll
            for (int k = 0; k < R; ++k) d = fma(v[k], v[k], d);
            d = d_rsqrt_nr(wave_sum_all(d));
#pragma unroll
            for (int k = 0; k < R; ++k)
                if (lane + 64 * k < n) at(lane + 64 * k, j + 1) = float(v[k] * d);
            wave_sync();
        }
    }
}

template <int NMAX>
__device__ __forceinline__ bool direct_close(const DirectArrays<NMAX>& D)
{
    uint64_t any = 0;
#pragma unroll
    for (int k = 0; k < (NMAX + 63) / 64; ++k) any |= D.close[k];
    return any != 0;
}

// The spectrum of T (S.ta, S.tb, set up); eigenvectors into Q0.  Returns whether
// solved.
template <typename T, int NMAX, int NT>
__device__ __forceinline__ bool direct_solve(Smem<T, NMAX, NT>& S, const int n, const int t,
                                             const bool want_q, T* __restrict__ Lc)
{
    constexpr int LPR = NT / NMAX;
    constexpr int LD = Smem<T, NMAX, NT>::LD;
    DirectArrays<NMAX>& D = S.u.d.t;
    if (!direct_eigenvalues<NMAX, NT>(D, S.u.d.g, n, t, want_q, Lc)) return false;
    if (!want_q) return true;
    constexpr bool WIDE = DirectWide<T, NMAX, NT>::value;
    auto factors = [&](const int q) {
        if constexpr (WIDE) return q ? S.fm.l : S.u.d.f.l;
        else return q ? S.Q1 : S.Q0;
    };
    direct_factors<NMAX, NT, NMAX, LPR, LD>(D, factors(0), factors(1), n, t, 0);
    team_sync<NT>();
    BED_PHASE(6);
    {
        constexpr int SG = NMAX / LPR;
        const int j = t / LPR, i0 = (t % LPR) * SG;
        const bool act = j < n;
        const int e = act ? j : 0;
        float z[SG];
        direct_vector<NMAX, LPR, LD>(D, factors(0) + e, factors(1) + e, e, act, n, t, z);
        wave_sync();
        if (act) {
#pragma unroll
            for (int s = 0; s < SG; ++s)
                if (i0 + s < n) S.Q0[(i0 + s) * LD + e] = z[s];
        }
    }
    team_sync<NT>();
    if (direct_close(D)) {
        if (t < 64)
            direct_orthogonal(D, n, t, [&](const int i, const int j) -> T& { return S.Q0[i * LD + j]; });
        team_sync<NT>();
    }
    BED_PHASE(7);
    return true;
}

// TRI: the input is already tridiagonal, given as its diagonal a (n values)
// followed by its off-diagonal b (n - 1 values) at Ain; there is no reduction
// and Q_H is the identity, so Q is Q_T (no back-transform).  ends_out (TRI,
// eigenvalues only): the first and last rows of Q_T, all that a merge above
// reads (Eq. (5)), as 2n values.
template <typename T, int NMAX, int NT, bool TRI = false>
__device__ __forceinline__ void syevd_team(const T* __restrict__ Ain, const int n,
                                           T* __restrict__ lam_out, T* __restrict__ Q_out,
                                           int* __restrict__ info_out, Smem<T, NMAX, NT>& S,
                                           const int t, const int leaf_arg = 0,
                                           T* __restrict__ ends_out = nullptr)
{
    static_assert(NMAX <= 64 && (NMAX & (NMAX - 1)) == 0, "NMAX: power of two <= 64");
    static_assert(NT % 64 == 0 && NT >= NMAX && NT % NMAX == 0, "team geometry");
    constexpr int LD = Smem<T, NMAX, NT>::LD;
    constexpr int NW = NT / 64;
    constexpr int LPR = NT / NMAX;
    const int lane = t & 63;
    const int wave = __builtin_amdgcn_readfirstlane(t >> 6);
    const T u = fp<T>::u;
    const int leaf = leaf_arg > 0 ? leaf_arg : leaf_default(NMAX);

    BED_PHASE(0);
    // ------------------------------------------------------------ load
    // 16-byte loads when the rows allow it (n a multiple of the vector width
    // and A 16-byte aligned), else one element per thread and step.  A
    // non-finite entry of the lower triangle is flagged per wave by a ballot,
    // and the largest magnitude's exponent is kept for the scaling below.
    {
        constexpr int VW = 16 / sizeof(T);
        bool bad = false;
        T amax = T(0);
        if constexpr (TRI) {
            for (int e = t; e < 2 * n - 1; e += NT) {
                const T v = Ain[e];
                bad = bad || !f_finite(v);
                amax = f_max(amax, f_abs(v));
                if (e < n) S.a[e] = v;
                else S.b[e - n] = v;
            }
        } else if (n % VW == 0 && (reinterpret_cast<uintptr_t>(Ain) & 15) == 0) {
            typedef T vec_t __attribute__((ext_vector_type(VW)));
            const vec_t* Av = reinterpret_cast<const vec_t*>(Ain);
            const int nv = n * n / VW;
            for (int e = t; e < nv; e += NT) {
                const vec_t v = Av[e];
                const int i = (e * VW) / n, j = (e * VW) % n;
#pragma unroll
                for (int q = 0; q < VW; ++q) {
                    if (j + q <= i && !f_finite(v[q])) bad = true;
                    amax = (j + q <= i) ? f_max(amax, f_abs(v[q])) : amax;
                    S.M[i * LD + j + q] = v[q];
                }
            }
        } else {
            for (int i = t / n, j = t % n, e = t; e < n * n; e += NT) {
                T v = Ain[e];
                if (j <= i && !f_finite(v)) bad = true;  // lower triangle only
                amax = (j <= i) ? f_max(amax, f_abs(v)) : amax;
                S.M[i * LD + j] = v;
                j += NT % n;
                i += NT / n;
                if (j >= n) {
                    j -= n;
                    ++i;
                }
            }
        }
        const bool wbad = __ballot(bad) != 0;
        const int wexp = group_max<64>(exp_field(amax), lane);
        if (lane == 0) {
            S.badw[wave] = wbad ? 1 : 0;
            S.expw[wave] = wexp;
        }
        if (t == 0) S.capped = 0;
    }
    team_sync<NT>();
    int anybad = 0;
#pragma unroll
    for (int w = 0; w < NW; ++w) anybad |= S.badw[w];
    if (anybad) {
        if (Q_out)
            for (int e = t; e < n * n; e += NT) Q_out[e] = f_nan<T>();
        for (int e = t; e < n; e += NT) lam_out[e] = f_nan<T>();
        if (t == 0 && info_out) *info_out = -1;
        return;
    }
    BED_PHASE(1);

    // ------------------------------------------------------------ Householder
    constexpr int AW = QH_WAVES<T, NMAX, NT>::value;
    constexpr int QW = HhWaves<T, NMAX, NT>::first_qh;
    const bool qh_wave = AW > 0 && wave >= QW && wave < QW + AW && Q_out != nullptr;
    T qh[QhShape<T, NMAX, NT>::VPL];
    int qj;
    if constexpr (TRI) {
        // exact power-of-two scaling of the given diagonals (the same threads
        // wrote them); Q_H = I is never formed
        const T sc = fexp<T>::pow2(input_shift(S));
        for (int e = t; e < 2 * n - 1; e += NT) {
            if (e < n) S.a[e] *= sc;
            else S.b[e - n] = coupling(S.b[e - n] * sc);
        }
        qj = n - 2;
    } else {
        qj = householder<T, NMAX, NT>(S, n, lane, wave, Q_out != nullptr,
                                      fexp<T>::pow2(input_shift(S)), qh);
    }
    team_sync<NT>();
    if constexpr (AW > 0 && !TRI) {
        // reflectors written after the last barrier of the reduction
        if (qh_wave)
            for (; qj < n - 2; ++qj) qh_apply<T, NMAX, NT>(S, lane, qj, qh);
    }
    constexpr bool DIRECT = std::is_same<T, float>::value && !TRI && LPR >= 4;
    const bool direct = DIRECT && leaf_arg == 0;
    if constexpr (DIRECT) {
        if (direct && wave == 0) direct_setup<NMAX, NT / NMAX>(S.u.d.t, S.ta, S.tb, n, lane, Q_out != nullptr);
    }
    team_sync<NT>();
    if constexpr (AW > 0 && !TRI) {
        // every reflector has been read: Q_H replaces them
        if (qh_wave) {
            constexpr int RW = QhShape<T, NMAX, NT>::RW;
            constexpr int VPL = QhShape<T, NMAX, NT>::VPL;
            constexpr int VLD = Smem<T, NMAX, NT>::VLD;
            constexpr int VW = 16 / sizeof(T);
            typedef T vec_t __attribute__((ext_vector_type(VW)));
            const int row = (wave - QW) * RW + lane % RW, c0 = (lane / RW) * VPL;
            vec_t* qp = reinterpret_cast<vec_t*>(S.Vt + row * VLD + c0);
#pragma unroll
            for (int q = 0; q < VPL / VW; ++q) {
                vec_t x;
#pragma unroll
                for (int e = 0; e < VW; ++e) x[e] = qh[q * VW + e];
                qp[q] = x;
            }
        }
    }
    BED_PHASE(2);

    T* Qc = S.Q0;
    T* Qn = S.Q1;
    T* Lc = S.lam0;
    T* Ln = S.lam1;
    // the direct solver takes the matrix unless its spectrum is too close
    bool solved = false;
    if constexpr (DIRECT) {
        if (direct) solved = direct_solve(S, n, t, Q_out != nullptr, Lc);
    }
    if (!solved) {
    // ------------------------------------------------------------ tear + leaves
    // The staging buffer becomes the merge matrix M: clear it so that entries
    // outside every node block (never written by a merge) are zero -- the MFMA
    // back-multiplication reads them against zero A entries.
    for (int e = t; e < NMAX * LD; e += NT) S.M[e] = T(0);
    if constexpr (!TRI) {  // T in the storage type
        for (int e = t; e < n; e += NT) {
            S.a[e] = T(S.ta[e]);
            S.b[e] = coupling(T(e + 1 < n ? S.tb[e] : 0.0));
        }
    }
    team_sync<NT>();
    int D = 0;  // depth of the smallest leaves
    while (((n + (1 << D) - 1) >> D) > leaf) ++D;
    if (wave == 0) {
        const int e = lane;
        T ae = (e < n) ? S.a[e] : T(0);
        // Eq. (3): every split s of a node with more than `leaf` elements
        // subtracts |b_{s-1}| from a_{s-1} and a_s (branch-free: every depth's
        // coupling is read from a clamped address and applied by a select)
        for (int d = 0; d < D; ++d) {
            const Node nd = node_of(e < n ? e : 0, d, n);
            const bool split = nd.hi - nd.lo > leaf && (e == nd.s - 1 || e == nd.s);
            const T bs = S.b[nd.s >= 1 ? nd.s - 1 : 0];
            ae -= (e < n && split) ? f_abs(bs) : T(0);
        }
        if (e < n) S.a[e] = ae;  // torn diagonal
        wave_sync();
        if (leaf <= 2) jacobi_leaves<2>(S, n, D, lane, Qc, Lc);
        else if (leaf <= 4) jacobi_leaves<4>(S, n, D, lane, Qc, Lc);
        else jacobi_leaves<8>(S, n, D, lane, Qc, Lc);
    }
    team_sync<NT>();
    BED_PHASE(3);

    // ------------------------------------------------------------ merges
    for (int d = D - 1; d >= 0; --d) {
        // ---- M1: node structure (data-independent) on the last wave while
        // wave 0 forms z, sorts, deflates and compacts --------------------------
        if (wave == NW - 1) {
            const int e = lane;
            const Node nd = node_of(e < n ? e : 0, d, n);
            const bool act = (e < n) && (nd.hi - nd.lo > leaf);
            const int lo = act ? nd.lo : e, hi = act ? nd.hi : e, s = nd.s;
            {
                // Rows of a leaf that is not merged at this depth pass through
                // the back-multiplication unchanged: their child block is the
                // leaf itself and M is the identity on it.
                const bool leaf = (e < n) && !act;
                const int kl = act ? (e < s ? lo : s) : (leaf ? nd.lo : NMAX);
                const int kh = act ? (e < s ? s : hi) : (leaf ? nd.hi : 0);
                if (e < NMAX) {
                    S.u.m.nlo[e] = (e < n) ? nd.lo : e;
                    S.u.m.nhi[e] = (e < n) ? nd.hi : e;
                    S.u.m.ckl[e] = kl;
                    S.u.m.ckh[e] = kh;
                }
                if (leaf)
                    for (int cc = nd.lo; cc < nd.hi; ++cc) S.M[e * LD + cc] = (cc == e) ? T(1) : T(0);
                const int tkl = group_min<16>(kl, lane), tkh = group_max<16>(kh, lane);
                const int tnl = group_min<16>((e < n) ? nd.lo : NMAX, lane);
                const int tnh = group_max<16>((e < n) ? nd.hi : 0, lane);
                if ((e & 15) == 0 && e < NMAX) {
                    S.u.m.tklo[e >> 4] = tkl;
                    S.u.m.tkhi[e >> 4] = tkh;
                    S.u.m.tnlo[e >> 4] = tnl;
                    S.u.m.tnhi[e >> 4] = tnh;
                }
            }
        }
        if (wave == 0) {
            const int e = lane;
            const Node nd = node_of(e < n ? e : 0, d, n);
            BED_MARK(d, 8);
            const bool act = (e < n) && (nd.hi - nd.lo > leaf);
            const int lo = act ? nd.lo : e, hi = act ? nd.hi : e, s = nd.s;
            const T bet = act ? S.b[s - 1] : T(0);
            const T rho = f_abs(bet);
            const T sgm = (bet < T(0)) ? T(-1) : T(1);
            BED_MARK(d, 9);
            // largest power of two <= the largest child size at this depth
            const int cmax = (((n + (1 << d) - 1) >> d) + 1) >> 1;
            const int sstep = 1 << (31 - __builtin_clz(cmax > 0 ? cmax : 1));
            if (act) {
                const T de = Lc[e];
                const T ze = (e < s) ? sgm * Qc[(s - 1) * LD + e] : Qc[s * LD + e];
                // rank among the sibling's sorted values (one chain per lane:
                // left elements count right ones strictly below, right
                // elements count left ones below or equal -- a stable merge)
                const bool left = e < s;
                const int pos = (left ? e - lo : e - s) +
                                count_below_steps<NMAX>(Lc + (left ? s : lo), left ? hi - s : s - lo,
                                                        de, !left, sstep);
                S.u.m.sd[lo + pos] = de;
                S.u.m.sz[lo + pos] = ze;
                S.u.m.sperm[lo + pos] = e;
            }
            wave_sync();
            BED_MARK(d, 10);
            T dp = act ? S.u.m.sd[e] : T(0);
            T zp = act ? S.u.m.sz[e] : T(0);
            // node sums over [lo, hi) from wave prefix sums: z^T z, d^T (z o z),
            // d^T d; max |d| from the sorted end points
            const T pz = wave_prefix_sum(zp * zp);
            const T pdz = wave_prefix_sum(dp * zp * zp);
            const T pd2 = wave_prefix_sum(dp * dp);
            const int ilo = (lo > 0) ? lo - 1 : 0, ihi = (hi > lo) ? hi - 1 : e;
            const T zz0 = __shfl(pz, ihi) - (lo > 0 ? __shfl(pz, ilo) : T(0));
            const T dz = __shfl(pdz, ihi) - (lo > 0 ? __shfl(pdz, ilo) : T(0));
            const T d2 = __shfl(pd2, ihi) - (lo > 0 ? __shfl(pd2, ilo) : T(0));
            const T dmax = act ? f_max(f_abs(S.u.m.sd[lo]), f_abs(S.u.m.sd[hi - 1])) : T(0);
            BED_MARK(d, 11);
            const T nmax = f_max(dmax, rho * zz0), tol = T(8) * u * nmax;
            // A node below 2^-20 of the matrix's scale is merged as 2^s times itself
            // (exact): the squares and reciprocals of its small differences would
            // leave the range.
            const int ns = fexp<T>::BIAS - exp_field(nmax);
            const int nsh = ns > 20 ? min(ns, fexp<T>::SMAX) : 0;
            const T nsc = fexp<T>::pow2(nsh);
            // Frobenius norm of the node (Eq. (10)), from D + rho z z^T
            const T fro2 = d2 + T(2) * rho * dz + rho * rho * zz0 * zz0;
            bool defl = act && (rho * f_abs(zp) <= tol);  // type 1
            const int n_type1 = __popcll(__ballot(defl));
            if (defl) zp = T(0);
            // type 2 candidates against the previous non-deflated component
            const uint64_t live = __ballot(act && !defl);
            const uint64_t below = live & lane_range(lo, e);
            const int prev = below ? 63 - __clzll(below) : e;
            const T zpr = __shfl(zp, prev), dpr = __shfl(dp, prev);
            bool cand = false;
            if (act && !defl && prev != e) {
                // |z| >= tol/rho here (no under/overflow in the squares).  This
                // test rounds differently from the exact one of the scan below
                // (reciprocal square root against hypot and division), so it
                // allows a factor 2: every pair that passes the exact test is
                // a candidate, and the scan decides each candidate exactly.
                const T ir = f_rcp(f_sqrt(fma(zpr, zpr, zp * zp)));
                cand = f_abs((dp - dpr) * (zp * ir) * (zpr * ir)) <= T(2) * tol;
            }
            const uint64_t cmask = __ballot(cand);
            BED_MARK(d, 12);
            if (act) {
                S.u.m.rpart[e] = -1;
                S.u.m.sdefl[e] = defl ? 1 : 0;
                S.u.m.sz[e] = zp;
            }
            bool hasrot = false;
            int my_nrot = 0;
            if (cmask) {
                // Rare path: the exact sequential Givens scan for nodes that
                // have a type-2 candidate (one lane per such node).
                wave_sync();
                const bool mine = act && e == lo && (cmask & lane_range(lo, hi));
                if (mine) {
                    // The scan over consecutive live pairs (last, p) changes
                    // something only at a pair that passes the test.  A pair
                    // whose `last` no rotation has touched and that is not a
                    // candidate fails it (the candidate test is looser), so
                    // only candidates and the successor of each rotated
                    // element are visited, in ascending order, each decided
                    // by the exact test: the decisions of the full scan.
                    uint64_t lv = live & lane_range(lo, hi);
                    uint64_t cm = cmask & lane_range(lo, hi);
                    int mod = -1;  // element changed by the latest rotation
                    for (;;) {
                        const uint64_t after = (mod >= 0) ? (lv & ~lane_range(0, mod + 1)) : 0;
                        const int succ = after ? __builtin_ctzll(after) : 64;
                        const int cnd = cm ? __builtin_ctzll(cm) : 64;
                        const int p = succ < cnd ? succ : cnd;
                        if (p >= hi) break;
                        cm &= ~(1ull << p);
                        const uint64_t bl = lv & lane_range(lo, p);
                        if (!bl) {
                            mod = -1;
                            continue;
                        }
                        const int last = 63 - __clzll(bl);
                        const T zl = S.u.m.sz[last], zi = S.u.m.sz[p];
                        const T dl = S.u.m.sd[last], di = S.u.m.sd[p];
                        const T rr = f_hypot(zl, zi);
                        const T c = zi / rr, sn = zl / rr;
                        if (f_abs((di - dl) * c * sn) <= tol) {
                            S.u.m.sd[last] = dl * c * c + di * sn * sn;
                            S.u.m.sd[p] = dl * sn * sn + di * c * c;
                            S.u.m.sz[last] = T(0);
                            S.u.m.sz[p] = rr;
                            S.u.m.sdefl[last] = 1;
                            S.u.m.rc[last] = c;
                            S.u.m.rs[last] = sn;
                            S.u.m.rpart[last] = p;
                            S.u.m.rlist[lo + my_nrot++] = last;
                            lv &= ~(1ull << last);
                            mod = p;
                        } else {
                            mod = -1;
                        }
                    }
                }
                wave_sync();
                if (act) {
                    dp = S.u.m.sd[e];
                    zp = S.u.m.sz[e];
                    defl = S.u.m.sdefl[e] != 0;
                }
                hasrot = (cmask & lane_range(lo, hi)) != 0;
            }
            const uint64_t live2 = __ballot(act && !defl);
            BED_MARK(d, 13);
            const uint64_t dead = __ballot(act && defl);
            const int k = __popcll(live2 & lane_range(lo, hi));
            if (act) {
                const int row = S.u.m.sperm[e];
                if (!defl) {
                    const int idx = __popcll(live2 & lane_range(lo, e));
                    S.u.m.dk[lo + idx] = nsc * dp;
                    S.u.m.zk[lo + idx] = zp;
                    S.u.m.ndrow[lo + idx] = row;
                } else {
                    const int idx = k + __popcll(dead & lane_range(lo, e));
                    S.u.m.itv[lo + idx] = dp;
                    S.u.m.itrow[lo + idx] = row;
                }
            }
            const T pzz = wave_prefix_sum((act && !defl) ? zp * zp : T(0));
            BED_MARK(d, 14);
            const T zz = __shfl(pzz, ihi) - (lo > 0 ? __shfl(pzz, ilo) : T(0));
            if (act && e == lo) {
                S.u.m.nk[lo] = k;
                S.u.m.nrho[lo] = nsc * rho;
                S.u.m.nzz[lo] = zz;
                S.u.m.nfro[lo] = nsc * f_sqrt(f_max(fro2, T(0)));
                S.u.m.nback[lo] = fexp<T>::pow2(-nsh);
                S.u.m.nrot[lo] = my_nrot;
            }
            const bool anyrot = __ballot(hasrot) != 0;
            if (e == 0) S.anyrot = anyrot ? 1 : 0;
            BED_DEFL(n_type1, (int)wave_total(float(act && e == lo ? my_nrot : 0)));
            (void)n_type1;
            BED_MARK(d, 15);
        }
        team_sync<NT>();
        BED_PHASE(10 + 8 * d + 0);

        {
            // poles (and items) per lane at this depth: ceil(max node size / LPR)
            const int need = ((((n + (1 << d) - 1) >> d)) + LPR - 1) / LPR;
            roots_vectors_dispatch<T, NMAX, NT, 1>(S, n, d, t, Ln, need, leaf);
        }
        BED_PHASE(10 + 8 * d + 4);

        // ---- M6: back-multiplication Q_next = blockdiag(Q1, Q2) M (Eq. (4)) --
        // 16x16 MFMA tiles.  A = Q_cur restricted to each row's child block,
        // B = M (zero outside the node blocks, the identity on unmerged
        // leaves), so every computed entry is final: the product of a row and
        // a column of different nodes is exactly zero, and such entries are
        // never read.  A wave loads the A operand of its row tile once and
        // reuses it for every column tile that meets the tile's nodes.  The
        // K loop has a fixed length (4, 8 or 16 steps, chosen once per row
        // tile) and operands come from clamped addresses, so the tile has no
        // per-step branches.
        if (!Q_out) {
            // Eigenvalues only: the next depth's z (Eq. (5)) reads the last
            // row of each left child and the first row of each right child,
            // i.e. the end rows of this depth's nodes -- and an end row of a
            // node is the matching end row of one child times M.  So only the
            // two end rows of every node are formed (2 m^2 flops per node
            // instead of the block product), wave w taking rows w, w + NW, ...
            // with one lane per column; unmerged leaves pass theirs through M
            // = I.  The other rows of the buffers are never read again.
            for (int r = wave; r < n; r += NW) {
                const int nlo = S.u.m.nlo[r], nhi = S.u.m.nhi[r];
                if (r != nlo && r != nhi - 1) continue;
                const int c = lane;
                if (c < nlo || c >= nhi) continue;
                const int kl = S.u.m.ckl[r], kh = S.u.m.ckh[r];
                T acc = T(0);
                for (int k = kl; k < kh; ++k) acc = fma(Qc[r * LD + k], S.M[k * LD + c], acc);
                Qn[r * LD + c] = acc;
            }
            for (int e = t; e < n; e += NT) {
                if (S.u.m.nhi[e] - S.u.m.nlo[e] <= leaf) Ln[e] = Lc[e];
            }
        } else {
            constexpr int RT = NMAX / 16;
            constexpr int CG = (NW >= RT) ? NW / RT : 1;    // column groups per row tile
            BED_MARK(d, 0);
            for (int idx = wave; idx < RT * CG; idx += NW) {
                const int rt = idx % RT, cg = idx / RT;
                const int r0 = 16 * rt;
                if (r0 >= n) continue;
                const int klo = S.u.m.tklo[rt], khi = S.u.m.tkhi[rt];
                const int nlo = S.u.m.tnlo[rt], nhi = S.u.m.tnhi[rt];
                BED_MARK(d, 4);
                if (klo >= khi) continue;
                const int kb0 = klo & ~3;
                const int nks = __builtin_amdgcn_readfirstlane((khi - kb0 + 3) >> 2);
                BED_MARK(d, 5);
                if (nks <= 4)
                    backmul_rowtile<T, NMAX, NT, 4>(S, Qc, Qn, n, lane, r0, cg, CG, kb0, nlo, nhi);
                else if (nks <= 8)
                    backmul_rowtile<T, NMAX, NT, 8>(S, Qc, Qn, n, lane, r0, cg, CG, kb0, nlo, nhi);
                else
                    backmul_rowtile<T, NMAX, NT, NMAX / 4>(S, Qc, Qn, n, lane, r0, cg, CG, kb0, nlo,
                                                           nhi);
            }
            BED_MARK(d, 2);
            // eigenvalues of nodes not merged at this depth
            for (int e = t; e < n; e += NT) {
                if (S.u.m.nhi[e] - S.u.m.nlo[e] <= leaf) Ln[e] = Lc[e];
            }
            BED_MARK(d, 3);
        }
        team_sync<NT>();
        BED_PHASE(10 + 8 * d + 5);
        T* tq = Qc; Qc = Qn; Qn = tq;
        T* tl = Lc; Lc = Ln; Ln = tl;
    }
    }

    if (!Q_out) {  // eigenvalues only
        for (int e = t; e < n; e += NT) lam_out[e] = fexp<T>::pow2(-input_shift(S)) * Lc[e];
        if (t == 0 && info_out) *info_out = S.capped;
        if constexpr (TRI) {
            // the root's end rows, carried through every depth
            if (ends_out)
                for (int e = t; e < 2 * n; e += NT)
                    ends_out[e] = (e < n) ? Qc[e] : Qc[(n - 1) * LD + e - n];
        }
        return;
    }

    // ------------------------------------------------------------ back-transform
    // (TRI: Q_H = I, the compact-WY branch with no reflectors stores Q_T)
    if constexpr (AW > 0 && !TRI) {
        // Q_A = Q_H Q_T on 16x16x4 MFMA tiles: wave w computes row tiles
        // [p RPW, p RPW + RPW) of column tile w % CT (p = w / CT).  Lane group kk
        // covers k in [kk KS, kk KS + KS), so each lane reads a contiguous
        // slice of its Q_H row.  The product goes to Qn unsigned; each wave
        // leaves, per column, its entry of largest magnitude (lowest row on
        // ties) for the sign rule applied by the store.
        using MF = Mf<T>;
        constexpr int CT = NMAX / 16;
        constexpr int RT = NMAX / 16;
        static_assert(NW >= CT, "one wave per column tile at least");
        constexpr int WPC = (NW / CT > RT) ? RT : NW / CT;  // waves per column tile
        constexpr int RPW = RT / WPC;
        constexpr int KS = NMAX / 4;
        constexpr int VLD = Smem<T, NMAX, NT>::VLD;
        constexpr int VW = 16 / sizeof(T);
        static_assert(WPC * NMAX <= int(sizeof(S.u.b.gram) / sizeof(T)), "sign candidates");
        typedef T vec_t __attribute__((ext_vector_type(VW)));
        const int i16 = lane & 15, kk = lane >> 4;
        if (wave < CT * WPC) {
            const int ct = wave % CT, part = wave / CT;
            const int c = 16 * ct + i16;
            T bq[KS];
#pragma unroll
            for (int s4 = 0; s4 < KS; ++s4) {
                const int k = kk * KS + s4;
                bq[s4] = (k < n) ? Qc[k * LD + c] : T(0);
            }
            typename MF::acc q[RPW];
#pragma unroll
            for (int pr = 0; pr < RPW; ++pr) {
                const int rt = part * RPW + pr;
                const vec_t* ap = reinterpret_cast<const vec_t*>(S.Vt + (16 * rt + i16) * VLD + kk * KS);
                T a[KS];
#pragma unroll
                for (int q4 = 0; q4 < KS / VW; ++q4) {
                    const vec_t x = ap[q4];
#pragma unroll
                    for (int e = 0; e < VW; ++e) a[q4 * VW + e] = x[e];
                }
                q[pr] = MF::zero();
#pragma unroll
                for (int s4 = 0; s4 < KS; ++s4) q[pr] = MF::mma(a[s4], bq[s4], q[pr]);
            }
            T best = T(-1), bval = T(0);
            int brow = 1 << 20;
#pragma unroll
            for (int pr = 0; pr < RPW; ++pr) {
#pragma unroll
                for (int v = 0; v < 4; ++v) {
                    const int row = 16 * (part * RPW + pr) + MF::crow(lane, v);
                    const T av = f_abs(q[pr][v]);
                    const bool take = row < n && (av > best || (av == best && row < brow));
                    best = take ? av : best;
                    brow = take ? row : brow;
                    bval = take ? q[pr][v] : bval;
                    if (row < n && c < n) Qn[row * LD + c] = q[pr][v];
                }
            }
            {
                const T ob = xmove<16>(best, lane);
                const int orow = xmove<16>(brow, lane);
                const T oval = xmove<16>(bval, lane);
                const bool take = ob > best || (ob == best && orow < brow);
                best = take ? ob : best;
                brow = take ? orow : brow;
                bval = take ? oval : bval;
            }
            {
                const T ob = xmove<32>(best, lane);
                const int orow = xmove<32>(brow, lane);
                const T oval = xmove<32>(bval, lane);
                const bool take = ob > best || (ob == best && orow < brow);
                bval = take ? oval : bval;
            }
            if (kk == 0) S.u.b.gram[part * NMAX + c] = bval;
        }
        team_sync<NT>();
        BED_PHASE(4);
        // Sign of column j: parts in increasing row order, a later part wins
        // only when strictly larger in magnitude.  16-byte stores when the
        // rows allow them, as for the load.
        auto colsign = [&](const int j) {
            T bv = S.u.b.gram[j];
#pragma unroll
            for (int pp = 1; pp < WPC; ++pp) {
                const T o = S.u.b.gram[pp * NMAX + j];
                bv = (f_abs(o) > f_abs(bv)) ? o : bv;
            }
            return bv;
        };
        if (n % VW == 0 && (reinterpret_cast<uintptr_t>(Q_out) & 15) == 0) {
            vec_t* Qv = reinterpret_cast<vec_t*>(Q_out);
            const int nv = n * n / VW;
            for (int e = t; e < nv; e += NT) {
                const int i = (e * VW) / n, j = (e * VW) % n;
                vec_t x;
#pragma unroll
                for (int q4 = 0; q4 < VW; ++q4) {
                    const T y = Qn[i * LD + j + q4];
                    x[q4] = (colsign(j + q4) < T(0)) ? -y : y;
                }
                Qv[e] = x;
            }
        } else {
            for (int i = t / n, j = t % n, e = t; e < n * n; e += NT) {
                const T x = Qn[i * LD + j];
                Q_out[e] = (colsign(j) < T(0)) ? -x : x;
                j += NT % n;
                i += NT / n;
                if (j >= n) {
                    j -= n;
                    ++i;
                }
            }
        }
        for (int e = t; e < n; e += NT) lam_out[e] = fexp<T>::pow2(-input_shift(S)) * Lc[e];
        if (t == 0 && info_out) *info_out = S.capped;
        BED_PHASE(5);
        return;
    } else {
    // Q_A = H_0 H_1 ... H_{n-3} Q_T in compact-WY blocks of 16 reflectors,
    // H_{16b} ... H_{16b+15} = I - V_b T_b V_b^T (T_b upper triangular), applied
    // for b = last .. 0.  Each wave keeps whole 16-column tiles of Q in MFMA
    // accumulators for all blocks, so the update needs no team barrier.
    {
        using MF = Mf<T>;
        constexpr int RT = NMAX / 16;
        constexpr int VLD = Smem<T, NMAX, NT>::VLD;
        const int nb = (!TRI && n > 2) ? n - 2 : 0;  // reflectors
        const int NB = (nb + 15) / 16;
        const int i16 = lane & 15;
        BED_MARK(7, 0);
        // Gram matrices G_b = V_b^T V_b (one wave per block); one MFMA chain
        // per row tile, summed at the end (independent chains overlap)
        for (int bk = wave; bk < NB; bk += NW) {
            const int k0 = 16 * bk;
            const bool okr = k0 + i16 < nb;
            typename MF::acc g = MF::zero();
            typename MF::acc gt[RT];
#pragma unroll
            for (int rt = 0; rt < RT; ++rt) {
                gt[rt] = MF::zero();
                if (rt < bk) continue;  // rows above the block's first reflector are zero
#pragma unroll
                for (int s4 = 0; s4 < 4; ++s4) {
                    const int row = 16 * rt + MF::crow(lane, s4);
                    const T vv = okr ? S.Vt[(k0 + i16) * VLD + row] : T(0);
                    gt[rt] = MF::mma(vv, vv, gt[rt]);
                }
            }
#pragma unroll
            for (int rt = 0; rt < RT; ++rt)
                if (rt >= bk) g += gt[rt];
#pragma unroll
            for (int v = 0; v < 4; ++v) S.u.b.gram[bk * 272 + MF::crow(lane, v) * 17 + i16] = g[v];
            wave_sync();
            // T_b: T(j, j) = tau_j, T(0:j, j) = -tau_j T(0:j, 0:j) G(0:j, j)
            BED_MARK(7, 1);
            if (lane < 16) {
                T trow[16];
#pragma unroll
                for (int j = 0; j < 16; ++j) {
                    const T tj = (k0 + j < nb) ? S.tau[k0 + j] : T(0);
                    T acc = T(0);
#pragma unroll
                    for (int kk = 0; kk < j; ++kk) acc = fma(trow[kk], S.u.b.gram[bk * 272 + kk * 17 + j], acc);
                    trow[j] = (lane < j) ? -tj * acc : (lane == j ? tj : T(0));
                }
#pragma unroll
                for (int j = 0; j < 16; ++j) S.u.b.tf[bk * 272 + lane * 17 + j] = trow[j];
            }
        }
        BED_MARK(7, 2);
        team_sync<NT>();
        constexpr int NBMAX = (NMAX + 13) / 16;  // blocks for n = NMAX
        for (int ct = wave; ct < RT; ct += NW) {
            const int c0 = 16 * ct;
            if (c0 >= n) continue;
            BED_MARK(7, 3);
            const int c = c0 + i16;
            typename MF::acc q[RT];
#pragma unroll
            for (int rt = 0; rt < RT; ++rt) {
#pragma unroll
                for (int v = 0; v < 4; ++v) {
                    const int row = 16 * rt + MF::crow(lane, v);
                    q[rt][v] = (row < n && c < n) ? Qc[row * LD + c] : T(0);
                }
            }
            // blocks last to first, unrolled so that the zero row tiles of
            // each V_b (below its first reflector) are skipped at compile time
#pragma unroll
            for (int bi = 0; bi < NBMAX; ++bi) {
                const int bk = NBMAX - 1 - bi;
                if (bk >= NB) continue;
                const int k0 = 16 * bk;
                const bool okr = k0 + i16 < nb;
                // operands of this block, loaded before the MFMA chains
                T va[RT][4], vb[RT][4], tv[4];
#pragma unroll
                for (int rt = 0; rt < RT; ++rt) {
#pragma unroll
                    for (int s4 = 0; s4 < 4; ++s4) {
                        const int row = 16 * rt + MF::crow(lane, s4);
                        const int kr = k0 + MF::crow(lane, s4);
                        va[rt][s4] = okr ? S.Vt[(k0 + i16) * VLD + row] : T(0);
                        vb[rt][s4] = (kr < nb) ? -S.Vt[kr * VLD + 16 * rt + i16] : T(0);
                    }
                }
#pragma unroll
                for (int s4 = 0; s4 < 4; ++s4) tv[s4] = S.u.b.tf[bk * 272 + i16 * 17 + MF::crow(lane, s4)];
                // X = V_b^T Q (16 x 16 tile of this column block): one chain
                // per row tile at or below the block, then summed
                typename MF::acc xt[RT];
#pragma unroll
                for (int rt = 0; rt < RT; ++rt) {
                    xt[rt] = MF::zero();
                    if (rt < bk) continue;
#pragma unroll
                    for (int s4 = 0; s4 < 4; ++s4) xt[rt] = MF::mma(va[rt][s4], q[rt][s4], xt[rt]);
                }
                typename MF::acc x = xt[RT - 1];
#pragma unroll
                for (int rt = 0; rt < RT - 1; ++rt)
                    if (rt >= bk) x += xt[rt];
                // Y = T_b X
                typename MF::acc y = MF::zero();
#pragma unroll
                for (int s4 = 0; s4 < 4; ++s4) y = MF::mma(tv[s4], x[s4], y);
                // Q -= V_b Y, the row tiles' chains interleaved
#pragma unroll
                for (int s4 = 0; s4 < 4; ++s4) {
#pragma unroll
                    for (int rt = 0; rt < RT; ++rt)
                        if (rt >= bk) q[rt] = MF::mma(vb[rt][s4], y[s4], q[rt]);
                }
            }
            BED_MARK(7, 4);
            // sign canonicalization: largest |.| entry positive, lowest row on ties
            T best = T(-1), bval = T(0);
            int brow = 1 << 20;
#pragma unroll
            for (int rt = 0; rt < RT; ++rt) {
#pragma unroll
                for (int v = 0; v < 4; ++v) {
                    const int row = 16 * rt + MF::crow(lane, v);
                    const T av = f_abs(q[rt][v]);
                    if (row < n && (av > best || (av == best && row < brow))) {
                        best = av;
                        brow = row;
                        bval = q[rt][v];
                    }
                }
            }
            {
                const T ob = xmove<16>(best, lane);
                const int orow = xmove<16>(brow, lane);
                const T oval = xmove<16>(bval, lane);
                if (ob > best || (ob == best && orow < brow)) {
                    best = ob;
                    brow = orow;
                    bval = oval;
                }
            }
            {
                const T ob = xmove<32>(best, lane);
                const int orow = xmove<32>(brow, lane);
                const T oval = xmove<32>(bval, lane);
                if (ob > best || (ob == best && orow < brow)) {
                    best = ob;
                    brow = orow;
                    bval = oval;
                }
            }
            const T sgn = (bval < T(0)) ? T(-1) : T(1);
#pragma unroll
            for (int rt = 0; rt < RT; ++rt) {
#pragma unroll
                for (int v = 0; v < 4; ++v) {
                    const int row = 16 * rt + MF::crow(lane, v);
                    if (row < n && c < n) Qn[row * LD + c] = sgn * q[rt][v];
                }
            }
        }
    }
    team_sync<NT>();
    BED_PHASE(4);
    for (int i = t / n, j = t % n, e = t; e < n * n; e += NT) {
        Q_out[e] = Qn[i * LD + j];
        j += NT % n;
        i += NT / n;
        if (j >= n) {
            j -= n;
            ++i;
        }
    }
    for (int e = t; e < n; e += NT) lam_out[e] = fexp<T>::pow2(-input_shift(S)) * Lc[e];
    if (t == 0 && info_out) *info_out = S.capped;
    BED_PHASE(5);
    }
}

}  // namespace bed
