// Exact click probabilities (Methods, Probability of any sample; the click
// projector of Methods, Model), in double-double on one MI355X.
//
//   p(C) = det(Q)^{-1/2} sum_{Z subset C} (-1)^{n-|Z|} det(A_Z)^{-1/2},  A = (Q^{-1})_CC
//
// The subsets form a binary include/exclude tree over the clicked modes.
// Including a mode takes its two quadratures out of the remaining matrix by a
// 2x2 Cholesky step (l = the factor of the mode's own block, y = l^{-1} times
// its rows, a_ij -= y_i y_j) and multiplies the subset's term by
// det(l)^{-1}; excluding it drops its rows.  A matrix is stored with the last
// mode first, so that what remains after a mode, in either branch, is a
// prefix of what was there: excluded children need no storage of their own.
// Work split of a row of n clicks, R = min(n, EX_R) (one wavefront per item):
//   - the first h = n - R modes: 2^h assignments z0, dealt to at most 2^EX_LGI
//     items per row in contiguous ranges.  The high bits of z0 are conditioned
//     on in LDS, from the gathered matrix; the result, of R + EX_IN modes, is
//     held in registers for the 2^EX_IN assignments that share it;
//   - the next R - S - 1 modes: breadth first in LDS, each level's included
//     children in one pass over (node, pair of modes);
//   - the last S + 1 modes: one lane per node and choice of the first of them
//     (lanes 0..31 without it, 32..63 with it), which then walks the tree of
//     the other S modes in registers.
// A lane's signed sum is kept in three words, the lanes' and parts' sums in
// double-double, in a fixed order; kappa = sum|terms| / |sum| is returned.
// Against binary128 the rms error at 3 / 6 / 8 / 10 / 11 clicks and kappa of
// 1e18 is 0.183 / 0.070 / 0.037 / 0.018 / 0.013 kappa 2^-106; with sums in two
// words and inverse roots off by a few units it was 0.258 / 0.099 / 0.050 /
// 0.035 / 0.023, with full double-double operations at every step of a Schur
// complement by inverse blocks 0.206 / 0.106 / 0.053 / 0.026 / 0.019.
//
// What bounds it: the fp64 vector ALUs (about 410 operations per subset, the
// Schur complements 7 entries of them at 27 each; 693 issued per subset with
// the levels' redundant factors and the lanes that carry an excluded mode).
// The breadth-first levels of 64 lanes' nodes take 39 KB of LDS, so that one
// wavefront sits on each SIMD with 512 registers.  At 30 clicks the counters
// read VALU issue in 62 % of a SIMD's cycles and LDS in 7 %; the wavefront
// issues something in 77 % and waits for its own results in the rest.  Against
// levels that end with three modes per node, copy excluded children and pay
// 122 operations per entry (43 KB, three wavefronts per compute unit): one row
// of 30 clicks 502 -> 32.5 ms (3.3e10 subsets/s), 4096 rows of 6-14 clicks at
// 20 modes 8.60 -> 0.67 ms.
#include <algorithm>
#include <cstring>
#include <mutex>

#include "internal.h"

#define EX_R 10         // modes handled inside one prefix assignment
#define EX_S 4          // of these, walked in registers by one lane (R = EX_R)
#define EX_IN 3         // prefix modes whose assignments share one conditioned matrix
#define EX_LGI 12       // at most 2^12 work items per row
#define EX_SMALL 8      // rows of at most this many clicks take the small kernel

// packed dd entries of a symmetric matrix of k modes
__host__ __device__ constexpr int ex_e(int k) { return k * (2 * k + 1); }
// where the levels of R modes sit: level l's included children (l >= 1, 2^{l-1}
// matrices of R - l modes) follow each other, the root's matrix comes last
__host__ __device__ constexpr int ex_lev(int R, int l)
{
    int o = 0;
    for (int u = 1; u < l; ++u) o += (1 << (u - 1)) * ex_e(R - u);
    return o;
}
// At R = EX_R the last level's two last matrices take the place of those of the
// root's rows that are no longer read when they are written (the rows of the
// modes before the level's own): this brings four wavefronts' levels into a
// compute unit's 160 KB
#define EX_LMAX (EX_R - EX_S - 1)
#define EX_TUCK 2
#define EX_ROOT (ex_lev(EX_R, EX_LMAX + 1) - EX_TUCK * ex_e(EX_S + 1))
static_assert(ex_e(EX_R - EX_LMAX + 1) + EX_TUCK * ex_e(EX_S + 1) <= ex_e(EX_R), "the tucked matrices lie in the root's dead rows");
#define EX_CAP (EX_ROOT + ex_e(EX_R))
static_assert(ex_e(GBS_MAX_N_EXACT) <= EX_CAP, "the prefix's matrix is conditioned in the levels' place");
static_assert(EX_LMAX == 5, "32 nodes, one lane for each choice of their first mode");
#define EX_CAP_SMALL (ex_lev(EX_SMALL, 6) + ex_e(EX_SMALL))

namespace {

__device__ __forceinline__ dd sel(bool c, dd x) { return dd{c ? x.hi : 0.0, c ? x.lo : 0.0}; }

// 2x2 Cholesky factor of a mode's block [[a, b], [b, d]]: inverse diagonal and
// the off-diagonal entry; det^{-1/2} = i0 i1
struct Piv {
    dd i0, l, i1;
};
__device__ __forceinline__ Piv factor(dd a, dd b, dd d)
{
    Piv f;
    f.i0 = dd_rsqrt(a);
    f.l = dd_mul(b, f.i0);
    f.i1 = dd_rsqrt(dd_fms(d, f.l, f.l));
    return f;
}
__device__ __forceinline__ dd rdet(dd a, dd b, dd d) { return dd_rsqrt(dd_fms(dd_mul(a, d), b, b)); }

// A lane's signed sum in three words, hi + mid + lo: the terms cancel by up to
// 1e20, and every rounding of the sum counts in full.  Adding a term loses
// nothing above 2^-159 of the sum, for the operations of one dd_add.
struct Sum {
    double hi, mid, lo, ab;  // ab: the sum of the terms' moduli
};
__device__ __forceinline__ void add_term(dd v, Sum &s)
{
    const dd a = two_sum(s.hi, v.hi);
    const dd b = two_sum(s.mid, a.lo);
    const dd c = two_sum(b.hi, v.lo);
    s.hi = a.hi;
    s.mid = c.hi;
    s.lo += b.lo + c.lo;
    s.ab += fabs(v.hi);
}
__device__ __forceinline__ dd sum_dd(const Sum &s)
{
    const dd a = two_sum(s.hi, s.mid);
    return quick_two_sum(a.hi, a.lo + s.lo);
}

// The first of K modes held in registers (packed, last mode first) taken out of
// the others' matrix; returns its -det^{-1/2}.
template <int K>
__device__ __forceinline__ dd step(const dd (&A)[ex_e(K)], dd (&B)[ex_e(K - 1)])
{
    constexpr int Y = ex_e(K - 1), D = Y + 4 * (K - 1);  // the first mode's rows, its own block
    const Piv f = factor(A[D], A[D + 1], A[D + 2]);
    dd y[K - 1][4];  // per mode: y0 (x, p), y1 (x, p)
#pragma unroll
    for (int j = 0; j < K - 1; ++j)
#pragma unroll
        for (int c = 0; c < 2; ++c) {
            y[j][c] = dd_mul(A[Y + 4 * j + c], f.i0);
            y[j][2 + c] = dd_mul(dd_fms(A[Y + 4 * j + 2 + c], f.l, y[j][c]), f.i1);
        }
#pragma unroll
    for (int i = 0; i < K - 1; ++i) {
#pragma unroll
        for (int j = 0; j < i; ++j)
#pragma unroll
            for (int t = 0; t < 4; ++t) {
                const int e = ex_e(i) + 4 * j + t, r = t >> 1, c = t & 1;
                B[e] = dd_fms2(A[e], y[i][r], y[j][c], y[i][2 + r], y[j][2 + c]);
            }
#pragma unroll
        for (int t = 0; t < 3; ++t) {
            const int e = ex_e(i) + 4 * i + t, r = t == 2, c = t > 0;
            B[e] = dd_fms2(A[e], y[i][r], y[i][c], y[i][2 + r], y[i][2 + c]);
        }
    }
    return dd_neg(dd_mul(f.i0, f.i1));
}

// The subsets of K modes held in registers; acc: the product of the inverse
// roots so far with the subset's sign.
template <int K>
__device__ __forceinline__ void walk(const dd (&A)[ex_e(K)], dd acc, Sum &sum)
{
    if constexpr (K == 1) {
        add_term(acc, sum);
        add_term(dd_neg(dd_mul(acc, rdet(A[0], A[1], A[2]))), sum);
    } else {
        dd B[ex_e(K - 1)];
        const dd r = step<K>(A, B);
        walk<K - 1>(B, dd_mul(acc, r), sum);
#pragma unroll
        for (int e = 0; e < ex_e(K - 1); ++e) B[e] = A[e];
        walk<K - 1>(B, acc, sum);
    }
}

__device__ __forceinline__ dd ld(const double2 *p)
{
    const double2 v = *p;
    return dd{v.x, v.y};
}
__device__ __forceinline__ void st(double2 *p, dd v) { *p = make_double2(v.hi, v.lo); }

// block (i, j), j <= i, of the lower triangle from its index i (i + 1)/2 + j
__device__ __forceinline__ void tri_ij(int t, int &i, int &j)
{
    i = (int)(0.5f * (sqrtf(8.0f * (float)t + 1.0f) - 1.0f));
    if ((i + 1) * (i + 2) / 2 <= t) ++i;
    if (i * (i + 1) / 2 > t) --i;
    j = t - i * (i + 1) / 2;
}

// y of mode block j in the rows of mode i of the matrix at m, in place
__device__ __forceinline__ void make_y(double2 *m, int i, int j, const Piv &f)
{
    double2 *q = m + ex_e(i) + 4 * j;
#pragma unroll
    for (int c = 0; c < 2; ++c) {
        const dd y0 = dd_mul(ld(q + c), f.i0);
        const dd y1 = dd_mul(dd_fms(ld(q + 2 + c), f.l, y0), f.i1);
        st(q + c, y0);
        st(q + 2 + c, y1);
    }
}
// the child's block (i, j) from the parent's, yr: the parent's row of y
__device__ __forceinline__ void update(const double2 *src, const double2 *yr, double2 *dst, int i, int j)
{
    const double2 *yi = yr + 4 * i, *yj = yr + 4 * j;
    const dd i0 = ld(yi), i1 = ld(yi + 1), i2 = ld(yi + 2), i3 = ld(yi + 3);
    const dd j0 = ld(yj), j1 = ld(yj + 1), j2 = ld(yj + 2), j3 = ld(yj + 3);
    const int e = ex_e(i) + 4 * j;
    if (i != j) {
        const dd a0 = dd_fms2(ld(src + e), i0, j0, i2, j2), a1 = dd_fms2(ld(src + e + 1), i0, j1, i2, j3);
        const dd a2 = dd_fms2(ld(src + e + 2), i1, j0, i3, j2), a3 = dd_fms2(ld(src + e + 3), i1, j1, i3, j3);
        st(dst + e, a0);
        st(dst + e + 1, a1);
        st(dst + e + 2, a2);
        st(dst + e + 3, a3);
    } else {
        const dd a0 = dd_fms2(ld(src + e), i0, i0, i2, i2), a1 = dd_fms2(ld(src + e + 1), i0, i1, i2, i3);
        const dd a2 = dd_fms2(ld(src + e + 2), i1, i1, i3, i3);
        st(dst + e, a0);
        st(dst + e + 1, a1);
        st(dst + e + 2, a2);
    }
}
__device__ __forceinline__ Piv factor_at(const double2 *m, int i)
{
    const double2 *q = m + ex_e(i) + 4 * i;
    return factor(ld(q), ld(q + 1), ld(q + 2));
}

// One wavefront conditions the matrix at m on the mode of its row i, in place
// (the rows above are left as they are); returns -det^{-1/2}.
__device__ __forceinline__ dd condition(double2 *m, int i, int lane)
{
    const Piv f = factor_at(m, i);
    __syncthreads();
    if (lane < i) make_y(m, i, lane, f);
    __syncthreads();
    for (int t = lane; t < i * (i + 1) / 2; t += 64) {
        int r, c;
        tri_ij(t, r, c);
        update(m, m + ex_e(i), m, r, c);
    }
    __syncthreads();
    return dd_neg(dd_mul(f.i0, f.i1));
}

// The matrix of K modes of a lane's node: the prefix of its parent's matrix at
// m, less the terms of the parent's first mode (row K, whose y stand there)
// where inc
template <int K>
__device__ __forceinline__ void load_node(dd (&A)[ex_e(K)], const double2 *m, bool inc, bool one)
{
    dd y[K][4];
#pragma unroll
    for (int j = 0; j < K; ++j)
#pragma unroll
        for (int t = 0; t < 4; ++t) y[j][t] = one ? dd_make(0.0) : sel(inc, ld(m + ex_e(K) + 4 * j + t));
#pragma unroll
    for (int i = 0; i < K; ++i) {
#pragma unroll
        for (int j = 0; j < i; ++j)
#pragma unroll
            for (int t = 0; t < 4; ++t) {
                const int e = ex_e(i) + 4 * j + t, r = t >> 1, c = t & 1;
                A[e] = dd_fms2(ld(m + e), y[i][r], y[j][c], y[i][2 + r], y[j][2 + c]);
            }
#pragma unroll
        for (int t = 0; t < 3; ++t) {
            const int e = ex_e(i) + 4 * i + t, r = t == 2, c = t > 0;
            A[e] = dd_fms2(ld(m + e), y[i][r], y[i][c], y[i][2 + r], y[i][2 + c]);
        }
    }
}

// Modes of a row of R = min(n, EX_R) that one lane walks in registers: few for
// the short rows (64 lanes then share the row's nodes: latency), EX_S for the
// long ones (the levels of 32 nodes fill the LDS)
__device__ __forceinline__ int ex_s(int R) { return R >= EX_R ? EX_S : R == 9 ? 3 : R >= 2 ? 2 : 1; }

__device__ __forceinline__ dd wave_dd_sum(dd v)
{
    for (int m = 32; m > 0; m >>= 1) {
        dd o = dd{__shfl_xor(v.hi, m), __shfl_xor(v.lo, m)};
        v = dd_add(v, o);
    }
    return v;
}

// whether a row's modes are in [0, M) and ascend (n <= 64; every lane gets it)
__device__ __forceinline__ bool wave_row_ok(const int *__restrict__ row, int n, int M, int lane)
{
    bool bad = false;
    if (lane < n) {
        const int m = row[lane];
        bad = m < 0 || m >= M || (lane > 0 && m <= row[lane - 1]);
    }
    return __ballot(bad) == 0ull;
}

// One work item: row p = block >> lgG, part g of the at most 2^lgG parts of its
// 2^h prefix assignments (rows of more than maxn clicks, or with modes outside
// [0, M) or not ascending, are left to k_exact_final, which flags them).
// SMALL: rows of at most EX_SMALL clicks only (fewer registers, less LDS).
template <bool SMALL>
__global__ __launch_bounds__(64) void k_exact(int M, const double *__restrict__ qi_hi,
                                              const double *__restrict__ qi_lo,
                                              const int *__restrict__ offsets,
                                              const int *__restrict__ modes, int lgG, int maxn,
                                              double *__restrict__ part)
{
    __shared__ double2 buf[SMALL ? EX_CAP_SMALL : EX_CAP];
    __shared__ double2 nacc[32];
    __shared__ short gidx[32];
    const int lane = threadIdx.x;
    const long long item = blockIdx.x;
    const int p = (int)(item >> lgG), ip = (int)(item & ((1LL << lgG) - 1));
    const int o = offsets[p], n = offsets[p + 1] - o;
    if (n <= 0 || n > maxn) return;
    const int h = SMALL ? 0 : max(n - EX_R, 0), R = n - h;
    const int lgP = min(h, lgG);  // this row's parts: 2^lgP
    if (ip >= (1 << lgP)) return;
    if (!wave_row_ok(modes + o, n, M, lane)) return;
    const int lgZ = h - lgP, nin = min(lgZ, EX_IN);  // assignments per part: 2^lgZ
    const int D = 2 * M, S = ex_s(R), L = max(R - S - 1, 0);
    const int root = SMALL ? ex_lev(R, L + 1) : R == EX_R ? EX_ROOT : ex_lev(R, L + 1);
    constexpr int NREG = (ex_e(EX_R + EX_IN) + 63) / 64;
    const dd sign = dd_make(n & 1 ? -1.0 : 1.0);
    Sum sum = {0.0, 0.0, 0.0, 0.0};
    for (int zm = 0; zm < (1 << (lgZ - nin)); ++zm) {
        const int z0 = (ip << lgZ) | (zm << nin);
        // the last R modes, then the nin inner prefix modes, then the other
        // included prefix modes: rows 0, 1, ... of the matrix
        int k = R + nin;
        if (lane < k) gidx[lane] = (short)modes[o + (lane < R ? n - 1 - lane : lane - R)];
        for (int b = nin; b < h; ++b)
            if (z0 >> b & 1) {
                if (lane == 0) gidx[k] = (short)modes[o + b];
                ++k;
            }
        __syncthreads();
        double2 *m0 = buf + (h > 0 ? 0 : root);
        for (int t = lane; t < k * (k + 1) / 2; t += 64) {
            int i, j;
            tri_ij(t, i, j);
            const int gi = gidx[i], gj = gidx[j];
            double2 *q = m0 + ex_e(i) + 4 * j;
            const long x = (long)gi * D + gj, y = (long)(gi + M) * D + gj;
            q[0] = make_double2(qi_hi[x], qi_lo[x]);
            q[1] = i == j ? make_double2(qi_hi[y], qi_lo[y]) : make_double2(qi_hi[x + M], qi_lo[x + M]);
            q[2] = i == j ? make_double2(qi_hi[y + M], qi_lo[y + M]) : make_double2(qi_hi[y], qi_lo[y]);
            if (i != j) q[3] = make_double2(qi_hi[y + M], qi_lo[y + M]);
        }
        __syncthreads();
        dd acc0 = sign;
        for (int i = k - 1; i >= R + nin; --i) acc0 = dd_mul(acc0, condition(m0, i, lane));
        double2 mr[NREG];
        if (!SMALL && nin > 0)
#pragma unroll
            for (int t = 0; t < NREG; ++t) mr[t] = buf[min(lane + 64 * t, ex_e(R + nin) - 1)];
        for (int zi = 0; zi < (1 << nin); ++zi) {
            dd acc = acc0;
            if (!SMALL && h > 0) {
                __syncthreads();
                if (nin > 0 && zi > 0) {
#pragma unroll
                    for (int t = 0; t < NREG; ++t)
                        if (lane + 64 * t < ex_e(R + nin)) buf[lane + 64 * t] = mr[t];
                    __syncthreads();
                }
                for (int b = nin - 1; b >= 0; --b)
                    if (zi >> b & 1) acc = dd_mul(acc, condition(buf, R + b, lane));
                // the root's matrix into its place (the two do not overlap)
                static_assert(EX_ROOT >= ex_e(EX_R), "");
                for (int e = lane; e < ex_e(EX_R); e += 64) buf[EX_ROOT + e] = buf[e];
            }
            if (lane == 0) nacc[0] = make_double2(acc.hi, acc.lo);
            __syncthreads();
            // where node v's matrix stands: that of its last included level
            auto node_at = [&](int v) {
                if (v == 0) return root;
                const int l = 32 - __clz(v), s = v - (1 << (l - 1));
                int at = 0, e = 0;
#pragma unroll
                for (int u = 1; u <= EX_LMAX; ++u) {
                    if (u < l) at += (1 << (u - 1)) * ex_e(R - u);
                    if (u == l) e = ex_e(R - u);
                }
                at += s * e;
                if (!SMALL && R == EX_R && l == EX_LMAX && s >= (1 << (EX_LMAX - 1)) - EX_TUCK)
                    at += ex_e(EX_S + 2);  // (tucked into the root's dead rows)
                return at;
            };
            // breadth first: level lev takes mode row kr of its 2^lev nodes (a lane
            // keeps its node over a level: 64 is a multiple of their number)
            for (int lev = 0, to = 0; lev < L; ++lev) {
                const int kr = R - 1 - lev, nodes = 1 << lev, v = lane & (nodes - 1);
                double2 *m = buf + node_at(v);
                for (int j = lane >> lev; j < kr; j += 64 >> lev) {
                    const Piv f = factor_at(m, kr);
                    make_y(m, kr, j, f);
                    if (j == 0) {
                        const dd a = dd_neg(dd_mul(ld(&nacc[v]), dd_mul(f.i0, f.i1)));
                        st(&nacc[v + nodes], a);
                    }
                }
                __syncthreads();
                double2 *ch = buf + to + v * ex_e(kr);
                if (!SMALL && R == EX_R && lev == EX_LMAX - 1 && v >= nodes - EX_TUCK) ch += ex_e(EX_S + 2);
                for (int t = lane >> lev; t < kr * (kr + 1) / 2; t += 64 >> lev) {
                    int i, j;
                    tri_ij(t, i, j);
                    update(m, m + ex_e(kr), ch, i, j);
                }
                to += ex_e(kr) << lev;
                __syncthreads();
            }
            // the last S + 1 modes: lane v without the first of them, lane 32 + v with
            const bool one = R <= S;  // (no level: a single lane walks the root)
            const int v = lane & 31, nodes = 1 << L;
            const bool inc = lane >= 32, on = one ? lane == 0 : v < nodes;
            const double2 *m = buf + node_at(on ? v : 0);
            dd a = ld(&nacc[on ? v : 0]);
            if (!one) {
                const Piv f = factor_at(m, S);
                if (inc) a = dd_neg(dd_mul(a, dd_mul(f.i0, f.i1)));
                double2 *q = buf + node_at(lane & (nodes - 1));
                for (int j = lane >> L; j < S; j += 64 >> L) {
                    const Piv g = factor_at(q, S);
                    make_y(q, S, j, g);
                }
                __syncthreads();
            }
            if (on) {
                if (S <= 2) {
                    if (S == 2) {
                        dd A[ex_e(2)];
                        load_node<2>(A, m, inc, one);
                        walk<2>(A, a, sum);
                    } else {
                        dd A[ex_e(1)];
                        load_node<1>(A, m, inc, one);
                        walk<1>(A, a, sum);
                    }
                } else if constexpr (!SMALL) {
                    // (R = 9 walks three modes, R = 10 four: the first of these
                    // included, then not)
                    dd A[ex_e(EX_S)], B[ex_e(EX_S - 1)];
                    dd aa = a;
                    if (S == EX_S) {
                        load_node<EX_S>(A, m, inc, one);
                        aa = dd_mul(a, step<EX_S>(A, B));
                    } else {
                        load_node<EX_S - 1>(B, m, inc, one);
                    }
#pragma unroll 1
                    for (int half = S == EX_S ? 2 : 1; half > 0; --half) {
                        walk<EX_S - 1>(B, aa, sum);
#pragma unroll
                        for (int e = 0; e < ex_e(EX_S - 1); ++e) B[e] = A[e];
                        aa = a;
                    }
                }
            }
            __syncthreads();
        }
    }
    const dd tot = wave_dd_sum(sum_dd(sum));
    double ab = sum.ab;
    for (int mm = 32; mm > 0; mm >>= 1) ab += __shfl_xor(ab, mm);
    if (lane == 0) {
        part[3 * item] = tot.hi;
        part[3 * item + 1] = tot.lo;
        part[3 * item + 2] = ab;
    }
}

// Per row (one wavefront): the CSR check, the fixed-order sum of the parts,
// times det(Q)^{-1/2}.  Outputs: p, status (required), logp, kappa (nullable).
__global__ __launch_bounds__(256) void k_exact_final(int P, int M, const int *__restrict__ offsets,
                                                     const int *__restrict__ modes, int lgG, int maxn,
                                                     const double *__restrict__ part,
                                                     const double *__restrict__ scal, double *__restrict__ p_out,
                                                     double *__restrict__ logp_out, double *__restrict__ kappa_out,
                                                     int *__restrict__ status_out)
{
    const int p = blockIdx.x * 4 + (threadIdx.x >> 6), lane = threadIdx.x & 63;
    if (p >= P) return;
    const int o = offsets[p], n = offsets[p + 1] - o;
    if (n < 0 || n > maxn || !wave_row_ok(modes + o, n, M, lane)) {
        if (lane == 0) {
            p_out[p] = NAN;
            if (logp_out) logp_out[p] = NAN;
            if (kappa_out) kappa_out[p] = NAN;
            status_out[p] = GBS_PS_BADROW;
        }
        return;
    }
    const int h = n > EX_R ? n - EX_R : 0;
    const int ni = 1 << (h < lgG ? h : lgG);
    const long long i0 = (long long)p << lgG;
    dd s = dd_make(0.0);
    double ab = 0.0;
    if (n > 0)
        for (int i = lane; i < ni; i += 64) {
            s = dd_add(s, dd{part[3 * (i0 + i)], part[3 * (i0 + i) + 1]});
            ab += part[3 * (i0 + i) + 2];
        }
    s = wave_dd_sum(s);
    for (int mm = 32; mm > 0; mm >>= 1) ab += __shfl_xor(ab, mm);
    if (lane != 0) return;
    if (n == 0) {
        s = dd_make(1.0);
        ab = 1.0;
    }
    const dd rq = dd{scal[1], scal[2]};
    const dd pr = dd_mul(s, rq);
    const double kappa = s.hi != 0.0 ? ab / fabs(s.hi) : INFINITY;
    int st = 0;
    // double-double terms carry ~1e-30 relative error; the sum is resolved to
    // 1e-10 unless it cancels by more than 1e20
    if (!(kappa < 1e20) || !(pr.hi > 0.0)) st = GBS_PS_CANCEL;
    p_out[p] = st ? NAN : pr.hi;
    if (logp_out) logp_out[p] = st ? NAN : log(pr.hi) + pr.lo / pr.hi;
    if (kappa_out) kappa_out[p] = kappa;
    status_out[p] = st;
}

}  // namespace

// Partial sums that a batch of rows of at most maxn clicks may take:
// P << exact_lgs(maxn) (the size of the buffers and the limit of the fixed one)
int exact_lgs(int maxn)
{
    const int h = maxn > 9 ? maxn - 9 : 0;
    return h < EX_LGI ? h : EX_LGI;
}

// Parts per row, 2^lg: enough for about 2^14 work items (1024 run at a time; the
// rows' unequal shares then even out, while the blocks of short rows that find
// nothing to do cost 7 ns each: 4096 rows of 6-14 clicks take 764, 752, 939 and
// 1430 us with 2^13 .. 2^16 items, model build included), at most one per prefix
// assignment and 2^EX_LGI, and for large batches of long rows no fewer than
// leave a part 2^14 assignments (half a second).
static int exact_lgg(int P, int maxn)
{
    const int h = maxn > EX_R ? maxn - EX_R : 0, most = std::min(h, EX_LGI);
    int lgP = 0;
    while (lgP < 30 && (1LL << lgP) < P) ++lgP;
    return std::min(most, std::max(14 - lgP, std::max(most - 6, 0)));
}

// The exact path on device CSR: partials in d_part (3 doubles per part, at
// least P << exact_lgs(maxn) of them), results into the device outputs.
int exact_launch(gbs_ctx *ctx, int P, const int32_t *d_off, const int32_t *d_modes, int maxn, double *d_part,
                 double *p_dev, double *logp_dev, double *kappa_dev, int32_t *status_dev)
{
    if (P == 0) return 0;
    DevModel &m = ctx->model;
    hipStream_t st = ctx->stream;
    if (((long long)P << exact_lgs(maxn)) > 0x7fffffffLL)
        return set_err(ctx, GBS_E_INVAL, "exact: too many work items (rows x 2^12)");
    const int lgG = exact_lgg(P, maxn);
    const unsigned nitems = (unsigned)P << lgG;
    const int ts = timer_begin(ctx, TG_EXACT);
    if (maxn > EX_SMALL)
        hipLaunchKernelGGL(k_exact<false>, dim3(nitems), dim3(64), 0, st, m.M, m.qi_hi, m.qi_lo, d_off, d_modes,
                           lgG, maxn, d_part);
    else if (maxn > 0)
        hipLaunchKernelGGL(k_exact<true>, dim3(nitems), dim3(64), 0, st, m.M, m.qi_hi, m.qi_lo, d_off, d_modes,
                           lgG, maxn, d_part);
    hipLaunchKernelGGL(k_exact_final, dim3((P + 3) / 4), dim3(256), 0, st, P, m.M, d_off, d_modes, lgG, maxn,
                       d_part, m.scal, p_dev, logp_dev, kappa_dev, status_dev);
    timer_end(ctx, ts);
    HIP_TRY(ctx, hipGetLastError());
    return 0;
}

// ---------------------------------------------------------------------------
// Fixed scratch for gbs_prob_exact_dev_noalloc: the partial sums of up to
// EX_NOALLOC_ITEMS work items (3 doubles each, 24 MiB), one copy per GPU that
// the library runs on, held until the process ends.  Host code never passes
// the array's name to a kernel (on the host it is only a stand-in for the
// symbol): its device address is taken once per device, with that device
// current, and kept in scratch_ptr.
// ---------------------------------------------------------------------------
#define EX_NOALLOC_ITEMS (1 << 20)
#define EX_MAX_DEVICES 64
static __device__ __align__(256) double scratch[3 * EX_NOALLOC_ITEMS];

namespace {
std::mutex scratch_mu;
double *scratch_ptr[EX_MAX_DEVICES] = {};
}  // namespace

// Once per device (the caller has made it current): the device address of
// `scratch`.  Returns a HIP error code.
int exact_scratch_init(int device)
{
    if (device < 0 || device >= EX_MAX_DEVICES) return (int)hipErrorInvalidDevice;
    std::lock_guard<std::mutex> lk(scratch_mu);
    if (scratch_ptr[device]) return 0;
    void *ptr = nullptr;
    const hipError_t e = hipGetSymbolAddress(&ptr, HIP_SYMBOL(scratch));
    if (e != hipSuccess) return (int)e;
    scratch_ptr[device] = (double *)ptr;
    return 0;
}

long long exact_noalloc_items() { return EX_NOALLOC_ITEMS; }

double *exact_scratch(int device)
{
    if (device < 0 || device >= EX_MAX_DEVICES) return nullptr;
    std::lock_guard<std::mutex> lk(scratch_mu);
    return scratch_ptr[device];
}

// Host CSR (already checked): one copy in, one launch, one copy out, in a block
// of the context's pool.
int exact_run(gbs_ctx *ctx, int P, const int32_t *offsets, const int32_t *modes, double *p,
              double *logp, double *kappa, int32_t *status)
{
    if (P == 0) return 0;
    hipStream_t st = ctx->stream;
    int maxn = 0;
    for (int r = 0; r < P; ++r) maxn = std::max(maxn, offsets[r + 1] - offsets[r]);
    const long long nitems = (long long)P << exact_lgs(maxn);
    const size_t nnz = offsets[P], n = P;
    // the block: p, log p, kappa and status of every row; the rows; the partial sums
    const size_t back = n * (3 * sizeof(double) + sizeof(int32_t)), in = (n + 1 + nnz) * sizeof(int32_t);
    const size_t o_part = (back + in + 15) & ~(size_t)15;
    size_t got = 0;
    char *blk = (char *)ctx->pool->take(o_part + std::max(nitems, 1LL) * 3 * sizeof(double), &got, false);
    if (!blk) return set_err(ctx, GBS_E_NOMEM, "exact: device allocation failed");
    double *d_out = (double *)blk;
    int32_t *d_st = (int32_t *)(d_out + 3 * n), *d_off = d_st + n, *d_modes = d_off + n + 1;
    ctx->stage.resize(std::max(in, back));
    std::memcpy(ctx->stage.data(), offsets, (n + 1) * sizeof(int32_t));
    if (nnz) std::memcpy(ctx->stage.data() + (n + 1) * sizeof(int32_t), modes, nnz * sizeof(int32_t));
    int rc = 0;
    hipError_t e = hipMemcpyAsync(d_off, ctx->stage.data(), in, hipMemcpyHostToDevice, st);
    if (e == hipSuccess)
        rc = exact_launch(ctx, P, d_off, d_modes, maxn, (double *)(blk + o_part), d_out, d_out + n, d_out + 2 * n, d_st);
    // (the upload is done before its host copy takes the results)
    if (e == hipSuccess) e = hipStreamSynchronize(st);
    if (!rc && e == hipSuccess) e = hipMemcpyAsync(ctx->stage.data(), blk, back, hipMemcpyDeviceToHost, st);
    if (e == hipSuccess) e = hipStreamSynchronize(st);
    ctx->pool->give(blk, got);
    if (e == hipSuccess && !rc) {
        const double *out = (const double *)ctx->stage.data();
        std::copy(out, out + n, p);
        if (logp) std::copy(out + n, out + 2 * n, logp);
        if (kappa) std::copy(out + 2 * n, out + 3 * n, kappa);
        std::memcpy(status, out + 3 * n, n * sizeof(int32_t));
    }
    stage_done(ctx);
    if (e != hipSuccess) return set_err(ctx, GBS_E_HIP, std::string("exact: ") + hipGetErrorString(e));
    return rc;
}
