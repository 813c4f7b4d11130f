// Per-row set-up of the order-j estimate: A = (Q^{-1})_CC = V diag(alpha) V^T,
// one workgroup per row.
//
//   1. Householder reduction of A to tridiagonal form (symmetric rank-2
//      updates of the trailing block, Golub & Van Loan, Matrix Computations,
//      section 8.3.1), the reflectors kept in the rows they annihilate;
//   2. the orthogonal factor accumulated in their place, last reflector first;
//   3. implicit symmetric QR steps with Wilkinson shifts on the tridiagonal
//      matrix (ibid., section 8.3): wavefront 0 chases the bulge of a step with
//      plane rotations and records them, while the other wavefronts apply the
//      rotations of the step before to the rows of the factor;
//   4. the contour plan of the row from its spectrum, by wavefront 0.
// The factor comes out column-major, which is the layout the contour kernels
// read (eigenvector k contiguous).
//
// What bounds it: serial chains.  A Householder step is two reductions over the
// trailing block's columns between two barriers (about 2500 cycles at 28
// columns); a QR step is a chain of rotations, about 45 instructions each that a
// single wavefront issues every 8 cycles, and 1.7 such steps per eigenvalue
// follow one another.  So the columns' sums are split over the wavefronts and
// met in LDS with one barrier, norms and inner products are formed by every
// wavefront for itself on the DPP paths, the chase takes one inverse root per
// rotation and no memory access, and the factor's update runs beside it.  Rows
// of up to GBS_NSMALL clicks hold the matrix in LDS (57 KB at 40 clicks, 8 KB at
// 14); larger ones in global memory (L2).  Against the matrix in global memory
// for every row, one lane's chase with two divisions and a root between memory
// accesses, the factor's update after it, and the plan's bisection in one
// thread (us): 64 rows of 6-14 clicks 395 -> 167, one of 30 clicks 1030 -> 285,
// 4096 of 15-40 clicks 7750 -> 4900, 512 of 40-110 clicks 22200 -> 10100.
// The spectrum is as accurate as theirs: rms errors of alpha at 9 / 27 / 40 / 64 /
// 110 clicks 5.8 / 9.1 / 8.7 / 10.0 / 8.4e-16 against 6.7 / 10.1 / 9.3 / 11.2 /
// 10.1e-16.
#include "contour_common.h"

namespace {

// bytes of LDS: each wavefront's partial sums, a reflector and its partner (in
// their place two steps' rotations later), diagonal, couplings, and the matrix
// of the small rows
__host__ __device__ constexpr int eig_lds(int N, int waves, bool mat)
{
    return 8 * ((waves + 2) * N + 2 * N + (mat ? N * (N + 1) : 0));
}

// The active block [lo, hi] of the tridiagonal matrix below top: hi the highest
// index at or below top whose coupling to the row above is not negligible (the
// negligible ones set to zero), lo the lowest index joined to hi by
// non-negligible couplings (its own set to zero); 64 candidates per ballot.
// hi = 0: none is left.
__device__ __forceinline__ void active_block(const double *dg, double *ed, int top, int lane, int &lo, int &hi)
{
    const double eps = 2.220446049250313e-16;
    hi = lo = 0;
    bool have = false;
    for (int base = top; base >= 0; base -= 64) {
        // lane: index idx, whether it is joined to the one above (ed[i] is
        // negligible when |ed[i]| <= eps (|dg[i]| + |dg[i+1]|))
        const int idx = base - lane, i = max(idx, 1);
        const double e = fabs(ed[i - 1]), g = fabs(dg[i - 1]) + fabs(dg[i]);
        const bool joined = idx > 0 && !(e <= eps * g);
        unsigned long long bal = __ballot(joined);
        int from = 0;  // lanes before this one are done with
        if (!have) {
            if (bal == 0ull) continue;
            from = __ffsll((long long)bal) - 1;
            hi = base - from;
            have = true;
        }
        const unsigned long long open = ~bal & (~0ull << from);
        if (open != 0ull) {
            lo = base - (__ffsll((long long)open) - 1);
            break;
        }
    }
    for (int idx = hi + 1 + lane; idx <= top; idx += 64) ed[idx - 1] = 0.0;
    if (lo > 0 && lane == 0) ed[lo - 1] = 0.0;
}

// 1/sqrt(x), x normal: the hardware's estimate (about 24 bits) and one
// third-order step, its e = 1 - x y^2 with the rounding of x y kept (half an ulp;
// without it one, and the spectrum's errors are a tenth to a third larger)
__device__ __forceinline__ double rsq_nr(double x)
{
    const double y = __builtin_amdgcn_rsq(x);
    const double h = x * y, hl = fma(x, y, -h);
    const double e = fma(-hl, y, fma(-h, y, 1.0));
    return fma(y * e, fma(0.375, e, 0.5), y);
}
// sqrt(x), x normal, within half an ulp and a little: s = x / sqrt(x) corrected once
__device__ __forceinline__ double sqrt_nr(double x)
{
    const double y = rsq_nr(x), s = x * y;
    return fma(fma(-s, s, x), 0.5 * y, s);
}

__device__ __forceinline__ double lane_value(double x, int l)
{
    return __hiloint2double(__builtin_amdgcn_readlane(__double2hiint(x), l),
                            __builtin_amdgcn_readlane(__double2loint(x), l));
}

// One implicit QR step on [lo, hi] (hi > lo, uniform) by one wavefront, every
// lane following the same chain; the rotations into rot.  64 steps of the chain
// at a time, the block's entries come from and the results go to registers,
// lane k those of the chunk's step k, so that no memory access stands in it.
__device__ __forceinline__ void chase(double *dg, double *ed, int lo, int hi, int lane, double2 *rot)
{
    // Wilkinson shift: the eigenvalue of the trailing 2 x 2 block closer to its
    // last diagonal entry
    const double e = ed[hi - 1], dh = dg[hi], dd = 0.5 * (dg[hi - 1] - dh);
    const double q2 = fma(dd, dd, e * e);  // (> 0: e is not negligible)
    const double den = dd + copysign(q2 > 1e-290 ? sqrt_nr(q2) : sqrt(q2), dd);
    const double mu = fabs(den) > 1e-290 ? fma(-e * e, rcp_nr(den), dh) : dh;
    // a = dg[k] and b = ed[k] as rotated by the previous step
    double a = dg[lo], b = ed[lo];
    double x = a - mu, z = b;
    for (int cb = lo; cb < hi; cb += 64) {
        const int k0 = cb + lane, len = min(64, hi - cb);
        // step k's d = dg[k + 1], en = ed[k + 1] (0 at the block's end)
        const double dv = k0 < hi ? dg[k0 + 1] : 0.0, ev = k0 + 1 < hi ? ed[k0 + 1] : 0.0;
        double nd = 0.0, nr = 0.0, nc = 1.0, ns = 0.0;
        for (int k = 0; k < len; ++k) {
            const double d = lane_value(dv, k), en = lane_value(ev, k);
            // G_k on (k, k+1): c = x/r, s = z/r, r = (x^2 + z^2)^{1/2}; the next
            // step's entries come from x, z and 1/r^2 directly
            const double xx = x * x, zz = z * z, r2 = fma(x, x, zz), xz = x * z;
            const double y = rsq_nr(r2), yy = y * y, rc = fma(yy, fma(-r2, yy, 1.0), yy);
            double c = x * y, sn = z * y, r = r2 * y;
            double ek = fma(xz, d - a, (xx - zz) * b) * rc;
            double dn = fma(-2.0 * xz, b, fma(xx, d, zz * a)) * rc;
            if (!(r2 > 1e-290)) {
                // (both entries negligible, or their squares out of range)
                r = hypot(x, z);
                c = r != 0.0 ? x / r : 1.0;
                sn = r != 0.0 ? z / r : 0.0;
                ek = fma(c * sn, d - a, (c * c - sn * sn) * b);
                dn = fma(-2.0 * c * sn, b, fma(c * c, d, sn * sn * a));
            }
            const double nk = (a + d) - dn;
            const bool me = lane == k;
            nd = me ? nk : nd;
            nr = me ? r : nr;
            nc = me ? c : nc;
            ns = me ? sn : ns;
            x = ek;
            z = sn * en;
            b = c * en;
            a = dn;
        }
        if (lane < len) {
            dg[k0] = nd;
            rot[k0] = make_double2(nc, ns);
            if (k0 > lo) ed[k0 - 1] = nr;  // the bulge is gone
        }
    }
    if (lane == 0) {
        dg[hi] = a;
        ed[hi - 1] = x;
    }
}

// ---------------------------------------------------------------------------
// eig_ordered: rows of up to EIG_TINY clicks, by one wavefront of k_eig, and
// whole devices of up to GBS_NSMALL modes (k_eig_whole).
// Lossless rows hold sectors whose last moments, or whose weights, lie at the
// transform's rounding: there a fit takes one moment more or less by the sign of
// an error.  With a perturbation of 1e-16 of Q (8 and 12 modes, orders 1 to 4) the
// estimates of rows of 3 / 4 / 5 / 6 / 7 / 8 clicks moved by up to 5e-7 / 3e-8 /
// 5e-9 / 2e-10 / 1e-11 / 9e-13: by more than 1e-9 where at most order + 1 clicks
// leave the moments to determine the distribution, and by nothing that is seen
// beyond EIG_TINY.  Between two ways to take the sums, 39 of 300 batches of 16
// rows of 2-6 clicks moved by more than 1e-9, and 6 of 100 distributions.  So
// here every value has one rounding that no split over lanes changes: sums run in
// index order or by one tree over the index, the
// rotations' quotients and roots are correctly rounded, and the radius comes from
// the halvings of [0, 0.98 R_b], six at a time: the lanes evaluate the 63
// midpoints that six halvings can meet.
// The matrix, then the factor, are in LDS; lanes take columns, then the factor's
// rows; the wavefronts share the rank-2 update's rows, and those after the first
// apply a step's rotations while the first chases the next.
// 16 rows of 2-6 clicks 73 us (115 with a thread per column and the matrix
// in memory; 55 with the sums split), a device of 30 modes 415 us (1030; 285).
// ---------------------------------------------------------------------------
#define EIG_ORDERED_LDS(N) ((9 * (N) + 2 * (N) * ((N) + 1)) * 8)

// c = x/r, sn = z/r, r = (x^2 + z^2)^{1/2}, each rounded to nearest: the root by
// Goldschmidt's coupled iteration for r and 1/(2r) from the estimate of 1/r, with
// the remainder r2 - g g formed by fused multiply-adds, and the quotients by 1/r
// with one correction by their remainder (Markstein, IBM J. Res. Dev. 34, 1990).
__device__ __forceinline__ void rotation(double x, double z, double &c, double &sn, double &r)
{
    const double r2 = fma(x, x, z * z), ax = fabs(x), az = fabs(z);
    const bool in = r2 > 1e-200 && r2 < 1e200 && (ax > 1e-200 || ax == 0.0) && (az > 1e-200 || az == 0.0);
    if (in) {
        const double y0 = __builtin_amdgcn_rsq(r2);
        double g = r2 * y0, h = 0.5 * y0;
        const double e = fma(-h, g, 0.5);
        g = fma(g, e, g);
        h = fma(h, e, h);
        g = fma(fma(-g, g, r2), h, g);
        r = fma(fma(-g, g, r2), h, g);
        double y = h + h;
        y = fma(y, fma(-r, y, 1.0), y);
        const double qx = x * y, qz = z * y;
        c = fma(fma(-r, qx, x), y, qx);
        sn = fma(fma(-r, qz, z), y, qz);
    } else {
        r = sqrt(r2);
        c = 1.0;
        sn = 0.0;
        if (r != 0.0) {
            c = x / r;
            sn = z / r;
        }
    }
}

// chase with these rotations
__device__ __forceinline__ void chase_ordered(double *dg, double *ed, int lo, int hi, int lane, double2 *rot)
{
    const double e = ed[hi - 1];
    const double dd = 0.5 * (dg[hi - 1] - dg[hi]);
    const double den = dd + copysign(sqrt(fma(dd, dd, e * e)), dd);
    const double mu = den != 0.0 ? dg[hi] - e * e / den : dg[hi];
    double a = dg[lo], b = ed[lo];
    double x = a - mu, z = b;
    for (int cb = lo; cb < hi; cb += 64) {
        const int k0 = cb + lane, len = min(64, hi - cb);
        const double dv = k0 < hi ? dg[k0 + 1] : 0.0, ev = k0 + 1 < hi ? ed[k0 + 1] : 0.0;
        double nd = 0.0, nr = 0.0, nc = 1.0, ns = 0.0;
        for (int k = 0; k < len; ++k) {
            const double d = lane_value(dv, k), en = lane_value(ev, k);
            double c, sn, r;
            rotation(x, z, c, sn, r);
            const double cs = c * sn, c2 = c * c, s2 = sn * sn;
            const double dk = c2 * a + 2.0 * cs * b + s2 * d;
            const double dn = s2 * a - 2.0 * cs * b + c2 * d;
            const double ek = cs * (d - a) + (c2 - s2) * b;
            const bool me = lane == k;
            nd = me ? dk : nd;
            nr = me ? r : nr;
            nc = me ? c : nc;
            ns = me ? sn : ns;
            x = ek;
            z = sn * en;
            b = c * en;
            a = dn;
        }
        if (lane < len) {
            dg[k0] = nd;
            rot[k0] = make_double2(nc, ns);
            if (k0 > lo) ed[k0 - 1] = nr;  // the bulge is gone
        }
    }
    if (lane == 0) {
        dg[hi] = a;
        ed[hi - 1] = x;
    }
}

// NT threads take part (64: the others of the workgroup have left); N <= 128
template <int NT>
__device__ __forceinline__ void eig_ordered(int M, const double *__restrict__ qi, const double *__restrict__ scal,
                                            const int *__restrict__ modes, int n, double *__restrict__ alpha_out,
                                            double *__restrict__ Qf, RowPlan *__restrict__ row, int frozen,
                                            double *sh)
{
    constexpr int NW = NT / 64, NJ = NT > 64 ? 2 : 1;  // wavefronts, columns per lane
    __shared__ int s_lo[2], s_hi[2];
    const int tid = threadIdx.x, lane = tid & 63, wid = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int N = 2 * n, D = 2 * M, LD = N + 1;
    double2 *rot = (double2 *)sh;  // two steps', N each
    double *v = sh + 4 * N, *w = v + N, *dg = w + N, *ed = dg + N, *tau = ed + N;
    double *W = tau + N, *Q = W + N * LD;
    auto sync = [] {
        if (NT > 64) {
            __syncthreads();
        } else {
            // LDS of one wavefront: its accesses keep their order
            __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
            __builtin_amdgcn_wave_barrier();
        }
    };
    // a tree over the index, 64 and above onto 0.. first
    auto tree = [&](const double *x) {
        double s = x[0];
        if (NJ > 1) s += x[NJ - 1];
        for (int m = 32; m > 0; m >>= 1) s += __shfl_xor(s, m);
        return s;
    };
    for (int idx = tid; idx < N * N; idx += NT) {
        const int i = idx / N, j = idx - i * N;
        const int ri = i < n ? modes[i] : modes[i - n] + M;
        const int rj = j < n ? modes[j] : modes[j - n] + M;
        W[i * LD + j] = qi[(long)ri * D + rj];
    }
    sync();
    for (int k = 0; k + 2 < N; ++k) {
        const int m = N - k - 1;
        double *Wk = W + k * LD + k + 1, *W2 = Wk + LD;
        double x[NJ], q[NJ];
#pragma unroll
        for (int u = 0; u < NJ; ++u) {
            const int i = lane + 64 * u;
            x[u] = i < m ? Wk[i] : 0.0;
            q[u] = i > 0 ? fma(x[u], x[u], 0.0) : 0.0;  // (rounded before the tree)
        }
        const double sg = tree(q);
        const double x0 = lane_value(x[0], 0);
        double tk = 0.0, al = x0;
        if (sg != 0.0) {
            al = -copysign(sqrt(x0 * x0 + sg), x0);
            const double v0 = x0 - al;
            tk = 2.0 / (v0 * v0 + sg);
            if (lane == 0) x[0] = v0;
        }
#pragma unroll
        for (int u = 0; u < NJ; ++u)
            if (wid == 0 && lane + 64 * u < m) v[lane + 64 * u] = x[u];
        if (wid == 0 && lane == 0) {
            dg[k] = W[k * LD + k];
            ed[k] = al;
            tau[k] = tk;
        }
        sync();
        if (wid == 0)
            for (int i = lane; i < m; i += 64) Wk[i] = v[i];
        if (tk != 0.0) {
            // column sums in index order, a column per thread of the workgroup
            if (tid < m) {
                double s = 0.0;
#pragma unroll 8
                for (int i = 0; i < m; ++i) s = fma(W2[i * LD + tid], v[i], s);
                w[tid] = tk * s;
            }
            sync();
            double pj[NJ];
#pragma unroll
            for (int u = 0; u < NJ; ++u) {
                const int j = lane + 64 * u;
                pj[u] = j < m ? w[j] : 0.0;
                q[u] = fma(pj[u], x[u], 0.0);
            }
            const double kk = 0.5 * tk * tree(q);
            sync();
#pragma unroll
            for (int u = 0; u < NJ; ++u) {
                const int j = lane + 64 * u;
                pj[u] -= kk * x[u];
                if (wid == 0 && j < m) w[j] = pj[u];
            }
            sync();
#pragma unroll
            for (int u = 0; u < NJ; ++u) {
                const int j = lane + 64 * u;
                if (j >= m) continue;
#pragma unroll 4
                for (int i = wid; i < m; i += NW) W2[i * LD + j] -= v[i] * pj[u] + w[i] * x[u];
            }
        }
        sync();
    }
    if (tid == 0) {
        if (N >= 2) {
            dg[N - 2] = W[(N - 2) * LD + N - 2];
            ed[N - 2] = W[(N - 2) * LD + N - 1];
        }
        if (N >= 1) {
            dg[N - 1] = W[(N - 1) * LD + N - 1];
            ed[N - 1] = 0.0;
        }
    }
    // the factor, column-major: Q[c * LD + r]
    for (int idx = tid; idx < N * N; idx += NT) {
        const int c = idx / N, r = idx - c * N;
        Q[c * LD + r] = r == c ? 1.0 : 0.0;
    }
    sync();
    for (int k = N - 3; k >= 0; --k) {
        const double tk = tau[k];
        if (tk == 0.0) continue;
        const int m = N - k - 1;
        const double *vk = W + k * LD + k + 1;
        double *Q2 = Q + (k + 1) * LD + k + 1;
        if (tid < m) {
            const double *col = Q2 + tid * LD;
            double s = 0.0;
#pragma unroll 8
            for (int i = 0; i < m; ++i) s = fma(col[i], vk[i], s);
            w[tid] = tk * s;
        }
        sync();
#pragma unroll
        for (int u = 0; u < NJ; ++u) {
            const int i = lane + 64 * u;
            if (i >= m) continue;
            const double vi = vk[i];
#pragma unroll 4
            for (int j = wid; j < m; j += NW) Q2[j * LD + i] -= vi * w[j];
        }
        sync();
    }
    bool fail = false;
    int top = N - 1;
    for (int t = 0;; ++t) {
        const int b = t & 1;
        int lo = 0, hi = 0;
        if (wid == 0) {
            if (t < 60 * N + 60)
                active_block(dg, ed, top, lane, lo, hi);
            else
                fail = top > 0;
            lo = __builtin_amdgcn_readfirstlane(lo);
            hi = __builtin_amdgcn_readfirstlane(hi);
            __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
            __builtin_amdgcn_wave_barrier();
            if (hi > 0) chase_ordered(dg, ed, lo, hi, lane, rot + b * N);
            top = hi;
            if (NT > 64 && lane == 0) {
                s_lo[b] = lo;
                s_hi[b] = hi;
            }
        }
        // this step's rotations (one wavefront), or the step before's
        const bool apply = NT > 64 ? wid > 0 && t > 0 : hi > 0;
        if (NT == 64) sync();
        if (apply) {
            const int p = NT > 64 ? b ^ 1 : b;
            if (NT > 64) {
                lo = s_lo[p];
                hi = s_hi[p];
            }
            const double2 *g = rot + p * N;
            for (int r = NT > 64 ? tid - 64 : tid; r < N; r += NT > 64 ? NT - 64 : 64) {
                double qk = Q[lo * LD + r];
#pragma unroll 4
                for (int k = lo; k < hi; ++k) {
                    const double qn = Q[(k + 1) * LD + r];
                    const double c = g[k].x, sn = g[k].y;
                    Q[k * LD + r] = c * qk + sn * qn;
                    qk = c * qn - sn * qk;
                }
                Q[hi * LD + r] = qk;
            }
        }
        sync();
        if ((NT > 64 ? s_hi[b] : top) == 0) break;
    }
    for (int idx = tid; idx < N * N; idx += NT) {
        const int c = idx / N, r = idx - c * N;
        Qf[idx] = Q[c * LD + r];
    }
    if (wid != 0) return;
    double lg[NJ], amin = 1e300, dev = 0.0;
#pragma unroll
    for (int u = 0; u < NJ; ++u) {
        const int i = lane + 64 * u;
        lg[u] = 0.0;
        if (i >= N) continue;
        const double a = dg[i];
        alpha_out[i] = a;
        lg[u] = log(a);
        amin = fmin(amin, a);
        dev = fmax(dev, fabs(a - 1.0));
    }
    const double logdetA = tree(lg);
    amin = -wave_max(-amin);
    dev = wave_max(dev);
    RowPlan rp = *row;
    row_plan<true>(rp, n, dg, lane, scal[0], logdetA, amin, dev, scal[3] != 0.0 || fail, frozen & 1,
                   (frozen & 2) != 0);
    if (lane == 0) *row = rp;
}

__device__ __noinline__ void eig_tiny(int M, const double *__restrict__ qi, const double *__restrict__ scal,
                                      const int *__restrict__ modes, int n, double *__restrict__ alpha_out,
                                      double *__restrict__ Qf, RowPlan *__restrict__ row, int frozen, double *sh)
{
    eig_ordered<64>(M, qi, scal, modes, n, alpha_out, Qf, row, frozen, sh);
}

// one row: every mode
__global__ __launch_bounds__(256) void k_eig_whole(int M, const double *__restrict__ qi,
                                                   const double *__restrict__ scal,
                                                   const int *__restrict__ offsets, const int *__restrict__ modes,
                                                   double *__restrict__ alpha_out, double *__restrict__ vt_out,
                                                   RowPlan *__restrict__ rows, int frozen)
{
    extern __shared__ __attribute__((aligned(16))) double sh[];
    eig_ordered<256>(M, qi, scal, modes, offsets[1] - offsets[0], alpha_out, vt_out, rows, frozen, sh);
}

// MAT: the matrix in LDS, row-major with odd stride N + 1 (rows of up to
// GBS_NSMALL clicks); else in wbuf (row-major, stride N), and the factor in
// place in vt_out from step 3 on.
template <bool MAT, int THREADS>
__global__ __launch_bounds__(THREADS) void k_eig(
    int M, const double *__restrict__ qi, const double *__restrict__ scal,
    const int *__restrict__ offsets, const int *__restrict__ modes, const int *__restrict__ perm,
    const long long *__restrict__ voff, double *__restrict__ wbuf, double *__restrict__ alpha_out,
    double *__restrict__ vt_out, RowPlan *__restrict__ rows, int frozen)
{
    constexpr int NW = THREADS / 64;
    constexpr int NJ = ((MAT ? 2 * GBS_NSMALL : 2 * GBS_MAX_N_APPROX) + 63) / 64;  // columns per lane
    extern __shared__ __attribute__((aligned(16))) double sh[];
    __shared__ int s_lo[2], s_hi[2];
    const int p = perm[blockIdx.x];
    const int o = offsets[p], n = offsets[p + 1] - o, N = 2 * n;
    const int tid = threadIdx.x, lane = tid & 63, wid = __builtin_amdgcn_readfirstlane(tid >> 6);
    const long long vo = voff[p];
    if (MAT && n <= EIG_TINY) {
        if (wid == 0)
            eig_tiny(M, qi, scal, modes + o, n, alpha_out + 2 * o, vt_out + vo, rows + p, frozen, sh);
        return;
    }
    static_assert(NW >= 4, "two steps' rotations fit the partial sums' place");
    static_assert(EIG_TINY >= 1 && GBS_NSMALL >= 1, "(from here on N >= 4)");
    double *part = sh;                       // NW x N partial sums
    double *v = part + NW * N, *w = v + N;   // the reflector, its partner in the rank-2
                                             // update (every wavefront writes both, alike)
    double2 *rot = (double2 *)sh;            // two steps', N each
    double *dg = w + N, *ed = dg + N;
    double *W = MAT ? ed + N : wbuf + 2 * vo;
    const int ld = MAT ? N + 1 : N;
    double *Qf = vt_out + vo;  // orthogonal factor, column-major: Qf[c * N + r]
    const int D = 2 * M;
    for (int idx = tid; idx < N * N; idx += THREADS) {
        const int i = idx / N, j = idx - i * N;
        const int ri = i < n ? modes[o + i] : modes[o + i - n] + M;
        const int rj = j < n ? modes[o + j] : modes[o + j - n] + M;
        W[i * ld + j] = qi[(long)ri * D + rj];
    }
    __syncthreads();
    // 1. reduction: step k annihilates W[k][k+2..], reflector v (length m = N-k-1)
    //    stored in row k right of the diagonal, its tau on the diagonal (dg, ed
    //    hold the tridiagonal matrix); lanes take the trailing block's columns,
    //    wavefronts its rows in turn
    for (int k = 0; k + 2 < N; ++k) {
        const int m = N - k - 1;
        double *Wk = W + (long)k * ld + k + 1, *W2 = Wk + ld;
        double sg = 0.0;
        for (int i = lane; i < m; i += 64) {
            const double x = Wk[i];
            if (i > 0) {
                v[i] = x;
                sg = fma(x, x, sg);
            }
        }
        sg = wave_sum_dpp(sg);
        const double x0 = Wk[0];
        double tk = 0.0, al = x0, v0 = x0;
        if (sg != 0.0) {
            // (any al and tau as consistent as these to rounding will do: H is
            // orthogonal to the rounding of tau, and couples row k by al)
            const double r2 = fma(x0, x0, sg);
            al = -copysign(r2 > 1e-290 ? sqrt_nr(r2) : sqrt(r2), x0);
            v0 = x0 - al;
            const double vv = fma(v0, v0, sg);
            tk = vv > 1e-290 ? 2.0 * rcp_nr(vv) : 2.0 / vv;
        }
        if (lane == 0) v[0] = v0;
        if (tk != 0.0) {
            // p = tau W2 v (W2 symmetric: column sums), then w = p - (tau/2)(p.v) v
            for (int j = lane; j < m; j += 64) {
                double s[4] = {0.0, 0.0, 0.0, 0.0};
                int i = wid;
                for (; i + 3 * NW < m; i += 4 * NW) {
                    double x[4], y[4];
#pragma unroll
                    for (int u = 0; u < 4; ++u) {
                        x[u] = W2[i * ld + j + u * NW * ld];
                        y[u] = v[i + u * NW];
                    }
#pragma unroll
                    for (int u = 0; u < 4; ++u) s[u] = fma(x[u], y[u], s[u]);
                }
                for (; i < m; i += NW) s[0] = fma(W2[i * ld + j], v[i], s[0]);
                part[wid * N + j] = (s[0] + s[1]) + (s[2] + s[3]);
            }
        }
        __syncthreads();  // (also: row k has been read by every wavefront)
        if (wid == 0) {
            for (int i = lane; i < m; i += 64) Wk[i] = v[i];
            if (lane == 0) {
                dg[k] = W[(long)k * ld + k];
                ed[k] = al;
                W[(long)k * ld + k] = tk;
            }
        }
        if (tk != 0.0) {
            // (w is written once, when it is final: all wavefronts write it)
            double pj[NJ], pv = 0.0;
#pragma unroll
            for (int u = 0; u < NJ; ++u) {
                const int j = lane + 64 * u;
                pj[u] = 0.0;
                if (j >= m) continue;
                double s = part[j];
#pragma unroll
                for (int t = 1; t < NW; ++t) s += part[t * N + j];
                pj[u] = tk * s;
                pv = fma(pj[u], v[j], pv);
            }
            pv = wave_sum_dpp(pv);
            const double kk = 0.5 * tk * pv;
#pragma unroll
            for (int u = 0; u < NJ; ++u) {
                const int j = lane + 64 * u;
                if (j < m) w[j] = pj[u] - kk * v[j];
            }
            // (the change first: one rounding of the entry, which is near one on the
            // diagonal, where two of them made the spectrum's errors a tenth larger)
            for (int j = lane; j < m; j += 64) {
                const double vj = v[j], wj = w[j];
                int i = wid;
                for (; i + 3 * NW < m; i += 4 * NW) {
                    double x[4];
#pragma unroll
                    for (int u = 0; u < 4; ++u) x[u] = W2[i * ld + j + u * NW * ld];
#pragma unroll
                    for (int u = 0; u < 4; ++u)
                        W2[i * ld + j + u * NW * ld] = x[u] - fma(v[i + u * NW], wj, w[i + u * NW] * vj);
                }
                for (; i < m; i += NW) W2[i * ld + j] -= fma(v[i], wj, w[i] * vj);
            }
        }
        __syncthreads();
    }
    if (tid == 0) {
        dg[N - 2] = W[(long)(N - 2) * ld + N - 2];
        ed[N - 2] = W[(long)(N - 2) * ld + N - 1];
        dg[N - 1] = W[(long)(N - 1) * ld + N - 1];
        ed[N - 1] = 0.0;
    }
    __syncthreads();
    // 2. factor H_0 H_1 ... H_{N-3}, in place: after step k the block of rows and
    //    columns from k + 1 on holds H_k ... H_{N-3} (the identity's first row and
    //    column of each block, still occupied by a used reflector, are put in on
    //    the way); then the first row and column
    if (tid < 4) {
        const int i = N - 2 + (tid >> 1), j = N - 2 + (tid & 1);
        W[(long)i * ld + j] = i == j ? 1.0 : 0.0;
    }
    __syncthreads();
    for (int k = N - 3; k >= 0; --k) {
        const int m = N - k - 1;
        double *Wk = W + (long)k * ld + k + 1, *W2 = Wk + ld;
        const double tk = W[(long)k * ld + k];
        const bool fresh = k < N - 3;  // (the last block, 2 x 2, was set above)
        for (int i = lane; i < m; i += 64) v[i] = Wk[i];
        // u_j = tau sum_i v_i Q2[i][j]; Q2[i][j] -= v_i u_j
        auto q2 = [&](int i, int j) {
            const double x = W2[i * ld + j];
            return fresh && (i == 0 || j == 0) ? (i == j ? 1.0 : 0.0) : x;
        };
        for (int j = lane; j < m; j += 64) {
            double s[4] = {0.0, 0.0, 0.0, 0.0};
            int i = wid;
            for (; i + 3 * NW < m; i += 4 * NW) {
                double x[4], y[4];
#pragma unroll
                for (int u = 0; u < 4; ++u) {
                    x[u] = q2(i + u * NW, j);
                    y[u] = v[i + u * NW];
                }
#pragma unroll
                for (int u = 0; u < 4; ++u) s[u] = fma(x[u], y[u], s[u]);
            }
            for (; i < m; i += NW) s[0] = fma(q2(i, j), v[i], s[0]);
            part[wid * N + j] = (s[0] + s[1]) + (s[2] + s[3]);
        }
        __syncthreads();
        for (int j = lane; j < m; j += 64) {
            double u = part[j];
#pragma unroll
            for (int t = 1; t < NW; ++t) u += part[t * N + j];
            u *= tk;
            int i = wid;
            for (; i + 3 * NW < m; i += 4 * NW) {
                double x[4];
#pragma unroll
                for (int t = 0; t < 4; ++t) x[t] = q2(i + t * NW, j);
#pragma unroll
                for (int t = 0; t < 4; ++t) W2[(i + t * NW) * ld + j] = fma(-v[i + t * NW], u, x[t]);
            }
            for (; i < m; i += NW) W2[i * ld + j] = fma(-v[i], u, q2(i, j));
        }
        __syncthreads();
    }
    for (int i = tid; i < N; i += THREADS) W[(long)i * ld] = W[i] = i == 0 ? 1.0 : 0.0;
    __syncthreads();
    if (!MAT) {
        // (the sweeps' rows are lanes: column-major)
        for (int idx = tid; idx < N * N; idx += THREADS) {
            const int c = idx / N, r = idx - c * N;
            Qf[idx] = W[(long)r * N + c];
        }
        __syncthreads();
    }
    // 3. implicit symmetric QR steps on (dg, ed); ed[i] couples i and i+1
    bool fail = false;
    int top = N - 1;
    for (int t = 0;; ++t) {
        const int b = t & 1;
        if (wid == 0) {
            int lo = 0, hi = 0;
            if (t < 60 * N + 60)
                active_block(dg, ed, top, lane, lo, hi);
            else
                fail = top > 0;
            lo = __builtin_amdgcn_readfirstlane(lo);
            hi = __builtin_amdgcn_readfirstlane(hi);
            if (hi > 0) chase(dg, ed, lo, hi, lane, rot + b * N);
            top = hi;
            if (lane == 0) {
                s_lo[b] = lo;
                s_hi[b] = hi;
            }
        } else if (t > 0) {
            // the step before: columns k and k+1 rotated for k = lo .. hi-1, one
            // row per lane
            const int lo = s_lo[b ^ 1], hi = s_hi[b ^ 1];
            const double2 *g = rot + (b ^ 1) * N;
            for (int r = tid - 64; r < N; r += THREADS - 64) {
                double *q = MAT ? W + (long)r * ld : Qf + r;
                const int st = MAT ? 1 : N;
                double qk = q[(long)lo * st];
                int k = lo;
                for (; k + 4 <= hi; k += 4) {
                    double qn[4];
                    double2 cs[4];
#pragma unroll
                    for (int u = 0; u < 4; ++u) {
                        qn[u] = q[(long)(k + u + 1) * st];
                        cs[u] = g[k + u];
                    }
#pragma unroll
                    for (int u = 0; u < 4; ++u) {
                        q[(long)(k + u) * st] = fma(cs[u].x, qk, cs[u].y * qn[u]);
                        qk = fma(cs[u].x, qn[u], -cs[u].y * qk);
                    }
                }
                for (; k < hi; ++k) {
                    const double qn = q[(long)(k + 1) * st];
                    const double2 cs = g[k];
                    q[(long)k * st] = fma(cs.x, qk, cs.y * qn);
                    qk = fma(cs.x, qn, -cs.y * qk);
                }
                q[(long)hi * st] = qk;
            }
        }
        __syncthreads();
        if (s_hi[b] == 0) break;
    }
    if (MAT)
        for (int idx = tid; idx < N * N; idx += THREADS) {
            const int c = idx / N, r = idx - c * N;
            Qf[idx] = W[r * ld + c];
        }
    // 4. spectrum and plan
    if (wid != 0) return;
    double lsum = 0.0, amin = 1e300, dev = 0.0;
    for (int i = lane; i < N; i += 64) {
        const double a = dg[i];
        alpha_out[2 * o + i] = a;
        lsum += log(a);
        amin = fmin(amin, a);
        dev = fmax(dev, fabs(a - 1.0));
    }
    const double logdetA = wave_sum(lsum);
    amin = -wave_max(-amin);
    dev = wave_max(dev);
    RowPlan rp = rows[p];
    row_plan<false>(rp, n, dg, lane, scal[0], logdetA, amin, dev, scal[3] != 0.0 || fail, frozen & 1, (frozen & 2) != 0);
    if (lane == 0) rows[p] = rp;
}

}  // namespace

int eig_rows(gbs_ctx *ctx, gbs_plan *pl)
{
    if (pl->P == 0) return 0;
    const int fz = (pl->frozen ? 1 : 0) | (pl->whole ? 2 : 0);
    if (pl->whole && pl->nbig == 0) {
        const int lds = EIG_ORDERED_LDS(2 * pl->max_n);
        if (int rc = func_lds_limit(ctx, (const void *)k_eig_whole, lds)) return rc;
        hipLaunchKernelGGL(k_eig_whole, dim3(1), dim3(256), lds, ctx->stream, ctx->model.M, ctx->model.qi_hi,
                           ctx->model.scal, pl->d_offsets, pl->d_modes, pl->d_alpha, pl->d_v, pl->d_rows, fz);
        HIP_TRY(ctx, hipGetLastError());
        return 0;
    }
    // (rows by decreasing click count; the larger ones are perm[0..nbig))
    if (pl->nbig > 0) {
        const void *fn = (const void *)k_eig<false, 512>;
        const int lds = eig_lds(2 * pl->max_n, 8, false);
        if (int rc = func_lds_limit(ctx, fn, lds)) return rc;
        hipLaunchKernelGGL((k_eig<false, 512>), dim3(pl->nbig), dim3(512), lds, ctx->stream, ctx->model.M,
                           ctx->model.qi_hi, ctx->model.scal, pl->d_offsets, pl->d_modes, pl->d_perm, pl->d_voff,
                           pl->d_wbig, pl->d_alpha, pl->d_v, pl->d_rows, fz);
    }
    // The small rows, largest first: one launch, or for batches of more rows than
    // run at a time one per class of click counts, so that each class's LDS lets
    // as many of its workgroups as possible share a compute unit (2 above 36
    // clicks, then 3, 4 and 6).
    constexpr int tops[] = {GBS_NSMALL, 36, 31, 25, EIG_TINY, -1};
    const bool classes = pl->P - pl->nbig > 4 * ctx->num_cu;
    for (int i = pl->nbig, c = 0; i < pl->P; ++c) {
        const int below = classes ? tops[c + 1] : -1, n0 = pl->h_n[pl->h_perm[i]];
        int e = i;
        while (e < pl->P && pl->h_n[pl->h_perm[e]] > below) ++e;
        if (e == i) continue;
        const int lds = std::max(eig_lds(2 * n0, 4, true), EIG_ORDERED_LDS(2 * EIG_TINY));
        if (int rc = func_lds_limit(ctx, (const void *)k_eig<true, 256>, lds)) return rc;
        hipLaunchKernelGGL((k_eig<true, 256>), dim3(e - i), dim3(256), lds, ctx->stream, ctx->model.M,
                           ctx->model.qi_hi, ctx->model.scal, pl->d_offsets, pl->d_modes, pl->d_perm + i,
                           pl->d_voff, pl->d_wbig, pl->d_alpha, pl->d_v, pl->d_rows, fz);
        i = e;
    }
    HIP_TRY(ctx, hipGetLastError());
    return 0;
}
