// Model build on the device, in double-double (Methods, Model; loss added).
//
//   sigma = D O diag(e^{-2r}, e^{2r}) O^T D / 2 + (I - D^2)/2,   Q = sigma + I/2
//   O = [[Re U, -Im U], [Im U, Re U]],  D = diag(sqrt eta, sqrt eta)
//
// Q is inverted by symmetric Gauss-Jordan sweeps over blocks of 16 rows, one
// launch per block, every 16 x 16 tile a workgroup: with P = L diag(d) L^T the
// block's own tile and Y_i = A_is L^{-T},
//   A_ss <- -P^{-1},  A_is <- A_is P^{-1},  A_ij <- A_ij - Y_i diag(1/d) Y_j^T,
// after the last block -Q^{-1}.  The Schur complements are thus those of the
// factorisation Q = L D L^T step by step, and the pivots its own; formed with
// P^{-1} instead, A_ij - (A_is P^{-1}) A_sj, they lose a factor cond(Q): against
// binary128 the rms error of Q^{-1} at 12 modes and r = 1.6 / 3 / 8 was 3.3 / 1170
// / 1.6e13 2^-106, now 2.0 / 43 / 3.9e6 (a Cholesky factor and triangular
// solves: 1.9 / 40 / 3.5e6).  The pivots d_k give
// positive definiteness, log det Q = sum log d_k and det(Q)^{-1/2} =
// prod d_k^{-1/2}.  Everything stays in HBM as hi/lo fp64 planes, row-major
// (2M)^2, xxpp order.
//
// What bounds it: the chain of 2M pivots (a double-double reciprocal, a product,
// up to three updates and a barrier each, 0.3 to 0.5 us), which every workgroup
// of a launch walks for itself so that no other launch stands between the
// blocks.  Blocks of 16 keep the tiles' products (16 terms per entry) below that
// chain.  Against a column-by-column Cholesky factor in one workgroup and a pair
// of triangular solves per column of the inverse, the inversion takes 8 / 34 /
// 96 / 257 us instead of 38 / 101 / 1160 / 8040 at M = 8 / 20 / 70 / 144 (a launch
// per block is 8 to 14 us; with P^{-1} in the Schur complements 8 to 12), and the
// assembly of Q 3 / 7 / 17 / 30 instead of 9 / 19 / 68 / 157.
#include "internal.h"

#define SWB 16

namespace {

__device__ __forceinline__ dd ld_dd(const double *hi, const double *lo, long i)
{
    return dd{hi[i], lo[i]};
}
__device__ __forceinline__ void st_dd(double *hi, double *lo, long i, dd v)
{
    hi[i] = v.hi;
    lo[i] = v.lo;
}

// The caller's U, r, eta into the model's own copy (where they are not there
// already), and e^{-2 r_k}, e^{2 r_k} (dd) and sqrt(eta_k) (dd).  Layout of expd:
// [0,2M) hi of d, [2M,4M) lo of d, [4M,5M) hi of s, [5M,6M) lo of s.
__global__ void k_model_scalars(int M, const double *ure, const double *uim, const double *r, const double *eta,
                                double *params, double *__restrict__ expd)
{
    const int k = blockIdx.x * blockDim.x + threadIdx.x, nt = gridDim.x * blockDim.x, D = 2 * M;
    if (k < D) {  // (a thread per exponential)
        const int m = k < M ? k : k - M;
        const double rk = r[m], ek = eta[m];
        const dd e = dd_exp(dd_make(k < M ? -2.0 * rk : 2.0 * rk));
        expd[k] = e.hi;
        expd[D + k] = e.lo;
        if (k < M) {
            const dd s = ek > 0.0 ? dd_sqrt(dd_make(ek)) : dd_make(0.0);
            expd[2 * D + k] = s.hi;
            expd[2 * D + M + k] = s.lo;
        }
        if (ure != params) params[2 * M * M + k] = k < M ? rk : ek;
    }
    if (ure != params)
        for (int i = k; i < M * M; i += nt) {
            params[i] = ure[i];
            params[M * M + i] = uim[i];
        }
}

__device__ __forceinline__ double o_entry(int M, const double *ure, const double *uim, int i,
                                          int k)
{
    if (i < M) return k < M ? ure[i * M + k] : -uim[i * M + k - M];
    return k < M ? uim[(i - M) * M + k] : ure[(i - M) * M + k - M];
}

// One 16 x 16 tile (ti >= tj) of Q per workgroup, one entry per thread, written
// with its mirror image; the rows of O and of O diag(e^{-2r}, e^{2r}) staged in
// LDS 16 columns at a time.
__global__ __launch_bounds__(256) void k_build_q(int M, const double *__restrict__ ure,
                                                 const double *__restrict__ uim,
                                                 const double *__restrict__ eta, const double *__restrict__ expd,
                                                 const double *__restrict__ sigma, double *__restrict__ q_hi,
                                                 double *__restrict__ q_lo)
{
    const int ti = blockIdx.x, tj = blockIdx.y;
    if (ti < tj) return;
    __shared__ double oa[SWB][SWB + 1];
    __shared__ double2 ob[SWB][SWB + 1];
    const int D = 2 * M, r = threadIdx.x >> 4, c = threadIdx.x & 15;
    const int i = ti * SWB + r, j = tj * SWB + c;
    dd q = dd_make(0.0);
    if (sigma) {
        if (i < D && j < D) {
            q = dd_make(sigma[(long)i * D + j]);
            if (i == j) q = dd_add_d(q, 0.5);
        }
    } else {
        dd acc = dd_make(0.0);
        const int jr = tj * SWB + r;  // (this thread stages row r of either side)
        for (int k0 = 0; k0 < D; k0 += SWB) {
            const int k = k0 + c;
            const bool kok = k < D;
            oa[r][c] = kok && i < D ? o_entry(M, ure, uim, i, k) : 0.0;
            const dd b = dd_mul_d(dd{kok ? expd[k] : 0.0, kok ? expd[D + k] : 0.0},
                                  kok && jr < D ? o_entry(M, ure, uim, jr, k) : 0.0);
            ob[r][c] = make_double2(b.hi, b.lo);
            __syncthreads();
#pragma unroll
            for (int t = 0; t < SWB; ++t) {
                // (error-free leading product and sum; what is below them in one
                // fp64 sum, folded back once per 16 terms)
                const double a = oa[r][t];
                const double2 v = ob[c][t];
                const dd f = two_prod(a, v.x);
                const dd s = two_sum(acc.hi, f.hi);
                acc.hi = s.hi;
                acc.lo += s.lo + fma(a, v.y, f.lo);
            }
            acc = quick_two_sum(acc.hi, acc.lo);
            __syncthreads();
        }
        if (i < D && j < D) {
            acc = dd_mul_d(acc, 0.5);
            dd si = dd{expd[2 * D + (i % M)], expd[2 * D + M + (i % M)]};
            dd sj = dd{expd[2 * D + (j % M)], expd[2 * D + M + (j % M)]};
            q = dd_mul(dd_mul(acc, si), sj);
            // diagonal: (1 - eta)/2 from the loss channel plus 1/2 = 1 - eta/2
            if (i == j) q = dd_add(q, two_sum(1.0, -0.5 * eta[i % M]));
        }
    }
    if (i < D && j <= i) {
        st_dd(q_hi, q_lo, (long)i * D + j, q);
        if (i != j) st_dd(q_hi, q_lo, (long)j * D + i, q);
    }
}

__device__ __forceinline__ dd wave_dd_prod(dd v)
{
    for (int m = 32; m > 0; m >>= 1) v = dd_mul(v, dd{__shfl_xor(v.hi, m), __shfl_xor(v.lo, m)});
    return v;
}

// a - p q - r s as dd_fms2, what is below the leading words added up as a short
// tree (29 operations against 27; Q^{-1}'s error is a tenth smaller)
__device__ __forceinline__ dd fms2(dd a, dd p, dd q, dd r, dd s)
{
    const dd f = two_prod(p.hi, q.hi), g = two_prod(r.hi, s.hi);
    const dd t = two_sum(f.hi, g.hi);
    const dd u = two_sum(a.hi, -t.hi);
    const double c = fma(p.hi, q.lo, p.lo * q.hi), d = fma(r.hi, s.lo, r.lo * s.hi);
    return quick_two_sum(u.hi, (a.lo - ((f.lo + g.lo) + t.lo)) + (u.lo - (c + d)));
}

// 1/x (x normal) by the hardware estimate and two Newton steps, within an ulp
__device__ __forceinline__ double rcp_nr(double x)
{
    double r = __builtin_amdgcn_rcp(x);
    r = fma(r, fma(-x, r, 1.0), r);
    return fma(r, fma(-x, r, 1.0), r);
}

// One sweep over block s, from src to dst (both full; a workgroup per tile
// ti >= tj, one entry per thread, written with its mirror image; rows past 2M
// act as rows of the identity).  P = L diag(d) L^T by right-looking steps that
// carry W = L^{-1} (in the lower part's place) and the rows of A_is and A_js
// along, which become Y = A L^{-T}: a block's inverse is formed for its own
// tiles alone.  ONE: a matrix of one block (nothing is carried along).
// scal: [0] log det Q, [1],[2] det(Q)^{-1/2} (dd), [3] 1 if not positive
// definite (dst is then the identity after the last block, so that no later
// kernel meets what the sweeps left), [8 .. 8+2D) the pivots as dd (hi then lo
// planes).
template <bool ONE>
__global__ __launch_bounds__(256) void k_sweep(int D, int s, int last, const double *__restrict__ s_hi,
                                               const double *__restrict__ s_lo, double *__restrict__ d_hi,
                                               double *__restrict__ d_lo, double *__restrict__ scal)
{
    const int ti = blockIdx.x, tj = blockIdx.y;
    if (ti < tj) return;
    // column k of P, row k of W, column k of either side's rows, as step k finds them
    __shared__ double2 pc[2][SWB], wr[2][SWB], ic[2][SWB], jc[2][SWB];
    __shared__ double2 piv[SWB], inv[SWB], w[SWB][SWB + 1], zi[SWB][SWB + 1], yj[SWB][SWB + 1];
    const int r = threadIdx.x >> 4, c = threadIdx.x & 15;
    const int i = ti * SWB + r, j = tj * SWB + c;
    const bool di = !ONE && ti != s, dc = !ONE && tj != s;
    bool bad = s > 0 && scal[3] != 0.0;
    // (read at a valid place and then chosen: no branch keeps the loads apart)
    auto at = [&](int a, int b) {
        const dd v = ld_dd(s_hi, s_lo, (long)min(a, D - 1) * D + min(b, D - 1)), e = dd_make(a == b ? 1.0 : 0.0);
        const bool in = a < D && b < D;
        return dd{in ? v.hi : e.hi, in ? v.lo : 0.0};
    };
    auto get = [](const double2 &v) { return dd{v.x, v.y}; };
    auto put = [](dd v) { return make_double2(v.hi, v.lo); };
    const int sr = s * SWB + r, sc = s * SWB + c;
    dd p = at(sr, sc), vi = at(i, sc), vj = at(tj * SWB + r, sc);
    const dd mine = at(i, j);
    if (c == 0) {
        pc[0][r] = put(p);
        ic[0][r] = put(vi);
        jc[0][r] = put(vj);
    }
    __syncthreads();
#pragma unroll 1
    for (int k = 0; k < SWB; ++k) {
        // (all of a step's operands first: the chain then waits for LDS once)
        const int b = k & 1;
        const bool right = c > k;
        const dd d = get(pc[b][k]), pr = get(pc[b][r]), pcc = get(pc[b][c]), wc = get(wr[b][c]);
        const dd ir = ONE ? pr : get(ic[b][r]), jr = ONE ? pr : get(jc[b][r]);
        bad = bad || !(d.hi > 0.0);
        // 1/d: the fp64 value y and y e (1 + e), e = 1 - d y
        const double y = rcp_nr(d.hi);
        const double e = fma(-d.lo, y, fma(-d.hi, y, 1.0));
        const dd id = quick_two_sum(y, y * fma(e, e, e));
        // one product by 1/d serves all: l_c of L's column k (entries right of k:
        // a_rc - a_rk l_c, also along the carried rows), l_r for W's row r
        const dd l = dd_mul(dd{right ? pcc.hi : pr.hi, right ? pcc.lo : pr.lo}, id);
        const dd q = dd_fms(p, l, dd{right ? pr.hi : wc.hi, right ? pr.lo : wc.lo});
        if (!ONE) {
            const dd zi_ = dd_fms(vi, ir, l), zj = dd_fms(vj, jr, l);
            vi = dd{right ? zi_.hi : vi.hi, right ? zi_.lo : vi.lo};
            vj = dd{right ? zj.hi : vj.hi, right ? zj.lo : vj.lo};
        }
        if (r > k && c <= r) p = c == k ? dd_neg(l) : q;
        if (threadIdx.x == 0) {
            piv[k] = put(d);
            inv[k] = put(id);
        }
        if (c == k + 1) {
            pc[b ^ 1][r] = put(p);
            if (!ONE) {
                ic[b ^ 1][r] = put(vi);
                jc[b ^ 1][r] = put(vj);
            }
        }
        if (r == k + 1 && c <= k) wr[b ^ 1][c] = put(p);
        __syncthreads();
    }
    // Z = Y diag(1/d) of the tile's rows, Y (beside the block's own rows Z) of its
    // columns; in the block's own tile diag(1/d) W
    const dd wv = r > c ? p : dd_make(r == c ? 1.0 : 0.0);
    const double2 dcl = inv[c], drw = inv[r];
    w[r][c] = put(wv);
    zi[r][c] = put(di ? dd_mul(vi, get(dcl)) : dd_mul(wv, get(drw)));
    yj[r][c] = put(di ? vj : dd_mul(vj, get(dcl)));
    __syncthreads();
    // A_ij - Z_i Y_j^T; Z_i W (its sign turned below), the new A_is; its mirror
    // image in the block's rows, (Z_j W)^T; -P^{-1} = -(diag(1/d) W)^T W
    const double2 *pa = di ? zi[r] : dc ? yj[c] : &zi[0][r], *pb = di && dc ? yj[c] : &w[0][dc ? r : c];
    const int sa = di || dc ? 1 : SWB + 1, sb = di && dc ? 1 : SWB + 1;
    dd out = di && dc ? mine : dd_make(0.0), more = dd_make(0.0);  // (two chains)
#pragma unroll
    for (int k = 0; k < SWB; k += 4) {
        out = fms2(out, get(pa[k * sa]), get(pb[k * sb]), get(pa[(k + 1) * sa]), get(pb[(k + 1) * sb]));
        more = fms2(more, get(pa[(k + 2) * sa]), get(pb[(k + 2) * sb]), get(pa[(k + 3) * sa]), get(pb[(k + 3) * sb]));
    }
    out = dd_add(out, more);
    if (di != dc) out = dd_neg(out);
    if (last) out = bad ? dd_make(i == j ? 1.0 : 0.0) : dd_neg(out);
    if (i < D && j <= i) {
        st_dd(d_hi, d_lo, (long)i * D + j, out);
        if (i != j) st_dd(d_hi, d_lo, (long)j * D + i, out);
    }
    if (ti == s && tj == s && threadIdx.x < 64) {
        const int lane = threadIdx.x, n0 = s * SWB;
        if (lane < SWB && n0 + lane < D) {
            scal[8 + n0 + lane] = piv[lane].x;
            scal[8 + D + n0 + lane] = piv[lane].y;
        }
        if (lane == 0 && (bad || s == 0)) scal[3] = bad ? 1.0 : 0.0;
        if (last) {
            double ld = 0.0;
            dd rd = dd_make(1.0);
            for (int k = lane; k < D; k += 64) {
                const dd d = k < n0 ? dd{scal[8 + k], scal[8 + D + k]} : get(piv[k - n0]);
                ld += log(d.hi) + d.lo / d.hi;
                rd = dd_mul(rd, dd_rsqrt(d));
            }
            for (int m = 32; m > 0; m >>= 1) ld += __shfl_xor(ld, m);
            rd = wave_dd_prod(rd);
            if (lane == 0) {
                scal[0] = ld;
                scal[1] = rd.hi;
                scal[2] = rd.lo;
            }
        }
    }
}

}  // namespace

static void free_model(DevModel &m)
{
    double **ptrs[] = {&m.q_hi, &m.q_lo, &m.qi_hi, &m.qi_lo, &m.work_hi, &m.work_lo,
                       &m.params, &m.scal, &m.expd};
    for (double **p : ptrs) {
        if (*p) (void)hipFree(*p);
        *p = nullptr;
    }
}

// Allocate model buffers for M modes (reallocating when M changes).
int model_alloc(gbs_ctx *ctx, int M)
{
    DevModel &m = ctx->model;
    if (m.M == M && m.q_hi) return 0;
    free_model(m);
    m.M = M;
    m.have = false;
    size_t D = 2 * (size_t)M, DD = D * D * sizeof(double);
    double **mats[] = {&m.q_hi, &m.q_lo, &m.qi_hi, &m.qi_lo, &m.work_hi, &m.work_lo};
    for (double **p : mats)
        if (ctx->pool->alloc((void **)p, DD) != hipSuccess) {
            free_model(m);
            m.M = 0;
            return set_err(ctx, -3, "model: device allocation failed");
        }
    if (ctx->pool->alloc((void **)&m.params, (2 * (size_t)M * M + 2 * M) * sizeof(double)) != hipSuccess ||
        ctx->pool->alloc((void **)&m.scal, (8 + 2 * D) * sizeof(double)) != hipSuccess ||
        ctx->pool->alloc((void **)&m.expd, 6 * (size_t)M * sizeof(double)) != hipSuccess) {
        free_model(m);
        m.M = 0;
        return set_err(ctx, -3, "model: device allocation failed");
    }
    return 0;
}

void model_release(gbs_ctx *ctx) { free_model(ctx->model); ctx->model.M = 0; }

// Build Q and its inverse.  ure, uim, r, eta: device arrays (the model's own
// copy ctx->model.params, or the caller's, which are copied there), ignored
// where sigma_dev is given.
int model_build_dev(gbs_ctx *ctx, const double *ure, const double *uim, const double *r, const double *eta,
                    const double *sigma_dev, bool sync)
{
    DevModel &m = ctx->model;
    int M = m.M, D = 2 * M;
    hipStream_t st = ctx->stream;
    const int tslot = timer_begin(ctx, TG_MODEL);
    if (!sigma_dev)
        hipLaunchKernelGGL(k_model_scalars, dim3((M * M + 255) / 256), dim3(256), 0, st, M, ure, uim, r, eta, m.params,
                           m.expd);
    const int T = (D + SWB - 1) / SWB;
    hipLaunchKernelGGL(k_build_q, dim3(T, T), dim3(256), 0, st, M, m.params, m.params + (size_t)M * M,
                       m.params + 2 * (size_t)M * M + M, m.expd, sigma_dev, m.q_hi, m.q_lo);
    // (the sweeps go back and forth between the work matrix and Q^{-1}'s place,
    // the last one into the latter)
    const double *sh = m.q_hi, *sl = m.q_lo;
    for (int s = 0; s < T; ++s) {
        const bool home = ((T - 1 - s) & 1) == 0;
        double *dh = home ? m.qi_hi : m.work_hi, *dl = home ? m.qi_lo : m.work_lo;
        hipLaunchKernelGGL((T > 1 ? k_sweep<false> : k_sweep<true>), dim3(T, T), dim3(256), 0, st, D, s, s == T - 1,
                           sh, sl, dh, dl, m.scal);
        sh = dh;
        sl = dl;
    }
    timer_end(ctx, tslot);
    HIP_TRY(ctx, hipGetLastError());
    if (!sync) {
        m.have = true;  // a non-PD Q is flagged on the device and reported per row
        return 0;
    }
    double flag = 0.0;
    HIP_TRY(ctx, hipMemcpyAsync(&flag, m.scal + 3, sizeof(double), hipMemcpyDeviceToHost, st));
    HIP_TRY(ctx, hipStreamSynchronize(st));
    if (flag != 0.0) {
        m.have = false;
        return set_err(ctx, -2, "covariance + I/2 is not positive definite");
    }
    m.have = true;
    return 0;
}
