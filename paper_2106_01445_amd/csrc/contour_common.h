// Device helpers shared by the forward (approx.hip) and adjoint (grad.hip)
// kernels of the order-j estimate: block reductions, the principal complex
// inverse square root, the LDS layout of M(w) per contour point, the radix-2
// FFT and the per-sector max-entropy fit.
#pragma once
#include "cplx.h"
#include "internal.h"

#define CONT_THREADS 512
#define FIT_THREADS 256
// Rounding of a contour value relative to the largest value of its transform:
// fp64 throughout (a few units of 2^-53), and the cluster sums of the mixed
// precision tier, whose eliminations run in fp32 (a few units of 2^-24).
#define ROUND_FP64 2e-16
#define ROUND_FP32 2e-7
// Mixed precision: a row whose estimated error exceeds the tier's target is
// run again in fp64 (GBS_PS_ESCALATED).
#ifndef MIXED_BOUND
#define MIXED_BOUND 1e-5
#endif
#define FIT_MAXIT 100
// largest odd factor of a contour size (K = r 2^a, r odd <= DFT_RMAX)
#ifndef DFT_RMAX
#define DFT_RMAX 15
#endif
// rows of up to this many clicks are decomposed by eig_ordered (eig.hip)
#define EIG_TINY 8

namespace {

__device__ __forceinline__ double wave_sum(double v)
{
    for (int m = 32; m > 0; m >>= 1) v += __shfl_xor(v, m);
    return v;
}
__device__ __forceinline__ double wave_max(double v)
{
    for (int m = 32; m > 0; m >>= 1) v = fmax(v, __shfl_xor(v, m));
    return v;
}
// the sum over a wavefront on the DPP paths (four steps within rows of 16
// lanes, two across them), from lane 63 to every lane
__device__ __forceinline__ double wave_sum_dpp(double x)
{
#define DPP_ADD(ctrl, rows)                                                                                  \
    {                                                                                                        \
        const int lo = __builtin_amdgcn_update_dpp(0, __double2loint(x), ctrl, rows, 0xf, true);             \
        const int hi = __builtin_amdgcn_update_dpp(0, __double2hiint(x), ctrl, rows, 0xf, true);             \
        x += __hiloint2double(hi, lo);                                                                       \
    }
    DPP_ADD(0x111, 0xf)  // row_shr 1, 2, 4, 8
    DPP_ADD(0x112, 0xf)
    DPP_ADD(0x114, 0xf)
    DPP_ADD(0x118, 0xf)
    DPP_ADD(0x142, 0xa)  // row_bcast 15, 31
    DPP_ADD(0x143, 0xc)
#undef DPP_ADD
    return __hiloint2double(__builtin_amdgcn_readlane(__double2hiint(x), 63),
                            __builtin_amdgcn_readlane(__double2loint(x), 63));
}
// sum and maximum over a workgroup (red: one entry per wavefront)
__device__ double block_sum(double v, double *red)
{
    v = wave_sum(v);
    if ((threadIdx.x & 63) == 0) red[threadIdx.x >> 6] = v;
    __syncthreads();
    double r = 0.0;
    for (int w = 0; w < (int)(blockDim.x >> 6); ++w) r += red[w];
    __syncthreads();
    return r;
}

__device__ double block_max(double v, double *red)
{
    v = wave_max(v);
    if ((threadIdx.x & 63) == 0) red[threadIdx.x >> 6] = v;
    __syncthreads();
    double r = red[0];
    for (int w = 1; w < (int)(blockDim.x >> 6); ++w) r = fmax(r, red[w]);
    __syncthreads();
    return r;
}

// log-sums over a workgroup of C pairs (largest exponent m, sum s of
// exp(. - m)) per thread, each as such a pair (red: 2 C entries per wavefront)
template <int C>
__device__ __forceinline__ void block_lse(double (&m)[C], double (&s)[C], double *red)
{
    const int w = threadIdx.x >> 6, nw = blockDim.x >> 6;
    double mx[C];
#pragma unroll
    for (int i = 0; i < C; ++i) mx[i] = wave_max(m[i]);
    if ((threadIdx.x & 63) == 0)
#pragma unroll
        for (int i = 0; i < C; ++i) red[w * C + i] = mx[i];
    __syncthreads();
#pragma unroll
    for (int i = 0; i < C; ++i) {
        mx[i] = red[i];
        for (int u = 1; u < nw; ++u) mx[i] = fmax(mx[i], red[u * C + i]);
        s[i] = wave_sum(m[i] == -INFINITY ? 0.0 : s[i] * exp(m[i] - mx[i]));
    }
    if ((threadIdx.x & 63) == 0)
#pragma unroll
        for (int i = 0; i < C; ++i) red[(nw + w) * C + i] = s[i];
    __syncthreads();
#pragma unroll
    for (int i = 0; i < C; ++i) {
        m[i] = mx[i];
        s[i] = 0.0;
        for (int u = 0; u < nw; ++u) s[i] += red[(nw + u) * C + i];
    }
    __syncthreads();
}

__device__ __forceinline__ cplx warp_csum(cplx v)
{
    for (int m = 32; m > 0; m >>= 1) {
        v.re += __shfl_xor(v.re, m);
        v.im += __shfl_xor(v.im, m);
    }
    return v;
}

// product over the 64 lanes of a wavefront (butterfly; every lane gets it)
__device__ __forceinline__ cplx warp_cprod(cplx v)
{
    for (int m = 32; m > 0; m >>= 1) {
        const cplx o = cplx{__shfl_xor(v.re, m), __shfl_xor(v.im, m)};
        v = cplx{fma(v.re, o.re, -v.im * o.im), fma(v.re, o.im, v.im * o.re)};
    }
    return v;
}

// z^{-1/2} on the principal branch, from |z| and the half-angle: with
// r = |z|, A = (|Re z| + r)/2, sqrt(z) = (sqrt A, Im z/(2 sqrt A)) for Re z >= 0
// and (|Im z|/(2 sqrt A), sign(Im z) sqrt A) otherwise; 1/sqrt(z) = conj(sqrt z)/r.
__device__ __forceinline__ cplx crsqrt_p(cplx z)
{
    const double s2 = fma(z.re, z.re, z.im * z.im);
    const double q = rsqrt(s2);          // 1/r
    const double r = s2 * q;
    const double A = 0.5 * (fabs(z.re) + r);
    const double w = rsqrt(A);
    const double big = A * w, small = 0.5 * fabs(z.im) * w;
    double sr, si;
    if (z.re >= 0.0) { sr = big; si = copysign(small, z.im); }
    else { sr = small; si = copysign(big, z.im); }
    return cmk(sr * q, -si * q);
}

// the same in fp32
__device__ __forceinline__ cplxf crsqrt_p(cplxf z)
{
    const float s2 = fmaf(z.re, z.re, z.im * z.im);
    const float q = rsqrtf(s2);
    const float r = s2 * q;
    const float A = 0.5f * (fabsf(z.re) + r);
    const float w = rsqrtf(A);
    const float big = A * w, small = 0.5f * fabsf(z.im) * w;
    float sr, si;
    if (z.re >= 0.0f) { sr = big; si = copysignf(small, z.im); }
    else { sr = small; si = copysignf(big, z.im); }
    return cmkf(sr * q, -si * q);
}

constexpr int CONT_MAXG = 8;
static_assert(CONT_MAXG <= CONT_THREADS / 64, "one wavefront per contour point of a pass");

// 2n rounded up to whole 16-wide tiles: rows kept in LDS hold V zero-padded to
// cont_tp x cont_tp (row stride cont_tp + 1) and d zero-padded to cont_tp
// entries, so that the M(w) tiles fetch their operands without masks
__host__ __device__ __forceinline__ int cont_tp(int n) { return 16 * ((2 * n + 15) / 16); }
// V (padded) and alpha (2n)
__host__ __device__ __forceinline__ int cont_vbytes(int n)
{
    return 8 * (cont_tp(n) * (cont_tp(n) + 1) + 2 * n);
}
// bytes of one slot: d (fp64 complex, cont_tp entries), z^{-1/2} (2n) and the
// 2x2 mode blocks of M(w) (3n + 4 n(n-1)/2 entries of the block type C),
// 16-byte aligned
template <class C = cplx>
__host__ __device__ __forceinline__ int cont_mbytes(int n)
{
    return 16 * (cont_tp(n) + 2 * n) + (((int)sizeof(C) * (2 * n * n + n) + 15) & ~15);
}
__host__ __device__ __forceinline__ int cont_fixed() { return 16 * (CONT_THREADS / 64) * 4 + 16 * CONT_MAXG; }

// Contour plan of one row from the spectrum alpha of A, run by one wavefront
// (every lane gets it): log P_vac(Cbar), and unless the plan is
// frozen the radius rho (the saddle point of the photon-number generating
// function at n photons, capped at 0.98 of the convergence radius
// 1/max|alpha - 1|) and the size K (the smallest r 2^a, r odd <= DFT_RMAX,
// a >= 1, that is >= 2n + 32 and whose aliasing factor (rho/R_b)^K is below
// 1e-16, at most GBS_KMAX); then log G_0(rho).
// (The radius thus tilts towards max(n, untilted mean).)
// A frozen radius is kept only while it still lies inside the current
// convergence disc with an aliasing factor (rho max|alpha - 1|)^K <= 1e-14 (the
// rule above with a margin, so that small changes of the model keep the plan);
// otherwise the row is planned afresh and flagged GBS_PS_CONTOUR.
// With target > 0 the tilted mean is set to target instead (the re-tilt of a
// row whose estimate lies in sectors far from the first target); the target
// used is kept in kbar.
// ORDERED: the radius by halvings alone and sums in index order (see
// eig_ordered).
template <bool ORDERED>
__device__ __forceinline__ void row_plan(RowPlan &rp, int n, const double *alpha, int lane,
                                         double logdetQ, double logdetA, double amin, double dev,
                                         bool nonpd, int frozen, bool whole = false, double target_in = 0.0)
{
    const int N = 2 * n;
    rp.status = 0;
    rp.flags = 0;
    rp.logdet_a = logdetA;
    rp.log_pvac = -0.5 * (logdetQ + logdetA);
    if (!(amin > 0.0) || nonpd) {
        rp.status = GBS_PS_PIVOT;
        return;
    }
    if (frozen) {
        const double x = rp.rho * dev;
        if (!(rp.K > 0 && rp.K <= GBS_KMAX) || !(x < 1.0) || (x > 0.0 && rp.K * log(x) > log(1e-14))) {
            frozen = 0;
            rp.flags = GBS_PS_CONTOUR;
        }
    }
    if (!frozen) {
        const double rb = dev > 1e-300 ? 1.0 / dev : 1e300;
        double hi = 0.98 * rb;
        // the tilted mean (increasing in rho) and its slope
        auto mfun = [&](double rho, double &slope) {
            double s = 0.0, d = 0.0;
            if (ORDERED) {
                slope = 0.0;
                for (int i = 0; i < N; ++i) {
                    const double a = alpha[i];
                    s += 0.5 * rho * (1.0 - a) / (1.0 + rho * (a - 1.0));
                }
                return s;
            }
            for (int i = lane; i < N; i += 64) {
                const double b = 1.0 - alpha[i], q = 1.0 / (1.0 - rho * b);
                s += 0.5 * rho * b * q;
                d += 0.5 * b * q * q;
            }
            slope = wave_sum_dpp(d);
            return wave_sum_dpp(s);
        };
        // the tilted mean photon number is set to n (the sectors of a click
        // pattern of n detectors start at n), or to the untilted mean where that
        // is larger (then the sectors that carry the estimate lie at and above
        // the untilted mean, and a radius below 1 would push them under the
        // transform's rounding floor); for the whole distribution, to the
        // untilted mean: rho = 1, every sector at its own weight
        double slope;
        const double target = target_in > 0.0 ? target_in : whole ? mfun(1.0, slope) : fmax((double)n, mfun(1.0, slope));
        double rho;
        if (dev < 1e-300) rho = 1.0;
        else if (mfun(hi, slope) <= target) rho = hi;
        else if (ORDERED) {
            // (at most 200 halvings, to the last few bits of rho)
            double lo = 0.0;
            for (int it = 0; it < 200 && hi - lo > 4e-16 * hi;) {
                // lane l > 0 is node l of a binary tree of halvings: the bits of l
                // below its leading one are the turns from the root, 1 for the
                // upper half
                double l = lo, h = hi;
                for (int b = 30 - __clz(lane | 1); b >= 0; --b) {
                    const double mid = 0.5 * (l + h);
                    if (lane >> b & 1) l = mid;
                    else h = mid;
                }
                const unsigned long long up = __ballot(mfun(0.5 * (l + h), slope) < target);
                for (int node = 1; node < 64 && it < 200 && hi - lo > 4e-16 * hi; ++it) {
                    const double mid = 0.5 * (lo + hi);
                    const int right = (int)(up >> node & 1ull);
                    if (right) lo = mid;
                    else hi = mid;
                    node = 2 * node + right;
                }
            }
            rho = 0.5 * (lo + hi);
        } else {
            // Newton steps inside the bracket, halved where they leave it or gain
            // less than a bit, to the last few bits of rho (a wavefront's lanes
            // take the terms: the 52 halvings of plain bisection, with the sums in
            // one thread, took 220 us at 40 clicks)
            double lo = 0.0;
            rho = 0.5 * hi;
            double last = hi;
            for (int it = 0; it < 200 && hi - lo > 4e-16 * hi; ++it) {
                const double f = mfun(rho, slope) - target;
                if (f < 0.0) lo = rho;
                else hi = rho;
                double next = rho - f / slope;
                double step = fabs(next - rho);
                const bool in = next > lo && next < hi;
                if (step <= 1e-12 * rho) {  // (quadratic convergence: the next is below rounding)
                    if (in) rho = next;
                    break;
                }
                if (!in || !(step < 0.5 * last)) {
                    next = 0.5 * (lo + hi);
                    step = fabs(next - rho);
                }
                last = step;
                rho = next;
            }
        }
        double kneed = 2.0 * n + 32.0;
        if (dev >= 1e-300) kneed = fmax(kneed, log(1e-16) / log(rho / rb));
        // the smallest r 2^a (r odd <= DFT_RMAX, a >= 1; the sizes dft_lds
        // takes) >= kneed
        int K = GBS_KMAX;
        for (int r = 1; r <= DFT_RMAX; r += 2) {
            int k = 2 * r;
            while (k < kneed && k < GBS_KMAX) k *= 2;
            if (k >= kneed && k < K) K = k;
        }
        rp.rho = rho;
        rp.kbar = target;
        rp.rconv = rb;
        rp.K = K;
        rp.log_rho = log(rho);
    }
    double s = 0.0;
    if (ORDERED) {
        // (each lane's terms, added in index order)
        for (int b = 0; b < N; b += 64) {
            const double t = b + lane < N ? log1p(rp.rho * (alpha[b + lane] - 1.0)) : 0.0;
            for (int i = 0; i < min(64, N - b); ++i) s += __shfl(t, i);
        }
    } else {
        for (int i = lane; i < N; i += 64) s += log1p(rp.rho * (alpha[i] - 1.0));
        s = wave_sum_dpp(s);
    }
    rp.log_g_rho = 0.5 * logdetA - 0.5 * s;
}

typedef double dbl4 __attribute__((ext_vector_type(4)));
// One 16x16x4 fp64 MFMA step, D += A B.  Lane l supplies A[l%16][l/16] and
// B[l/16][l%16]; element e of D sits at row 4e + l/16, column l%16.
__device__ __forceinline__ dbl4 mfma4(double a, double b, dbl4 c)
{
    return __builtin_amdgcn_mfma_f64_16x16x4f64(a, b, c, 0, 0, 0);
}

// Position of the pair (a, b), a < b, inside one plane of pair blocks.  Column
// layout (DIAG false): b(b-1)/2 + a, so that pairs sharing b are adjacent.
// Diagonal layout (DIAG true): the pairs of each distance b - a in turn, so
// that (a, b), (a+1, b+1), ... are adjacent.
template <bool DIAG>
__device__ __forceinline__ int pair_pos(int n, int a, int b)
{
    if (!DIAG) return b * (b - 1) / 2 + a;
    const int d = b - a;
    return (d - 1) * n - (((d - 1) * d) >> 1) + a;
}

// Store one 16x16 tile (it <= jt) of M(w) (2n x 2n, quadrature-major rows
// x_0..x_{n-1}, p_0..p_{n-1}) from the MFMA layout into the 2x2 mode-block
// layout at blk: every entry i <= j of the upper triangle is one block entry,
// diagonal blocks (x_a x_a, x_a p_a, p_a p_a) at a, n + a, 2n + a, pair blocks
// a < b (x_a x_b, x_a p_b, p_a x_b, p_a p_b) at 3n + t np + pair_pos(a, b).
// With FIX the arrays sit at the strides of a GBS_NSMALL-click row instead
// (GBS_NSMALL for the diagonal-block arrays, its pair count for the others).
template <class C, bool DIAG = false, bool FIX = false>
__device__ __forceinline__ void m_store(int n, int it, int jt, const dbl4 &mre, const dbl4 &mim,
                                        C *blk, int lane)
{
    const int N = 2 * n;
    const int ds = FIX ? GBS_NSMALL : n, np = FIX ? GBS_NSMALL * (GBS_NSMALL - 1) / 2 : n * (n - 1) / 2;
    const int l16 = lane & 15, lq = lane >> 4;
    const int j = jt * 16 + l16;
    if (j >= N) return;
#pragma unroll
    for (int e = 0; e < 4; ++e) {
        const int ii = it * 16 + 4 * e + lq;
        if (ii > j) continue;
        int off;
        if (j < n) {
            off = ii == j ? ii : 3 * ds + pair_pos<DIAG>(n, ii, j);
        } else if (ii < n) {
            const int a = ii, b = j - n;
            off = a == b ? ds + a : (a < b ? 3 * ds + np + pair_pos<DIAG>(n, a, b)
                                           : 3 * ds + 2 * np + pair_pos<DIAG>(n, b, a));
        } else {
            const int a = ii - n, b = j - n;
            off = a == b ? 2 * ds + a : 3 * ds + 3 * np + pair_pos<DIAG>(n, a, b);
        }
        blk[off] = from_d<C>(cmk(mre[e], mim[e]));
    }
}

// A BS x BS block of 16x16 tiles of M(w) = V diag(d) V^T on the matrix cores, by
// one wavefront: tiles (BS ib + s, BS jb + t), those with it <= jt stored.  Vt
// holds the eigenvectors as rows (entry i of eigenvector k at k*vs + i).  Each
// operand fetched per k-step serves BS tiles (BS = 2 halves the loads per MFMA
// where V is read from L2).
// With PAD, Vt and d are zero beyond 2n up to the tile edge, and no fetch is
// masked; FIX selects the fixed-stride block layout of m_store.
template <int BS, class C = cplx, bool DIAG = false, bool PAD = false, bool FIX = false>
__device__ __forceinline__ void m_block_mfma(int n, int ib, int jb, const double *Vt, int vs,
                                             const cplx *d, C *blk, int lane)
{
    const int N = 2 * n, KS = (N + 3) >> 2;
    const int l16 = lane & 15, lq = lane >> 4;
    int iv[BS], jv[BS];
#pragma unroll
    for (int s = 0; s < BS; ++s) {
        iv[s] = (BS * ib + s) * 16 + l16;
        jv[s] = (BS * jb + s) * 16 + l16;
    }
    dbl4 mre[BS][BS], mim[BS][BS];
#pragma unroll
    for (int s = 0; s < BS; ++s)
#pragma unroll
        for (int t = 0; t < BS; ++t) mre[s][t] = mim[s][t] = dbl4{0.0, 0.0, 0.0, 0.0};
#pragma unroll 2
    for (int ks = 0; ks < KS; ++ks) {
        const int k = ks * 4 + lq;
        const bool kok = PAD || k < N;
        const cplx dl = d[kok ? k : 0];
        double ar[BS], ai[BS], bv[BS];
#pragma unroll
        for (int s = 0; s < BS; ++s) {
            const bool aok = PAD || (kok && iv[s] < N), bok = PAD || (kok && jv[s] < N);
            const double va = Vt[aok ? k * vs + iv[s] : 0], vb = Vt[bok ? k * vs + jv[s] : 0];
            ar[s] = aok ? va * dl.re : 0.0;
            ai[s] = aok ? va * dl.im : 0.0;
            bv[s] = bok ? vb : 0.0;
        }
#pragma unroll
        for (int s = 0; s < BS; ++s)
#pragma unroll
            for (int t = 0; t < BS; ++t) {
                mre[s][t] = mfma4(ar[s], bv[t], mre[s][t]);
                mim[s][t] = mfma4(ai[s], bv[t], mim[s][t]);
            }
    }
#pragma unroll
    for (int s = 0; s < BS; ++s)
#pragma unroll
        for (int t = 0; t < BS; ++t)
            if (BS * ib + s <= BS * jb + t)
                m_store<C, DIAG, FIX>(n, BS * ib + s, BS * jb + t, mre[s][t], mim[s][t], blk, lane);
}

// tile u of the column-major list of upper tiles (it <= jt)
__device__ __forceinline__ void upper_tile(int u, int &it, int &jt)
{
    jt = 0;
    while ((jt + 1) * (jt + 2) / 2 <= u) ++jt;
    it = u - jt * (jt + 1) / 2;
}

template <class C>
struct SlotMT {
    cplx *d, *rz;
    C *d0, *d1, *d2, *o0, *o1, *o2, *o3;
};
using SlotM = SlotMT<cplx>;

template <class C = cplx>
__device__ __forceinline__ SlotMT<C> slot_view(cplx *base, int n)
{
    const int N = 2 * n, np = n * (n - 1) / 2;
    SlotMT<C> m;
    m.d = base;
    m.rz = base + cont_tp(n);
    m.d0 = (C *)(m.rz + N);
    m.d1 = m.d0 + n;
    m.d2 = m.d1 + n;
    m.o0 = m.d2 + n;
    m.o1 = m.o0 + np;
    m.o2 = m.o1 + np;
    m.o3 = m.o2 + np;
    return m;
}

// ---------------------------------------------------------------------------
// Sector fits.  Four lanes (a quad) work on one sector: each takes every fourth
// term of the support, and the sums over it meet by quad permutations, so that
// all four lanes hold the same values and take the same branches.
// What bounds them: the chain of Newton steps, each a sum of n exponentials.
// One evaluation per step serves its line search, the next step's Hessian and,
// at the last point, the sensitivity; a quarter of the terms per lane shortens
// it; neighbouring sectors' parameters start most fits (k_dft_fit).
// ---------------------------------------------------------------------------
#define FIT_G 4  // lanes per sector
typedef const __attribute__((address_space(3))) double *LdsTab;  // (a table in LDS)

__device__ __forceinline__ double quad_xor(double x, int ctrl1)
{
    int lo = __double2loint(x), hi = __double2hiint(x);
    if (ctrl1) {
        lo = __builtin_amdgcn_mov_dpp(lo, 0xB1, 0xf, 0xf, true);  // lanes 1, 0, 3, 2
        hi = __builtin_amdgcn_mov_dpp(hi, 0xB1, 0xf, 0xf, true);
    } else {
        lo = __builtin_amdgcn_mov_dpp(lo, 0x4E, 0xf, 0xf, true);  // lanes 2, 3, 0, 1
        hi = __builtin_amdgcn_mov_dpp(hi, 0x4E, 0xf, 0xf, true);
    }
    return __hiloint2double(hi, lo);
}
__device__ __forceinline__ double quad_sum(double x)
{
    x += quad_xor(x, 1);
    return x + quad_xor(x, 0);
}
__device__ __forceinline__ double quad_max(double x)
{
    x = fmax(x, quad_xor(x, 1));
    return fmax(x, quad_xor(x, 0));
}

// 1/x (x normal) by the hardware estimate and two Newton steps, within an ulp
__device__ __forceinline__ double rcp_nr(double x)
{
    double r = __builtin_amdgcn_rcp(x);
    r = fma(r, fma(-x, r, 1.0), r);
    return fma(r, fma(-x, r, 1.0), r);
}

// The basis on the support, phi[4 v + t - 1] = C(v, t) / C(n-1, t) for v = n - n'
// empty modes, t = 1..4 (zero where C(n-1, t) is), by the whole workgroup
__device__ __forceinline__ void fit_basis(int n, double *phi)
{
    const double ib[4] = {n > 1 ? 1.0 / (n - 1.0) : 0.0, n > 2 ? 2.0 / ((n - 1.0) * (n - 2.0)) : 0.0,
                          n > 3 ? 6.0 / ((n - 1.0) * (n - 2.0) * (n - 3.0)) : 0.0,
                          n > 4 ? 24.0 / ((n - 1.0) * (n - 2.0) * (n - 3.0) * (n - 4.0)) : 0.0};
    for (int v = threadIdx.x; v < n; v += blockDim.x) {
        phi[4 * v] = v * ib[0];
        phi[4 * v + 1] = 0.5 * v * (v - 1) * ib[1];
        phi[4 * v + 2] = v * (v - 1.0) * (v - 2.0) / 6.0 * ib[2];
        phi[4 * v + 3] = v * (v - 1.0) * (v - 2.0) * (v - 3.0) / 24.0 * ib[3];
    }
}

// Log-partition sum of the exp-polynomial with parameters c on n' = 1..n - v0,
// and about f0, its JP features at its largest term: the mean E[phi - f0] and the
// second moments E2 (upper triangle, row-major); gl: this lane's place in its
// quad.  JP is a template argument so that every array index is static (kept in
// registers).  Weights and features are taken relative to the largest term,
// found in a pass of its own: a distribution that has shrunk to one point then
// has a covariance of exactly zero, which ends the fit (with the rounding of w / w
// in its place moments that no distribution has take all FIT_MAXIT steps: a
// 30-mode device's sectors 5.7 ms instead of 0.3), and on a short support, where
// four features are nearly dependent, the covariance E2 - E E' loses least.
// SEQ (cut supports, v0 > 0, of up to FIT_SEQ points): every lane adds up the whole support in
// index order, f0 = 0.  There three or four moments determine the distribution
// almost, the covariance is singular but for rounding, and whether the last
// moment can be used hangs on the last bits of these sums (split over the quad,
// 3 of 300 devices' distributions moved by up to 5e-4 at order 4).
#define FIT_SEQ 10
template <int JP, bool SEQ>
__device__ __forceinline__ void fit_eval(int n, int v0, LdsTab phi, int gl, const double *c, double &lse,
                                         double *f0, double *E, double *E2)
{
    double zmax = -1e300, s = 0.0, e[JP], e2[JP * (JP + 1) / 2];
    int vm = v0;
    for (int v = v0 + (SEQ ? 0 : gl); v < n; v += SEQ ? 1 : FIT_G) {
        double z = 0.0;
#pragma unroll
        for (int t = 0; t < JP; ++t) z -= c[t] * phi[4 * v + t];
        if (z > zmax) {
            zmax = z;
            vm = v;
        }
    }
    if (!SEQ) {
        const double zq = quad_max(zmax);
        vm = (int)quad_max(zmax == zq ? (double)vm : (double)v0);
        zmax = zq;
    }
#pragma unroll
    for (int t = 0; t < JP; ++t) {
        e[t] = 0.0;
        f0[t] = SEQ ? 0.0 : phi[4 * vm + t];
    }
#pragma unroll
    for (int t = 0; t < JP * (JP + 1) / 2; ++t) e2[t] = 0.0;
    for (int v = v0 + (SEQ ? 0 : gl); v < n; v += SEQ ? 1 : FIT_G) {
        double f[JP], z = 0.0;
#pragma unroll
        for (int t = 0; t < JP; ++t) {
            f[t] = phi[4 * v + t];
            z -= c[t] * f[t];
            if (!SEQ) f[t] -= f0[t];
        }
        const double w = exp(z - zmax);
        s += w;
        int k = 0;
#pragma unroll
        for (int t = 0; t < JP; ++t) {
            const double wf = w * f[t];
            e[t] += wf;
#pragma unroll
            for (int u = t; u < JP; ++u) e2[k++] += wf * f[u];
        }
    }
    if (SEQ) {
        lse = zmax + log(s);
#pragma unroll
        for (int t = 0; t < JP; ++t) E[t] = e[t] / s;
#pragma unroll
        for (int k = 0; k < JP * (JP + 1) / 2; ++k) E2[k] = e2[k] / s;
        return;
    }
    s = quad_sum(s);
    lse = zmax + log(s);
    const double is = rcp_nr(s);
#pragma unroll
    for (int t = 0; t < JP; ++t) E[t] = quad_sum(e[t]) * is;
#pragma unroll
    for (int k = 0; k < JP * (JP + 1) / 2; ++k) E2[k] = quad_sum(e2[k]) * is;
}

// Solve of the JP x JP system H x = r (H from E, E2 as the covariance of the
// features, damped by 1e-14 of its trace) by L D L^T, or L L^T with SEQ; false if
// H is not positive.
template <int JP, bool SEQ>
__device__ __forceinline__ bool fit_solve(const double *E, const double *E2, const double *r, double *x)
{
    double H[JP][JP], L[JP][JP], tr = 0.0;
    int k = 0;
#pragma unroll
    for (int t = 0; t < JP; ++t)
#pragma unroll
        for (int u = t; u < JP; ++u) H[u][t] = E2[k++] - E[t] * E[u];
#pragma unroll
    for (int t = 0; t < JP; ++t) tr += H[t][t];
    if (!(tr > 0.0)) return false;
#pragma unroll
    for (int t = 0; t < JP; ++t) H[t][t] += 1e-14 * tr;
    if (SEQ) {
#pragma unroll
        for (int j = 0; j < JP; ++j) {
            double d = H[j][j];
#pragma unroll
            for (int l = 0; l < j; ++l) d -= L[j][l] * L[j][l];
            if (!(d > 0.0)) return false;
            L[j][j] = sqrt(d);
#pragma unroll
            for (int i = j + 1; i < JP; ++i) {
                double v = H[i][j];
#pragma unroll
                for (int l = 0; l < j; ++l) v -= L[i][l] * L[j][l];
                L[i][j] = v / L[j][j];
            }
        }
        double y[JP];
#pragma unroll
        for (int i = 0; i < JP; ++i) {
            double v = r[i];
#pragma unroll
            for (int l = 0; l < i; ++l) v -= L[i][l] * y[l];
            y[i] = v / L[i][i];
        }
#pragma unroll
        for (int i = JP - 1; i >= 0; --i) {
            double v = y[i];
#pragma unroll
            for (int l = i + 1; l < JP; ++l) v -= L[l][i] * x[l];
            x[i] = v / L[i][i];
        }
        return true;
    }
    // column j: H[i][j] <- L_ij d_j, L[i][j] = L_ij
#pragma unroll
    for (int j = 0; j < JP; ++j) {
#pragma unroll
        for (int l = 0; l < j; ++l)
#pragma unroll
            for (int i = j; i < JP; ++i) H[i][j] -= L[j][l] * H[i][l];
        if (!(H[j][j] > 0.0)) return false;
#pragma unroll
        for (int i = j + 1; i < JP; ++i) L[i][j] = H[i][j] / H[j][j];
    }
#pragma unroll
    for (int i = 0; i < JP; ++i) {
        x[i] = r[i];
#pragma unroll
        for (int l = 0; l < i; ++l) x[i] -= L[i][l] * x[l];
    }
#pragma unroll
    for (int i = JP - 1; i >= 0; --i) {
        x[i] /= H[i][i];  // (of a distribution near one point, down to 1e-308)
#pragma unroll
        for (int l = i + 1; l < JP; ++l) x[i] -= L[l][i] * x[l];
    }
    return true;
}

// Max-entropy fit on n' = 1..n - v0 (v = n - n' empty modes, v >= v0) of the JP
// moments m[] by Newton's method on the convex dual, from the parameters c;
// returns 1 if a Hessian is singular, 2 after FIT_MAXIT steps, else 0, minus
// the log-partition sum (log q(n) when v0 = 0), the parameters in c and the
// sensitivity u = H^{-1} E[phi] (H the covariance of the basis under the fit;
// 1e300 where H is singular) on success.
template <int JP, bool SEQ>
__device__ __forceinline__ int fit_newton(int n, int v0, LdsTab phi, int gl, const double *m, double *c,
                                          double &logq, double *u)
{
    double lse, f0[JP], E[JP], E2[JP * (JP + 1) / 2];
    fit_eval<JP, SEQ>(n, v0, phi, gl, c, lse, f0, E, E2);
    for (int it = 0; it <= FIT_MAXIT; ++it) {
        double mg[JP], slope = 0.0, L0 = lse;
        bool conv = true;
#pragma unroll
        for (int t = 0; t < JP; ++t) {
            mg[t] = (f0[t] - m[t]) + E[t];
            L0 += c[t] * m[t];
            if (!(fabs(mg[t]) <= 1e-15 + 1e-12 * fabs(m[t]))) conv = false;
        }
        // Newton step H x = -g, g = m - E, H the covariance of the features
        double x[JP], cn[JP];
        if (!fit_solve<JP, SEQ>(E, E2, mg, x)) return 1;
#pragma unroll
        for (int t = 0; t < JP; ++t) slope -= mg[t] * x[t];
        // (Armijo, while the predicted decrease is above the rounding of the
        // objective.  After convergence one polishing step, kept only if the
        // objective does not rise: with a moment below the tolerance, whose
        // feature has no weight at c, the covariance says nothing about it and
        // the step may lead anywhere)
        double st = 1.0;
        const double noise = 1e-13 * fmax(1.0, fabs(L0));
        for (;;) {
#pragma unroll
            for (int t = 0; t < JP; ++t) cn[t] = st > 0.0 ? c[t] + st * x[t] : c[t];
            fit_eval<JP, SEQ>(n, v0, phi, gl, cn, lse, f0, E, E2);
            if (!conv && !(-slope > noise)) break;
            double l2 = lse;
#pragma unroll
            for (int t = 0; t < JP; ++t) l2 += cn[t] * m[t];
            if (l2 <= L0 + (conv ? noise : 1e-4 * st * slope) || !(st > 1e-12)) break;
            st = conv ? 0.0 : 0.5 * st;
        }
#pragma unroll
        for (int t = 0; t < JP; ++t) c[t] = cn[t];
        if (conv) {
            if (!(fabs(lse) < INFINITY)) return 1;
            logq = -lse;
            // d log q / dm = -H^{-1} E[phi], the fit's own moments
#pragma unroll
            for (int t = 0; t < JP; ++t) mg[t] = f0[t] + E[t];
            if (!fit_solve<JP, SEQ>(E, E2, mg, u))
#pragma unroll
                for (int t = 0; t < JP; ++t) u[t] = 1e300;
            return 0;
        }
    }
    return 2;
}

__device__ __forceinline__ void lse_add(double &mx, double &s, double v)
{
    if (v == -INFINITY) return;
    if (v > mx) {
        s = s * exp(mx - v) + 1.0;
        mx = v;
    } else {
        s += exp(v - mx);
    }
}

// exp(2 pi i q / K), q >= 0, with the angle reduced to the nearest quarter
// turn in integers first: 2q/K = k/2 + x, k = round(4q/K), x = (4q - kK)/(2K)
// in [-1/4, 1/4], so that the only rounding is that of x.  Points near -1 (on
// a contour, w = -rho, next to the generating function's singularity on the
// negative axis) and near +-1, +-i then carry phase errors of ~1e-17 rad for
// every K, where rounding 2q/K itself would cost ~3e-16 rad whenever K is not
// a power of two.
__device__ __forceinline__ cplx unit_root(long long q, int K)
{
    const long long k = (4 * q + K / 2) / K;
    const double x = (double)(4 * q - k * K) / (2.0 * (double)K);
    double s, c;
    sincospi(x, &s, &c);
    switch ((int)(k & 3)) {
    case 0: return cplx{c, s};
    case 1: return cplx{-s, c};
    case 2: return cplx{-c, -s};
    default: return cplx{s, -c};
    }
}

// Sector transforms.  A contour has K = r 2^a points, r odd and at most
// DFT_RMAX, a >= 1 (the smallest such K that meets the aliasing rule, so that
// fewer points are evaluated than with powers of two alone).  The forward DFT
// X[k] = sum_q x[q] W^{qk}, W = exp(-2 pi i / K), runs in LDS by decimation in
// time: the r interleaved subsequences x[j + r m] (j < r) are transformed by
// radix-2 stages, each in its own block of L = K / r entries, and combined by
// r-point DFTs: X[m + s L] = sum_j W^{j m} F_j[m] W^{j s L} (s < r).
struct DftShape {
    int K, r, L, lgL;
};
__device__ __forceinline__ DftShape dft_shape(int K)
{
    DftShape d;
    d.K = K;
    d.r = K >> __builtin_ctz((unsigned)K);  // the odd part
    d.L = K / d.r;
    d.lgL = 0;
    while ((1 << d.lgL) < d.L) ++d.lgL;
    return d;
}
// Where input sample q goes: block q mod r, bit-reversed position q div r.
__device__ __forceinline__ int dft_pos(const DftShape &d, int q)
{
    const int j = q % d.r, m = q / d.r;
    return j * d.L + (int)(__brev((unsigned)m) >> (32 - d.lgL));
}
// W^e for 0 <= e < K from the half table W[m] = exp(-2 pi i m / K), m < K/2.
__device__ __forceinline__ cplx dft_tw(const cplx *W, int K, int e)
{
    return e < K / 2 ? W[e] : cneg(W[e - K / 2]);
}
// In-place forward DFT of X[0..K) in LDS, input placed by dft_pos, output in
// natural order.  All threads of the block (at least DFT_MINT) take part; in
// the r-point combines each thread takes outputs o = tid, tid + nt, ..., held
// until every input has been read.
#define DFT_MINT 256
__device__ void dft_lds(cplx *X, const cplx *W, const DftShape &d)
{
    const int tid = threadIdx.x, nt = blockDim.x;
    const int K = d.K, L = d.L;
    for (int lh = 0; lh < d.lgL; ++lh) {
        // W_L^{pos L / (2 half)} = W^{pos r L / (2 half)}, half = 2^lh (b counts
        // the butterflies over all blocks: whole groups of 2 half entries)
        const int half = 1 << lh, tstep = d.r << (d.lgL - lh - 1);
        for (int b = tid; b < K / 2; b += nt) {
            const int pos = b & (half - 1);
            const int i = ((b >> lh) << (lh + 1)) + pos, j = i + half;
            const cplx w = W[pos * tstep];
            const cplx u = X[i], v = cmul(w, X[j]);
            X[i] = cadd(u, v);
            X[j] = csub(u, v);
        }
        __syncthreads();
    }
    if (d.r > 1) {
        // twiddles in place, then the r-point sums (each of their roots W^{e}, e
        // a multiple of L, is a root of unity of order r)
        for (int o = tid + L; o < K; o += nt) {
            const int j = o >> d.lgL, m = o & (L - 1);
            X[o] = cmul(dft_tw(W, K, j * m), X[o]);
        }
        __syncthreads();
        cplx out[GBS_KMAX / DFT_MINT];
#pragma unroll
        for (int i = 0; i < GBS_KMAX / DFT_MINT; ++i) {
            const int o = tid + i * nt;
            if (o >= K) continue;
            const int m = o & (L - 1), step = o - m;
            cplx acc = X[m];
            int e = 0;  // (j o / L mod r) L
#pragma unroll 4
            for (int j = 1; j < d.r; ++j) {
                e += step;
                if (e >= K) e -= K;
                acc = cadd(acc, cmul(dft_tw(W, K, e), X[j * L + m]));
            }
            out[i] = acc;
        }
        __syncthreads();
#pragma unroll
        for (int i = 0; i < GBS_KMAX / DFT_MINT; ++i)
            if (tid + i * nt < K) X[tid + i * nt] = out[i];
        __syncthreads();
    }
}

// Result of one sector fit with at most JM moments: log q(n), the fitted
// parameters, the moments (zero past the ones used) and the sensitivity of log
// q(n) to them (d log q / d m_t = -u_t, u = H^{-1} E[phi]; zero past the ones used),
// how many moments were used, and bad != 0 if no fit succeeded.
template <int JM>
struct SectorFitT {
    double lq;
    double c[JM], m[JM], u[JM];
    int jr, bad;
};

template <int JM, bool SEQ>
__device__ __forceinline__ int fit_moments(int jr, int n, int v0, LdsTab phi, int gl, const double *m, double *c,
                                           double &logq, double *u)
{
    switch (jr) {
    case 1: return fit_newton<1, SEQ>(n, v0, phi, gl, m, c, logq, u);
    case 2: return fit_newton<2, SEQ>(n, v0, phi, gl, m, c, logq, u);
    case 3: return fit_newton<3, SEQ>(n, v0, phi, gl, m, c, logq, u);
    default: return fit_newton<JM >= 4 ? 4 : 1, SEQ>(n, v0, phi, gl, m, c, logq, u);
    }
}

// Fit one sector by a quad from its tilted moments t0..t4 (t0 > 0; moments past
// JM are ignored) on n' = 1..n - v0 (v0 > 0: a sector with fewer photons than
// modes): the moments m_t = tau_t / (tau_0 C(n-1,t)) are used up to the
// longest feasible prefix (0 < m_t < 1, decreasing in t, since
// 0 <= phi_{t+1} <= phi_t <= 1).  A moment whose true value lies below the
// transform's rounding floor can come out infeasible; it is then dropped, and
// so is the next one if the fit fails.  With m_1 <= 0 every clicked mode
// fires: q(n) = 1.
// The fit starts from cs where that holds the parameters of js = jr moments (a
// neighbouring sector's), else from the geometric distribution with the first
// moment (its limit for a long support), and again from c = 0 where a Hessian
// on the way was singular: the dual is convex, so the start only sets the
// number of steps (measured with orders 2 / 3: 11 / 14 from c = 0, 7 / 12 from
// the geometric one, 4 from a neighbour's).  js < 0, or a cut support (CUT: v0
// may be positive) of up to FIT_SEQ points: from c = 0 alone.  The moments
// arrive by value and the fit runs out of line, so that callers index nothing
// at run time.
template <int JM, bool CUT>
__device__ __noinline__ SectorFitT<JM> fit_sector(int n, int v0, int jp, LdsTab phi, int gl, double t0,
                                                  double t1, double t2, double t3, double t4, int js, double c1,
                                                  double c2, double c3, double c4)
{
    SectorFitT<JM> r;
    const double binv[4] = {1.0 / (n - 1.0), 2.0 / ((n - 1.0) * (n - 2.0)),
                            6.0 / ((n - 1.0) * (n - 2.0) * (n - 3.0)),
                            24.0 / ((n - 1.0) * (n - 2.0) * (n - 3.0) * (n - 4.0))};
    const double tau[4] = {t1, t2, t3, t4}, cs[4] = {c1, c2, c3, c4};
#pragma unroll
    for (int t = 0; t < JM; ++t) {
        r.m[t] = t < jp ? tau[t] / t0 * binv[t] : 0.0;
        r.c[t] = r.u[t] = 0.0;
    }
    int jr = 0;
#pragma unroll
    for (int t = 1; t <= JM; ++t)
        if (jr == t - 1 && t <= jp && r.m[t - 1] > 0.0 && r.m[t - 1] < 1.0 &&
            (t == 1 || r.m[t - 1] < r.m[t - 2]))
            jr = t;
    r.lq = 0.0;
    if (jp == 0) {
        r.jr = 0;
        r.bad = 0;
        return r;
    }
    const bool seq = CUT && v0 > 0 && n - v0 <= FIT_SEQ;
    int bad = 1;
    while (jr >= 1 && bad) {
        // starts: 2 a neighbour's, 1 geometric, 0 zero
        const double mu = r.m[0] * (n - 1.0);
        bad = 1;
        for (int start = seq || js < 0 ? 0 : js == jr ? 2 : 1; start >= 0 && bad == 1; --start) {
            if (start == 1 && (v0 > 0 || !(mu < 0.5 * (n - 1.0)))) continue;
#pragma unroll
            for (int t = 0; t < JM; ++t) r.c[t] = start == 2 && t < jr ? cs[t] : 0.0;
            if (start == 1) r.c[0] = (n - 1.0) * log1p(1.0 / mu);
            if (CUT && seq)
                bad = fit_moments<JM, true>(jr, n, v0, phi, gl, r.m, r.c, r.lq, r.u);
            else
                bad = fit_moments<JM, false>(jr, n, v0, phi, gl, r.m, r.c, r.lq, r.u);
        }
        if (bad) --jr;
    }
    if (jr == 0) {
        bad = r.m[0] <= 0.0 ? 0 : 1;
        r.lq = 0.0;
#pragma unroll
        for (int t = 0; t < JM; ++t) r.c[t] = 0.0;
    }
#pragma unroll
    for (int t = 0; t < JM; ++t)
        if (t >= jr) r.u[t] = 0.0;
    r.jr = jr;
    r.bad = bad;
    return r;
}

}  // namespace
