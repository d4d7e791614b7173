// Precomputation of the local scattering matrices, FP64 on the GPU (Sec. 3.2:
// "we can pre-compute and store the block diagonal matrix A~^{-1}").
//
// For one generating contour (NG nodes, p-point Gauss panels) and modes
// m = 0..M the modal Nystrom matrix is A~_m = 1/2 I + K_m with
//   far entries   K_m(i, j) = k^G_m(y_i, y_j) r_j |gamma'_j| w_j,
//   near entries  K_m(i, j) = int_{-1}^{1} k^G_m(y_i, y(s)) l_j(s) r(s) |gamma'(s)| ds
// on the target's own panel, its neighbours and any panel closer to y_i than
// that panel's arc length (the paper cites Kolm-Rokhlin corrected quadrature
// for this step; here it is product integration with a graded Gauss rule:
// geometric bisection towards the (near-)singular parameter, 10 Gauss points or
// more per level, see the constants below for how far it goes).
// On a near panel the curve is the polynomial interpolant of the node
// positions and its derivative gives the normal and line element; on the
// target's own panel the displacement y(s) - y_i is formed from the Lagrange
// form with the exact factor (s - s_i), so n'.(y' - y) keeps full relative
// accuracy as y' -> y.
//
// The modal kernel k^G_m = (k^D_m + gamma k^S_m) / (4 pi) is evaluated exactly
// (gamma = i eta for kappa > 0; eta at kappa = 0, the Laplace equation of Sec. 6.1):
//   k^S_m = sum_l c_l q_{m-l} + i s_m,  c_l, s_m: Fourier coefficients of the
//   entire functions cos(kR(t)) and sin(kR)/R (sampled at Nt points),
//   q_m = 2 Q_{|m|-1/2}(chi) / sqrt(r r') with Q the toroidal harmonic
//   (AGM elliptic integrals, then the three-term recurrence: forward near
//   chi = 1, backward otherwise);
//   k^D_m = normal derivative at the source of the same expression.
// Pipeline per batch of target rows:
//   gen_far / gen_near  -> evaluation points (source data + weight)
//   toroidal_kernel     -> q_mu per point                        (thread per point)
//   modal_kernel        -> k^G_m * weight per point, m = 0..M    (16 points a workgroup)
//   scatter / near_reduce -> entries of A~_m
// (with the 1/2 on the diagonal), and S_m = A~_m^{-1} by Gauss-Jordan elimination
// with partial pivoting.  Shapes with the same p, M and Nt go through the pipeline
// together: three small shapes one after the other leave most of the chip idle.
#include <algorithm>
#include <cmath>
#include <memory>

#include "axs_internal.h"
#include "fp64_math.h"

namespace axs {

// Gauss points per level: the interpolation l_j(s) times the curve's own
// polynomial has degree 2p and more, which 10 points do not integrate for p > 10
// (with 10 the largest error of an entry is 2e-12 at p = 11, 1e-11 at 12 and
// 1e-8 at 16; with p points the kernel values' noise, 1e-12).  kl: the shape's longest panel
// in units of 1/kappa; the kernel's own oscillation takes one more for every two
// beyond 5 (with 10 the error is 1e-10 at kl = 9).
static int level_points(int p, double kl) {
    return std::max(p, 10 + (int)std::ceil(std::min(std::max(0.0, 0.5 * (kl - 5.0)), 54.0)));
}
constexpr int PMAX = 16;       // max nodes per panel supported
// Levels of the graded rule.  Every kernel value costs the same, so the points
// are what the precomputation pays for; 46 levels on both sides of every near
// panel (920 points) resolved far more than is there:
//  - own panel (the target is a node of it): a logarithmic singularity at the
//    node, a(s) log|s - s_i| + b(s) with a, b analytic.  OWN_LEV levels, then the
//    remaining interval [0, h] under x = h u^OWN_Q with OWN_NQ Gauss points,
//    which integrates polynomials and polynomials times log x to rounding: 134
//    points a side for p <= 10.
//  - other near panels: the integrand is analytic at the split point, its
//    singularity at least the target's distance d away, so the halving stops
//    where the innermost interval is shorter than d / 8 and that interval is one
//    level (10 Gauss points leave (16 + sqrt(255))^-20); 90 to 110 points a side,
//    none on a side of length zero.
// In FP64 the two rules agree with the 46-level one to the noise of the kernel
// values (1e-13 to 4e-12 of the largest entry, where 46 levels are as far from a
// tanh-sinh rule) for spheres of 1 to 20 panels, spheroids, a 10 : 1 needle and
// bowls, p = 3 to 16.
// 2760 -> 480 points per target node of a smooth contour.
constexpr int OWN_LEV = 11, OWN_Q = 8, OWN_NQ = 24;
constexpr int MAX_LEV = 46;

typedef double gj_f64x4 __attribute__((ext_vector_type(4)));

struct Pts {
    double *rt, *rp, *dr, *dz, *nr, *nz, *wj;   // [P]
    double *lag;                                 // [near points][p]
};

// target node i against near panel P, split at sstar: n0 points on the side
// towards -1 and n1 towards 1, from near point `first` of the batch on
struct NearDesc {
    int32_t i, P;
    double sstar;
    int32_t n0, n1, first, shape;
};

// target node i and panel P, their nodes all taken as far points
struct FarDesc {
    int32_t i, P, shape;
};

// where a shape's matrices go; nodes and panels are numbered through all shapes
// that are set up together.  Its rules, in the table of constants: `ngl` Gauss points a
// level from gl on and their weights behind, own_pts(ngl) of the own panel from own on
// and their weights behind.
struct ShapeRef {
    double2 *A;
    int32_t NG, node0;
    int32_t ngl, gl, own, pad;
};
__host__ __device__ inline int own_pts(int ngl) { return OWN_LEV * ngl + OWN_NQ; }

// ---------------------------------------------------------------------------
// evaluation points
// ---------------------------------------------------------------------------
// far points: pair (i, P) of target node and panel, its p nodes in turn
__global__ void gen_far_kernel(const FarDesc *__restrict__ pairs, int n, int p, const double *__restrict__ r,
                               const double *__restrict__ z, const double *__restrict__ nr,
                               const double *__restrict__ nz, const double *__restrict__ aw, Pts pts) {
    int o = blockIdx.x * blockDim.x + threadIdx.x;
    if (o >= n * p) return;
    const FarDesc pr = pairs[o / p];
    const int i = pr.i, j = pr.P * p + o % p;
    pts.rt[o] = r[i];
    pts.rp[o] = r[j];
    pts.dr[o] = r[j] - r[i];
    pts.dz[o] = z[j] - z[i];
    pts.nr[o] = nr[j];
    pts.nz[o] = nz[j];
    pts.wj[o] = aw[j];
}

// one workgroup per near pair.  rd, zd: derivative of each panel's interpolant at its
// nodes, so that the curve and its tangent both come from the Lagrange basis.  The
// basis is formed from running products kept in registers (p <= PMAX, unrolled).
// With the products in scratch memory and p^3 of them for the tangent the three shapes of
// 8 mixed bodies took 3 x 153 us, in one launch 15 now.
__global__ __launch_bounds__(128) void gen_near_kernel(const NearDesc *__restrict__ desc, int p,
                                                       const double *__restrict__ snode,
                                                       const double *__restrict__ lden,
                                                       const ShapeRef *__restrict__ shapes,
                                                       const double *__restrict__ tab, const double *__restrict__ r,
                                                       const double *__restrict__ z, const double *__restrict__ rd,
                                                       const double *__restrict__ zd, Pts pts, int64_t base) {
    const NearDesc d = desc[blockIdx.x];
    const ShapeRef sh = shapes[d.shape];
    const int ngl = sh.ngl;
    const double *glu = tab + sh.gl, *glw = glu + ngl, *ownx = tab + sh.own, *ownw = ownx + own_pts(ngl);
    const int own = (d.i / p) == d.P;
    const int iloc = own ? d.i - d.P * p : -1;
    const double *rP = r + d.P * p, *zP = z + d.P * p, *rdP = rd + d.P * p, *zdP = zd + d.P * p;
    const double ri = r[d.i], zi = z[d.i];
    for (int idx = threadIdx.x; idx < d.n0 + d.n1; idx += blockDim.x) {
        const int side = idx >= d.n0;
        const int q = side ? idx - d.n0 : idx;
        const int64_t o = base + d.first + idx;
        const double sst = d.sstar;
        const double dir = side == 0 ? -1.0 : 1.0;
        const double Ls = side == 0 ? sst + 1.0 : 1.0 - sst;
        double *lag = pts.lag + (int64_t)(d.first + idx) * p;
        double off, wq;
        if (own) {
            off = Ls * ownx[q];
            wq = Ls * ownw[q];
        } else {
            const int lev = q / ngl, kq = q % ngl, nlev = (side ? d.n1 : d.n0) / ngl;
            const double hi = Ls * ldexp(1.0, -lev);
            const double lo = lev == nlev - 1 ? 0.0 : 0.5 * hi;
            off = lo + (hi - lo) * 0.5 * (glu[kq] + 1.0);
            wq = glw[kq] * 0.5 * (hi - lo);
        }
        const double s = sst + dir * off;
        // Lagrange basis at s; on the own panel the factor (s - s_iloc) is the
        // exact signed offset.  L[k]: first the product of the factors before k.
        double L[PMAX], diff[PMAX], run = 1.0;
#pragma unroll
        for (int k = 0; k < PMAX; ++k)
            if (k < p) {
                diff[k] = k == iloc ? dir * off : s - snode[k];
                L[k] = run;
                run *= diff[k];
            }
        double rp = 0, zp = 0, rs = 0, zs = 0, dr = 0, dz = 0;
        run = 1.0;
#pragma unroll
        for (int k = PMAX - 1; k >= 0; --k)
            if (k < p) {
                const double l = L[k] * run * lden[k];
                run *= diff[k];
                lag[k] = l;
                rp = fma(l, rP[k], rp);
                zp = fma(l, zP[k], zp);
                rs = fma(l, rdP[k], rs);
                zs = fma(l, zdP[k], zs);
                dr = fma(l, rP[k] - ri, dr);   // own panel: the target node's term is exactly 0
                dz = fma(l, zP[k] - zi, dz);
            }
        if (!own) {
            dr = rp - ri;
            dz = zp - zi;
        }
        const double sp = sqrt(rs * rs + zs * zs);
        const bool ok = rp > 1e-13 && (dr * dr + dz * dz) > 0.0;
        pts.rt[o] = ri;
        pts.rp[o] = ok ? rp : -1.0;     // rp < 0 marks a point that contributes nothing
        pts.dr[o] = dr;
        pts.dz[o] = dz;
        pts.nr[o] = -zs / sp;
        pts.nz[o] = rs / sp;
        pts.wj[o] = ok ? wq * rp * sp : 0.0;
    }
}

// ---------------------------------------------------------------------------
// toroidal harmonics: q_mu = 2 Q_{mu-1/2}(chi)/sqrt(r r') = scale e^{-decay mu} f_mu
// ---------------------------------------------------------------------------
// lane j's value of x, in scalar registers
__device__ __forceinline__ double lane_value(double x, int j) {
    return __hiloint2double(__builtin_amdgcn_readlane(__double2hiint(x), j),
                            __builtin_amdgcn_readlane(__double2loint(x), j));
}

// One point per thread, f[mu][point].  Bound: the serial recurrence, up to 10 nq
// steps of two dependent multiply-adds in some wavefront or other.
//  - nq eta <= 2 (chi = cosh eta): forward from the elliptic integrals, which
//    amplifies rounding by e^2 at most.  With c = chi - 1 and e_mu = (mu - 1/2)
//    (f_mu - f_{mu-1}) the three-term recurrence is
//      e_{mu+1} = e_mu + 2 mu c f_mu,   f_{mu+1} = f_mu + e_{mu+1} / (mu + 1/2),
//    free of the rounding of 1 + c, which at small c is most of the error.
//  - otherwise backward, with the decay taken out, Q_{mu-1/2} ~ t^mu g_mu, t = e^{-eta}
//    (and 2 chi t = 1 + t^2), and h_mu = (mu - 1/2) (g_{mu-1} - g_mu):
//      h_mu = t^2 h_{mu+1} + (1 - t^2) g_mu / 2,   g_{mu-1} = g_mu + h_mu / (mu - 1/2),
//    all terms positive and no size beyond a power of mu; started at h = g / 2,
//    its limit, 18 / eta steps above nq (an error there shrinks by t^2 a step).
// All lanes of a wavefront take the same mu, each from its own start on, so the
// reciprocals come from one division per 64 steps.  With a division a step and the
// values of a point in a row of memory the three shapes of 8 mixed bodies took 3 x 233
// us, in one launch 54 now; 112,000 points of one shape (nq = 104) 381 and 62.
__global__ __launch_bounds__(64) void toroidal_kernel(Pts pts, int64_t npts, int nq, double *__restrict__ f,
                                                      double *__restrict__ scale, double *__restrict__ decay) {
    const int64_t pt = (int64_t)blockIdx.x * 64 + threadIdx.x;
    const int lane = threadIdx.x;
    const double rp = pt < npts ? pts.rp[pt] : -1.0;
    const bool active = rp > 0.0;
    double chim1 = 1.0, eta = 1.0, Q0 = 0.0, d1 = 0.0, srr = 1.0;
    if (active) {
        const double rt = pts.rt[pt], dr = pts.dr[pt], dz = pts.dz[pt];
        const double rr = rt * rp;
        srr = sqrt(rr);
        chim1 = (dr * dr + dz * dz) / (2.0 * rr);
        const double chi = 1.0 + chim1;
        const double pm = chim1 / (chi + 1.0);           // 1 - m, m = 2/(chi+1)
        // complete elliptic integrals K(m), E(m) by the arithmetic-geometric mean
        double a = 1.0, b = sqrt(pm), csum = 0.5 * (1.0 - pm), pw = 0.5;
        for (int it = 0; it < 64; ++it) {
            const double an = 0.5 * (a + b), cn = 0.5 * (a - b);
            b = sqrt(a * b);
            a = an;
            pw *= 2.0;
            csum += pw * cn * cn;
            if (fabs(cn) <= 1e-17 * a) break;
        }
        const double K = M_PI / (2.0 * a);
        const double E = K * (1.0 - csum);
        Q0 = sqrt(2.0 / (chi + 1.0)) * K;
        d1 = chim1 * Q0 - sqrt(2.0 * (chi + 1.0)) * E;   // Q_{1/2} - Q_{-1/2}
        eta = 2.0 * asinh(sqrt(0.5 * chim1));
    }
    double *q = f + pt;
    const bool backward = active && nq * eta > 2.0, forward = active && !backward;   // a NaN goes forward
    // backward starts: whole blocks of 64 above nq
    const int first = backward ? (int)(ceil(18.0 / eta) + 20.0 + 63.0) / 64 : 0;
    int wfirst = first;
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) wfirst = max(wfirst, __shfl_xor(wfirst, o, 64));
    wfirst = __builtin_amdgcn_readfirstlane(wfirst);
    double norm = 1.0;
    if (wfirst > 0) {
        const double t2 = exp(-2.0 * eta), w = -0.5 * expm1(-2.0 * eta);
        double v = 1.0, h = 0.5;
        for (int blk = wfirst; blk > 0; --blk) {
            const int mu0 = nq + 64 * blk;
            if (blk == first) {   // what a lane did ahead of its start is not used
                v = 1.0;
                h = 0.5;
            }
            const double rec = 1.0 / ((mu0 - lane) - 0.5);
#pragma unroll 16
            for (int j = 0; j < 64; ++j) {
                h = fma(w, v, t2 * h);
                v = fma(h, lane_value(rec, j), v);
            }
        }
        for (int mu0 = nq; mu0 >= 1; mu0 -= 64) {
            const double rec = 1.0 / ((mu0 - lane) - 0.5);
            for (int j = 0; j < min(64, mu0); ++j) {
                h = fma(w, v, t2 * h);
                v = fma(h, lane_value(rec, j), v);
                if (backward) q[(mu0 - j - 1) * npts] = v;
            }
        }
        norm = Q0 / v;
    }
    if (__any(forward)) {
        double v = Q0 + d1, e = 0.5 * d1;
        if (forward) {
            q[0] = Q0;
            q[npts] = v;
        }
        for (int mu0 = 1; mu0 + 1 < nq; mu0 += 64) {
            const double rec = 1.0 / ((mu0 + lane) + 0.5);
            for (int j = 0; j < min(64, nq - 1 - mu0); ++j) {
                e = fma(2.0 * (mu0 + j) * chim1, v, e);
                v = fma(e, lane_value(rec, j), v);
                if (forward) q[(mu0 + j + 1) * npts] = v;
            }
        }
    }
    if (active) {
        scale[pt] = 2.0 / srr * (backward ? norm : 1.0);
        decay[pt] = backward ? eta : 0.0;
    }
}

// ---------------------------------------------------------------------------
// modal kernel values
// ---------------------------------------------------------------------------
// (x cos x - sin x) / x^3 = sum_{k>=1} (-1)^k 2k x^{2k-2} / (2k+1)!  for |x| <= 0.2
// (the first term left out is below 2e-21)
__device__ __forceinline__ double tcos_series(double x) {
    const double y = x * x;
    double t = 1.0 / 518918400.0;
    t = fma(t, y, -1.0 / 3991680.0);
    t = fma(t, y, 1.0 / 45360.0);
    t = fma(t, y, -1.0 / 840.0);
    t = fma(t, y, 1.0 / 30.0);
    return fma(t, y, -1.0 / 3.0);
}

// sin x and cos x for 0 <= x < 1e5: x less the nearest multiple n of pi/2, whose second part
// leaves n 1.5e-33, and the Taylor series on [-pi/4, pi/4] (first terms left out below 9e-20 and 4e-21)
__device__ __forceinline__ void sincos_small(double x, double &s, double &c) {
    const double n = rint(x * 0.636619772367581343);
    double r = fma(-n, 1.5707963267948966, x);
    r = fma(-n, 6.123233995736766e-17, r);
    const double y = r * r;
    double a = 1.0 / 355687428096000.0, b = -1.0 / 6402373705728000.0;
    a = fma(a, y, -1.0 / 1307674368000.0);
    b = fma(b, y, 1.0 / 20922789888000.0);
    a = fma(a, y, 1.0 / 6227020800.0);
    b = fma(b, y, -1.0 / 87178291200.0);
    a = fma(a, y, -1.0 / 39916800.0);
    b = fma(b, y, 1.0 / 479001600.0);
    a = fma(a, y, 1.0 / 362880.0);
    b = fma(b, y, -1.0 / 3628800.0);
    a = fma(a, y, -1.0 / 5040.0);
    b = fma(b, y, 1.0 / 40320.0);
    a = fma(a, y, 1.0 / 120.0);
    b = fma(b, y, -1.0 / 720.0);
    a = fma(a, y, -1.0 / 6.0);
    b = fma(b, y, 1.0 / 24.0);
    b = fma(b, y, -0.5);
    const double sn = fma(a * y, r, r), cs = fma(b, y, 1.0);
    const int q = (int)n;
    s = (q & 1) ? cs : sn;
    c = (q & 1) ? sn : cs;
    if (q & 2) s = -s;
    if ((q + 1) & 2) c = -c;
}

// Sizes and LDS of modal_kernel for PT points a workgroup (in doubles)
struct ModalSize {
    int Nt, M, H, KP, L, nq, Lc;
    __host__ __device__ ModalSize(int Nt_, int M_)
        : Nt(Nt_), M(M_), H(Nt_ / 2), KP((H / 2 + 4) / 4 * 4), L(H - 1), nq(M_ + H), Lc(L > M_ ? L : M_) {}
    __host__ __device__ int shared(int PT) const {
        return Nt + H + 2 + PT * ((8 * KP > 2 * nq ? 8 * KP : 2 * nq) + 2 * (L + 1) + 2 * (M + 1));
    }
};

// k^G_m (times the point's weight) for m = 0..M of PT points per workgroup, in three parts:
//  - the four even functions of t (cos kR, sin(kR)/R and their normal
//    derivatives) at t_k = 2 pi k / Nt, k = 0..H = Nt/2, weighted for the cosine series
//      f_l = sum_k g_k cos(2 pi l k / Nt)
//    and folded at H/2, where cos changes by (-1)^l: e_k = g_k + g_{H-k} for even
//    l, o_k = g_k - g_{H-k} for odd;
//  - the series as a product on the FP64 matrix cores: the cosines of 16 l of
//    one parity times the folded samples of 4 PT columns;
//  - the convolution over l with q_{m-l}, per thread one point and MB values of
//    m: c_0 q_m + sum_l c_l (q_{|m-l|} + q_{m+l}), the MB pairs (q, dq) on either side
//    kept in registers and moved on by one per l.
// Bound by VALU issue (69 % of the cycles with two workgroups a CU), about half of it
// in the last part.  One wavefront per point, with five LDS reads per four
// multiply-adds of the series, took 3 x 184 us for the three shapes of 8 mixed bodies (M =
// 20), this 224 in one launch; 112,000 points with M = 40: 677 and 278.
template <int PT, int MB>
__global__ __launch_bounds__(256) void modal_kernel(Pts pts, int64_t npts, int Nt, int M, const double *__restrict__ f,
                                                    const double *__restrict__ scale, const double *__restrict__ decay,
                                                    double kappa, double gam_re, double gam_im,
                                                    double2 *__restrict__ kout) {
    extern __shared__ __attribute__((aligned(16))) double sm[];
    const ModalSize z(Nt, M);
    const int H = z.H, KP = z.KP, L = z.L, nq = z.nq;
    constexpr int CW = 4 * PT, CT = PT / 4, NPAR = 256 / PT;
    double *cosT = sm, *s2T = sm + Nt;               // cos(2 pi j / Nt); sin^2(pi j / Nt), j <= H
    double *ev = s2T + H + 2, *od = ev + KP * CW;    // folded samples [KP][CW]
    double2 *qd = (double2 *)ev;                     // later (q_mu, dq_mu) [nq][PT]
    const int un = 8 * KP > 2 * nq ? 8 * KP : 2 * nq;
    double2 *cd = (double2 *)(ev + PT * un);         // series of cos and its derivative [L + 1][PT]
    double2 *ss = cd + (L + 1) * PT;                 // of sin / R and its derivative [M + 1][PT], then the results
    const int tid = threadIdx.x, wave = tid >> 6, lane = tid & 63, g = lane >> 4, l16 = lane & 15;
    const int pl = tid % PT, par = tid / PT;         // this thread's point and its share of the work on it
    const int64_t pt0 = (int64_t)blockIdx.x * PT, pt = pt0 + pl;
    for (int j = tid; j < Nt; j += 256) cosT[j] = cospi(2.0 * j / Nt);
    for (int j = tid; j <= H; j += 256) {
        const double sh = sinpi((double)j / Nt);
        s2T[j] = sh * sh;
    }
    const double rp = pt < npts ? pts.rp[pt] : -1.0;
    const bool active = rp > 0.0;                    // rp <= 0 marks a point without contribution
    double rt = 0, dr = 0, dz = 0, nrp = 0, nzp = 0, wj = 0;
    if (active) {
        rt = pts.rt[pt];
        dr = pts.dr[pt];
        dz = pts.dz[pt];
        nrp = pts.nr[pt];
        nzp = pts.nz[pt];
        wj = pts.wj[pt];
    }
    const double rr = rt * rp, d0sq = dr * dr + dz * dz, ndel = nrp * dr + nzp * dz;
    __syncthreads();
    // samples (all factors are even in t)
    for (int k = par; k < KP; k += NPAR) {
        double e[4] = {0, 0, 0, 0}, o[4] = {0, 0, 0, 0};
        if (active && 2 * k <= H)
            for (int side = 0; side < (2 * k < H ? 2 : 1); ++side) {
                const int kk = side ? H - k : k;
                const double s2 = s2T[kk];               // sin^2(t/2)
                const double d2 = fma(4.0 * rr, s2, d0sq);
                const double inv = rsq(d2);
                double R = d2 * inv;
                R = d2 > 0.0 ? fma(0.5 * inv, fma(-R, R, d2), R) : 0.0;
                const double x = kappa * R;
                double sn, cs;
                if (x < 1e5) sincos_small(x, sn, cs);
                else sincos(x, &sn, &cs);
                const double sd = R > 0.0 ? sn * inv : kappa;
                const double T = x > 0.2 ? (x * cs - sn) * (inv * inv * inv) : kappa * kappa * kappa * tcos_series(x);
                const double gg = ndel + 2.0 * nrp * rt * s2;
                const double w = (k == 0 ? 1.0 : 2.0) / Nt;
                const double v[4] = {cs * w, sd * w, -kappa * sd * gg * w, T * gg * w};
#pragma unroll
                for (int c = 0; c < 4; ++c) {
                    e[c] += v[c];
                    o[c] += side ? -v[c] : (2 * k < H ? v[c] : 0.0);   // cos(pi l / 2) = 0 for odd l
                }
            }
#pragma unroll
        for (int c = 0; c < 4; ++c) {
            // rows 128 bytes apart in the banks, so that the four k of a fragment do not collide
            const int col = PT == 16 ? 16 * (c ^ (k & 1)) + pl : PT * c + pl;
            ev[k * CW + col] = e[c];
            od[k * CW + col] = o[c];
        }
    }
    __syncthreads();
    // cosine series, 16 l of one parity per wavefront and turn
    const int ntile = 2 * ((z.Lc / 2 + 16) / 16);
    for (int tile = wave; tile < ntile; tile += 4) {
        const int odd = tile & 1, l0 = 32 * (tile >> 1) + odd;
        const double *src = odd ? od : ev;
        gj_f64x4 acc[CT];
#pragma unroll
        for (int c = 0; c < CT; ++c) acc[c] = (gj_f64x4){0, 0, 0, 0};
        const int l = l0 + 2 * l16;
        int idx = l * g % Nt;
        const int step = 4 * l % Nt;
        for (int k = 0; k < KP; k += 4) {
            const double a = cosT[idx];
            idx += step;
            if (idx >= Nt) idx -= Nt;
#pragma unroll
            for (int c = 0; c < CT; ++c) {
                const int col = (PT == 16 ? 16 * (c ^ (g & 1)) : 16 * c) + l16;
                acc[c] = __builtin_amdgcn_mfma_f64_16x16x4f64(a, src[(k + g) * CW + col], acc[c], 0, 0, 0);
            }
        }
#pragma unroll
        for (int c = 0; c < CT; ++c) {
            const int fct = (16 * c + l16) / PT, p2 = (16 * c + l16) % PT;
#pragma unroll
            for (int v = 0; v < 4; ++v) {
                const int ll = l0 + 2 * (g + 4 * v);
                if (fct % 2 == 0) {
                    if (ll <= L) (fct ? cd[ll * PT + p2].y : cd[ll * PT + p2].x) = acc[c][v];
                } else if (ll <= M) {
                    (fct == 3 ? ss[ll * PT + p2].y : ss[ll * PT + p2].x) = acc[c][v] * (2.0 * M_PI);
                }
            }
        }
    }
    __syncthreads();
    // q_mu and its normal derivative
    {
        const double chim1 = d0sq / (2.0 * rr), c2m1 = chim1 * (chim1 + 2.0);
        const double ndchi = ndel / rr - nrp * d0sq / (2.0 * rr * rp);
        const double ca = ndchi / c2m1, cb = nrp / (2.0 * rp);
        const double sc = active ? scale[pt] : 0.0, de = active ? decay[pt] : 0.0, t = exp(-de);
        const double *fp = f + min(pt, npts - 1);
        // consecutive mu per thread, eight loads in flight
        const int ch = (nq + NPAR - 1) / NPAR, mu1 = min(nq, (par + 1) * ch);
        int mu = par * ch;
        double pw = sc * exp(-de * mu);
        double prev = mu > 0 ? sc * exp(-de * (mu - 1)) * fp[min(mu - 1, nq - 1) * npts] : sc * t * fp[npts];   // Q_{-3/2} = Q_{1/2}
        for (; mu < mu1; mu += 8) {
            double v[8];
#pragma unroll
            for (int i = 0; i < 8; ++i) v[i] = fp[min(mu + i, nq - 1) * npts];
#pragma unroll
            for (int i = 0; i < 8; ++i)
                if (mu + i < mu1) {
                    const double q = pw * v[i];
                    const double dq = (mu + i - 0.5) * fma(chim1, q, q - prev) * ca - cb * q;
                    qd[(mu + i) * PT + pl] = active ? make_double2(q, dq) : make_double2(0.0, 0.0);
                    prev = q;
                    pw *= t;
                }
        }
    }
    __syncthreads();
    const double inv4pi = 0.25 / M_PI;
    for (int m0 = par * MB; m0 <= M; m0 += NPAR * MB) {
        double2 lo[MB], hi[MB];   // (q, dq) of |m0 + j - l| in slot (j - l) mod MB, of m0 + j + l in (j + l) mod MB
        double sr[MB], sd[MB];
        const double2 c0 = cd[pl];
#pragma unroll
        for (int j = 0; j < MB; ++j) {
            lo[j] = hi[j] = qd[min(m0 + j, nq - 1) * PT + pl];
            sr[j] = c0.x * lo[j].x;
            sd[j] = fma(c0.y, lo[j].x, c0.x * lo[j].y);
        }
        for (int l0 = 0; l0 < L; l0 += MB)
#pragma unroll
            for (int u = 1; u <= MB; ++u) {
                const int l = l0 + u;
                if (l > L) break;
                lo[(MB - u) % MB] = qd[abs(m0 - l) * PT + pl];
                hi[(MB - 1 + u) % MB] = qd[min(m0 + MB - 1 + l, nq - 1) * PT + pl];
                const double2 c = cd[l * PT + pl];
#pragma unroll
                for (int j = 0; j < MB; ++j) {
                    const double2 a = lo[(j + MB - u) % MB], b = hi[(j + u) % MB];
                    const double q = a.x + b.x;
                    sr[j] = fma(c.x, q, sr[j]);
                    sd[j] = fma(c.y, q, fma(c.x, a.y + b.y, sd[j]));
                }
            }
#pragma unroll
        for (int j = 0; j < MB; ++j)
            if (m0 + j <= M) {
                double2 &o = ss[(m0 + j) * PT + pl];
                const double si = o.x, di = o.y;
                // (kD + gamma kS) / (4 pi)
                const double re = (sd[j] + gam_re * sr[j] - gam_im * si) * inv4pi;
                const double im = (di + gam_re * si + gam_im * sr[j]) * inv4pi;
                o = active ? make_double2(re * wj, im * wj) : make_double2(0.0, 0.0);
            }
    }
    __syncthreads();
    for (int i = tid; i < PT * (M + 1); i += 256) {
        const int q = i / (M + 1);
        if (pt0 + q < npts) kout[pt0 * (M + 1) + i] = ss[i % (M + 1) * PT + q];
    }
}

static void require_modal_size(int Nt, int M) {
    AXS_REQUIRE(Nt <= 16384 && (size_t)ModalSize(Nt, M).shared(4) * sizeof(double) <= 160 * 1024, AXS_EINVAL,
                "mode count or wavenumber too large for the modal kernel");
}

// Values of m = 0..M for npts points.  16 points a workgroup while two workgroups
// share a CU's LDS, else 4 (large kappa r or M); of 2, 3 and 4 values of m a thread the one that leaves the
// fewest turns idle.
static void modal_launch(Ctx &c, Pts pts, int64_t npts, int Nt, int M, double *f, double *scale, double *decay,
                         double kappa, double gam_re, double gam_im, double2 *kout) {
    const ModalSize z(Nt, M);
    const int PT = (size_t)z.shared(16) * sizeof(double) <= 80 * 1024 ? 16 : 4;
    const size_t shm = (size_t)z.shared(PT) * sizeof(double);
    require_modal_size(Nt, M);
    hipLaunchKernelGGL(toroidal_kernel, dim3(ceil_div(npts, 64)), dim3(64), 0, c.stream, pts, npts, z.nq, f, scale,
                       decay);
    AXS_HIP(hipGetLastError());
    int MB = 3;
    if (PT == 16) {
        double best = 1e300;
        for (int b : {4, 3, 2}) {
            const double cost = (double)ceil_div(M + 1, 16 * b) * (b + 1.5);   // the loads of c and the new pairs cost as much as 1.5 values
            if (cost < best) best = cost, MB = b;
        }
    }
    const dim3 grid((unsigned)ceil_div(npts, PT)), blk(256);
    if (PT == 4)
        hipLaunchKernelGGL((modal_kernel<4, 3>), grid, blk, shm, c.stream, pts, npts, Nt, M, f, scale, decay,
                           kappa, gam_re, gam_im, kout);
    else if (MB == 2)
        hipLaunchKernelGGL((modal_kernel<16, 2>), grid, blk, shm, c.stream, pts, npts, Nt, M, f, scale, decay,
                           kappa, gam_re, gam_im, kout);
    else if (MB == 3)
        hipLaunchKernelGGL((modal_kernel<16, 3>), grid, blk, shm, c.stream, pts, npts, Nt, M, f, scale, decay,
                           kappa, gam_re, gam_im, kout);
    else
        hipLaunchKernelGGL((modal_kernel<16, 4>), grid, blk, shm, c.stream, pts, npts, Nt, M, f, scale, decay,
                           kappa, gam_re, gam_im, kout);
    AXS_HIP(hipGetLastError());
}

// ---------------------------------------------------------------------------
// assembly of A~_m
// ---------------------------------------------------------------------------
__global__ void scatter_far_kernel(const FarDesc *__restrict__ pairs, int n, int p, int M,
                                   const ShapeRef *__restrict__ shapes, const double2 *__restrict__ kval) {
    int64_t idx = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (idx >= (int64_t)n * p * (M + 1)) return;
    const int o = (int)(idx / (M + 1)), m = (int)(idx % (M + 1));
    const FarDesc pr = pairs[o / p];
    const ShapeRef sh = shapes[pr.shape];
    sh.A[((int64_t)m * sh.NG + pr.i - sh.node0) * sh.NG + pr.P * p + o % p - sh.node0] = kval[idx];
}

// Entries of the near pairs: sum over a pair's points of the kernel values
// (M + 1 complex numbers a point: 2 (M + 1) rows) times the p basis values, on the FP64
// matrix cores, 16 rows per workgroup with the points split between its four
// wavefronts.  One thread per entry read every kernel value p times: 3 x 75 us for the
// three shapes of 8 mixed bodies, 14 now.  The target's own entry takes the 1/2 of 1/2 I + K.
__global__ __launch_bounds__(256) void near_reduce_kernel(const NearDesc *__restrict__ desc, int M, int p,
                                                          const ShapeRef *__restrict__ shapes,
                                                          const double2 *__restrict__ kval,
                                                          const double *__restrict__ lag, int64_t base) {
    __shared__ double s_acc[4][16][17];
    const NearDesc d = desc[blockIdx.x];
    const int per = d.n0 + d.n1, R = 2 * (M + 1), row0 = blockIdx.y * 16;
    const double *kv = (const double *)(kval + (base + d.first) * (M + 1));
    const double *lg = lag + (int64_t)d.first * p;
    const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63, g = lane >> 4, l16 = lane & 15;
    const bool row_in = row0 + l16 < R, col_in = l16 < p;
    const int row = min(row0 + l16, R - 1), col = min(l16, p - 1);
    gj_f64x4 acc = {0, 0, 0, 0};
    for (int q0 = wave * 16; q0 < per; q0 += 64) {
        double a[4], b[4];   // clamped, not conditional: eight loads in flight
#pragma unroll
        for (int u = 0; u < 4; ++u) {
            const int q = min(q0 + 4 * u + g, per - 1);
            a[u] = kv[(int64_t)q * R + row];
            b[u] = lg[q * p + col];
        }
#pragma unroll
        for (int u = 0; u < 4; ++u) {
            const bool in = q0 + 4 * u + g < per;
            acc = __builtin_amdgcn_mfma_f64_16x16x4f64(in && row_in ? a[u] : 0.0, in && col_in ? b[u] : 0.0, acc, 0, 0, 0);
        }
    }
#pragma unroll
    for (int v = 0; v < 4; ++v) s_acc[wave][g + 4 * v][l16] = acc[v];
    __syncthreads();
    const int comp = threadIdx.x & 1, j = (threadIdx.x >> 1) & 15, rl = 2 * (threadIdx.x >> 5) + comp;
    const int m = (row0 + rl) / 2;
    if (m <= M && j < p) {
        const ShapeRef sh = shapes[d.shape];
        double v = (s_acc[0][rl][j] + s_acc[1][rl][j]) + (s_acc[2][rl][j] + s_acc[3][rl][j]);
        if (comp == 0 && d.i == d.P * p + j) v += 0.5;
        ((double *)(sh.A + ((int64_t)m * sh.NG + d.i - sh.node0) * sh.NG + d.P * p + j - sh.node0))[comp] = v;
    }
}

// Inverses of all matrices (every shape, every mode) by in-place Gauss-Jordan
// elimination with partial pivoting (largest entry of the column among the rows
// not yet used as pivots; ties -> lowest row).  Rows are never moved: pivot row
// r_j belongs to column j, and the end result B gives A^{-1}[j][r_c] =
// B[r_j][c] (gj_finish_kernel).
//
// Blocked by GJB = 16 columns so that the work runs over the whole chip
// instead of one workgroup per matrix.  In the columns K of a block the
// elimination leaves T = A[:, K] (A[R, K])^{-1} with the pivot rows R holding
// the inverse itself and the others its negated product; all other columns
// then need A <- A (pivot rows zeroed) + T A_old[R, :], one product with an
// inner dimension of 16.  Products are summed up by themselves and then added to the
// entry, one rounding at its size per block, not 32: relative error of the inverses of
// 10 to 200 rows 4.5e-16 on average, 6.4e-16 with the entry as the sum's first term,
// 5.1e-16 by gauss_jordan_kernel.
//   gj_panel_kernel  - one workgroup per matrix, one row per thread held in
//                      registers; bound by its 16 serial steps (one barrier each:
//                      every wavefront offers its candidate row);
//   gj_update_kernel - a 16 x 16 tile per wavefront on the FP64 matrix cores,
//                      read from one copy of the matrix and written to the other
//                      (the pivot rows are read by every tile).
// 41 matrices of 200 x 200 (MI355X): 26 launches, 0.51 ms (13 x 25 us + 13 x 14
// us); one workgroup per matrix over global memory took 19.97 ms.  Blocks of 32
// columns: 7 x 69 + 7 x 19 us (a panel step reads and writes twice as much LDS).
struct GJItem {
    const double2 *A;   // NG x NG, row-major
    double2 *b0, *b1;   // two copies of NG x NG the blocks alternate between
    double2 *T;         // NG x GJB
    int32_t *prow;      // [NG] pivot row of each column
    int32_t *col;       // [NG] column of each row, -1 while it is no pivot
    double2 *S;         // NG x NG, row-major: A^{-1}
    int32_t NG, pad;
};
constexpr int GJB = 16;
constexpr int GJ_ROWS = 1024;   // one thread per row: larger matrices take gauss_jordan_kernel

__device__ __forceinline__ const double2 *gj_src(const GJItem &it, int step) {
    return step == 0 ? it.A : (step & 1) ? it.b0 : it.b1;
}

// largest x of the wavefront, by moves between neighbouring lanes (ds_bpermute takes
// ten times as long in this chain)
__device__ __forceinline__ int wave_max(int x) {
    x = max(x, __builtin_amdgcn_update_dpp(x, x, 0x111, 0xf, 0xf, false));   // row_shr:1
    x = max(x, __builtin_amdgcn_update_dpp(x, x, 0x112, 0xf, 0xf, false));   // row_shr:2
    x = max(x, __builtin_amdgcn_update_dpp(x, x, 0x114, 0xf, 0xf, false));   // row_shr:4
    x = max(x, __builtin_amdgcn_update_dpp(x, x, 0x118, 0xf, 0xf, false));   // row_shr:8
    x = max(x, __builtin_amdgcn_update_dpp(x, x, 0x142, 0xf, 0xf, false));   // row_bcast:15
    x = max(x, __builtin_amdgcn_update_dpp(x, x, 0x143, 0xf, 0xf, false));   // row_bcast:31
    return __builtin_amdgcn_readlane(x, 63);
}

template <int BS>
__global__ __launch_bounds__(BS) void gj_panel_kernel(const GJItem *__restrict__ items, int step) {
    const GJItem it = items[blockIdx.x];
    const int NG = it.NG, k0 = step * GJB;
    if (k0 >= NG) return;
    const int nb = min(GJB, NG - k0);
    const int r = threadIdx.x, lane = r & 63, wave = r >> 6;
    constexpr int NW = BS / 64;
    __shared__ int s_max[2][NW], s_row[2][NW];
    __shared__ double2 s_cand[2][NW][GJB];   // each wavefront's candidate row
    const bool live = r < NG;
    // clamped, not conditional, so that all loads are in flight together
    const double2 *src = gj_src(it, step) + (int64_t)min(r, NG - 1) * NG + k0;
    double ar[GJB], ai[GJB];
#pragma unroll
    for (int j = 0; j < GJB; ++j) {
        const double2 v = src[min(j, nb - 1)];
        ar[j] = v.x;
        ai[j] = v.y;
    }
    int mycol = step == 0 ? -1 : it.col[min(r, NG - 1)];
    if (!live) mycol = 0;
    // The column of a step is always the first register, and every step moves the row
    // on by one, in the assignments it makes anyway: a rolled loop with constant
    // indices (unrolled, its 40 KB of code are fetched as slowly as they are run).
    // Steps past the last column only move the row.
#pragma unroll 1
    for (int c = 0; c < GJB; ++c) {
        // the upper half of |a|^2 orders the candidates to 1e-6, plenty for a pivot
        int mag = -1;
        if (mycol < 0) {
            const double v = ar[0] * ar[0] + ai[0] * ai[0];
            mag = v >= 0.0 ? __double2hiint(v) : 0;   // NaN: the result is NaN whatever the pivot
        }
        const int wm = wave_max(mag);
        const int first = __ffsll((unsigned long long)__ballot(mag == wm)) - 1;
        if (lane == first) {
            s_max[c & 1][wave] = wm;
            s_row[c & 1][wave] = r;
#pragma unroll
            for (int j = 0; j < GJB; ++j) s_cand[c & 1][wave][j] = make_double2(ar[j], ai[j]);
        }
        __syncthreads();
        int best = s_max[c & 1][0], bw = 0;
#pragma unroll
        for (int w = 1; w < NW; ++w)
            if (s_max[c & 1][w] > best) {
                best = s_max[c & 1][w];
                bw = w;
            }
        const bool step_in = c < nb, mine = step_in && r == s_row[c & 1][bw];
        const double2 *u = s_cand[c & 1][bw];
        const double2 pv = u[0];
        const double den = 1.0 / (pv.x * pv.x + pv.y * pv.y);
        const double vr = pv.x * den, vi = -pv.y * den;   // 1 / pivot
        // row r: a - f u with f = a_0 / pivot, -f in the column itself; pivot row:
        // u / pivot, 1 / pivot in the column, which is 0 - g u with g = -1 / pivot
        double fr = ar[0] * vr - ai[0] * vi, fi = ar[0] * vi + ai[0] * vr;
        if (mine) {
            fr = -vr;
            fi = -vi;
            mycol = k0 + c;
        }
        const double a0r = step_in ? -fr : ar[0], a0i = step_in ? -fi : ai[0];
        if (!step_in) fr = fi = 0.0;
#pragma unroll
        for (int j = 1; j < GJB; ++j) {
            const double2 x = u[j];
            ar[j - 1] = (mine ? 0.0 : ar[j]) - fma(fr, x.x, -(fi * x.y));
            ai[j - 1] = (mine ? 0.0 : ai[j]) - fma(fr, x.y, fi * x.x);
        }
        ar[GJB - 1] = a0r;
        ai[GJB - 1] = a0i;
    }
    if (!live) return;
    it.col[r] = mycol;
    if (mycol >= k0) it.prow[mycol] = r;   // here, not in the loop, whose barriers would wait for the store
#pragma unroll
    for (int j = 0; j < GJB; ++j) it.T[(int64_t)r * GJB + j] = make_double2(ar[j], ai[j]);
}

__global__ __launch_bounds__(256) void gj_update_kernel(const GJItem *__restrict__ items, int step) {
    const GJItem it = items[blockIdx.z];
    const int NG = it.NG, k0 = step * GJB;
    if (k0 >= NG) return;
    const int nb = min(GJB, NG - k0);
    const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63, q = lane >> 4;
    const int r0 = blockIdx.y * 32 + (wave >> 1) * 16, c0 = blockIdx.x * 32 + (wave & 1) * 16;
    if (r0 >= NG || c0 >= NG) return;
    const double2 *src = gj_src(it, step);
    double2 *dst = (step & 1) ? it.b1 : it.b0;
    const int col = c0 + (lane & 15);
    if (c0 == k0) {   // the block's own columns
#pragma unroll
        for (int v = 0; v < 4; ++v) {
            const int row = r0 + q + 4 * v;
            if (row < NG && col < NG) dst[(int64_t)row * NG + col] = it.T[(int64_t)row * GJB + (lane & 15)];
        }
        return;
    }
    // rows and columns past the edge are clamped and not stored: no load waits for a branch
    const int colc = min(col, NG - 1);
    gj_f64x4 accr = {0, 0, 0, 0}, acci = {0, 0, 0, 0};
    double2 own[4];
#pragma unroll
    for (int v = 0; v < 4; ++v) {
        const int row = min(r0 + q + 4 * v, NG - 1);
        own[v] = src[(int64_t)row * NG + colc];
        if (it.col[row] >= k0) own[v] = make_double2(0.0, 0.0);   // a pivot row of this block
    }
    const int arow = min(r0 + (lane & 15), NG - 1);
#pragma unroll
    for (int k = 0; k < GJB; k += 4) {
        double2 a = it.T[(int64_t)arow * GJB + k + q];
        double2 b = src[(int64_t)it.prow[k0 + min(k + q, nb - 1)] * NG + colc];
        if (k + q >= nb) a = b = make_double2(0.0, 0.0);
        accr = __builtin_amdgcn_mfma_f64_16x16x4f64(a.x, b.x, accr, 0, 0, 0);
        acci = __builtin_amdgcn_mfma_f64_16x16x4f64(a.x, b.y, acci, 0, 0, 0);
        accr = __builtin_amdgcn_mfma_f64_16x16x4f64(-a.y, b.y, accr, 0, 0, 0);
        acci = __builtin_amdgcn_mfma_f64_16x16x4f64(a.y, b.x, acci, 0, 0, 0);
    }
#pragma unroll
    for (int v = 0; v < 4; ++v) {
        const int row = r0 + q + 4 * v;
        if (row < NG && col < NG) dst[(int64_t)row * NG + col] = make_double2(own[v].x + accr[v], own[v].y + acci[v]);
    }
}

// S[j][r_c] = B[r_j][c]
__global__ __launch_bounds__(256) void gj_finish_kernel(const GJItem *__restrict__ items) {
    const GJItem it = items[blockIdx.y];
    const int NG = it.NG;
    const int64_t t = (int64_t)blockIdx.x * 256 + threadIdx.x;
    if (t >= (int64_t)NG * NG) return;
    const int j = (int)(t / NG), c = (int)(t % NG);
    const double2 *B = gj_src(it, (NG + GJB - 1) / GJB);
    it.S[(int64_t)j * NG + it.prow[c]] = B[(int64_t)it.prow[j] * NG + c];
}

// Gauss-Jordan inverse with partial pivoting (ties -> lowest row), one block
// per matrix, in global memory: matrices of more than GJ_ROWS rows, which one
// workgroup of the blocked elimination cannot hold at a row per thread.  The
// work array (NG x 2 NG) is b0 followed by b1.
template <int BS>
__global__ __launch_bounds__(BS) void gauss_jordan_kernel(const GJItem *__restrict__ items) {
    const GJItem it = items[blockIdx.x];
    const int NG = it.NG;
    const int W = 2 * NG;
    const double2 *a = it.A;
    double2 *g = it.b0;
    double2 *s = it.S;
    __shared__ double rmax[BS];
    __shared__ int ridx[BS];
    __shared__ double2 piv_inv;
    extern __shared__ double2 fac[];   // [NG]
    for (int64_t t = threadIdx.x; t < (int64_t)NG * W; t += BS) {
        const int r = (int)(t / W), c = (int)(t % W);
        g[t] = c < NG ? a[(int64_t)r * NG + c] : make_double2(c - NG == r ? 1.0 : 0.0, 0.0);
    }
    __syncthreads();
    for (int k = 0; k < NG; ++k) {
        double best = -1.0;
        int bi = k;
        for (int r = k + threadIdx.x; r < NG; r += BS) {
            const double2 v = g[(int64_t)r * W + k];
            const double mag = fabs(v.x) + fabs(v.y) > 0 ? hypot(v.x, v.y) : 0.0;
            if (mag > best) {
                best = mag;
                bi = r;
            }
        }
        rmax[threadIdx.x] = best;
        ridx[threadIdx.x] = bi;
        __syncthreads();
        for (int o = BS / 2; o > 0; o >>= 1) {
            if (threadIdx.x < o) {
                const double b2 = rmax[threadIdx.x + o];
                const int i2 = ridx[threadIdx.x + o];
                if (b2 > rmax[threadIdx.x] || (b2 == rmax[threadIdx.x] && i2 < ridx[threadIdx.x])) {
                    rmax[threadIdx.x] = b2;
                    ridx[threadIdx.x] = i2;
                }
            }
            __syncthreads();
        }
        const int pr = ridx[0];
        if (pr != k) {
            for (int c = k + threadIdx.x; c < W; c += BS) {
                const double2 t0 = g[(int64_t)k * W + c];
                g[(int64_t)k * W + c] = g[(int64_t)pr * W + c];
                g[(int64_t)pr * W + c] = t0;
            }
        }
        __syncthreads();
        if (threadIdx.x == 0) {
            const double2 pv = g[(int64_t)k * W + k];
            const double den = pv.x * pv.x + pv.y * pv.y;
            piv_inv = make_double2(pv.x / den, -pv.y / den);
        }
        __syncthreads();
        const double2 pinv = piv_inv;
        for (int c = k + threadIdx.x; c < W; c += BS) {
            const double2 v = g[(int64_t)k * W + c];
            g[(int64_t)k * W + c] = make_double2(v.x * pinv.x - v.y * pinv.y, v.x * pinv.y + v.y * pinv.x);
        }
        for (int r = threadIdx.x; r < NG; r += BS) fac[r] = g[(int64_t)r * W + k];
        __syncthreads();
        for (int64_t t = threadIdx.x; t < (int64_t)NG * (W - k); t += BS) {
            const int r = (int)(t / (W - k)), c = k + (int)(t % (W - k));
            if (r == k) continue;
            const double2 f = fac[r], u = g[(int64_t)k * W + c];
            double2 v = g[(int64_t)r * W + c];
            v.x -= f.x * u.x - f.y * u.y;
            v.y -= f.x * u.y + f.y * u.x;
            g[(int64_t)r * W + c] = v;
        }
        __syncthreads();
    }
    for (int64_t t = threadIdx.x; t < (int64_t)NG * NG; t += BS) {
        const int r = (int)(t / NG), c = (int)(t % NG);
        s[t] = g[(int64_t)r * W + NG + c];
    }
}

// Planar column-major copies (element (i, k) at k NG + i) of the matrices, S_m in FP64 and
// FP32 and A~_m (where given) in FP64: 32 x 32 tiles turned in LDS, so that
// reads and writes both run along rows (without, the reads of 41 matrices of 200 x 200
// took 28 us of each 29 us launch).
__global__ __launch_bounds__(256) void split_planar_kernel(const PlanarMat *__restrict__ mats, double *__restrict__ s64r,
                                                           double *__restrict__ s64i, float *__restrict__ s32r,
                                                           float *__restrict__ s32i, double *__restrict__ a64r,
                                                           double *__restrict__ a64i) {
    __shared__ double2 tile[32][33];
    const PlanarMat mt = mats[blockIdx.x];
    const int NG = mt.NG, nt = (NG + 31) / 32, x = threadIdx.x & 31, y = threadIdx.x >> 5;
    for (int t = blockIdx.y; t < nt * nt; t += gridDim.y) {
        const int i0 = t / nt * 32, k0 = t % nt * 32;
        for (int which = 0; which < (mt.A ? 2 : 1); ++which) {
            const double2 *src = which ? mt.A : mt.S;
            __syncthreads();
#pragma unroll
            for (int q = 0; q < 32; q += 8)
                if (i0 + y + q < NG && k0 + x < NG) tile[y + q][x] = src[(int64_t)(i0 + y + q) * NG + k0 + x];
            __syncthreads();
#pragma unroll
            for (int q = 0; q < 32; q += 8) {
                if (k0 + y + q >= NG || i0 + x >= NG) continue;
                const double2 v = tile[x][y + q];
                const int64_t o = mt.off + (int64_t)(k0 + y + q) * NG + i0 + x;
                if (which) {
                    a64r[o] = v.x;
                    a64i[o] = v.y;
                } else {
                    s64r[o] = v.x;
                    s64i[o] = v.y;
                    s32r[o] = (float)v.x;
                    s32i[o] = (float)v.y;
                }
            }
        }
    }
}

// ---------------------------------------------------------------------------
// host: Gauss-Legendre rule by Newton's method on the three-term recurrence
// ---------------------------------------------------------------------------
void gauss_legendre_rule(int n, std::vector<double> &x, std::vector<double> &w);
static void gauss_legendre(int n, std::vector<double> &x, std::vector<double> &w) { gauss_legendre_rule(n, x, w); }
void gauss_legendre_rule(int n, std::vector<double> &x, std::vector<double> &w) {
    x.assign(n, 0.0);
    w.assign(n, 0.0);
    for (int i = 0; i < n; ++i) {
        double t = std::cos(M_PI * (i + 0.75) / (n + 0.5));
        for (int it = 0; it < 100; ++it) {
            double p0 = 1.0, p1 = t;
            for (int k = 2; k <= n; ++k) {
                double p2 = ((2.0 * k - 1.0) * t * p1 - (k - 1.0) * p0) / k;
                p0 = p1;
                p1 = p2;
            }
            double dp = n * (t * p1 - p0) / (t * t - 1.0);
            double dt = p1 / dp;
            t -= dt;
            if (std::fabs(dt) < 1e-16) {
                // final derivative at the converged root
                p0 = 1.0;
                p1 = t;
                for (int k = 2; k <= n; ++k) {
                    double p2 = ((2.0 * k - 1.0) * t * p1 - (k - 1.0) * p0) / k;
                    p0 = p1;
                    p1 = p2;
                }
                dp = n * (t * p1 - p0) / (t * t - 1.0);
                break;
            }
        }
        double p0 = 1.0, p1 = t;
        for (int k = 2; k <= n; ++k) {
            double p2 = ((2.0 * k - 1.0) * t * p1 - (k - 1.0) * p0) / k;
            p0 = p1;
            p1 = p2;
        }
        double dp = n * (t * p1 - p0) / (t * t - 1.0);
        x[n - 1 - i] = t;                    // ascending
        w[n - 1 - i] = 2.0 / ((1.0 - t * t) * dp * dp);
    }
}

void gauss_legendre_public(int n, std::vector<double> &x, std::vector<double> &w) { gauss_legendre(n, x, w); }

static double interp_at(const std::vector<double> &sn, const double *f, int p, double s) {
    double v = 0;
    for (int j = 0; j < p; ++j) {
        double l = 1.0;
        for (int k = 0; k < p; ++k)
            if (k != j) l *= (s - sn[k]) / (sn[j] - sn[k]);
        v += l * f[j];
    }
    return v;
}

static int modal_nt(const Shape &s) {
    double rmax = 1e-3;
    for (double v : s.r) rmax = std::max(rmax, v);
    double need = 4.0 * s.kappa * rmax + 64.0;
    int nt = 64;
    while (nt < need) nt += 64;
    return nt;
}

// the evaluation points of shapes set up together: what their launches need, with
// the offsets of the tables in the upload
struct ShapePlan {
    Shape all;        // contour nodes of all of them (p, M, Nt, kappa and eta are common)
    size_t tab = 0, refs = 0;   // the doubles below and the shapes' rules, in one array; the ShapeRefs
    size_t o_sn = 0, o_lden = 0, o_r = 0, o_z = 0, o_nr = 0, o_nz = 0, o_aw = 0, o_rd = 0, o_zd = 0;
    struct Batch {   // target rows
        size_t far = 0, near = 0;
        int nfar = 0, nd = 0;
        int64_t nnear = 0;
    };
    std::vector<Batch> batches;
};

static ShapePlan plan_shapes(const std::vector<Shape *> &shapes, Upload &up) {
    ShapePlan plan;
    Shape &s = plan.all;
    s = *shapes[0];
    std::vector<ShapeRef> refs;
    std::vector<int> shape_of, first_panel;   // of each panel; of each shape, and one past the last
    s.NG = s.n_panels = 0;
    for (auto *v : {&s.r, &s.z, &s.dr, &s.dz, &s.gw}) v->clear();
    for (auto *q : shapes) {
        refs.push_back(ShapeRef{(double2 *)q->A64, q->NG, s.NG, 0, 0, 0, 0});
        first_panel.push_back(s.n_panels);
        shape_of.resize(s.n_panels + q->n_panels, (int)refs.size() - 1);
        s.NG += q->NG;
        s.n_panels += q->n_panels;
        s.r.insert(s.r.end(), q->r.begin(), q->r.end());
        s.z.insert(s.z.end(), q->z.begin(), q->z.end());
        s.dr.insert(s.dr.end(), q->dr.begin(), q->dr.end());
        s.dz.insert(s.dz.end(), q->dz.begin(), q->dz.end());
        s.gw.insert(s.gw.end(), q->gw.begin(), q->gw.end());
    }
    first_panel.push_back(s.n_panels);
    const int NG = s.NG, p = s.p, np_ = s.n_panels;

    std::vector<double> sn, sw;
    gauss_legendre(p, sn, sw);
    std::vector<double> lden(p);
    for (int j = 0; j < p; ++j) {
        double d = 1.0;
        for (int k = 0; k < p; ++k)
            if (k != j) d *= (sn[j] - sn[k]);
        lden[j] = 1.0 / d;
    }
    // node data
    std::vector<double> nr(NG), nz(NG), aw(NG), plen(np_, 0.0), smax(np_, 0.0);
    for (int i = 0; i < NG; ++i) {
        const double sp = std::hypot(s.dr[i], s.dz[i]);
        nr[i] = -s.dz[i] / sp;
        nz[i] = s.dr[i] / sp;
        aw[i] = s.r[i] * sp * s.gw[i];
        plen[i / p] += sp * s.gw[i];
        smax[i / p] = std::max(smax[i / p], sp);
    }
    std::vector<double> hc;   // the table of constants
    auto put = [&](const std::vector<double> &v) {
        const size_t o = hc.size();
        hc.insert(hc.end(), v.begin(), v.end());
        return o;
    };
    // every shape's rules by its own panels, so that its matrices are the same beside any
    // other shape; shapes of one rule share it
    std::vector<double> qu, qw;
    gauss_legendre(OWN_NQ, qu, qw);
    for (size_t k = 0; k < refs.size(); ++k) {
        const double longest = *std::max_element(plen.begin() + first_panel[k], plen.begin() + first_panel[k + 1]);
        const int ngl = level_points(p, s.kappa * longest);
        for (size_t o = 0; o < k; ++o)
            if (refs[o].ngl == ngl) refs[k].gl = refs[o].gl, refs[k].own = refs[o].own;
        refs[k].ngl = ngl;
        if (refs[k].own > 0) continue;
        std::vector<double> gu, gw, ownx, ownw;
        gauss_legendre(ngl, gu, gw);
        // the own-panel rule on [0, 1], singular at 0
        for (int lev = 0; lev < OWN_LEV; ++lev)
            for (int q = 0; q < ngl; ++q) {
                const double half = std::ldexp(0.25, -lev);   // half of [2^-(lev + 1), 2^-lev]
                ownx.push_back(2.0 * half + half * (gu[q] + 1.0));
                ownw.push_back(half * gw[q]);
            }
        for (int q = 0; q < OWN_NQ; ++q) {
            const double u = 0.5 * (qu[q] + 1.0), h = std::ldexp(1.0, -OWN_LEV);
            ownx.push_back(h * std::pow(u, OWN_Q));
            ownw.push_back(h * OWN_Q * std::pow(u, OWN_Q - 1) * 0.5 * qw[q]);
        }
        refs[k].gl = (int32_t)put(gu);
        put(gw);
        refs[k].own = (int32_t)put(ownx);
        put(ownw);
    }
    plan.refs = up.put(refs);
    // derivative of every panel's interpolant at its nodes
    std::vector<double> rd(NG, 0.0), zd(NG, 0.0);
    for (int i = 0; i < NG; ++i) {
        const int P0 = i / p * p, a = i - P0;
        for (int k = 0; k < p; ++k) {
            if (k == a) continue;
            const double w = lden[k] / (lden[a] * (sn[a] - sn[k]));
            rd[i] += w * (s.r[P0 + k] - s.r[i]);
            zd[i] += w * (s.z[P0 + k] - s.z[i]);
        }
    }
    // near panels and split points per target (host geometry)
    std::vector<std::vector<NearDesc>> near(NG);
    std::vector<double> endr(2 * np_), endz(2 * np_);
    for (int P = 0; P < np_; ++P) {
        endr[2 * P] = interp_at(sn, &s.r[P * p], p, -1.0);
        endr[2 * P + 1] = interp_at(sn, &s.r[P * p], p, 1.0);
        endz[2 * P] = interp_at(sn, &s.z[P * p], p, -1.0);
        endz[2 * P + 1] = interp_at(sn, &s.z[P * p], p, 1.0);
    }
    // circles around the panels' nodes and ends: most panels are beyond their length
    // from a target by these alone
    std::vector<double> cr(np_), cz(np_), crad(np_, 0.0);
    for (int P = 0; P < np_; ++P) {
        cr[P] = 0.5 * (endr[2 * P] + endr[2 * P + 1]);
        cz[P] = 0.5 * (endz[2 * P] + endz[2 * P + 1]);
        for (int k = -2; k < p; ++k) {
            const double a = k < 0 ? endr[2 * P + k + 2] : s.r[P * p + k], b = k < 0 ? endz[2 * P + k + 2] : s.z[P * p + k];
            crad[P] = std::max(crad[P], std::hypot(a - cr[P], b - cz[P]));
        }
    }
    // points on one side (length Ls in s) of a panel at distance d: halve until
    // the innermost interval is shorter than d / 8
    auto side_points = [&](double Ls, double d, double speed, int ngl) {
        if (!(Ls > 1e-14)) return 0;
        int n = 1;
        while (n < MAX_LEV && std::ldexp(Ls, 1 - n) * speed > 0.125 * d) ++n;
        return n * ngl;
    };
    for (int i = 0; i < NG; ++i) {
        const int own = i / p, sh = shape_of[own];
        for (int P = first_panel[sh]; P < first_panel[sh + 1]; ++P) {
            const double lim = (plen[P] + crad[P]) * (1.0 + 1e-12), ca = cr[P] - s.r[i], cb = cz[P] - s.z[i];
            if (std::abs(P - own) > 1 && ca * ca + cb * cb > lim * lim) continue;
            double best2 = 1e300, bs = 0;
            auto consider = [&](double rr, double zz, double sv) {
                const double a = rr - s.r[i], b = zz - s.z[i], d2 = a * a + b * b;
                if (d2 < best2) {
                    best2 = d2;
                    bs = sv;
                }
            };
            consider(endr[2 * P], endz[2 * P], -1.0);
            for (int k = 0; k < p; ++k) consider(s.r[P * p + k], s.z[P * p + k], sn[k]);
            consider(endr[2 * P + 1], endz[2 * P + 1], 1.0);
            const double best = std::sqrt(best2);
            const bool is_near = std::abs(P - own) <= 1 || best < plen[P];
            if (!is_near) continue;
            NearDesc d{};
            d.i = i;
            d.P = P;
            d.shape = sh;
            if (P == own) {
                d.sstar = sn[i - own * p];
                d.n0 = d.n1 = own_pts(refs[sh].ngl);
            } else {
                d.sstar = bs;
                d.n0 = side_points(bs + 1.0, best, smax[P], refs[sh].ngl);
                d.n1 = side_points(1.0 - bs, best, smax[P], refs[sh].ngl);
            }
            near[i].push_back(d);
        }
    }
    plan.o_sn = put(sn), plan.o_lden = put(lden), plan.o_r = put(s.r), plan.o_z = put(s.z), plan.o_nr = put(nr),
    plan.o_nz = put(nz), plan.o_aw = put(aw), plan.o_rd = put(rd), plan.o_zd = put(zd);
    plan.tab = up.put(hc);
    // batches of target rows, bounded number of evaluation points
    const int64_t max_pts = 1 << 19;
    int i0 = 0;
    while (i0 < NG) {
        int i1 = i0;
        int64_t npts = 0;
        std::vector<FarDesc> far;
        std::vector<NearDesc> nd;
        int64_t nnear = 0;
        while (i1 < NG) {
            const int sh = shape_of[i1 / p], P0 = first_panel[sh], P1 = first_panel[sh + 1];
            int64_t add = (int64_t)(P1 - P0 - (int)near[i1].size()) * p;
            for (auto &d : near[i1]) add += d.n0 + d.n1;
            if (i1 > i0 && npts + add > max_pts) break;
            npts += add;
            size_t k = 0;
            for (int P = P0; P < P1; ++P) {
                if (k < near[i1].size() && near[i1][k].P == P) {
                    NearDesc d = near[i1][k++];
                    d.first = (int32_t)nnear;
                    nnear += d.n0 + d.n1;
                    nd.push_back(d);
                } else {
                    far.push_back(FarDesc{i1, P, sh});
                }
            }
            ++i1;
        }
        ShapePlan::Batch bt;
        bt.nfar = (int)far.size();
        bt.nd = (int)nd.size();
        bt.nnear = nnear;
        bt.far = up.put(far);
        bt.near = up.put(nd);
        plan.batches.push_back(bt);
        i0 = i1;
    }
    return plan;
}

// A~_m of these shapes (every entry is written), queued without synchronisation
static void run_shapes(Ctx &c, const ShapePlan &plan, const Upload &up) {
    const Shape &s = plan.all;
    const int p = s.p, M = s.M, Nt = s.Nt, nq = M + Nt / 2;
    const double *dc = up.at<double>(plan.tab);
    const ShapeRef *refs = up.at<ShapeRef>(plan.refs);
    for (auto &bt : plan.batches) {
        const int64_t nfar = (int64_t)bt.nfar * p, nnear = bt.nnear, P = nfar + nnear;
        const FarDesc *d_far = up.at<FarDesc>(bt.far);
        const NearDesc *d_nd = up.at<NearDesc>(bt.near);
        // point storage
        double *pbuf = (double *)c.scratch(WS_MISC, ((size_t)P * 9 + (size_t)nnear * p) * sizeof(double));
        Pts pts{pbuf, pbuf + P, pbuf + 2 * P, pbuf + 3 * P, pbuf + 4 * P, pbuf + 5 * P, pbuf + 6 * P, pbuf + 9 * P};
        double *qv = (double *)c.scratch(WS_TMP, (size_t)P * nq * sizeof(double));
        double2 *kv = (double2 *)c.scratch(WS_TMP3, (size_t)P * (M + 1) * sizeof(double2));
        if (nfar) {
            hipLaunchKernelGGL(gen_far_kernel, dim3(ceil_div(nfar, 256)), dim3(256), 0, c.stream, d_far, bt.nfar, p,
                               dc + plan.o_r, dc + plan.o_z, dc + plan.o_nr, dc + plan.o_nz, dc + plan.o_aw, pts);
            AXS_HIP(hipGetLastError());
        }
        // a target's own panel is always near, so no batch is without near points
        hipLaunchKernelGGL(gen_near_kernel, dim3(bt.nd), dim3(128), 0, c.stream, d_nd, p, dc + plan.o_sn,
                           dc + plan.o_lden, refs, dc, dc + plan.o_r, dc + plan.o_z, dc + plan.o_rd, dc + plan.o_zd, pts, nfar);
        AXS_HIP(hipGetLastError());
        modal_launch(c, pts, P, Nt, M, qv, pbuf + 7 * P, pbuf + 8 * P, s.kappa, s.kappa > 0 ? 0.0 : s.eta,
                     s.kappa > 0 ? s.eta : 0.0, kv);
        if (nfar) {
            hipLaunchKernelGGL(scatter_far_kernel, dim3(ceil_div(nfar * (M + 1), 256)), dim3(256), 0, c.stream, d_far,
                               bt.nfar, p, M, refs, kv);
            AXS_HIP(hipGetLastError());
        }
        hipLaunchKernelGGL(near_reduce_kernel, dim3(bt.nd, (unsigned)ceil_div(2 * (M + 1), 16)), dim3(256), 0, c.stream,
                           d_nd, M, p, refs, kv, pts.lag, nfar);
        AXS_HIP(hipGetLastError());
    }
}

// give back blocks that queued kernels may still read
static void release(Ctx &c, std::vector<void *> &blocks) {
    AXS_HIP(hipStreamSynchronize(c.stream));
    for (void *p : blocks) c.dfree(p);
    blocks.clear();
}

// S_m = A~_m^{-1} for every shape and mode, in groups of shapes whose work
// arrays (about NG x 2 NG per matrix) stay within 4 GiB.  Per group one launch
// sequence over all its matrices: two launches per 16 columns, or one launch of
// gauss_jordan_kernel where a matrix has more rows than a workgroup has threads.
static void invert_shapes(Ctx &c, std::vector<std::unique_ptr<Upload>> &keep, std::vector<void *> &done) {
    constexpr size_t WORK_CAP = (size_t)4 << 30;
    auto per = [](const Shape &s) {   // work bytes per matrix
        return ((size_t)2 * s.NG * s.NG + (size_t)GJB * s.NG) * sizeof(double2) + (size_t)2 * s.NG * sizeof(int32_t);
    };
    size_t k = 0;
    while (k < c.shapes.size()) {
        size_t k1 = k, bytes = 0, nmat = 0;
        int maxNG = 0;
        const bool blocked = c.shapes[k].NG <= GJ_ROWS;
        while (k1 < c.shapes.size()) {
            const Shape &s = c.shapes[k1];
            const size_t b = (size_t)(s.M + 1) * per(s);
            if (k1 > k && (bytes + b > WORK_CAP || (s.NG <= GJ_ROWS) != blocked || nmat + s.M + 1 > 65535)) break;
            bytes += b;
            nmat += s.M + 1;
            maxNG = std::max(maxNG, s.NG);
            ++k1;
        }
        char *work = (char *)c.dalloc(bytes);
        std::vector<GJItem> items;
        size_t off = 0;
        for (size_t q = k; q < k1; ++q) {
            Shape &s = c.shapes[q];
            const int64_t nn = (int64_t)s.NG * s.NG;
            double2 *S = (double2 *)s.S64;
            for (int m = 0; m <= s.M; ++m) {
                GJItem g{};
                g.A = (const double2 *)s.A64 + m * nn;
                g.b0 = (double2 *)(work + off);
                g.b1 = g.b0 + nn;
                g.T = g.b1 + nn;
                g.S = S + m * nn;
                g.NG = s.NG;
                off += ((size_t)2 * nn + (size_t)GJB * s.NG) * sizeof(double2);
                items.push_back(g);
            }
        }
        for (auto &g : items) {
            g.prow = (int32_t *)(work + off);
            g.col = g.prow + g.NG;
            off += (size_t)2 * g.NG * sizeof(int32_t);
        }
        keep.emplace_back(new Upload(c));
        Upload &up = *keep.back();
        const size_t o_items = up.put(items);
        up.commit();
        const GJItem *d_items = up.at<GJItem>(o_items);
        const unsigned n = (unsigned)items.size();
        if (blocked) {
            const unsigned t32 = (unsigned)ceil_div(maxNG, 32);
            const int steps = (int)ceil_div(maxNG, GJB);
            for (int st = 0; st < steps; ++st) {
                if (maxNG <= 64)
                    hipLaunchKernelGGL(gj_panel_kernel<64>, dim3(n), dim3(64), 0, c.stream, d_items, st);
                else if (maxNG <= 256)
                    hipLaunchKernelGGL(gj_panel_kernel<256>, dim3(n), dim3(256), 0, c.stream, d_items, st);
                else if (maxNG <= 512)
                    hipLaunchKernelGGL(gj_panel_kernel<512>, dim3(n), dim3(512), 0, c.stream, d_items, st);
                else
                    hipLaunchKernelGGL(gj_panel_kernel<GJ_ROWS>, dim3(n), dim3(GJ_ROWS), 0, c.stream, d_items, st);
                hipLaunchKernelGGL(gj_update_kernel, dim3(t32, t32, n), dim3(256), 0, c.stream, d_items, st);
            }
            hipLaunchKernelGGL(gj_finish_kernel, dim3((unsigned)ceil_div((int64_t)maxNG * maxNG, 256), n), dim3(256), 0,
                               c.stream, d_items);
        } else {
            hipLaunchKernelGGL(gauss_jordan_kernel<256>, dim3(n), dim3(256), maxNG * sizeof(double2), c.stream, d_items);
        }
        AXS_HIP(hipGetLastError());
        done.push_back(up.dev);
        done.push_back(work);
        k = k1;
        if (k < c.shapes.size()) release(c, done);   // one group's work array at a time
    }
}

void precompute_shapes(Ctx &c) {
    std::vector<std::unique_ptr<Upload>> keep;   // host copies and device blocks, until the synchronisation
    std::vector<void *> done;
    keep.emplace_back(new Upload(c));
    Upload &up = *keep.back();
    // the matrices of all shapes in one block each, in the shapes' order
    size_t total = 0;
    for (auto &s : c.shapes) {
        AXS_REQUIRE(s.p <= PMAX, AXS_EINVAL, "at most 16 nodes per panel are supported");
        s.Nt = modal_nt(s);
        require_modal_size(s.Nt, s.M);   // before anything is allocated or queued
        total += (size_t)(s.M + 1) * s.NG * s.NG;
    }
    double2 *A = (double2 *)c.dalloc(total * sizeof(double2)), *S = (double2 *)c.dalloc(total * sizeof(double2));
    size_t off = 0;
    for (auto &s : c.shapes) {
        s.A64 = (double *)(A + off);
        s.S64 = (double *)(S + off);
        off += (size_t)(s.M + 1) * s.NG * s.NG;
    }
    std::vector<ShapePlan> plans;
    std::vector<char> taken(c.shapes.size(), 0);
    for (size_t k = 0; k < c.shapes.size(); ++k) {
        if (taken[k]) continue;
        std::vector<Shape *> group;
        for (size_t q = k; q < c.shapes.size(); ++q) {
            const Shape &a = c.shapes[k], &b = c.shapes[q];
            if (b.p != a.p || b.M != a.M || b.Nt != a.Nt || b.kappa != a.kappa || b.eta != a.eta) continue;
            taken[q] = 1;
            group.push_back(&c.shapes[q]);
        }
        plans.push_back(plan_shapes(group, up));
    }
    up.commit();
    for (auto &plan : plans) run_shapes(c, plan, up);
    done.push_back(up.dev);
    invert_shapes(c, keep, done);
    release(c, done);
    for (auto &k : keep) k->pending = false;
}

void modal_values(Ctx &c, double kappa, double gam_re, double gam_im, int M, int Nt,
                  const std::vector<double> &h, int64_t P, double2 *kout) {
    const int nq = M + Nt / 2;
    double *pbuf = (double *)c.scratch(WS_MISC, (size_t)P * 9 * sizeof(double));
    copy_in(c, pbuf, h.data(), (size_t)P * 7 * sizeof(double));
    Pts pts{pbuf, pbuf + P, pbuf + 2 * P, pbuf + 3 * P, pbuf + 4 * P, pbuf + 5 * P, pbuf + 6 * P, nullptr};
    double *qv = (double *)c.scratch(WS_TMP, (size_t)P * nq * sizeof(double));
    modal_launch(c, pts, P, Nt, M, qv, pbuf + 7 * P, pbuf + 8 * P, kappa, gam_re, gam_im, kout);
}

void split_planar(Ctx &c, const PlanarMat *mats, int n, int max_NG, double *s64r, double *s64i, float *s32r, float *s32i,
                  double *a64r, double *a64i) {
    const int64_t nt = ceil_div(max_NG, 32);
    hipLaunchKernelGGL(split_planar_kernel, dim3(n, (unsigned)std::min<int64_t>(nt * nt, 65535)), dim3(256), 0, c.stream,
                       mats, s64r, s64i, s32r, s32i, a64r, a64i);
    AXS_HIP(hipGetLastError());
}

}  // namespace axs
