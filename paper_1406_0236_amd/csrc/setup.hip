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
// geometric bisection towards the (near-)singular parameter, max(10, p) Gauss
// points per level, see the constants below for how far it goes).
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
//   chi = 1, backward continued fraction otherwise);
//   k^D_m = normal derivative at the source of the same expression.
// Pipeline per batch of target rows:
//   gen_far / gen_near  -> evaluation points (source data + weight)
//   toroidal_kernel     -> q_mu, n.grad q_mu per point            (thread per point)
//   modal_kernel        -> k^G_m * weight per point, m = 0..M    (wavefront per point)
//   scatter / near_reduce -> entries of A~_m
// then 1/2 on the diagonal and S_m = A~_m^{-1} by Gauss-Jordan elimination
// with partial pivoting (one workgroup per mode).
#include <cmath>

#include "axs_internal.h"

namespace axs {

// Gauss points per level: the interpolation l_j(s) times the curve's own
// polynomial has degree 2p and more, which 10 points do not integrate for p > 10
// (with 10 the largest error of an entry is 2e-12 at p = 11, 1e-11 at 12 and
// 1e-8 at 16; with p points the kernel values' noise, 1e-12)
static int level_points(int p) { return p > 10 ? p : 10; }
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
// bowls, p = 3 to 16.  2760 -> 480 points per target node of a smooth contour:
// precomputation of 8 mixed bodies 6.08 -> 2.71 ms, of 27 spheres (one shape of
// 200 contour nodes) 6.85 -> 2.73 ms.
constexpr int OWN_LEV = 11, OWN_Q = 8, OWN_NQ = 24;
constexpr int MAX_LEV = 46;

struct Pts {
    double *rt, *rp, *dr, *dz, *nr, *nz, *wj;   // [P]
    double *lag;                                 // [near points][p]
};

// target node i against near panel P, split at sstar: n0 points on the side
// towards -1 and n1 towards 1, from near point `first` of the batch on
struct NearDesc {
    int32_t i, P;
    double sstar;
    int32_t n0, n1, first, pad;
};

// ---------------------------------------------------------------------------
// evaluation points
// ---------------------------------------------------------------------------
// far points: pair (i, P) of target node and panel, its p nodes in turn
__global__ void gen_far_kernel(const int2 *__restrict__ pairs, int n, int p, const double *__restrict__ r,
                               const double *__restrict__ z, const double *__restrict__ nr,
                               const double *__restrict__ nz, const double *__restrict__ aw, Pts pts) {
    int o = blockIdx.x * blockDim.x + threadIdx.x;
    if (o >= n * p) return;
    const int2 pr = pairs[o / p];
    const int i = pr.x, j = pr.y * p + o % p;
    pts.rt[o] = r[i];
    pts.rp[o] = r[j];
    pts.dr[o] = r[j] - r[i];
    pts.dz[o] = z[j] - z[i];
    pts.nr[o] = nr[j];
    pts.nz[o] = nz[j];
    pts.wj[o] = aw[j];
}

// one workgroup per near pair
__global__ void gen_near_kernel(const NearDesc *__restrict__ desc, int p, const double *__restrict__ snode,
                                const double *__restrict__ lden, const double *__restrict__ glu,
                                const double *__restrict__ glw, int ngl, const double *__restrict__ ownx,
                                const double *__restrict__ ownw, const double *__restrict__ r,
                                const double *__restrict__ z, Pts pts, int64_t base) {
    const NearDesc d = desc[blockIdx.x];
    const int own = (d.i / p) == d.P;
    for (int idx = threadIdx.x; idx < d.n0 + d.n1; idx += blockDim.x) {
        const int side = idx >= d.n0;
        const int q = side ? idx - d.n0 : idx;
        const int64_t o = base + d.first + idx;
        const double sst = d.sstar;
        const double dir = side == 0 ? -1.0 : 1.0;
        const double Ls = side == 0 ? sst + 1.0 : 1.0 - sst;
        double* lag = pts.lag + (int64_t)(d.first + idx) * p;
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
        const int iloc = d.i - d.P * p;
        const double *rP = r + d.P * p, *zP = z + d.P * p;
        // Lagrange basis and its derivative at s; on the own panel the factor
        // (s - s_iloc) is the exact signed offset.
        double diff[PMAX];
        for (int k = 0; k < p; ++k) diff[k] = (own && k == iloc) ? dir * off : s - snode[k];
        double L[PMAX], D[PMAX];
        for (int j = 0; j < p; ++j) {
            double prod = lden[j];
            for (int k = 0; k < p; ++k)
                if (k != j) prod *= diff[k];
            L[j] = prod;
            double der = 0;
            for (int m = 0; m < p; ++m) {
                if (m == j) continue;
                double t = lden[j];
                for (int k = 0; k < p; ++k)
                    if (k != j && k != m) t *= diff[k];
                der += t;
            }
            D[j] = der;
        }
        double rp = 0, zp = 0, rs = 0, zs = 0, dr = 0, dz = 0;
        for (int k = 0; k < p; ++k) {
            rp += L[k] * rP[k];
            zp += L[k] * zP[k];
            rs += D[k] * rP[k];
            zs += D[k] * zP[k];
        }
        if (own) {
            for (int k = 0; k < p; ++k) {
                if (k == iloc) continue;
                dr += L[k] * (rP[k] - r[d.i]);
                dz += L[k] * (zP[k] - z[d.i]);
            }
        } else {
            dr = rp - r[d.i];
            dz = zp - z[d.i];
        }
        const double sp = sqrt(rs * rs + zs * zs);
        const bool ok = rp > 1e-13 && (dr * dr + dz * dz) > 0.0;
        pts.rt[o] = r[d.i];
        pts.rp[o] = ok ? rp : -1.0;     // rp < 0 marks a point that contributes nothing
        pts.dr[o] = dr;
        pts.dz[o] = dz;
        pts.nr[o] = -zs / sp;
        pts.nz[o] = rs / sp;
        pts.wj[o] = ok ? wq * rp * sp : 0.0;
        for (int k = 0; k < p; ++k) lag[k] = L[k];
    }
}

// ---------------------------------------------------------------------------
// toroidal harmonics: q_mu = 2 Q_{mu-1/2}(chi)/sqrt(r r') and its normal derivative
// ---------------------------------------------------------------------------
__global__ void toroidal_kernel(Pts pts, int64_t npts, int nmax, double *__restrict__ qv,
                                double *__restrict__ dqv) {
    int64_t pt = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (pt >= npts) return;
    const int nq = nmax + 1;
    double *q = qv + pt * nq, *dq = dqv + pt * nq;
    const double rp = pts.rp[pt];
    if (!(rp > 0.0)) {
        for (int mu = 0; mu < nq; ++mu) q[mu] = dq[mu] = 0.0;
        return;
    }
    const double rt = pts.rt[pt], dr = pts.dr[pt], dz = pts.dz[pt], nrp = pts.nr[pt], nzp = pts.nz[pt];
    const double rr = rt * rp;
    const double d0sq = dr * dr + dz * dz;
    const double chim1 = d0sq / (2.0 * rr);
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
    const double kk = sqrt(2.0 / (chi + 1.0));
    const double Q0 = kk * K;
    const double eta = chim1 < 1e-3 ? 2.0 * asinh(sqrt(0.5 * chim1)) : acosh(chi);
    q[0] = Q0;
    if (nq > 1) {
        if (!(2.0 * nq * eta > 2.0)) {       // forward recurrence (also taken for a NaN argument)
            double qa = Q0, qb = chi * kk * K - sqrt(2.0 * (chi + 1.0)) * E;
            q[1] = qb;
            for (int mu = 1; mu + 1 < nq; ++mu) {
                const double qc = (2.0 * mu * chi * qb - (mu - 0.5) * qa) / (mu + 0.5);
                q[mu + 1] = qc;
                qa = qb;
                qb = qc;
            }
        } else {
            // rho_mu = Q_{mu+1/2}/Q_{mu-1/2} by the backward recurrence
            // rho_{mu-1} = (mu - 1/2) / (2 mu chi - (mu + 1/2) rho_mu), started at e^{-eta}
            const int top = nq + (int)ceil(20.0 / eta) + 20;
            double rho = 1.0 / (chi + sqrt(chim1 * (chi + 1.0)));
            for (int mu = top; mu >= 1; --mu) {
                rho = (mu - 0.5) / (2.0 * mu * chi - (mu + 0.5) * rho);
                if (mu < nq) q[mu] = rho;            // slot mu holds rho_{mu-1}
            }
            for (int mu = 1; mu < nq; ++mu) q[mu] = q[mu - 1] * q[mu];
        }
    }
    const double c2m1 = chim1 * (chi + 1.0);
    const double srr = sqrt(rr);
    const double ndel = nrp * dr + nzp * dz;
    const double ndchi = ndel / rr - nrp * d0sq / (2.0 * rr * rp);
    const double q1 = nq > 1 ? q[1] : 0.0;   // Q_{-3/2} = Q_{1/2}
    double prev = q1;
    for (int mu = 0; mu < nq; ++mu) {
        const double Qm = q[mu];
        const double dQ = (mu - 0.5) * (chi * Qm - prev) / c2m1;
        prev = Qm;
        const double qq = 2.0 * Qm / srr;
        q[mu] = qq;
        dq[mu] = 2.0 * dQ * ndchi / srr - nrp * qq / (2.0 * rp);
    }
}

// ---------------------------------------------------------------------------
// modal kernel values per point: one wavefront per point
// ---------------------------------------------------------------------------
__device__ double tcos_series(double x) {
    // (x cos x - sin x) / x^3 = sum_{k>=1} (-1)^k 2k x^{2k-2} / (2k+1)!
    double x2 = x * x, term = 1.0, sum = 0.0;
    double fact = 6.0;  // (2k+1)! for k = 1
    for (int k = 1; k <= 11; ++k) {
        sum += ((k & 1) ? -1.0 : 1.0) * (2.0 * k) * term / fact;
        term *= x2;
        fact *= (2.0 * k + 2.0) * (2.0 * k + 3.0);
    }
    return sum;
}

template <int WPB>
__global__ __launch_bounds__(64 * WPB) void modal_kernel(Pts pts, int64_t npts, int Nt, int M,
                                                         const double *__restrict__ qv,
                                                         const double *__restrict__ dqv, double kappa,
                                                         double gam_re, double gam_im,
                                                         double2 *__restrict__ kout) {
    extern __shared__ double sm[];
    const int Nh = Nt / 2 + 1, L = Nt / 2 - 1, nq = M + L + 1;
    const int per = 4 * Nh + 2 * (L + 1) + 2 * (M + 1) + 2 * nq;
    double *cosT = sm;                               // [Nt]
    const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63;
    double *base = sm + Nt + wave * per;
    double *Cs = base, *Ss = Cs + Nh, *Dc = Ss + Nh, *Ds = Dc + Nh;
    double *cl = Ds + Nh, *dcl = cl + (L + 1), *sm_ = dcl + (L + 1), *dsm = sm_ + (M + 1);
    double *ql = dsm + (M + 1), *dql = ql + nq;
    for (int j = threadIdx.x; j < Nt; j += 64 * WPB) cosT[j] = cospi(2.0 * j / Nt);
    const int64_t pt = (int64_t)blockIdx.x * WPB + wave;
    const bool inrange = pt < npts;
    const double rp = inrange ? pts.rp[pt] : -1.0;
    const bool active = rp > 0.0;       // rp <= 0 marks a point without contribution
    double rt = 0, dr = 0, dz = 0, nrp = 0, nzp = 0, wj = 0;
    if (active) {
        rt = pts.rt[pt];
        dr = pts.dr[pt];
        dz = pts.dz[pt];
        nrp = pts.nr[pt];
        nzp = pts.nz[pt];
        wj = pts.wj[pt];
    }
    const double d0sq = dr * dr + dz * dz, ndel = nrp * dr + nzp * dz;
    // samples t_k = 2 pi k / Nt, k = 0..Nt/2 (all factors are even in t)
    if (active) {
        for (int k = lane; k < Nh; k += 64) {
            const double sh = sinpi((double)k / Nt);
            const double s2 = sh * sh;                   // sin^2(t/2)
            const double R = sqrt(d0sq + 4.0 * rt * rp * s2);
            const double x = kappa * R;
            double sn, cs;
            sincos(x, &sn, &cs);
            const double sd = R > 0.0 ? sn / R : kappa;
            const double T = x > 0.2 ? (x * cs - sn) / (R * R * R) : kappa * kappa * kappa * tcos_series(x);
            const double g = ndel + 2.0 * nrp * rt * s2;
            Cs[k] = cs;
            Ss[k] = sd;
            Dc[k] = -kappa * sd * g;
            Ds[k] = T * g;
        }
        for (int mu = lane; mu < nq; mu += 64) {
            ql[mu] = qv[pt * nq + mu];
            dql[mu] = dqv[pt * nq + mu];
        }
    }
    __syncthreads();
    // cosine-series coefficients:  f_l = (1/Nt) [f_0 + (-1)^l f_{Nt/2} + 2 sum_{k=1}^{Nt/2-1} f_k cos(2 pi l k / Nt)]
    if (active) {
        const int Lc = L > M ? L : M;
        for (int l = lane; l <= Lc; l += 64) {
            const double sgn = (l & 1) ? -1.0 : 1.0;
            double a0 = Cs[0] + sgn * Cs[Nh - 1], a1 = Ss[0] + sgn * Ss[Nh - 1];
            double a2 = Dc[0] + sgn * Dc[Nh - 1], a3 = Ds[0] + sgn * Ds[Nh - 1];
            double b0 = 0, b1 = 0, b2 = 0, b3 = 0;
            int idx = 0;
            for (int k = 1; k < Nh - 1; ++k) {
                idx += l;
                if (idx >= Nt) idx -= Nt;
                const double cw = cosT[idx];
                b0 = fma(Cs[k], cw, b0);
                b1 = fma(Ss[k], cw, b1);
                b2 = fma(Dc[k], cw, b2);
                b3 = fma(Ds[k], cw, b3);
            }
            const double inv = 1.0 / Nt;
            if (l <= L) {
                cl[l] = (a0 + 2.0 * b0) * inv;
                dcl[l] = (a2 + 2.0 * b2) * inv;
            }
            if (l <= M) {
                sm_[l] = (a1 + 2.0 * b1) * inv * (2.0 * M_PI);
                dsm[l] = (a3 + 2.0 * b3) * inv * (2.0 * M_PI);
            }
        }
    }
    __syncthreads();
    if (!inrange) return;
    double2 *out = kout + pt * (M + 1);
    const double inv4pi = 0.25 / M_PI;
    for (int m = lane; m <= M; m += 64) {
        if (!active) {
            out[m] = make_double2(0.0, 0.0);
            continue;
        }
        double sr = 0.0, dr_ = 0.0;
        for (int l = -L; l <= L; ++l) {
            const int al = l < 0 ? -l : l;
            const int mm = m - l < 0 ? l - m : m - l;
            sr = fma(cl[al], ql[mm], sr);
            dr_ = fma(dcl[al], ql[mm], fma(cl[al], dql[mm], dr_));
        }
        const double si = sm_[m], di = dsm[m];
        // (kD + gamma kS) / (4 pi)
        const double re = (dr_ + gam_re * sr - gam_im * si) * inv4pi;
        const double im = (di + gam_re * si + gam_im * sr) * inv4pi;
        out[m] = make_double2(re * wj, im * wj);
    }
}

// ---------------------------------------------------------------------------
// assembly of A~_m
// ---------------------------------------------------------------------------
__global__ void scatter_far_kernel(const int2 *__restrict__ pairs, int n, int p, int M, int NG,
                                   const double2 *__restrict__ kval, double2 *__restrict__ A) {
    int64_t idx = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (idx >= (int64_t)n * p * (M + 1)) return;
    const int o = (int)(idx / (M + 1)), m = (int)(idx % (M + 1));
    const int2 pr = pairs[o / p];
    A[((int64_t)m * NG + pr.x) * NG + pr.y * p + o % p] = kval[idx];
}

__global__ void near_reduce_kernel(const NearDesc *__restrict__ desc, int M, int NG, int p,
                                   const double2 *__restrict__ kval, const double *__restrict__ lag,
                                   int64_t base, double2 *__restrict__ A) {
    const NearDesc d = desc[blockIdx.x];
    const int per = d.n0 + d.n1;
    const double2 *kv = kval + (base + d.first) * (M + 1);
    const double *lg = lag + (int64_t)d.first * p;
    for (int t = threadIdx.x; t < (M + 1) * p; t += blockDim.x) {
        const int m = t / p, j = t % p;
        double re = 0, im = 0;
        for (int q = 0; q < per; ++q) {
            const double2 v = kv[(int64_t)q * (M + 1) + m];
            const double l = lg[(int64_t)q * p + j];
            re = fma(v.x, l, re);
            im = fma(v.y, l, im);
        }
        A[((int64_t)m * NG + d.i) * NG + d.P * p + j] = make_double2(re, im);
    }
}

__global__ void add_half_identity_kernel(double2 *A, int M, int NG) {
    int idx = blockIdx.x * blockDim.x + threadIdx.x;
    if (idx >= (M + 1) * NG) return;
    const int m = idx / NG, i = idx % NG;
    A[((int64_t)m * NG + i) * NG + i].x += 0.5;
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
// inner dimension of 16:
//   gj_panel_kernel  - one workgroup per matrix, one row per thread held in
//                      registers; bound by its 16 serial steps (two barriers each);
//   gj_update_kernel - a 16 x 16 tile per wavefront on the FP64 matrix cores,
//                      read from one copy of the matrix and written to the other
//                      (the pivot rows are read by every tile).
// 41 matrices of 200 x 200 (MI355X): 26 launches, 0.60 ms (13 x 30 us + 13 x 16
// us); one workgroup per matrix over global memory took 19.97 ms.
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

typedef double gj_f64x4 __attribute__((ext_vector_type(4)));

__device__ __forceinline__ const double2 *gj_src(const GJItem &it, int step) {
    return step == 0 ? it.A : (step & 1) ? it.b0 : it.b1;
}

template <int BS>
__global__ __launch_bounds__(BS) void gj_panel_kernel(const GJItem *__restrict__ items, int step) {
    const GJItem it = items[blockIdx.x];
    const int NG = it.NG, k0 = step * GJB;
    if (k0 >= NG) return;
    const int nb = min(GJB, NG - k0);
    const int r = threadIdx.x, lane = r & 63, wave = r >> 6;
    constexpr int NW = BS / 64;
    __shared__ double s_max[2][NW];
    __shared__ int s_row[2][NW];
    __shared__ double2 s_piv[2][GJB];
    const bool live = r < NG;
    const double2 *src = gj_src(it, step) + (int64_t)r * NG + k0;
    double ar[GJB], ai[GJB];
#pragma unroll
    for (int j = 0; j < GJB; ++j) {
        double2 v = make_double2(0.0, 0.0);
        if (live && j < nb) v = src[j];
        ar[j] = v.x;
        ai[j] = v.y;
    }
    int mycol = !live ? 0 : step == 0 ? -1 : it.col[r];
#pragma unroll
    for (int c = 0; c < GJB; ++c) {
        if (c >= nb) break;
        double mag = -1.0;
        if (mycol < 0) {
            mag = ar[c] * ar[c] + ai[c] * ai[c];
            if (!(mag >= 0.0)) mag = 0.0;   // NaN: the result is NaN whatever the pivot
        }
        double wm = mag;
#pragma unroll
        for (int o = 32; o > 0; o >>= 1) wm = fmax(wm, __shfl_xor(wm, o, 64));
        const int first = __ffsll((unsigned long long)__ballot(mag == wm)) - 1;
        if (lane == 0) {
            s_max[c & 1][wave] = wm;
            s_row[c & 1][wave] = wave * 64 + first;
        }
        __syncthreads();
        double best = s_max[c & 1][0];
        int pr = s_row[c & 1][0];
#pragma unroll
        for (int w = 1; w < NW; ++w)
            if (s_max[c & 1][w] > best) {
                best = s_max[c & 1][w];
                pr = s_row[c & 1][w];
            }
        if (r == pr) {
            const double den = ar[c] * ar[c] + ai[c] * ai[c];
            const double pr_ = ar[c] / den, pi_ = -ai[c] / den;
            ar[c] = 1.0;
            ai[c] = 0.0;
#pragma unroll
            for (int j = 0; j < GJB; ++j) {
                const double x = ar[j] * pr_ - ai[j] * pi_, y = ar[j] * pi_ + ai[j] * pr_;
                ar[j] = x;
                ai[j] = y;
                s_piv[c & 1][j] = make_double2(x, y);
            }
            mycol = k0 + c;
            it.prow[k0 + c] = r;
        }
        __syncthreads();
        if (r != pr) {
            const double fr = ar[c], fi = ai[c];
            ar[c] = 0.0;
            ai[c] = 0.0;
#pragma unroll
            for (int j = 0; j < GJB; ++j) {
                const double2 u = s_piv[c & 1][j];
                ar[j] = fma(-fr, u.x, fma(fi, u.y, ar[j]));
                ai[j] = fma(-fr, u.y, fma(-fi, u.x, ai[j]));
            }
        }
    }
    if (!live) return;
    it.col[r] = mycol;
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
    gj_f64x4 accr, acci;
#pragma unroll
    for (int v = 0; v < 4; ++v) {
        const int row = r0 + q + 4 * v;
        double2 x = make_double2(0.0, 0.0);
        if (row < NG && col < NG) {
            const int pc = it.col[row];
            if (pc < k0) x = src[(int64_t)row * NG + col];   // not a pivot row of this block
        }
        accr[v] = x.x;
        acci[v] = x.y;
    }
    const int arow = r0 + (lane & 15);
#pragma unroll
    for (int k = 0; k < GJB; k += 4) {
        double2 a = make_double2(0.0, 0.0), b = a;
        if (k + q < nb) {
            if (arow < NG) a = it.T[(int64_t)arow * GJB + k + q];
            if (col < NG) b = src[(int64_t)it.prow[k0 + k + q] * NG + col];
        }
        accr = __builtin_amdgcn_mfma_f64_16x16x4f64(a.x, b.x, accr, 0, 0, 0);
        acci = __builtin_amdgcn_mfma_f64_16x16x4f64(a.x, b.y, acci, 0, 0, 0);
        accr = __builtin_amdgcn_mfma_f64_16x16x4f64(-a.y, b.y, accr, 0, 0, 0);
        acci = __builtin_amdgcn_mfma_f64_16x16x4f64(a.y, b.x, acci, 0, 0, 0);
    }
#pragma unroll
    for (int v = 0; v < 4; ++v) {
        const int row = r0 + q + 4 * v;
        if (row < NG && col < NG) dst[(int64_t)row * NG + col] = make_double2(accr[v], acci[v]);
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

// S (complex128 row-major [M+1][NG][NG]) -> planar column-major FP64 and FP32 copies
__global__ void split_planar_kernel(const double2 *__restrict__ S, int M, int NG, double *__restrict__ r64,
                                    double *__restrict__ i64, float *__restrict__ r32,
                                    float *__restrict__ i32) {
    int64_t t = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    const int64_t nn = (int64_t)NG * NG;
    if (t >= (M + 1) * nn) return;
    const int64_t m = t / nn, e = t % nn;
    const int k = (int)(e / NG), i = (int)(e % NG);      // output (column-major): element (i, k) at k*NG + i
    const double2 v = S[m * nn + (int64_t)i * NG + k];
    r64[t] = v.x;
    i64[t] = v.y;
    if (r32) {
        r32[t] = (float)v.x;
        i32[t] = (float)v.y;
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

void precompute_shape(Ctx &c, Shape &s) {
    const int NG = s.NG, p = s.p, M = s.M, np_ = s.n_panels;
    AXS_REQUIRE(p <= PMAX, AXS_EINVAL, "at most 16 nodes per panel are supported");
    s.Nt = modal_nt(s);
    const int Nt = s.Nt, L = Nt / 2 - 1, nq = M + L + 1;

    std::vector<double> sn, sw, gu, gwq, qu, qw;
    gauss_legendre(p, sn, sw);
    const int ngl = level_points(p), own_pts = OWN_LEV * ngl + OWN_NQ;
    gauss_legendre(ngl, gu, gwq);
    gauss_legendre(OWN_NQ, qu, qw);
    std::vector<double> lden(p);
    for (int j = 0; j < p; ++j) {
        double d = 1.0;
        for (int k = 0; k < p; ++k)
            if (k != j) d *= (sn[j] - sn[k]);
        lden[j] = 1.0 / d;
    }
    // the own-panel rule on [0, 1], singular at 0
    std::vector<double> ownx, ownw;
    for (int lev = 0; lev < OWN_LEV; ++lev)
        for (int k = 0; k < ngl; ++k) {
            const double half = std::ldexp(0.25, -lev);   // half of [2^-(lev + 1), 2^-lev]
            ownx.push_back(2.0 * half + half * (gu[k] + 1.0));
            ownw.push_back(half * gwq[k]);
        }
    for (int k = 0; k < OWN_NQ; ++k) {
        const double u = 0.5 * (qu[k] + 1.0), h = std::ldexp(1.0, -OWN_LEV);
        ownx.push_back(h * std::pow(u, OWN_Q));
        ownw.push_back(h * OWN_Q * std::pow(u, OWN_Q - 1) * 0.5 * qw[k]);
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
    // near panels and split points per target (host geometry)
    std::vector<std::vector<NearDesc>> near(NG);
    std::vector<double> endr(2 * np_), endz(2 * np_);
    for (int P = 0; P < np_; ++P) {
        endr[2 * P] = interp_at(sn, &s.r[P * p], p, -1.0);
        endr[2 * P + 1] = interp_at(sn, &s.r[P * p], p, 1.0);
        endz[2 * P] = interp_at(sn, &s.z[P * p], p, -1.0);
        endz[2 * P + 1] = interp_at(sn, &s.z[P * p], p, 1.0);
    }
    // points on one side (length Ls in s) of a panel at distance d: halve until
    // the innermost interval is shorter than d / 8
    auto side_points = [&](double Ls, double d, double speed) {
        if (!(Ls > 1e-14)) return 0;
        int n = 1;
        while (n < MAX_LEV && std::ldexp(Ls, 1 - n) * speed > 0.125 * d) ++n;
        return n * ngl;
    };
    for (int i = 0; i < NG; ++i) {
        const int own = i / p;
        for (int P = 0; P < np_; ++P) {
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
            if (P == own) {
                d.sstar = sn[i - own * p];
                d.n0 = d.n1 = own_pts;
            } else {
                d.sstar = bs;
                d.n0 = side_points(bs + 1.0, best, smax[P]);
                d.n1 = side_points(1.0 - bs, best, smax[P]);
            }
            near[i].push_back(d);
        }
    }
    // device constants, one block
    std::vector<double> hc;
    auto put = [&](const std::vector<double> &v) {
        const size_t o = hc.size();
        hc.insert(hc.end(), v.begin(), v.end());
        return o;
    };
    const size_t o_sn = put(sn), o_lden = put(lden), o_gu = put(gu), o_gw = put(gwq), o_ox = put(ownx),
                 o_ow = put(ownw), o_r = put(s.r), o_z = put(s.z), o_nr = put(nr), o_nz = put(nz), o_aw = put(aw);
    double *dc = (double *)c.dalloc(hc.size() * sizeof(double));
    AXS_HIP(hipMemcpyAsync(dc, hc.data(), hc.size() * sizeof(double), hipMemcpyHostToDevice, c.stream));

    const int64_t nmat = (int64_t)(M + 1) * NG * NG;
    double2 *A = (double2 *)c.dalloc(nmat * sizeof(double2));   // every entry is written below
    s.A64 = (double *)A;

    // batches of target rows, bounded number of evaluation points
    const int64_t max_pts = 1 << 19;
    int i0 = 0;
    while (i0 < NG) {
        int i1 = i0;
        int64_t npts = 0;
        std::vector<int2> far;
        std::vector<NearDesc> nd;
        int64_t nnear = 0;
        while (i1 < NG) {
            int64_t add = (int64_t)(np_ - (int)near[i1].size()) * p;
            for (auto &d : near[i1]) add += d.n0 + d.n1;
            if (i1 > i0 && npts + add > max_pts) break;
            npts += add;
            size_t k = 0;
            for (int P = 0; P < np_; ++P) {
                if (k < near[i1].size() && near[i1][k].P == P) {
                    NearDesc d = near[i1][k++];
                    d.first = (int32_t)nnear;
                    nnear += d.n0 + d.n1;
                    nd.push_back(d);
                } else {
                    far.push_back(make_int2(i1, P));
                }
            }
            ++i1;
        }
        const int64_t nfar = (int64_t)far.size() * p;
        const int64_t P = nfar + nnear;
        // point storage
        double *pbuf = (double *)c.scratch(WS_MISC, ((size_t)P * 7 + (size_t)nnear * p) * sizeof(double));
        Pts pts{pbuf, pbuf + P, pbuf + 2 * P, pbuf + 3 * P, pbuf + 4 * P, pbuf + 5 * P, pbuf + 6 * P, pbuf + 7 * P};
        double *qv = (double *)c.scratch(WS_TMP, (size_t)P * nq * sizeof(double));
        double *dqv = (double *)c.scratch(WS_TMP2, (size_t)P * nq * sizeof(double));
        double2 *kv = (double2 *)c.scratch(WS_TMP3, (size_t)P * (M + 1) * sizeof(double2));
        int2 *d_far = (int2 *)c.scratch(WS_RED, far.size() * sizeof(int2));
        NearDesc *d_nd = (NearDesc *)c.scratch(WS_GEMM, nd.size() * sizeof(NearDesc));
        if (nfar) {
            AXS_HIP(hipMemcpyAsync(d_far, far.data(), far.size() * sizeof(int2), hipMemcpyHostToDevice, c.stream));
            hipLaunchKernelGGL(gen_far_kernel, dim3(ceil_div(nfar, 256)), dim3(256), 0, c.stream, d_far,
                               (int)far.size(), p, dc + o_r, dc + o_z, dc + o_nr, dc + o_nz, dc + o_aw, pts);
            AXS_HIP(hipGetLastError());
        }
        // a target's own panel is always near, so no batch is without near points
        AXS_HIP(hipMemcpyAsync(d_nd, nd.data(), nd.size() * sizeof(NearDesc), hipMemcpyHostToDevice, c.stream));
        hipLaunchKernelGGL(gen_near_kernel, dim3(nd.size()), dim3(128), 0, c.stream, d_nd, p, dc + o_sn, dc + o_lden,
                           dc + o_gu, dc + o_gw, ngl, dc + o_ox, dc + o_ow, dc + o_r, dc + o_z, pts, nfar);
        AXS_HIP(hipGetLastError());
        hipLaunchKernelGGL(toroidal_kernel, dim3(ceil_div(P, 64)), dim3(64), 0, c.stream, pts, P, nq - 1, qv,
                           dqv);
        AXS_HIP(hipGetLastError());
        constexpr int WPB = 4;
        const int per = 4 * (Nt / 2 + 1) + 2 * (L + 1) + 2 * (M + 1) + 2 * nq;
        const size_t shm = (Nt + WPB * per) * sizeof(double);
        AXS_REQUIRE(shm <= 160 * 1024, AXS_EINVAL, "mode count or wavenumber too large for the modal kernel");
        hipLaunchKernelGGL(modal_kernel<WPB>, dim3(ceil_div(P, WPB)), dim3(64 * WPB), shm, c.stream, pts, P, Nt,
                           M, qv, dqv, s.kappa, s.kappa > 0 ? 0.0 : s.eta, s.kappa > 0 ? s.eta : 0.0, kv);
        AXS_HIP(hipGetLastError());
        if (nfar) {
            hipLaunchKernelGGL(scatter_far_kernel, dim3(ceil_div(nfar * (M + 1), 256)), dim3(256), 0, c.stream,
                               d_far, (int)far.size(), p, M, NG, kv, A);
            AXS_HIP(hipGetLastError());
        }
        hipLaunchKernelGGL(near_reduce_kernel, dim3(nd.size()), dim3(256), 0, c.stream, d_nd, M, NG, p, kv, pts.lag,
                           nfar, A);
        AXS_HIP(hipGetLastError());
        i0 = i1;
        if (i0 >= NG) {
            hipLaunchKernelGGL(add_half_identity_kernel, dim3(ceil_div((M + 1) * NG, 256)), dim3(256), 0, c.stream, A,
                               M, NG);
            AXS_HIP(hipGetLastError());
        }
        AXS_HIP(hipStreamSynchronize(c.stream));   // far, nd (and hc) are pageable host memory
    }
    c.dfree(dc);
}

// S_m = A~_m^{-1} for every shape and mode, in groups of shapes whose work
// arrays (about NG x 2 NG per matrix) stay within 4 GiB.  Per group one launch
// sequence over all its matrices: two launches per 16 columns, or one launch of
// gauss_jordan_kernel where a matrix has more rows than a workgroup has threads.
void invert_shapes(Ctx &c) {
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
            double2 *S = (double2 *)c.dalloc((size_t)(s.M + 1) * nn * sizeof(double2));
            s.S64 = (double *)S;
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
        GJItem *d_items = (GJItem *)c.dalloc(items.size() * sizeof(GJItem));
        AXS_HIP(hipMemcpyAsync(d_items, items.data(), items.size() * sizeof(GJItem), hipMemcpyHostToDevice, c.stream));
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
        AXS_HIP(hipStreamSynchronize(c.stream));   // items is pageable host memory; the work array is released
        c.dfree(d_items);
        c.dfree(work);
        k = k1;
    }
}

void modal_values(Ctx &c, double kappa, double gam_re, double gam_im, int M, int Nt,
                  const std::vector<double> &h, int64_t P, double2 *kout) {
    const int L = Nt / 2 - 1, nq = M + L + 1;
    double *pbuf = (double *)c.scratch(WS_MISC, (size_t)P * 7 * sizeof(double));
    AXS_HIP(hipMemcpy(pbuf, h.data(), (size_t)P * 7 * sizeof(double), hipMemcpyHostToDevice));
    Pts pts{pbuf, pbuf + P, pbuf + 2 * P, pbuf + 3 * P, pbuf + 4 * P, pbuf + 5 * P, pbuf + 6 * P, nullptr};
    double *qv = (double *)c.scratch(WS_TMP, (size_t)P * nq * sizeof(double));
    double *dqv = (double *)c.scratch(WS_TMP2, (size_t)P * nq * sizeof(double));
    hipLaunchKernelGGL(toroidal_kernel, dim3(ceil_div(P, 64)), dim3(64), 0, c.stream, pts, P, nq - 1, qv, dqv);
    AXS_HIP(hipGetLastError());
    constexpr int WPB = 4;
    const int per = 4 * (Nt / 2 + 1) + 2 * (L + 1) + 2 * (M + 1) + 2 * nq;
    const size_t shm = (Nt + WPB * per) * sizeof(double);
    AXS_REQUIRE(shm <= 160 * 1024, AXS_EINVAL, "mode count or wavenumber too large for the modal kernel");
    hipLaunchKernelGGL(modal_kernel<WPB>, dim3(ceil_div(P, WPB)), dim3(64 * WPB), shm, c.stream, pts, P, Nt, M,
                       qv, dqv, kappa, gam_re, gam_im, kout);
    AXS_HIP(hipGetLastError());
}

void split_planar(Ctx &c, Shape &s, const double *src, double *r64, double *i64, float *r32, float *i32) {
    const int64_t nmat = (int64_t)(s.M + 1) * s.NG * s.NG;
    hipLaunchKernelGGL(split_planar_kernel, dim3(ceil_div(nmat, 256)), dim3(256), 0, c.stream,
                       (const double2 *)src, s.M, s.NG, r64, i64, r32, i32);
    AXS_HIP(hipGetLastError());
}

}  // namespace axs
