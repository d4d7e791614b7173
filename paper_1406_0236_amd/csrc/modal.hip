// The block-diagonal preconditioner D^{-1} = blockdiag(F* S F) (Sec. 3.2 eq.
// "singleinverse", Sec. 4 Remark on the cost of D^{-1} B sigma):
//   (1) forward DFT in the azimuth of every body,
//   (2) per Fourier mode, apply the stored S_|m| = A~_|m|^{-1} (A~_{-m} = A~_m),
//   (3) inverse DFT, optionally adding the identity term of eq. "precond".
// N_F = 2M + 1 is odd and small (41, 81), so the DFT is a direct sum with the
// twiddle table and the input rows staged in LDS (same result as an FFT).  The
// nodes l and N_F - l share their cosine and have opposite sines, and so do the
// modes k and -k: with a_l = w_l + w_{N_F - l}, b_l = w_l - w_{N_F - l} both modes come
// from the same M products a_l cos, b_l sin, a quarter of the plain sum's.
// Step (2) is a batched complex GEMM on the matrix cores: for each shape and
// |m| the columns are (+m, -m) x (bodies of that shape) x (right-hand sides),
// and the complex product is four real MFMA products on planar operands.
#include "axs_internal.h"

namespace axs {

template <typename R> struct CT;
template <> struct CT<float> { using T = float2; };
template <> struct CT<double> { using T = double2; };

// Contour nodes per DFT block: 16, or 4 where 16 would leave fewer than 1,024
// workgroups.  The forward transform also adds up the partial inter-body sums, which for
// a small system is most of its time: 8,200 nodes, FP64, 25 partial sums 5.4 us
// (a pass over 64 of them in 14 workgroups: 55 us).
constexpr int DFT_BS = 256;

__device__ __forceinline__ int64_t xelem(const BodyDev &b, int nrhs, int k, int c, int i) {
    const int m = k <= b.M ? k : k - b.NF;
    const int am = m < 0 ? -m : m;
    const int sgn = m < 0 ? 1 : 0;
    const int64_t colbase = (int64_t)b.nb * nrhs * (am == 0 ? 0 : 2 * am - 1);
    const int64_t col = (int64_t)(sgn * b.nb + b.local) * nrhs + c;
    return (int64_t)nrhs * b.xoff + (colbase + col) * b.NG + i;
}

// X[k][i] = sum_l w[i][l] e^{-2 pi i k l / N_F} for the body's contour nodes
// [i0, i0 + GI) and rhs c.  Input: sum over `splits` partial inter-body sums
// (from_vec = 0) or a complex128 vector (from_vec = 1).
template <typename R, int GI>
__global__ __launch_bounds__(DFT_BS) void dft_forward_kernel(
    const BodyDev *__restrict__ bodies, const typename CT<R>::T *__restrict__ part, int splits,
    const double2 *__restrict__ vec, int from_vec, int64_t N, int nrhs, const R *__restrict__ tw,
    R *__restrict__ Xr, R *__restrict__ Xi) {
    using R2 = typename CT<R>::T;
    constexpr int P = GI + 1;                   // row pitch: the rows are written along l
    extern __shared__ __align__(16) unsigned char smem[];
    R2 *w = (R2 *)smem;                         // [NF][P]
    const BodyDev b = bodies[blockIdx.z];
    const int c = blockIdx.y;
    const int i0 = blockIdx.x * GI;
    if (i0 >= b.NG) return;
    const int ni = min(GI, b.NG - i0);
    const int NF = b.NF, M = b.M;
    R2 *t = w + P * NF;                         // [NF] twiddles (cos, sin)(2 pi j / NF)
    for (int j = threadIdx.x; j < NF; j += DFT_BS) {
        t[j].x = tw[2 * (b.twoff + j)];
        t[j].y = tw[2 * (b.twoff + j) + 1];
    }
    const int64_t base = b.offset + (int64_t)i0 * NF;
    for (int idx = threadIdx.x; idx < ni * NF; idx += DFT_BS) {
        R2 v;
        if (from_vec) {
            double2 d = vec[(int64_t)c * N + base + idx];
            v.x = (R)d.x;
            v.y = (R)d.y;
        } else {
            v.x = R(0);
            v.y = R(0);
            const R2 *src = part + (int64_t)c * N + base + idx;
            const int64_t step = (int64_t)nrhs * N;
            int s = 0;
            for (; s + 8 <= splits; s += 8) {   // loads first, then the sum in order
                R2 p[8];
#pragma unroll
                for (int u = 0; u < 8; ++u) p[u] = src[(s + u) * step];
#pragma unroll
                for (int u = 0; u < 8; ++u) {
                    v.x += p[u].x;
                    v.y += p[u].y;
                }
            }
            for (; s < splits; ++s) {
                const R2 p = src[s * step];
                v.x += p.x;
                v.y += p.y;
            }
        }
        w[(idx % NF) * P + idx / NF] = v;
    }
    __syncthreads();
    for (int idx = threadIdx.x; idx < M * GI; idx += DFT_BS) {
        const int l = 1 + idx / GI, i = idx % GI;
        if (i >= ni) continue;
        const R2 x = w[l * P + i], y = w[(NF - l) * P + i];
        R2 s, d;
        s.x = x.x + y.x;
        s.y = x.y + y.y;
        d.x = x.x - y.x;
        d.y = x.y - y.y;
        w[l * P + i] = s;
        w[(NF - l) * P + i] = d;
    }
    __syncthreads();
    for (int idx = threadIdx.x; idx < (M + 1) * GI; idx += DFT_BS) {
        const int k = idx / GI, i = idx % GI;
        if (i >= ni) continue;
        R cr = w[i].x, ci = w[i].y, sr = 0, si = 0;
        int tj = 0;
        for (int l = 1; l <= M; ++l) {
            tj += k;
            if (tj >= NF) tj -= NF;
            const R2 s = w[l * P + i], d = w[(NF - l) * P + i], e = t[tj];
            cr = fma(s.x, e.x, cr);
            ci = fma(s.y, e.x, ci);
            sr = fma(d.x, e.y, sr);
            si = fma(d.y, e.y, si);
        }
        const int64_t o = xelem(b, nrhs, k, c, i0 + i);
        Xr[o] = cr + si;
        Xi[o] = ci - sr;
        if (k > 0) {
            const int64_t o2 = xelem(b, nrhs, NF - k, c, i0 + i);
            Xr[o2] = cr - si;
            Xi[o2] = ci + sr;
        }
    }
}

// y[c][node] = alpha sigma[c][node] + beta / N_F sum_k Y[k][i] e^{+2 pi i k l / N_F}
template <typename R, int GI>
__global__ __launch_bounds__(DFT_BS) void dft_inverse_kernel(
    const BodyDev *__restrict__ bodies, const R *__restrict__ Yr, const R *__restrict__ Yi, int64_t N,
    int nrhs, const R *__restrict__ tw, const double2 *__restrict__ sigma, double alpha, double beta,
    double2 *__restrict__ y) {
    using R2 = typename CT<R>::T;
    extern __shared__ __align__(16) unsigned char smem[];
    R2 *yh = (R2 *)smem;                        // [GI][NF]: Y_0, then Y_k + Y_-k at k, Y_k - Y_-k at N_F - k
    const BodyDev b = bodies[blockIdx.z];
    const int c = blockIdx.y;
    const int i0 = blockIdx.x * GI;
    if (i0 >= b.NG) return;
    const int ni = min(GI, b.NG - i0);
    const int NF = b.NF, M = b.M;
    R2 *t = yh + (GI + 1) * NF;
    for (int j = threadIdx.x; j < NF; j += DFT_BS) {
        t[j].x = tw[2 * (b.twoff + j)];
        t[j].y = tw[2 * (b.twoff + j) + 1];
    }
    for (int idx = threadIdx.x; idx < (M + 1) * GI; idx += DFT_BS) {
        const int k = idx / GI, i = idx % GI;
        if (i >= ni) continue;
        const int64_t o = xelem(b, nrhs, k, c, i0 + i);
        R2 s, d;
        s.x = Yr[o];
        s.y = Yi[o];
        if (k > 0) {
            const int64_t o2 = xelem(b, nrhs, NF - k, c, i0 + i);
            const R xr = Yr[o2], xi = Yi[o2];
            d.x = s.x - xr;
            d.y = s.y - xi;
            s.x += xr;
            s.y += xi;
            yh[i * NF + NF - k] = d;
        }
        yh[i * NF + k] = s;
    }
    __syncthreads();
    const double scale = beta / NF;
    const int64_t base = (int64_t)c * N + b.offset + (int64_t)i0 * NF;
    auto put = [&](int64_t g, R re, R im) {
        double2 out = make_double2(scale * (double)re, scale * (double)im);
        if (alpha != 0.0) {
            const double2 s = sigma[g];
            out.x += alpha * s.x;
            out.y += alpha * s.y;
        }
        y[g] = out;
    };
    for (int idx = threadIdx.x; idx < ni * (M + 1); idx += DFT_BS) {
        const int i = idx / (M + 1), l = idx - i * (M + 1);
        const R2 *row = yh + i * NF;
        R cr = row[0].x, ci = row[0].y, sr = 0, si = 0;
        int tj = 0;
        for (int k = 1; k <= M; ++k) {
            tj += l;
            if (tj >= NF) tj -= NF;
            const R2 s = row[k], d = row[NF - k], e = t[tj];
            cr = fma(s.x, e.x, cr);
            ci = fma(s.y, e.x, ci);
            sr = fma(d.x, e.y, sr);
            si = fma(d.y, e.y, si);
        }
        const int64_t g = base + (int64_t)i * NF;
        put(g + l, cr - si, ci + sr);
        if (l > 0) put(g + NF - l, cr + si, ci - sr);
    }
}

// ---------------------------------------------------------------------------
// batched complex GEMM on MFMA:  Y = S X  per (shape, |m|)
// S planar column-major (element (i, k) at k*NG + i); X, Y planar column-major
// with leading dimension NG.  16 x 16 tiles of the 16x16x4 MFMA, four k steps'
// operands loaded ahead of their products.  KS = 1: a 256-thread block computes
// a 32 x 32 tile, each wave a 16 x 16 tile.  KS = 4: a block computes one 16 x 16 tile,
// each wave a quarter of the inner dimension, added up in LDS; taken where
// 32 x 32 tiles would leave fewer than 1,024 workgroups (few bodies and right-
// hand sides), where the product is bound by the latency of its serial k loop
// (8,200 nodes, FP64: 15 us with KS = 1, 5 us with KS = 4).
// Operand layout of the 16x16x4 MFMA (one block of 16x16): lane l supplies
// A[l % 16][l / 16] and B[l / 16][l % 16]; it receives column l % 16 of D in
// four registers v = 0..3, rows 4 (l / 16) + v for FP32 and (l / 16) + 4 v for
// FP64 (the FP64 result is not row-grouped).
// ---------------------------------------------------------------------------
typedef float f32x4 __attribute__((ext_vector_type(4)));
typedef double f64x4 __attribute__((ext_vector_type(4)));

__device__ __forceinline__ f32x4 mfma16(float a, float b, f32x4 c) {
    return __builtin_amdgcn_mfma_f32_16x16x4f32(a, b, c, 0, 0, 0);
}
__device__ __forceinline__ f64x4 mfma16(double a, double b, f64x4 c) {
    return __builtin_amdgcn_mfma_f64_16x16x4f64(a, b, c, 0, 0, 0);
}
template <typename R> struct V4;
template <> struct V4<float> {
    using T = f32x4;
    static __device__ __forceinline__ int row(int lane, int v) { return 4 * (lane >> 4) + v; }
};
template <> struct V4<double> {
    using T = f64x4;
    static __device__ __forceinline__ int row(int lane, int v) { return (lane >> 4) + 4 * v; }
};

template <typename R, int KS>
__global__ __launch_bounds__(256) void modal_gemm_kernel(const GemmBatch *__restrict__ batches, int nrhs,
                                                         const R *__restrict__ Sr, const R *__restrict__ Si,
                                                         const R *__restrict__ Xr, const R *__restrict__ Xi,
                                                         R *__restrict__ Yr, R *__restrict__ Yi) {
    using V = typename V4<R>::T;
    const GemmBatch bt = batches[blockIdx.z];
    const int NG = bt.NG;
    const int ncols = bt.ncols * nrhs;
    const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63;
    const int r0 = KS == 1 ? blockIdx.x * 32 + (wave >> 1) * 16 : blockIdx.x * 16;
    const int c0 = KS == 1 ? blockIdx.y * 32 + (wave & 1) * 16 : blockIdx.y * 16;
    if (r0 >= NG || c0 >= ncols) return;   // with KS = 4 the whole block
    // rows and columns beyond the matrix repeat the last one; their results are not stored
    const int arow = min(r0 + (lane & 15), NG - 1), bcol = min(c0 + (lane & 15), ncols - 1);
    const int kk = lane >> 4;
    const int64_t xo = bt.x_off * nrhs;
    const R *Ar = Sr + bt.a_off + arow, *Ai = Si + bt.a_off + arow;
    const R *Br = Xr + xo + (int64_t)bcol * NG, *Bi = Xi + xo + (int64_t)bcol * NG;
    // this wave's k range: quarters in steps of 16
    const int quarter = KS == 1 ? NG : ((NG + 63) / 64) * 16;
    const int kb = KS == 1 ? 0 : wave * quarter, ke = min(NG, kb + quarter);
    V accr = {0, 0, 0, 0}, acci = {0, 0, 0, 0};
    auto step = [&](R ar, R ai, R br, R bi) {
        accr = mfma16(ar, br, accr);
        acci = mfma16(ar, bi, acci);
        accr = mfma16(ai, -bi, accr);
        acci = mfma16(ai, br, acci);
    };
    int k0 = kb;
    for (; k0 + 16 <= ke; k0 += 16) {
        R ar[4], ai[4], br[4], bi[4];
#pragma unroll
        for (int u = 0; u < 4; ++u) {
            const int k = k0 + 4 * u + kk;
            ar[u] = Ar[(int64_t)k * NG];
            ai[u] = Ai[(int64_t)k * NG];
            br[u] = Br[k];
            bi[u] = Bi[k];
        }
#pragma unroll
        for (int u = 0; u < 4; ++u) step(ar[u], ai[u], br[u], bi[u]);
    }
    for (; k0 < ke; k0 += 4) {
        const int k = k0 + kk;
        const bool kok = k < ke;
        const R ar = kok ? Ar[(int64_t)k * NG] : R(0), ai = kok ? Ai[(int64_t)k * NG] : R(0);
        const R br = kok ? Br[k] : R(0), bi = kok ? Bi[k] : R(0);
        step(ar, ai, br, bi);
    }
    if constexpr (KS > 1) {
        __shared__ R s_acc[KS - 1][8][64];
        if (wave > 0) {
#pragma unroll
            for (int v = 0; v < 4; ++v) {
                s_acc[wave - 1][v][lane] = accr[v];
                s_acc[wave - 1][4 + v][lane] = acci[v];
            }
        }
        __syncthreads();
        if (wave > 0) return;
#pragma unroll
        for (int q = 0; q < KS - 1; ++q)
#pragma unroll
            for (int v = 0; v < 4; ++v) {
                accr[v] += s_acc[q][v][lane];
                acci[v] += s_acc[q][4 + v][lane];
            }
    }
    const int ocol = c0 + (lane & 15);
    if (ocol < ncols) {
#pragma unroll
        for (int v = 0; v < 4; ++v) {
            const int orow = r0 + V4<R>::row(lane, v);
            if (orow < NG) {
                Yr[xo + (int64_t)ocol * NG + orow] = accr[v];
                Yi[xo + (int64_t)ocol * NG + orow] = acci[v];
            }
        }
    }
}

// ---------------------------------------------------------------------------
// host launchers
// ---------------------------------------------------------------------------
// contour nodes per DFT block (see above), and the block's LDS
static int dft_gi(const Ctx &c, int nrhs) {
    return ceil_div(c.max_NG, 16) * nrhs * (int64_t)c.bodies.size() < 1024 ? 4 : 16;
}
static size_t dft_smem(const Ctx &c, int gi, size_t elem) {
    int maxnf = 0;
    for (auto &s : c.shapes) maxnf = std::max(maxnf, s.NF);
    return (size_t)(gi + 2) * maxnf * elem;
}

template <typename R, int GI>
static void launch_forward(Ctx &c, int from_vec, const void *vec, int nrhs, int splits, const R *tw) {
    using R2 = typename CT<R>::T;
    const int64_t total = (int64_t)nrhs * c.N;
    R *Xr = (R *)c.scratch(WS_XR, total * sizeof(R)), *Xi = (R *)c.scratch(WS_XI, total * sizeof(R));
    hipLaunchKernelGGL((dft_forward_kernel<R, GI>),
                       dim3((unsigned)ceil_div(c.max_NG, GI), nrhs, (unsigned)c.bodies.size()), dim3(DFT_BS),
                       dft_smem(c, GI, sizeof(R2)), c.stream, c.body_dev, (const R2 *)c.scratch(WS_PART, 0), splits,
                       (const double2 *)vec, from_vec, c.N, nrhs, tw, Xr, Xi);
    AXS_HIP(hipGetLastError());
}

void dft_forward(Ctx &c, int prec, int from_vec, const void *vec, int nrhs, int splits) {
    const bool small = dft_gi(c, nrhs) == 4;
    if (prec == AXS_FP32) {
        if (small) launch_forward<float, 4>(c, from_vec, vec, nrhs, splits, c.tw32);
        else launch_forward<float, 16>(c, from_vec, vec, nrhs, splits, c.tw32);
    } else {
        if (small) launch_forward<double, 4>(c, from_vec, vec, nrhs, splits, c.tw64);
        else launch_forward<double, 16>(c, from_vec, vec, nrhs, splits, c.tw64);
    }
}

template <typename R>
static void launch_gemm(Ctx &c, int nrhs, const R *Sr, const R *Si) {
    const int64_t total = (int64_t)nrhs * c.N, cols = (int64_t)c.gemm_max_cols * nrhs;
    R *Yr = (R *)c.scratch(WS_YR, total * sizeof(R)), *Yi = (R *)c.scratch(WS_YI, total * sizeof(R));
    const R *Xr = (const R *)c.scratch(WS_XR, 0), *Xi = (const R *)c.scratch(WS_XI, 0);
    if (ceil_div(c.max_NG, 32) * ceil_div(cols, 32) * c.ngemm < 1024)
        hipLaunchKernelGGL((modal_gemm_kernel<R, 4>),
                           dim3((unsigned)ceil_div(c.max_NG, 16), (unsigned)ceil_div(cols, 16), (unsigned)c.ngemm),
                           dim3(256), 0, c.stream, c.gemm, nrhs, Sr, Si, Xr, Xi, Yr, Yi);
    else
        hipLaunchKernelGGL((modal_gemm_kernel<R, 1>),
                           dim3((unsigned)ceil_div(c.max_NG, 32), (unsigned)ceil_div(cols, 32), (unsigned)c.ngemm),
                           dim3(256), 0, c.stream, c.gemm, nrhs, Sr, Si, Xr, Xi, Yr, Yi);
    AXS_HIP(hipGetLastError());
}

void modal_gemm(Ctx &c, int prec, int nrhs, bool forward) {
    // all shapes' matrices live in one planar allocation per precision (see precompute)
    const Shape &s0 = c.shapes[0];
    if (forward && prec != AXS_FP64) throw Error{AXS_EINVAL, "the A~_m products exist in FP64 only"};
    if (prec == AXS_FP32)
        launch_gemm<float>(c, nrhs, s0.S32r, s0.S32i);
    else
        launch_gemm<double>(c, nrhs, forward ? s0.A64r : s0.S64r, forward ? s0.A64i : s0.S64i);
}

template <typename R, int GI>
static void launch_inverse(Ctx &c, const void *sigma, double alpha, double beta, void *y, int nrhs, const R *tw) {
    using R2 = typename CT<R>::T;
    hipLaunchKernelGGL((dft_inverse_kernel<R, GI>),
                       dim3((unsigned)ceil_div(c.max_NG, GI), nrhs, (unsigned)c.bodies.size()), dim3(DFT_BS),
                       dft_smem(c, GI, sizeof(R2)), c.stream, c.body_dev, (const R *)c.scratch(WS_YR, 0),
                       (const R *)c.scratch(WS_YI, 0), c.N, nrhs, tw, (const double2 *)sigma, alpha, beta,
                       (double2 *)y);
    AXS_HIP(hipGetLastError());
}

void dft_inverse(Ctx &c, int prec, const void *sigma, double alpha, double beta, void *y, int nrhs) {
    const bool small = dft_gi(c, nrhs) == 4;
    if (prec == AXS_FP32) {
        if (small) launch_inverse<float, 4>(c, sigma, alpha, beta, y, nrhs, c.tw32);
        else launch_inverse<float, 16>(c, sigma, alpha, beta, y, nrhs, c.tw32);
    } else {
        if (small) launch_inverse<double, 4>(c, sigma, alpha, beta, y, nrhs, c.tw64);
        else launch_inverse<double, 16>(c, sigma, alpha, beta, y, nrhs, c.tw64);
    }
}

}  // namespace axs
