// Fields of a density off the surface, FP64: the scattered field at points (eq.
// "intHelm1" with the surface rule) and the far-field pattern.
//
//   u[c][t] = sum_j K(t, j) q[c][j],   q = w sigma / 4 pi,
//   near:  K = e^{ikR}/R [ (n.d)(1 - i k R)/R^2 + gamma ],  d = x_t - x_j
//   far:   K = i (eta - k xh.n_j) e^{-i k xh.x_j}
//
// Bound: FP64 VALU issue (counted per target-node pair: near 44 instructions with one
// density, far 47 with four; 4 of them for each density), so a pair is evaluated once for all right-hand sides of a group of
// up to 8, its sin/cos come from the inter-body sums' LDS table, and nothing else
// is read per pair: targets sit in lanes (TPT per lane), and the nodes' records
// (position and normal, for the far field scaled, and the group's densities, packed
// once per call) pass
// through LDS 64 at a time and are read back as broadcasts (by scalar loads
// instead the kernels took 8 % longer, prefetched or not).  The nodes are cut
// into chunks so that even a few targets fill the chip; the chunks' partial sums
// are added in a fixed order.
// In a kernel trace, 20,000 directions x 18,860 nodes x 4 densities: 0.65 ms, 79 % of the
// FP64 issue rate at the clock it ran at; 1,024 points x 437,400 nodes: 0.77 ms, 80 % (the
// whole calls, untraced, 0.65 and 0.72 ms; with one workgroup per target and right-hand
// side and the library sincos 5.7 to 6.1 and 2.7 to 3.0).
// Small calls, and few targets with many densities, take field_direct_kernel: one
// workgroup per target and right-hand side after all, in one launch.
#include "axs_internal.h"
#include "fp64_math.h"

#include <algorithm>
#include <cmath>

namespace axs {

constexpr int FIELD_TILE = 64;   // node records in LDS at a time
constexpr size_t FIELD_SCRATCH = (size_t)256 << 20;   // records of one pass over groups of rhs, and its partial sums

enum FieldKind { FIELD_FAR = 0, FIELD_NEAR = 1, FIELD_LAPLACE = 2 };

// records of one batch of rhs groups: rec[g][j][6 + 2 nr], rhs c0 + g nr + i
// (zero densities beyond nrhs)
__global__ __launch_bounds__(256) void field_records_kernel(const double *__restrict__ g, int64_t N,
                                                            const double2 *__restrict__ sigma, int c0, int nrhs,
                                                            int nr, double sx, double sn, double *__restrict__ rec) {
    const int64_t j = (int64_t)blockIdx.x * 256 + threadIdx.x;
    if (j >= N) return;
    double *o = rec + ((int64_t)blockIdx.y * N + j) * (6 + 2 * nr);
#pragma unroll
    for (int a = 0; a < 3; ++a) {
        o[a] = g[a * N + j] * sx;
        o[3 + a] = g[(3 + a) * N + j] * sn;
    }
    const double w = g[6 * N + j] * (0.25 / M_PI);
    for (int i = 0; i < nr; ++i) {
        const int c = c0 + blockIdx.y * nr + i;
        double2 v = make_double2(0.0, 0.0);
        if (c < nrhs) v = sigma[(int64_t)c * N + j];
        o[6 + 2 * i] = v.x * w;
        o[7 + 2 * i] = v.y * w;
    }
}

// part[chunk][c - c0][t] for the pass's nc rhs from c0 on (u[c0 ..][t] where there is
// one chunk).  wide: phases may reach
// 2^39 revolutions, reduced to a fraction first.  Near: the distance comes from the
// differences of the coordinates as given, and k / 2 pi goes into R^2 (one
// multiplication a pair).  With records and targets scaled by k / 2 pi beforehand each
// carried a rounding of its own, which the difference of close points keeps: errors of
// 5e-14 of the field 1e-3 off a body at the origin and 3e-11 where the scene lay
// 1,000 away.
template <int KIND, int NR, int TPT>
__global__ __launch_bounds__(256) void field_kernel(const double *__restrict__ rec, int64_t N, int64_t chunk,
                                                    const double *__restrict__ tgt, int nt, double kappa,
                                                    double k2pi, double eta, int wide,
                                                    const double2 *__restrict__ sctab, int nc,
                                                    double2 *__restrict__ part) {
    constexpr int ST = 6 + 2 * NR;
    __shared__ __align__(16) double s_rec[FIELD_TILE * ST];
    __shared__ double2 s_tab[KIND == FIELD_LAPLACE ? 1 : SC_N];
    if constexpr (KIND != FIELD_LAPLACE) {
        for (int i = threadIdx.x; i < SC_N; i += blockDim.x) s_tab[i] = sctab[i];
    }
    const int t0 = blockIdx.x * blockDim.x * TPT + threadIdx.x;
    double tx[TPT], ty[TPT], tz[TPT], ar[TPT][NR], ai[TPT][NR];
#pragma unroll
    for (int k = 0; k < TPT; ++k) {
        const int t = min(t0 + k * (int)blockDim.x, nt - 1);
        tx[k] = tgt[3 * t];
        ty[k] = tgt[3 * t + 1];
        tz[k] = tgt[3 * t + 2];
#pragma unroll
        for (int c = 0; c < NR; ++c) ar[k][c] = ai[k][c] = 0.0;
    }
    const int64_t j0 = (int64_t)blockIdx.y * chunk, j1 = min(N, j0 + chunk);
    const double *__restrict__ base = rec + (int64_t)blockIdx.z * N * ST;
#pragma unroll 1
    for (int64_t jb = j0; jb < j1; jb += FIELD_TILE) {
        const int cnt = (int)min((int64_t)FIELD_TILE, j1 - jb);
        __syncthreads();   // (the first one publishes the table as well)
        for (int i = threadIdx.x; i < cnt * ST; i += blockDim.x) s_rec[i] = base[jb * ST + i];
        __syncthreads();
#pragma unroll 1
        for (int j = 0; j < cnt; ++j) {
            const double *r = s_rec + j * ST;
            const double x = r[0], y = r[1], z = r[2], nx = r[3], ny = r[4], nz = r[5];
#pragma unroll
            for (int k = 0; k < TPT; ++k) {
                double gr, gi;
                if constexpr (KIND == FIELD_FAR) {
                    double ph = fma(tx[k], x, fma(ty[k], y, tz[k] * z));
                    if (wide) ph -= rint(ph);
                    const double f = fma(tx[k], nx, fma(ty[k], ny, fma(tz[k], nz, eta)));
                    double s, c;
                    sincos_rev_tab(ph, s_tab, s, c);
                    gr = -f * s;
                    gi = f * c;
                } else {
                    const double dx = tx[k] - x, dy = ty[k] - y, dz = tz[k] - z;
                    const double r2 = fma(dx, dx, fma(dy, dy, dz * dz));
                    const double nd = fma(nx, dx, fma(ny, dy, nz * dz));
                    const double u = rsq(r2);
                    if constexpr (KIND == FIELD_LAPLACE) {
                        gr = u * fma(nd, u * u, eta);
                        gi = 0.0;
                    } else {
                        double s, c;
                        const double rk = r2 * k2pi;               // times u: R k / 2 pi
                        if (wide) {
                            const double ph = rk * u;
                            sincos_rev_tab(ph - rint(ph), s_tab, s, c);
                        } else {
                            sincos_phase(rk, u, 0.0, s_tab, s, c);
                        }
                        const double t = nd * (u * u);
                        const double P = t * u;                    // n.d / R^3
                        const double Q = fma(-kappa, t, eta * u);  // eta / R - k n.d / R^2
                        gr = fma(c, P, -s * Q);
                        gi = fma(c, Q, s * P);
                    }
                }
#pragma unroll
                for (int c = 0; c < NR; ++c) {
                    const double qr = r[6 + 2 * c], qi = r[7 + 2 * c];
                    if constexpr (KIND == FIELD_LAPLACE) {
                        ar[k][c] = fma(gr, qr, ar[k][c]);
                        ai[k][c] = fma(gr, qi, ai[k][c]);
                    } else {
                        ar[k][c] = fma(gr, qr, fma(-gi, qi, ar[k][c]));
                        ai[k][c] = fma(gr, qi, fma(gi, qr, ai[k][c]));
                    }
                }
            }
        }
    }
#pragma unroll
    for (int k = 0; k < TPT; ++k) {
        const int t = t0 + k * (int)blockDim.x;
        if (t >= nt) continue;
#pragma unroll
        for (int c = 0; c < NR; ++c) {
            const int cc = blockIdx.z * NR + c;
            if (cc < nc) part[((int64_t)blockIdx.y * nc + cc) * nt + t] = make_double2(ar[k][c], ai[k][c]);
        }
    }
}

// u[i] = sum over chunks of part[chunk][i], i < items: 16 items x 16 slices of
// the chunks per workgroup, then the slices in order
__global__ __launch_bounds__(256) void field_reduce_kernel(const double2 *__restrict__ part, int nchunk, int64_t items,
                                                           double2 *__restrict__ u) {
    __shared__ double2 s_sum[16][17];
    const int col = threadIdx.x & 15, sl = threadIdx.x >> 4;
    const int64_t i = (int64_t)blockIdx.x * 16 + col;
    double2 a = make_double2(0.0, 0.0);
    if (i < items)
        for (int k = sl; k < nchunk; k += 16) {
            const double2 v = part[(int64_t)k * items + i];
            a.x += v.x;
            a.y += v.y;
        }
    s_sum[sl][col] = a;
    __syncthreads();
    if (sl || i >= items) return;
#pragma unroll
    for (int k = 1; k < 16; ++k) {
        a.x += s_sum[k][col].x;
        a.y += s_sum[k][col].y;
    }
    u[i] = a;
}

// Small calls, and few targets with many densities: one workgroup per target and right-
// hand side straight from the node arrays, one launch without records, table and
// partial sums.  Bound by its own latency, a lane's pass over N / 256 nodes (30 us a
// call, and 1.7 us per 1,000 nodes; far 2.2), until some 600 workgroups fill the chip
// (then 6 ps a pair and density).
template <int KIND>
__global__ __launch_bounds__(256) void field_direct_kernel(const double *__restrict__ g, int64_t N,
                                                           const double2 *__restrict__ sigma,
                                                           const double *__restrict__ tgt, int nt, double kappa,
                                                           double eta, double2 *__restrict__ u) {
    __shared__ double2 s_sum[4];
    const int t = blockIdx.x, c = blockIdx.y;
    const double tx = tgt[3 * t], ty = tgt[3 * t + 1], tz = tgt[3 * t + 2];
    const double2 *q = sigma + (int64_t)c * N;
    double re = 0, im = 0;
    for (int64_t j = threadIdx.x; j < N; j += 256) {
        const double x = g[j], y = g[N + j], z = g[2 * N + j];
        const double nx = g[3 * N + j], ny = g[4 * N + j], nz = g[5 * N + j];
        double gr, gi;
        if constexpr (KIND == FIELD_FAR) {
            double sn, cs;
            sincos(-kappa * (tx * x + ty * y + tz * z), &sn, &cs);
            const double f = eta - kappa * (tx * nx + ty * ny + tz * nz);
            gr = -f * sn;
            gi = f * cs;
        } else {
            const double dx = tx - x, dy = ty - y, dz = tz - z;
            const double r2 = dx * dx + dy * dy + dz * dz, R = sqrt(r2);
            const double a = (nx * dx + ny * dy + nz * dz) / r2;
            if constexpr (KIND == FIELD_LAPLACE) {
                gr = (a + eta) / R;
                gi = 0.0;
            } else {
                double sn, cs;
                sincos(kappa * R, &sn, &cs);
                // e^{ikR}/R [a (1 - i k R) + i eta], a = n.d / R^2
                const double b = eta - a * kappa * R, er = cs / R, ei = sn / R;
                gr = er * a - ei * b;
                gi = er * b + ei * a;
            }
        }
        const double w = g[6 * N + j] * (0.25 / M_PI);
        const double qr = q[j].x * w, qi = q[j].y * w;
        re += gr * qr - gi * qi;
        im += gr * qi + gi * qr;
    }
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) {
        re += __shfl_xor(re, o, 64);
        im += __shfl_xor(im, o, 64);
    }
    if ((threadIdx.x & 63) == 0) s_sum[threadIdx.x >> 6] = make_double2(re, im);
    __syncthreads();
    if (threadIdx.x) return;
#pragma unroll
    for (int k = 1; k < 4; ++k) {
        re += s_sum[k].x;
        im += s_sum[k].y;
    }
    u[(int64_t)c * nt + t] = make_double2(re, im);
}

// The line between the two, from sweeps of 288 to 437,400 nodes, 1 to 1,024 targets and 1
// to 256 densities (us a call, direct / through records).
//  - Small calls.  The nodes set the direct kernel's latency: near, 1 and 8 densities,
//    3,060 nodes 34 / 41 and 34 / 54, 8,200 nodes 43 / 43 and 44 / 56; far 35 / 37 and 36 / 46,
//    48 / 40 and 48 / 48; zero frequency 34 / 34 and 34 / 53, 43 / 35 and 44 / 54; near, 64
//    densities, 16,400 nodes 59 / 113.  The work, counted with 256 nodes' worth for a
//    workgroup's start, sets the time beyond it: near, 840 nodes, 1 density, 1,024
//    targets 36 / 44; 4: 512 targets 40 / 43, 1,024 50 / 48; 64: 64 targets 49 / 55, 128 70 / 50.
//  - Few targets, many densities, any number of nodes: a lane of field_kernel is one
//    target and idle without, and the records are written and read for nothing: 65,280
//    nodes, 256 densities, 1 and 8 targets: near 236 / 1,410 and 819 / 1,411, far 338 /
//    1,164 and 615 / 1,157, zero frequency 235 / 935 and 718 / 934; 437,400 nodes, 64 densities,
//    8 targets: near 1,896 / 2,344, far 3,079 / 1,953, zero frequency 1,839 / 1,438.
template <int KIND>
static bool field_direct(int64_t N, int nt, int nrhs, int nr) {
    const int64_t nodes = (KIND == FIELD_NEAR ? 6144 + 768 * nr : 2048 + 1024 * nr) + 128 * std::min(nrhs, 64);
    const int64_t work = nr <= 4 ? 1 << (KIND == FIELD_LAPLACE ? 20 : 21) : KIND == FIELD_FAR ? 1 << 22 : 3 << 21;
    if (N <= nodes && (int64_t)nt * nrhs * (N + 256) <= work) return true;
    if (KIND == FIELD_NEAR) return nrhs >= 48 && nt <= (nrhs >= 128 ? 12 : nrhs >= 56 ? 8 : 4);
    if (KIND == FIELD_FAR) return nrhs >= 96 && nt <= 12;
    return nrhs >= 80 && nt <= (nrhs >= 128 ? 8 : 4);
}

// targets per lane where there are many: they share a node's LDS reads
constexpr int field_tpt(int nr) { return nr > 4 ? 2 : 4; }

// workgroups of 256 threads a CU holds at a time with many targets
template <int KIND, int NR>
static int field_resident() {
    static const int n = [] {
        int r = 0;
        AXS_HIP(hipOccupancyMaxActiveBlocksPerMultiprocessor(&r, field_kernel<KIND, NR, field_tpt(NR)>, 256, 0));
        return std::max(1, r);
    }();
    return n;
}

template <int KIND>
static int field_resident_for(int nr) {
    switch (nr) {
        case 1: return field_resident<KIND, 1>();
        case 2: return field_resident<KIND, 2>();
        case 3: return field_resident<KIND, 3>();
        case 4: return field_resident<KIND, 4>();
        case 5: return field_resident<KIND, 5>();
        case 6: return field_resident<KIND, 6>();
        case 7: return field_resident<KIND, 7>();
        default: return field_resident<KIND, 8>();
    }
}

template <int KIND, int NR>
static void launch_field(Ctx &c, dim3 grid, int bs, bool many, const double *rec, int64_t chunk, const double *tgt, int nt,
                         double eta, int wide, int nc, double2 *part) {
    constexpr int TPT = field_tpt(NR);
    if (many)
        hipLaunchKernelGGL((field_kernel<KIND, NR, TPT>), grid, dim3(bs), 0, c.stream, rec, c.N, chunk, tgt, nt,
                           c.kappa, c.kappa / (2.0 * M_PI), eta, wide, c.sctab, nc, part);
    else
        hipLaunchKernelGGL((field_kernel<KIND, NR, 1>), grid, dim3(bs), 0, c.stream, rec, c.N, chunk, tgt, nt,
                           c.kappa, c.kappa / (2.0 * M_PI), eta, wide, c.sctab, nc, part);
    AXS_HIP(hipGetLastError());
}

template <int KIND>
static void field_sums(Ctx &c, const void *sigma, int nrhs, const double *tgt, int nt, double sx, double sn,
                       double eta, int wide, void *u) {
    // groups of equal width, at most 8 rhs each
    const int groups = (int)ceil_div(nrhs, 8), nr = (int)ceil_div(nrhs, groups);
    if (field_direct<KIND>(c.N, nt, nrhs, nr)) {
        hipLaunchKernelGGL(field_direct_kernel<KIND>, dim3(nt, nrhs), dim3(256), 0, c.stream, c.g64, c.N,
                           (const double2 *)sigma, tgt, nt, c.kappa, eta, (double2 *)u);
        AXS_HIP(hipGetLastError());
        return;
    }
    const size_t rec_group = (size_t)c.N * (6 + 2 * nr) * sizeof(double);
    // groups of one pass: as many as have their records within FIELD_SCRATCH (at least one)
    const int gb = (int)std::max<size_t>(1, std::min<size_t>(groups, FIELD_SCRATCH / rec_group));
    // up to 64 targets: one wavefront per workgroup; from 1,024 targets on 4 per lane
    // (2 with more than 4 densities), if that leaves three workgroups a CU
    // (18,860 nodes: 1,024 targets 83 us with 4, 69 with 1; 3,000 targets the same)
    const int64_t most = std::max<int64_t>(1, std::min<int64_t>(1024, c.N / 64));   // chunks
    const bool many = nt >= 1024 && ceil_div(nt, 256 * field_tpt(nr)) * gb * most >= 768;
    const int bs = nt > 64 ? 256 : 64, tile = bs * (many ? field_tpt(nr) : 1);
    const int tiles = (int)ceil_div(nt, tile);
    // chunks of at least 64 nodes, at most 1,024.  Few targets: as many as make 1,024
    // workgroups of four wavefronts (4 per CU; more cost as much as they fill).  Many: as
    // fill whole rounds of the workgroups the CUs hold at a time, one or up to four
    // where the tiles do not divide a round well (20,000 directions, 4 densities: 38
    // chunks, 760 workgroups of the 768 held, 0.65 ms; 52 chunks, a round and a third, 0.70)
    const int64_t all = (int64_t)tiles * gb;
    int64_t want = std::max<int64_t>(1, std::min(most, ceil_div((int64_t)1024 * 256, all * bs)));
    if (many) {
        const int64_t round = 256 * (int64_t)field_resident_for<KIND>(nr);
        double fill = 0.0;
        for (int k = 1; k <= 4; ++k) {
            const int64_t n = std::max<int64_t>(1, std::min(most, k * round / all));
            const double f = (double)(all * n) / (double)(ceil_div(all * n, round) * round);
            if (f > fill + 0.03) fill = f, want = n;
        }
    }
    // a pass's partial sums stay within FIELD_SCRATCH too (8 rhs on 65,535 targets, the most
    // of one group, have room for 32 chunks)
    const size_t part_chunk = (size_t)std::min(nrhs, gb * nr) * nt * sizeof(double2);
    want = std::max<int64_t>(1, std::min<int64_t>(want, FIELD_SCRATCH / part_chunk));
    const int64_t chunk = ceil_div(c.N, want);
    const int nchunk = (int)ceil_div(c.N, chunk);
    double *rec = (double *)c.scratch(WS_TMP, rec_group * gb);
    double2 *sums = nchunk > 1 ? (double2 *)c.scratch(WS_TMP2, nchunk * part_chunk) : nullptr;
    for (int g0 = 0; g0 < groups; g0 += gb) {
        const int ng = std::min(gb, groups - g0), c0 = g0 * nr, nc = std::min(nrhs - c0, ng * nr);
        double2 *out = (double2 *)u + (int64_t)c0 * nt, *part = nchunk > 1 ? sums : out;
        hipLaunchKernelGGL(field_records_kernel, dim3((unsigned)ceil_div(c.N, 256), ng), dim3(256), 0, c.stream, c.g64,
                           c.N, (const double2 *)sigma, c0, nrhs, nr, sx, sn, rec);
        AXS_HIP(hipGetLastError());
        const dim3 grid(tiles, nchunk, ng);
        switch (nr) {
#define AXS_FIELD_NR(NR_)                                                                                      \
    case NR_:                                                                                                  \
        launch_field<KIND, NR_>(c, grid, bs, many, rec, chunk, tgt, nt, eta, wide, nc, part);                  \
        break;
            AXS_FIELD_NR(1)
            AXS_FIELD_NR(2)
            AXS_FIELD_NR(3)
            AXS_FIELD_NR(4)
            AXS_FIELD_NR(5)
            AXS_FIELD_NR(6)
            AXS_FIELD_NR(7)
            AXS_FIELD_NR(8)
#undef AXS_FIELD_NR
        }
        if (nchunk > 1) {
            const int64_t items = (int64_t)nc * nt;
            hipLaunchKernelGGL(field_reduce_kernel, dim3((unsigned)ceil_div(items, 16)), dim3(256), 0, c.stream, part,
                               nchunk, items, out);
            AXS_HIP(hipGetLastError());
        }
    }
}

// radius about the origin that holds every body
static double scene_radius(const Ctx &c) {
    double r = 0;
    for (auto &b : c.bodies)
        r = std::max(r, std::sqrt(b.centre[0] * b.centre[0] + b.centre[1] * b.centre[1] + b.centre[2] * b.centre[2]) +
                            b.bound_radius);
    return r;
}

// tmax: largest |target| (host); NaN or Inf there counts as wide
void eval_field_launch(Ctx &c, const void *sigma, int nrhs, const double *tgt_dev, int nt, double tmax, void *u) {
    if (c.kappa == 0) {
        field_sums<FIELD_LAPLACE>(c, sigma, nrhs, tgt_dev, nt, 1.0, 1.0, c.eta, 0, u);
        return;
    }
    const double k2pi = c.kappa / (2.0 * M_PI);
    const int wide = !((scene_radius(c) + tmax) * k2pi < 549755813888.0);   // 2^39 revolutions
    field_sums<FIELD_NEAR>(c, sigma, nrhs, tgt_dev, nt, 1.0, 1.0, c.eta, wide, u);
}

void far_field_launch(Ctx &c, const void *sigma, int nrhs, const double *xh_dev, int nd, double xmax, void *u) {
    const double k2pi = c.kappa / (2.0 * M_PI);
    const int wide = !(scene_radius(c) * xmax * k2pi < 549755813888.0);
    field_sums<FIELD_FAR>(c, sigma, nrhs, xh_dev, nd, -k2pi, -c.kappa, c.eta, wide, u);
}

}  // namespace axs
