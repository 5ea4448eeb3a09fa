// Per-bubble spherical-harmonic preconditioner for the single-layer system.
//
// On a sphere of radius R the single-layer operator is diagonal in spherical
// harmonics with eigenvalue R/(2n+1) for degree n. Every bubble here is a
// closed surface whose vertices carry the parametrisation of a template unit
// sphere (the (theta, phi) of the initial mesh, as for the paper's shape
// filter, Section 3.7), so an approximate inverse of L restricted to bubble b
// is
//   P_b^{-1} x = (1/R_b) [ c x + G diag(2n+1 - c) G+ x ],   c = 2 (nmax + 1) + 1,
// with G the real harmonics of degree <= nmax sampled at the template
// vertices, G+ = (G^T W G)^{-1} G^T W their weighted least-squares projector
// (W = template vertex areas), and R_b = sqrt(area_b / 4 pi). Degrees above
// nmax get the first unresolved eigenvalue. Applied as a right
// preconditioner inside GMRES, so the residual GMRES monitors is the true
// one and the solution is unchanged.
#include <algorithm>
#include <cmath>
#include <complex>
#include <type_traits>
#include <vector>

#include <condition_variable>
#include <exception>
#include <mutex>
#include <thread>

#include "ctx.h"

namespace bfm {

static unsigned nblk(int64_t n, int t) { return (unsigned)((n + t - 1) / t); }

// Real harmonics of degree 0..nmax at unit vector d, orthonormal on the
// unit sphere and without the Condon-Shortley phase: for each degree n the
// order-0 value, then the cos(m lon) and sin(m lon) parts of orders 1..n.
// The recurrence yields sqrt((n-m)!/(n+m)!) P_n^m(cos theta) e^{i m lon};
// the factor sqrt((2n+1)/4pi) (times sqrt(2) for m > 0) normalises it.
static void sh_row(int nmax, const double d[3], double *row) {
    using cplx = std::complex<double>;
    const double x = d[0], y = d[1], z = d[2];
    const double r2 = x * x + y * y + z * z;
    std::vector<cplx> col(nmax + 1);
    cplx diag(1.0, 0.0);
    for (int m = 0; m <= nmax; ++m) {
        if (m > 0) diag *= cplx(x, y) * std::sqrt((2.0 * m - 1.0) / (2.0 * m));
        cplx pr(0.0, 0.0), cr = diag;
        for (int n = m; n <= nmax; ++n) {
            if (n > m) {
                const double a = std::sqrt((double)(n - m) * (n + m));
                const double b = (n - m - 1 > 0) ? std::sqrt((double)(n - m - 1) * (n + m - 1)) : 0.0;
                const cplx nr = ((2.0 * n - 1.0) * z * cr - r2 * b * pr) / a;
                pr = cr;
                cr = nr;
            }
            const double f = std::sqrt((2.0 * n + 1.0) / (4.0 * 3.14159265358979323846)) *
                             (m > 0 ? std::sqrt(2.0) : 1.0);
            if (m == 0) {
                row[n * n] = f * cr.real();
            } else {
                row[n * n + 2 * m - 1] = f * cr.real();
                row[n * n + 2 * m] = f * cr.imag();
            }
        }
    }
}

// In-place Cholesky solve of S X = B (S n x n SPD, row-major; B n x k).
static void cholesky_solve(int n, std::vector<double> &S, std::vector<double> &B, int k) {
    for (int j = 0; j < n; ++j) {
        double d = S[(size_t)j * n + j];
        for (int p = 0; p < j; ++p) d -= S[(size_t)j * n + p] * S[(size_t)j * n + p];
        BFM_CHECK(d > 0.0, BFM_EINVAL, "template basis: Gram matrix not positive definite");
        d = std::sqrt(d);
        S[(size_t)j * n + j] = d;
        for (int i = j + 1; i < n; ++i) {
            double v = S[(size_t)i * n + j];
            for (int p = 0; p < j; ++p) v -= S[(size_t)i * n + p] * S[(size_t)j * n + p];
            S[(size_t)i * n + j] = v / d;
        }
    }
    for (int c = 0; c < k; ++c) {
        for (int i = 0; i < n; ++i) {  // forward
            double v = B[(size_t)i * k + c];
            for (int p = 0; p < i; ++p) v -= S[(size_t)i * n + p] * B[(size_t)p * k + c];
            B[(size_t)i * k + c] = v / S[(size_t)i * n + i];
        }
        for (int i = n - 1; i >= 0; --i) {  // backward
            double v = B[(size_t)i * k + c];
            for (int p = i + 1; p < n; ++p) v -= S[(size_t)p * n + i] * B[(size_t)p * k + c];
            B[(size_t)i * k + c] = v / S[(size_t)i * n + i];
        }
    }
}

// Uploads G (row-major [nd][nc] on the host) and its least-squares
// projector Gp = (G^T W G)^{-1} G^T W (W = diag(wv)) in the device layouts.
static void basis_upload(int nd, int nc, const std::vector<double> &G, const std::vector<double> &wv, ShBasis &B,
                         hipStream_t st) {
    std::vector<double> S((size_t)nc * nc, 0.0), R((size_t)nc * nd, 0.0);
    for (int i = 0; i < nc; ++i)
        for (int v = 0; v < nd; ++v) R[(size_t)i * nd + v] = G[(size_t)v * nc + i] * wv[v];
    for (int i = 0; i < nc; ++i)
        for (int j = 0; j <= i; ++j) {
            double s = 0.0;
            for (int v = 0; v < nd; ++v) s += R[(size_t)i * nd + v] * G[(size_t)v * nc + j];
            S[(size_t)i * nc + j] = S[(size_t)j * nc + i] = s;
        }
    cholesky_solve(nc, S, R, nd);
    // device layouts (column-major): G [nd x nc], Gp [nc x nd]
    std::vector<double> Gc((size_t)nd * nc), Gpc((size_t)nc * nd);
    for (int v = 0; v < nd; ++v)
        for (int i = 0; i < nc; ++i) {
            Gc[(size_t)i * nd + v] = G[(size_t)v * nc + i];
            Gpc[(size_t)v * nc + i] = R[(size_t)i * nd + v];
        }
    B.G.ensure(Gc.size());
    B.Gp.ensure(Gpc.size());
    BFM_HIP(hipMemcpyAsync(B.G.get(), Gc.data(), sizeof(double) * Gc.size(), hipMemcpyHostToDevice, st));
    BFM_HIP(hipMemcpyAsync(B.Gp.get(), Gpc.data(), sizeof(double) * Gpc.size(), hipMemcpyHostToDevice, st));
    BFM_HIP(hipStreamSynchronize(st));
    B.nc = nc;
    B.nd = nd;
}

// Real trigonometric basis of the torus angles (Section 3.7, spherical7: the
// real form of e^{i(n theta + m phi)}, |n|, |m| <= h): the products of
// {1, cos k theta, sin k theta : k = 1..h} with the same set in phi, theta
// functions slowest.
static void trig_row(int h, double th, double ph, double *row) {
    const int w = 2 * h + 1;
    std::vector<double> a(w), b(w);
    a[0] = b[0] = 1.0;
    for (int k = 1; k <= h; ++k) {
        a[2 * k - 1] = std::cos(k * th);
        a[2 * k] = std::sin(k * th);
        b[2 * k - 1] = std::cos(k * ph);
        b[2 * k] = std::sin(k * ph);
    }
    for (int i = 0; i < w; ++i)
        for (int j = 0; j < w; ++j) row[i * w + j] = a[i] * b[j];
}

void torus_basis_build(const Precond &P, int h, ShBasis &B, hipStream_t st) {
    const int nd = P.nd;
    BFM_CHECK(nd > 0 && P.genus == 1 && !P.ang_h.empty(), BFM_EINVAL, "no torus template set");
    const int nc = (2 * h + 1) * (2 * h + 1);
    BFM_CHECK(h >= 0 && nc <= nd, BFM_EINVAL, "trigonometric degree must satisfy (2 degree + 1)^2 <= vertices per bubble");
    if (B.genus == 1 && B.nmax == h && B.nd == nd && B.weighted == 0 && B.gen == P.gen) return;
    std::vector<double> G((size_t)nd * nc), wv(nd, 1.0);
    for (int v = 0; v < nd; ++v) trig_row(h, P.ang_h[2 * v], P.ang_h[2 * v + 1], &G[(size_t)v * nc]);
    basis_upload(nd, nc, G, wv, B, st);
    B.nmax = h;
    B.weighted = 0;
    B.genus = 1;
    B.gen = P.gen;
}

void sh_basis_build(const Precond &P, int nmax, ShBasis &B, hipStream_t st, bool weighted) {
    const int nd = P.nd;
    BFM_CHECK(nd > 0 && P.genus == 0 && !P.dirs_h.empty(), BFM_EINVAL, "no sphere template set");
    BFM_CHECK(nmax >= 0 && (nmax + 1) * (nmax + 1) <= nd, BFM_EINVAL,
              "harmonic degree must satisfy (degree + 1)^2 <= vertices per bubble");
    if (B.genus == 0 && B.nmax == nmax && B.nd == nd && B.weighted == (int)weighted && B.gen == P.gen) return;
    const int nc = (nmax + 1) * (nmax + 1);
    // weights: template vertex areas from the first bubble's triangles on the
    // unit directions, or all ones (plain least squares)
    std::vector<double> wv(nd, weighted ? 0.0 : 1.0);
    for (size_t k = 0; weighted && k + 2 < P.tri_h.size(); k += 3) {
        const double *a = &P.dirs_h[3 * P.tri_h[k]], *b = &P.dirs_h[3 * P.tri_h[k + 1]],
                     *d = &P.dirs_h[3 * P.tri_h[k + 2]];
        const double e1[3] = {b[0] - a[0], b[1] - a[1], b[2] - a[2]};
        const double e2[3] = {d[0] - a[0], d[1] - a[1], d[2] - a[2]};
        const double cx = e1[1] * e2[2] - e1[2] * e2[1], cy = e1[2] * e2[0] - e1[0] * e2[2],
                     cz = e1[0] * e2[1] - e1[1] * e2[0];
        const double A = 0.5 * std::sqrt(cx * cx + cy * cy + cz * cz);
        for (int t = 0; t < 3; ++t) wv[P.tri_h[k + t]] += A / 3.0;
    }
    std::vector<double> G((size_t)nd * nc);  // row-major [nd][nc]
    for (int v = 0; v < nd; ++v) sh_row(nmax, &P.dirs_h[3 * v], &G[(size_t)v * nc]);
    basis_upload(nd, nc, G, wv, B, st);
    B.nmax = nmax;
    B.weighted = (int)weighted;
    B.genus = 0;
    B.gen = P.gen;
}

void precond_build(bfm_ctx *c) {
    Precond &P = c->pre;
    const int nmax = c->opt.precond_degree;
    if (P.ready && P.nmax == nmax) return;
    sh_basis_build(P, nmax, P.basis, c->stream);
    const int nc = P.basis.nc;
    std::vector<double> fac(nc);
    const double cc = 2.0 * (nmax + 1) + 1.0;
    for (int n = 0; n <= nmax; ++n)
        for (int i = n * n; i < (n + 1) * (n + 1); ++i) fac[i] = (2.0 * n + 1.0) - cc;
    P.fac.ensure(nc);
    BFM_HIP(hipMemcpyAsync(P.fac.get(), fac.data(), sizeof(double) * nc, hipMemcpyHostToDevice, c->stream));
    BFM_HIP(hipStreamSynchronize(c->stream));
    P.nmax = nmax;
    P.nc = nc;
    P.cc = cc;
    P.ready = true;
}

// Per-bubble equivalent radius sqrt(area / 4 pi) from the vertex weights.
__global__ void k_bubble_radius(const double *s, int nd, double *R) {
    __shared__ double red[256];
    const int b = blockIdx.x;
    double a = 0.0;
    for (int v = threadIdx.x; v < nd; v += 256) a += s[(int64_t)b * nd + v];
    red[threadIdx.x] = a;
    __syncthreads();
    for (int st = 128; st > 0; st >>= 1) {
        if ((int)threadIdx.x < st) red[threadIdx.x] += red[threadIdx.x + st];
        __syncthreads();
    }
    if (threadIdx.x == 0) R[b] = sqrt(red[0] / (4.0 * 3.14159265358979323846));
}

// C = A B, column-major FP64 on MFMA
// (v_mfma_f64_16x16x4f64). A workgroup of 4 waves owns a 64 x 64 tile of C
// (each wave a 32 x 32 quarter, 2 x 2 MFMA blocks); K advances in chunks of
// 32 staged through LDS, the next chunk's elements loaded into registers
// while the current one is multiplied. C aliases neither A nor B.
// MFMA operand layout: lane l supplies A[l % 16][l / 16] and B[l / 16][l % 16]
// of a 16 x 4 by 4 x 16 product; element r of the result holds row
// l / 16 + 4 r, column l % 16.
typedef double dbl4 __attribute__((ext_vector_type(4)));

constexpr int kGemmKC = 32;  // K chunk

__global__ void __launch_bounds__(256) k_gemm_nn(int M, int N, int K, const double *A, int lda,
                                                 const double *B, int ldb, double *C, int ldc) {
    // A and B chunks ([k][row], [k][col]); after the products the same LDS
    // holds the 64 x 64 result tile ([col][row]) for coalesced stores
    __shared__ double sbuf[2 * kGemmKC * (64 + 1)];
    static_assert(2 * kGemmKC >= 64, "the result tile fits in the chunk buffers");
    double(*As)[64 + 1] = reinterpret_cast<double(*)[64 + 1]>(sbuf);
    double(*Bs)[64 + 1] = reinterpret_cast<double(*)[64 + 1]>(sbuf + kGemmKC * (64 + 1));
    double(*Cs)[64 + 1] = reinterpret_cast<double(*)[64 + 1]>(sbuf);
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int i0 = blockIdx.x * 64, j0 = blockIdx.y * 64;
    const int wi = (wave >> 1) * 32, wj = (wave & 1) * 32;
    dbl4 acc[2][2];
    for (int a = 0; a < 2; ++a)
        for (int b = 0; b < 2; ++b) acc[a][b] = dbl4{0.0, 0.0, 0.0, 0.0};
    // element e = tid + 256 u of a chunk: A (64 rows x 32 k, rows fastest),
    // B (32 k x 64 columns, k fastest)
    double ra[8], rb[8];
    auto load = [&](int k0) {
#pragma unroll
        for (int u = 0; u < 8; ++u) {
            const int e = tid + 256 * u;
            const int ii = e & 63, kk = e >> 6;
            const int gi = i0 + ii, gk = k0 + kk;
            ra[u] = (gi < M && gk < K) ? A[(int64_t)gk * lda + gi] : 0.0;
            const int kq = e & 31, jj = e >> 5;
            const int gj = j0 + jj, gk2 = k0 + kq;
            rb[u] = (gj < N && gk2 < K) ? B[(int64_t)gj * ldb + gk2] : 0.0;
        }
    };
    if (K > 0) load(0);
    for (int k0 = 0; k0 < K; k0 += kGemmKC) {
#pragma unroll
        for (int u = 0; u < 8; ++u) {
            const int e = tid + 256 * u;
            As[e >> 6][e & 63] = ra[u];
            Bs[e & 31][e >> 5] = rb[u];
        }
        __syncthreads();
        if (k0 + kGemmKC < K) load(k0 + kGemmKC);  // in flight during the products
#pragma unroll
        for (int k4 = 0; k4 < kGemmKC / 4; ++k4) {
            const int kk = 4 * k4 + lane / 16;
            double af[2], bf[2];
#pragma unroll
            for (int a = 0; a < 2; ++a) af[a] = As[kk][wi + 16 * a + lane % 16];
#pragma unroll
            for (int b = 0; b < 2; ++b) bf[b] = Bs[kk][wj + 16 * b + lane % 16];
#pragma unroll
            for (int a = 0; a < 2; ++a)
#pragma unroll
                for (int b = 0; b < 2; ++b)
                    acc[a][b] = __builtin_amdgcn_mfma_f64_16x16x4f64(af[a], bf[b], acc[a][b], 0, 0, 0);
        }
        __syncthreads();
    }
    // the tile through LDS, then each wave stores whole 64-row columns
    // (512 contiguous bytes) instead of 16 columns x 4 rows
    __syncthreads();
#pragma unroll
    for (int a = 0; a < 2; ++a)
#pragma unroll
        for (int b = 0; b < 2; ++b)
#pragma unroll
            for (int r = 0; r < 4; ++r) Cs[wj + 16 * b + lane % 16][wi + 16 * a + lane / 16 + 4 * r] = acc[a][b][r];
    __syncthreads();
    const int gi = i0 + lane;
#pragma unroll 4
    for (int cc = wave; cc < 64; cc += 4) {
        const int gj = j0 + cc;
        if (gi < M && gj < N) C[(int64_t)gj * ldc + gi] = Cs[cc][lane];
    }
}

void gemm_nn_f64(int M, int N, int K, const double *A, int lda, const double *B, int ldb, double *C, int ldc,
                 hipStream_t st) {
    if (M <= 0 || N <= 0) return;
    k_gemm_nn<<<dim3((M + 63) / 64, (N + 63) / 64), 256, 0, st>>>(M, N, K, A, lda, B, ldb, C, ldc);
    BFM_LAUNCHED();
}

// X[b][v] = in_s at vertex v of bubble b (caller order), with the bubble's sums
// xsum[0][b] = s . X, xsum[1][b] = U . X (U null: none). One workgroup per bubble.
__global__ void __launch_bounds__(256) k_pre_gather(const double *__restrict__ in_s, const int *__restrict__ iperm,
                                                    const double *__restrict__ s, const double *__restrict__ U, int nd,
                                                    int nb, double *__restrict__ X, double *__restrict__ xsum) {
    __shared__ double red[2][4];
    const int b = blockIdx.x;
    double a0 = 0.0, a1 = 0.0;
    for (int v = threadIdx.x; v < nd; v += 256) {
        const int64_t o = (int64_t)b * nd + v;
        const double x = in_s[iperm[o]];
        X[o] = x;
        if (U) {
            a0 = fma(s[o], x, a0);
            a1 = fma(U[o], x, a1);
        }
    }
    if (!U) return;
    for (int o = 32; o > 0; o >>= 1) {
        a0 += __shfl_xor(a0, o);
        a1 += __shfl_xor(a1, o);
    }
    if ((threadIdx.x & 63) == 0) {
        red[0][threadIdx.x >> 6] = a0;
        red[1][threadIdx.x >> 6] = a1;
    }
    __syncthreads();
    if (threadIdx.x < 2) {
        const double *r = red[threadIdx.x];
        xsum[(int64_t)threadIdx.x * nb + b] = ((r[0] + r[1]) + r[2]) + r[3];
    }
}

// Two doubles at any double's address, one load
struct __attribute__((packed, aligned(8))) PrePair {
    double x, y;
};

// A lane's B values of a row of K for B MFMA steps from position s on: the lane
// takes positions s + B (lane / 16) + 0 .. B - 1 (which k of a step a lane holds
// is free as long as both operands agree), so a row is read in runs of 8 B bytes
// by 16-byte loads. Near the row's end the run is moved back to stay inside
// (len >= B); v0 is its first position, and positions the lane does not own
// (below its first, or from `end` on) come as zeros.
template <int B>
__device__ inline void pre_run(const double *row, int s, int len, int end, double (&x)[B], int &v0) {
    const int first = s + B * (((int)threadIdx.x & 63) >> 4);
    v0 = min(first, len - B);
    if constexpr (B % 2 == 0) {
#pragma unroll
        for (int u = 0; u < B; u += 2) {
            const PrePair q = *reinterpret_cast<const PrePair *>(row + v0 + u);
            x[u] = q.x;
            x[u + 1] = q.y;
        }
    } else {
#pragma unroll
        for (int u = 0; u < B; ++u) x[u] = row[v0 + u];
    }
#pragma unroll
    for (int u = 0; u < B; ++u) x[u] = v0 + u >= first && v0 + u < end ? x[u] : 0.0;
}

// C[i][b] = fac[i] sum_v T(i, v) X[b][v] (fac null: 1), T(i, v) = T[v * sv + i * si],
// C column-major [nc x nb]. One tile of 16 NI coefficients x 16 NJ bubbles per
// workgroup, the sum over v split over its four waves. A product of this size
// (169 x 642 x 1000) is bound by the latency of a wave's chain of loads: 16 x 16
// tiles with four waves each give it 2772 short chains, of B steps' loads at a
// time. With many bubbles it is bound by reading the operands from L2 once per
// tile, and the tiles are wider (kCoefWide).
template <int NI, int NJ, int B>
__global__ void __launch_bounds__(256) k_pre_coef(int nc, int nb, int nd, const double *__restrict__ T, int sv, int si,
                                                  const double *__restrict__ X, const double *__restrict__ fac,
                                                  double *__restrict__ C) {
    __shared__ double red[3][NI * NJ * 4][64];
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6, kq = lane >> 4, rl = lane & 15;
    const int i0 = blockIdx.x * 16 * NI, b0 = blockIdx.y * 16 * NJ;
    const int steps = (nd + 3) / 4, s0 = 4 * (steps * wave / 4), s1 = min(nd, 4 * (steps * (wave + 1) / 4));
    dbl4 acc[NJ][NI];
#pragma unroll
    for (int j = 0; j < NJ; ++j)
#pragma unroll
        for (int i = 0; i < NI; ++i) acc[j][i] = dbl4{0.0, 0.0, 0.0, 0.0};
    for (int s = s0; s < s1; s += 4 * B) {
        double x[NJ][B], t[NI][B];
        int v0 = 0;
#pragma unroll
        for (int j = 0; j < NJ; ++j)
            pre_run<B>(X + (int64_t)min(b0 + 16 * j + rl, nb - 1) * nd, s, nd, s1, x[j], v0);
#pragma unroll
        for (int i = 0; i < NI; ++i)
#pragma unroll
            for (int u = 0; u < B; ++u)
                t[i][u] = T[(int64_t)(v0 + u) * sv + (int64_t)min(i0 + 16 * i + rl, nc - 1) * si];
#pragma unroll
        for (int u = 0; u < B; ++u)
#pragma unroll
            for (int j = 0; j < NJ; ++j)
#pragma unroll
                for (int i = 0; i < NI; ++i)
                    acc[j][i] = __builtin_amdgcn_mfma_f64_16x16x4f64(x[j][u], t[i][u], acc[j][i], 0, 0, 0);
    }
    if (wave > 0)
#pragma unroll
        for (int j = 0; j < NJ; ++j)
#pragma unroll
            for (int i = 0; i < NI; ++i)
#pragma unroll
                for (int r = 0; r < 4; ++r) red[wave - 1][(j * NI + i) * 4 + r][lane] = acc[j][i][r];
    __syncthreads();
    if (wave > 0) return;
#pragma unroll
    for (int j = 0; j < NJ; ++j)
#pragma unroll
        for (int i = 0; i < NI; ++i)
#pragma unroll
            for (int r = 0; r < 4; ++r) {  // bubble kq + 4 r, coefficient rl of the block
                const int e = (j * NI + i) * 4 + r, b = b0 + 16 * j + kq + 4 * r, ic = i0 + 16 * i + rl;
                const double v = ((acc[j][i][r] + red[0][e][lane]) + red[1][e][lane]) + red[2][e][lane];
                if (b < nb && ic < nc) C[(int64_t)b * nc + ic] = fac ? fac[ic] * v : v;
            }
}

// out_s at vertex v of bubble b (+)= ((G C + cc X)[v][b]) / R[b] (+ cy[b]); G
// column-major [nd x nc]. One wave per 32 vertices x 16 NJ bubbles, B steps'
// loads in flight, the result's places loaded ahead of them. Bound by the
// scattered result: wider tiles, which read less, change little (kOutWide).
template <int NJ, int B>
__global__ void __launch_bounds__(64) k_pre_out(int nc, int nb, int nd, const double *__restrict__ G,
                                                const double *__restrict__ C, double cc,
                                                const double *__restrict__ X, const double *__restrict__ R,
                                                const double *__restrict__ cy, const int *__restrict__ iperm, int add,
                                                double *__restrict__ out) {
    const int lane = threadIdx.x, kq = lane >> 4, rl = lane & 15;
    const int v0 = blockIdx.x * 32, b0 = blockIdx.y * 16 * NJ;
    const int va = min(v0 + rl, nd - 1), vb = min(v0 + 16 + rl, nd - 1);
    int at[NJ][2][4];
#pragma unroll
    for (int j = 0; j < NJ; ++j)
#pragma unroll
        for (int h = 0; h < 2; ++h)
#pragma unroll
            for (int r = 0; r < 4; ++r)
                at[j][h][r] = iperm[(int64_t)min(b0 + 16 * j + kq + 4 * r, nb - 1) * nd + (h ? vb : va)];
    dbl4 acc[NJ][2];
#pragma unroll
    for (int j = 0; j < NJ; ++j) acc[j][0] = acc[j][1] = dbl4{0.0, 0.0, 0.0, 0.0};
    for (int s = 0; s < nc; s += 4 * B) {
        double c[NJ][B], ga[B], gb[B];
        int c0 = 0;
#pragma unroll
        for (int j = 0; j < NJ; ++j)
            pre_run<B>(C + (int64_t)min(b0 + 16 * j + rl, nb - 1) * nc, s, nc, nc, c[j], c0);
#pragma unroll
        for (int u = 0; u < B; ++u) {
            ga[u] = G[(int64_t)(c0 + u) * nd + va];
            gb[u] = G[(int64_t)(c0 + u) * nd + vb];
        }
#pragma unroll
        for (int u = 0; u < B; ++u)
#pragma unroll
            for (int j = 0; j < NJ; ++j) {
                acc[j][0] = __builtin_amdgcn_mfma_f64_16x16x4f64(c[j][u], ga[u], acc[j][0], 0, 0, 0);
                acc[j][1] = __builtin_amdgcn_mfma_f64_16x16x4f64(c[j][u], gb[u], acc[j][1], 0, 0, 0);
            }
    }
#pragma unroll
    for (int j = 0; j < NJ; ++j)
#pragma unroll
        for (int h = 0; h < 2; ++h) {
            const int v = v0 + 16 * h + rl;
            if (v >= nd) continue;
#pragma unroll
            for (int r = 0; r < 4; ++r) {
                const int b = b0 + 16 * j + kq + 4 * r;
                if (b >= nb) continue;
                const double y = fma(cc, X[(int64_t)b * nd + v], acc[j][h][r]) / R[b] + (cy ? cy[b] : 0.0);
                double *d = out + at[j][h][r];
                *d = add ? *d + y : y;
            }
        }
}

// ---------------------------------------------------------------------------
// Coarse correction (two-level form). With Z the per-bubble indicator
// vectors and S = diag(s), the coarse matrix A_c = (S Z)^T L Z couples the
// bubbles' mean values: A_c[a][a] = sum_{i, j in a} s_i L_ij (exact, from
// the bubble's own pairs and the singular diagonal), A_c[a][b] =
// area_a area_b / (4 pi |c_a - c_b|) for a != b (each bubble seen from the
// other as a point monopole at its area centroid). After the block step
// x = P_b^{-1} v the correction adds Z A_c^{-1} (S Z)^T (v - L x), with the
// residual's bubble sums formed from the same model of L:
//   (S Z)^T L x |_a = U_a . x_a + area_a sum_{b != a} m_b / (4 pi |c_a - c_b|),
//   U_a = s_a^T L_aa (per vertex), m_b = sum_{j in b} s_j x_j.

// area and area-weighted centroid of every bubble
__global__ void k_coarse_geom(const double *xyz, const double *s, int nd, double *cen, double *area, double *usum) {
    __shared__ double red[4][256];
    const int b = blockIdx.x;
    double a[4] = {0, 0, 0, 0};
    for (int v = threadIdx.x; v < nd; v += 256) {
        const int64_t o = (int64_t)b * nd + v;
        const double w = s[o];
        a[0] += w * xyz[3 * o];
        a[1] += w * xyz[3 * o + 1];
        a[2] += w * xyz[3 * o + 2];
        a[3] += w;
    }
    for (int k = 0; k < 4; ++k) red[k][threadIdx.x] = a[k];
    __syncthreads();
    for (int st = 128; st > 0; st >>= 1) {
        if ((int)threadIdx.x < st)
            for (int k = 0; k < 4; ++k) red[k][threadIdx.x] += red[k][threadIdx.x + st];
        __syncthreads();
    }
    if (threadIdx.x == 0) {
        for (int k = 0; k < 3; ++k) cen[3 * b + k] = red[k][0] / red[3][0];
        area[b] = red[3][0];
        usum[b] = 0.0;  // summed by k_coarse_u
    }
}

// U_j = s_j (sum_{i in a, i != j} s_i / (4 pi r_ij) + L_jj) for vertex j of
// bubble a (caller order), with the singular diagonal L_jj in its
// translation-free form summed over the own bubble only:
//   L_jj = n_j . [sum_i M_ji (r_i - r_j) - sum_i L_ji n_i],
//   M_ji = s_i n_i . (r_j - r_i) / (4 pi r^3),  L_ji = s_i / (4 pi r).
// (The other bubbles' closed surfaces contribute only their discretisation
// error to these sums; the coarse space is a preconditioner, so the own
// bubble suffices and the build does not wait for the diagonal pass.)
// One workgroup per tile (vertex block of 256, bubble; a grid-stride loop
// over tiles: a capped grid that left wave slots free for the octree build
// beside it measured slower, its kernels started later); the bubble's points
// pass through LDS in chunks. The sums run in FP32 on coordinates relative to the
// bubble's centroid (formed in FP64): the coarse space only preconditions,
// and at a mesh spacing of a tenth of the radius the relative error of r_ij
// is about 1e-6. The pair i = j (r = 0) is masked. usum[b] += the tile's
// sum of U (the coarse matrix's diagonal).
__global__ void __launch_bounds__(256) k_coarse_u(const double *xyz, const double *s, const double *nrm, int64_t nv,
                                                  int nd, int nb, const double *cen, double *U, double *usum) {
    constexpr int CH = 256;
    __shared__ float4 sp[CH];  // x, y, z, s
    __shared__ float4 sn[CH];  // n_x, n_y, n_z
    __shared__ double red[4];
    const int nvb = (nd + 255) / 256;
    for (int64_t tile = blockIdx.x; tile < (int64_t)nvb * nb; tile += gridDim.x) {
        const int b = (int)(tile / nvb);
        const int j = (int)(tile - (int64_t)b * nvb) * 256 + threadIdx.x;
        const int64_t base = (int64_t)b * nd;
        const bool ok = j < nd;
        const int64_t oj = base + (ok ? j : 0);
        const double c0x = cen[3 * b], c0y = cen[3 * b + 1], c0z = cen[3 * b + 2];
        const float xj = (float)(xyz[3 * oj] - c0x), yj = (float)(xyz[3 * oj + 1] - c0y),
                    zj = (float)(xyz[3 * oj + 2] - c0z);
        float acc = 0.f, ax = 0.f, ay = 0.f, az = 0.f;  // sum s_i / r; sum M-type vector - L-type vector
        for (int c0 = 0; c0 < nd; c0 += CH) {
            const int cn = min(CH, nd - c0);
            __syncthreads();
            for (int t = threadIdx.x; t < cn; t += 256) {
                const int64_t o = base + c0 + t;
                sp[t] = make_float4((float)(xyz[3 * o] - c0x), (float)(xyz[3 * o + 1] - c0y),
                                    (float)(xyz[3 * o + 2] - c0z), (float)s[o]);
                sn[t] = make_float4((float)nrm[o], (float)nrm[nv + o], (float)nrm[2 * nv + o], 0.f);
            }
            __syncthreads();
            const int self = j - c0;  // position of the receiver in this chunk (masked)
            for (int t = 0; t < cn; ++t) {
                const float4 q = sp[t], m = sn[t];
                const float dx = xj - q.x, dy = yj - q.y, dz = zj - q.z;  // r_j - r_i
                const float r2 = dx * dx + dy * dy + dz * dz;
                const float inv = (t == self) ? 0.f : __builtin_amdgcn_rsqf(r2);
                const float si = q.w * inv;  // s_i / r
                acc += si;
                // s_i n_i.(r_j - r_i) / r^3 (r_i - r_j) - s_i / r n_i
                const float g = (m.x * dx + m.y * dy + m.z * dz) * si * inv * inv;
                ax -= g * dx + si * m.x;
                ay -= g * dy + si * m.y;
                az -= g * dz + si * m.z;
            }
        }
        double u = 0.0;
        if (ok) {
            const double k4 = 1.0 / (4.0 * 3.14159265358979323846);
            const double ljj =
                (nrm[oj] * (double)ax + nrm[nv + oj] * (double)ay + nrm[2 * nv + oj] * (double)az) * k4;
            u = s[oj] * ((double)acc * k4 + ljj);
            U[oj] = u;
        }
        // the tile's sum of U: wave sums, then one atomic
        for (int o = 32; o > 0; o >>= 1) u += __shfl_down(u, o);
        if ((threadIdx.x & 63) == 0) red[threadIdx.x >> 6] = u;
        __syncthreads();
        if (threadIdx.x == 0) atomicAdd(usum + b, red[0] + red[1] + red[2] + red[3]);
    }
}

// A (column-major nb x nb): off-diagonal point-monopole couplings; the
// diagonal from the bubble sums of U.
__global__ void k_coarse_matrix(const double *cen, const double *area, const double *usum, int nb, double *A) {
    int64_t e = blockIdx.x * (int64_t)blockDim.x + threadIdx.x;
    if (e >= (int64_t)nb * nb) return;
    const int a = (int)(e % nb), b = (int)(e / nb);
    if (a == b) {
        A[e] = usum[a];
        return;
    }
    const double dx = cen[3 * a] - cen[3 * b], dy = cen[3 * a + 1] - cen[3 * b + 1], dz = cen[3 * a + 2] - cen[3 * b + 2];
    A[e] = area[a] * area[b] / (4.0 * 3.14159265358979323846 * sqrt(dx * dx + dy * dy + dz * dz));
}

// Inverse of a symmetric positive definite matrix by the symmetric sweep
// operator in blocks of 128 pivots (no pivoting needed). Sweeping block K maps
//   A_KK -> -P, P = A_KK^{-1};  A_iK -> W_i = A_iK P;  A_ij -> A_ij - W_i A_jK^T
// for every i, j outside K, and all blocks swept give -A^{-1}. The matrix stays
// symmetric throughout, so only its lower triangle (column-major, row >= column)
// is kept and updated: n^3 flops, half of a Gauss-Jordan sweep's, and half its
// traffic. Three launches a block: the pivot block (one workgroup: a serial
// chain of 128 pivots), the panel, the rest of the triangle. Alone, n = 1000:
// 0.76 ms, 8 x (67 + 17 + 10) us, bound by the pivot chain; n = 5000: 6.5 ms,
// 40 x (66 + 19 + 76), the update at 41 Tflop/s. In the solve of 5000 bubbles,
// where it runs beside the octree and the diagonal pass, 55.3 -> 46.0 ms against
// a Gauss-Jordan sweep over the whole matrix in blocks of 64 and 256.
constexpr int kSweep = 128;      // pivots a block
constexpr int kSweepTile = 64;   // tile of the update
static_assert(kSweep == 2 * kSweepTile, "a pivot block is two tiles");

// P (kSweep x kSweep, identity outside bs x bs) = inverse of the diagonal block
// at (k0, k0); the block itself becomes -P. One pivot a step: its row, which by
// symmetry is also its column, goes through LDS (two buffers, one barrier a
// step), and every thread updates its 8 x 8 elements in registers: rows
// 32 q + 2 ty + e and columns 32 q + 2 tx + e, so that the reads of a wave
// touch each bank once.
__global__ void __launch_bounds__(256) k_sweep_pivot(double *__restrict__ A, int n, int k0, int bs,
                                                     double *__restrict__ P) {
    __shared__ __align__(16) double row[2][kSweep];
    const int tx = threadIdx.x & 15, ty = threadIdx.x >> 4;
    double a[8][8];
#pragma unroll
    for (int r = 0; r < 8; ++r)
#pragma unroll
        for (int c = 0; c < 8; ++c) {
            const int i = 32 * (r >> 1) + 2 * ty + (r & 1), j = 32 * (c >> 1) + 2 * tx + (c & 1);
            const int hi = max(i, j), lo = min(i, j);
            a[r][c] = hi < bs ? A[(int64_t)(k0 + lo) * n + k0 + hi] : (i == j ? 1.0 : 0.0);
        }
    // one pivot: row 2 t + e of quarter q, in register row R = 2 q + e
    auto pivot = [&](auto RC, int t) {
        constexpr int R = decltype(RC)::value;
        double *buf = row[R & 1];
        if (ty == t) {
#pragma unroll
            for (int q = 0; q < 4; ++q)
                *reinterpret_cast<double2 *>(buf + 32 * q + 2 * tx) = make_double2(a[R][2 * q], a[R][2 * q + 1]);
        }
        __syncthreads();
        // 1 / pivot: hardware reciprocal and two Newton steps
        const double piv = buf[32 * (R >> 1) + 2 * t + (R & 1)];
        double p = __builtin_amdgcn_rcp(piv);
        p = fma(p, fma(-piv, p, 1.0), p);
        p = fma(p, fma(-piv, p, 1.0), p);
        double ci[8], cj[8];
#pragma unroll
        for (int q = 0; q < 4; ++q) {
            const double2 u = *reinterpret_cast<const double2 *>(buf + 32 * q + 2 * ty);
            const double2 v = *reinterpret_cast<const double2 *>(buf + 32 * q + 2 * tx);
            ci[2 * q] = u.x;
            ci[2 * q + 1] = u.y;
            cj[2 * q] = v.x * p;
            cj[2 * q + 1] = v.y * p;
        }
        const bool mine = ty == t, col = tx == t;
#pragma unroll
        for (int r = 0; r < 8; ++r)
#pragma unroll
            for (int c = 0; c < 8; ++c) {
                a[r][c] = fma(-ci[r], cj[c], a[r][c]);
                if (r == R) a[r][c] = mine ? cj[c] : a[r][c];
                if (c == R) a[r][c] = col ? (r == R && mine ? -p : ci[r] * p) : a[r][c];
            }
    };
    auto quarter = [&](auto QC) {
        constexpr int Q = decltype(QC)::value;
#pragma unroll 1
        for (int t = 0; t < 16 && 32 * Q + 2 * t < bs; ++t) {  // identity pivots beyond bs change nothing
            pivot(std::integral_constant<int, 2 * Q>{}, t);
            pivot(std::integral_constant<int, 2 * Q + 1>{}, t);
        }
    };
    quarter(std::integral_constant<int, 0>{});
    quarter(std::integral_constant<int, 1>{});
    quarter(std::integral_constant<int, 2>{});
    quarter(std::integral_constant<int, 3>{});
#pragma unroll
    for (int r = 0; r < 8; ++r)
#pragma unroll
        for (int c = 0; c < 8; ++c) {
            const int i = 32 * (r >> 1) + 2 * ty + (r & 1), j = 32 * (c >> 1) + 2 * tx + (c & 1);
            P[j * kSweep + i] = -a[r][c];
            if (i >= j && i < bs) A[(int64_t)(k0 + j) * n + k0 + i] = a[r][c];
        }
}

// Panel: V_i = A_iK (kept for the update), W_i = V_i P, which replaces A_iK; 32
// rows a workgroup, wave w the columns 32 w .. of W. V and W are column-major
// n x kSweep (columns beyond bs zero). Rows above the block are held transposed,
// as A_Ki.
constexpr int kPanelRows = 32;
__global__ void __launch_bounds__(256) k_sweep_panel(double *__restrict__ A, int n, int k0, int bs,
                                                     const double *__restrict__ P, double *__restrict__ V,
                                                     double *__restrict__ W) {
    __shared__ double Vs[kSweep][kPanelRows + 1];
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    // the grid counts the rows outside the block; k0 is a multiple of the tile
    int i0 = blockIdx.x * kPanelRows;
    const bool below = i0 >= k0;
    if (below) i0 += bs;
    const int rows = below ? min(kPanelRows, n - i0) : kPanelRows;
#pragma unroll 4
    for (int u = 0; u < kSweep * kPanelRows / 256; ++u) {
        const int e = tid + 256 * u;
        const int i = below ? e % kPanelRows : e / kSweep, k = below ? e / kPanelRows : e % kSweep;
        const int ic = min(i, rows - 1), kc = min(k, bs - 1);
        const double v = below ? A[(int64_t)(k0 + kc) * n + i0 + ic] : A[(int64_t)(i0 + ic) * n + k0 + kc];
        Vs[k][i] = k < bs ? v : 0.0;
    }
    __syncthreads();
#pragma unroll 4
    for (int u = 0; u < kSweep * kPanelRows / 256; ++u) {
        const int e = tid + 256 * u, i = e % kPanelRows, k = e / kPanelRows;
        if (i < rows) V[(int64_t)k * n + i0 + i] = Vs[k][i];
    }
    // 32 x 32 of W^T a wave: result rows are columns of W, its columns rows
    dbl4 acc[2][2];
    for (int a = 0; a < 2; ++a)
        for (int b = 0; b < 2; ++b) acc[a][b] = dbl4{0.0, 0.0, 0.0, 0.0};
#pragma unroll 8
    for (int k4 = 0; k4 < kSweep / 4; ++k4) {
        const int k = 4 * k4 + lane / 16;
        double pf[2], vf[2];
#pragma unroll
        for (int a = 0; a < 2; ++a) pf[a] = P[k * kSweep + 32 * wave + 16 * a + lane % 16];  // P is symmetric
#pragma unroll
        for (int b = 0; b < 2; ++b) vf[b] = Vs[k][16 * b + lane % 16];
#pragma unroll
        for (int a = 0; a < 2; ++a)
#pragma unroll
            for (int b = 0; b < 2; ++b) acc[a][b] = __builtin_amdgcn_mfma_f64_16x16x4f64(pf[a], vf[b], acc[a][b], 0, 0, 0);
    }
    __syncthreads();  // V has been read
#pragma unroll
    for (int a = 0; a < 2; ++a)
#pragma unroll
        for (int b = 0; b < 2; ++b)
#pragma unroll
            for (int r = 0; r < 4; ++r) Vs[32 * wave + 16 * a + lane / 16 + 4 * r][16 * b + lane % 16] = acc[a][b][r];
    __syncthreads();
#pragma unroll 4
    for (int u = 0; u < kSweep * kPanelRows / 256; ++u) {
        const int e = tid + 256 * u, i = e % kPanelRows, k = e / kPanelRows;
        if (i >= rows) continue;
        W[(int64_t)k * n + i0 + i] = Vs[k][i];
        if (below && k < bs) A[(int64_t)(k0 + k) * n + i0 + i] = Vs[k][i];
    }
    if (!below) {
#pragma unroll 4
        for (int u = 0; u < kSweep * kPanelRows / 256; ++u) {
            const int e = tid + 256 * u, i = e / kSweep, k = e % kSweep;
            if (k < bs) A[(int64_t)(i0 + i) * n + k0 + k] = Vs[k][i];
        }
    }
}

// Update of the lower triangle's tiles outside block K: A_ij -= W_i V_j^T, K =
// 128 in four chunks of 32 through LDS, the next chunk's loads in flight during
// the products. A wave owns a 32 x 32 quarter and computes its transpose, whose
// result lanes run down the columns of A, so the tile is read into the
// accumulators and stored from them in 128-byte pieces. The stash's odd rows
// are held with their halves of 32 columns' 16s exchanged: both rows that a
// half-wave reads fall on different banks.
__global__ void __launch_bounds__(256, 4) k_sweep_update(double *__restrict__ A, int n, int k0, int bs,
                                                         const double *__restrict__ V, const double *__restrict__ W) {
    constexpr int KC = 32, T = kSweepTile;
    __shared__ double Ws[KC][T], Vs[KC][T];
    int ti = (int)((sqrtf(8.0f * (float)blockIdx.x + 1.0f) - 1.0f) * 0.5f);  // tile row: ti (ti + 1) / 2 <= block
    while ((int64_t)(ti + 1) * (ti + 2) / 2 <= (int64_t)blockIdx.x) ++ti;
    while ((int64_t)ti * (ti + 1) / 2 > (int64_t)blockIdx.x) --ti;
    const int tj = (int)((int64_t)blockIdx.x - (int64_t)ti * (ti + 1) / 2);
    const int i0 = T * ti, j0 = T * tj;
    if ((i0 >= k0 && i0 < k0 + bs) || (j0 >= k0 && j0 < k0 + bs)) return;  // the panel's
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int wi = (wave >> 1) * 32, wj = (wave & 1) * 32;
    // rows of W and V that this lane loads (the last row again beyond n)
    const int ri = min(i0 + lane, n - 1), rj = min(j0 + lane, n - 1);
    double rw[KC / 4], rv[KC / 4];
    auto load = [&](int c) {
#pragma unroll
        for (int u = 0; u < KC / 4; ++u) {
            const int64_t k = (int64_t)(KC * c + wave + 4 * u) * n;
            rw[u] = W[k + ri];
            rv[u] = V[k + rj];
        }
    };
    load(0);
    dbl4 acc[2][2];  // [column block][row block]
#pragma unroll
    for (int a = 0; a < 2; ++a)
#pragma unroll
        for (int b = 0; b < 2; ++b)
#pragma unroll
            for (int r = 0; r < 4; ++r) {
                const int i = min(i0 + wi + 16 * b + lane % 16, n - 1), j = min(j0 + wj + 16 * a + lane / 16 + 4 * r, n - 1);
                acc[a][b][r] = A[(int64_t)j * n + i];
            }
#pragma unroll 1
    for (int c = 0; c < kSweep / KC; ++c) {
#pragma unroll
        for (int u = 0; u < KC / 4; ++u) {
            const int k = wave + 4 * u, x = lane ^ (16 * (k & 1));
            Ws[k][x] = -rw[u];
            Vs[k][x] = rv[u];
        }
        __syncthreads();
        if (c + 1 < kSweep / KC) load(c + 1);
#pragma unroll
        for (int k4 = 0; k4 < KC / 4; ++k4) {
            const int k = 4 * k4 + lane / 16, sw = 16 * (k & 1);
            double vf[2], wf[2];
#pragma unroll
            for (int a = 0; a < 2; ++a) vf[a] = Vs[k][(wj + 16 * a + lane % 16) ^ sw];
#pragma unroll
            for (int b = 0; b < 2; ++b) wf[b] = Ws[k][(wi + 16 * b + lane % 16) ^ sw];
#pragma unroll
            for (int a = 0; a < 2; ++a)
#pragma unroll
                for (int b = 0; b < 2; ++b)
                    acc[a][b] = __builtin_amdgcn_mfma_f64_16x16x4f64(vf[a], wf[b], acc[a][b], 0, 0, 0);
        }
        __syncthreads();
    }
#pragma unroll
    for (int a = 0; a < 2; ++a)
#pragma unroll
        for (int b = 0; b < 2; ++b)
#pragma unroll
            for (int r = 0; r < 4; ++r) {
                const int i = i0 + wi + 16 * b + lane % 16, j = j0 + wj + 16 * a + lane / 16 + 4 * r;
                if (i < n && j < n) A[(int64_t)j * n + i] = acc[a][b][r];
            }
}

// A := -A on the lower triangle, mirrored to the upper one.
__global__ void __launch_bounds__(256) k_sweep_mirror(double *__restrict__ A, int n) {
    constexpr int T = 32;
    if (blockIdx.x < blockIdx.y) return;
    __shared__ double t[T][T + 1];
    const int i0 = T * blockIdx.x, j0 = T * blockIdx.y, x = threadIdx.x & 31;
    for (int y = threadIdx.x >> 5; y < T; y += 8) {
        const int i = i0 + x, j = j0 + y;
        if (i < n && j < n) t[y][x] = -A[(int64_t)j * n + i];
    }
    __syncthreads();
    for (int y = threadIdx.x >> 5; y < T; y += 8) {
        const int i = i0 + x, j = j0 + y;
        if (i < n && j < n && i >= j) A[(int64_t)j * n + i] = t[y][x];
        const int i2 = j0 + x, j2 = i0 + y;  // the transposed place
        if (i2 < n && j2 < n && i2 < j2) A[(int64_t)j2 * n + i2] = t[x][y];
    }
}

// Coarse right-hand side of the residual v - L x, x = (G C + cc v) / R on each
// bubble, one wave per bubble a:
//   m_a = s . x, U . x from the coefficients (TS = G^T s, TU = G^T U per bubble)
//   and the sums of v; t_a = m_a / area_a;
//   rc_a = s . v - U . x + A_c[a][a] t_a.
// The monopole sum over the other bubbles is A_c's own off-diagonal part
// applied to t, (A_c t)_a - A_c[a][a] t_a, so it needs no pass over pairs:
// A_c^{-1} of the whole right-hand side is A_c^{-1} rc - t.
__global__ void __launch_bounds__(256) k_coarse_rhs(const double *__restrict__ C, const double *__restrict__ TS,
                                                    const double *__restrict__ TU, int nc, int nb, double cc,
                                                    const double *__restrict__ R, const double *__restrict__ xsum,
                                                    const double *__restrict__ area, const double *__restrict__ usum,
                                                    double *__restrict__ rc, double *__restrict__ t) {
    const int lane = threadIdx.x & 63, a = blockIdx.x * 4 + (threadIdx.x >> 6);
    if (a >= nb) return;
    double m = 0.0, u = 0.0;
    for (int i = lane; i < nc; i += 64) {
        const int64_t o = (int64_t)a * nc + i;
        const double c = C[o];
        m = fma(TS[o], c, m);
        u = fma(TU[o], c, u);
    }
    for (int o = 32; o > 0; o >>= 1) {
        m += __shfl_xor(m, o);
        u += __shfl_xor(u, o);
    }
    if (lane == 0) {
        const double sv = xsum[a], ir = 1.0 / R[a];
        const double ta = fma(cc, sv, m) * ir / area[a];
        t[a] = ta;
        rc[a] = sv - fma(cc, xsum[(int64_t)nb + a], u) * ir + usum[a] * ta;
    }
}

// y = A x - t for symmetric A (nb x nb): row a read as column a; one block per row
__global__ void __launch_bounds__(256) k_dense_mv(const double *__restrict__ A, const double *__restrict__ x,
                                                  const double *__restrict__ t, int nb, double *__restrict__ y) {
    __shared__ double red[4];
    const int a = blockIdx.x;
    const double *col = A + (int64_t)a * nb;
    double v = 0.0;
#pragma unroll 4
    for (int b = threadIdx.x; b < nb; b += 256) v = fma(col[b], x[b], v);
    for (int o = 32; o > 0; o >>= 1) v += __shfl_xor(v, o);
    if ((threadIdx.x & 63) == 0) red[threadIdx.x >> 6] = v;
    __syncthreads();
    if (threadIdx.x == 0) y[a] = ((red[0] + red[1]) + red[2]) + red[3] - t[a];
}

void precond_radii(bfm_ctx *c) {
    Precond &P = c->pre;
    P.R.ensure(c->nb);
    k_bubble_radius<<<c->nb, 256, 0, c->stream>>>(c->s.get(), P.nd, P.R.get());
    BFM_LAUNCHED();
}

// Bubbles from which the coefficients take tiles of 48 x 16 (least time of 16 x 16
// and 48 x 16 tiles: 12 bubbles 6.3 and 10.1 us, 1000 bubbles 17.4 and 11.6, 5000
// bubbles 69 and 39; 32 x 32, 64 x 32 and 48 x 64 lie above 48 x 16 at 1000) and
// from which the result takes 32 bubbles a wave (16 and 32: 1000 bubbles 17 and
// 20 us, 5000 bubbles 65 and 58).
constexpr int kCoefWide = 512, kOutWide = 2048;
static void pre_coef(int nc, int nb, int nd, const double *T, int sv, int si, const double *X, const double *fac,
                     double *C, hipStream_t st) {
    if (nd < 14)  // no run of a lane fits the row
        k_pre_coef<1, 1, 1><<<dim3(nblk(nc, 16), nblk(nb, 16)), 256, 0, st>>>(nc, nb, nd, T, sv, si, X, fac, C);
    else if (nb < kCoefWide)
        k_pre_coef<1, 1, 14><<<dim3(nblk(nc, 16), nblk(nb, 16)), 256, 0, st>>>(nc, nb, nd, T, sv, si, X, fac, C);
    else
        k_pre_coef<3, 1, 8><<<dim3(nblk(nc, 48), nblk(nb, 16)), 256, 0, st>>>(nc, nb, nd, T, sv, si, X, fac, C);
    BFM_LAUNCHED();
}

// Five launches (three without the coarse correction) in place of eleven,
// 75 us of kernels at 1000 bubbles: gather with the sums of the input,
// coefficients, coarse right-hand side, its dense product, result.
void precond_apply(bfm_ctx *c, const double *in_s, double *out_s, bool add) {
    Precond &P = c->pre;
    hipStream_t st = c->stream;
    const int nd = P.nd, nc = P.nc, nb = c->nb;
    const bool coarse = c->opt.precond == BFM_PRECOND_SH_COARSE;
    const int *iperm = c->tree.iperm.get();
    double *X = P.X.ensure((size_t)nd * nb);
    double *Cm = P.C.ensure((size_t)nc * nb);
    k_pre_gather<<<nb, 256, 0, st>>>(in_s, iperm, c->s.get(), coarse ? P.U.get() : nullptr, nd, nb, X, P.csum.get());
    BFM_LAUNCHED();
    // C = diag(2n+1 - c) G+ X
    pre_coef(nc, nb, nd, P.basis.Gp.get(), nc, 1, X, P.fac.get(), Cm, st);
    const double *cy = nullptr;
    if (coarse) {
        double *rc = P.csum.get() + 2 * (int64_t)nb, *t = rc + nb;
        k_coarse_rhs<<<nblk(nb, 4), 256, 0, st>>>(Cm, P.TS.get(), P.TU.get(), nc, nb, P.cc, P.R.get(), P.csum.get(),
                                                  P.carea.get(), P.cusum.get(), rc, t);
        BFM_LAUNCHED();
        k_dense_mv<<<nb, 256, 0, st>>>(P.Ainv.get(), rc, t, nb, P.cy.get());
        BFM_LAUNCHED();
        cy = P.cy.get();
    }
    auto out = nc < 12 ? k_pre_out<1, 1> : (nb < kOutWide ? k_pre_out<1, 12> : k_pre_out<2, 4>);
    const int wide = nc >= 12 && nb >= kOutWide ? 32 : 16;
    out<<<dim3(nblk(nd, 32), nblk(nb, wide)), 64, 0, st>>>(nc, nb, nd, P.basis.G.get(), Cm, P.cc, X, P.R.get(), cy,
                                                           iperm, add ? 1 : 0, out_s);
    BFM_LAUNCHED();
}

// In-place inverse of a symmetric positive definite n x n matrix (column-major;
// its lower triangle is read) by the blocked symmetric sweep.
void spd_inverse(double *A, int n, DevBuf<double> &piv, DevBuf<double> &row, DevBuf<double> &col, hipStream_t st) {
    double *P = piv.ensure((size_t)kSweep * kSweep);
    double *V = row.ensure((size_t)kSweep * n), *W = col.ensure((size_t)kSweep * n);
    const int64_t tiles = nblk(n, kSweepTile);
    for (int k0 = 0; k0 < n; k0 += kSweep) {
        const int bs = std::min(kSweep, n - k0);
        k_sweep_pivot<<<1, 256, 0, st>>>(A, n, k0, bs, P);
        BFM_LAUNCHED();
        if (bs == n) break;
        k_sweep_panel<<<nblk(n - bs, kPanelRows), 256, 0, st>>>(A, n, k0, bs, P, V, W);
        BFM_LAUNCHED();
        k_sweep_update<<<(unsigned)(tiles * (tiles + 1) / 2), 256, 0, st>>>(A, n, k0, bs, V, W);
        BFM_LAUNCHED();
    }
    const unsigned m = (unsigned)nblk(n, 32);
    k_sweep_mirror<<<dim3(m, m), 256, 0, st>>>(A, n);
    BFM_LAUNCHED();
}

void coarse_build(bfm_ctx *c, hipStream_t st) {
    Precond &P = c->pre;
    const int nd = P.nd, nb = c->nb;
    P.csum.ensure(4 * (size_t)nb);  // used by precond_apply
    P.cy.ensure(nb);
    const int nc = P.nc;  // (precond_build has run)
    double *cen = P.ccen.ensure(3 * (size_t)nb), *area = P.carea.ensure(nb), *usum = P.cusum.ensure(nb);
    k_coarse_geom<<<nb, 256, 0, st>>>(c->xyz.get(), c->s.get(), nd, cen, area, usum);
    BFM_LAUNCHED();
    double *U = P.U.ensure((size_t)nd * nb);
    const int64_t tiles = (int64_t)nblk(nd, 256) * nb;
    k_coarse_u<<<(unsigned)tiles, 256, 0, st>>>(c->xyz.get(), c->s.get(), c->nrm.get(), c->nv, nd, nb, cen, U, usum);
    BFM_LAUNCHED();
    // G^T s and G^T U of every bubble
    pre_coef(nc, nb, nd, P.basis.G.get(), 1, nd, c->s.get(), nullptr, P.TS.ensure((size_t)nc * nb), st);
    pre_coef(nc, nb, nd, P.basis.G.get(), 1, nd, U, nullptr, P.TU.ensure((size_t)nc * nb), st);
    double *A = P.Ainv.ensure((size_t)nb * nb);
    k_coarse_matrix<<<nblk((int64_t)nb * nb, 256), 256, 0, st>>>(cen, area, usum, nb, A);
    BFM_LAUNCHED();
    spd_inverse(A, nb, P.sweep_p, P.sweep_v, P.sweep_w, st);
}

static void coarse_worker_wait(CoarseWorker *w);

void coarse_join(bfm_ctx *c) {
    if (!c->coarse_pending) return;
    c->coarse_pending = false;
    if (c->coarse_worker) coarse_worker_wait(c->coarse_worker);  // the build and its event are queued
    BFM_HIP(hipStreamWaitEvent(c->stream, c->ev_coarse, 0));
}

void coarse_mark(bfm_ctx *c) {
    coarse_join(c);  // an earlier build that nobody waited for (a solve that failed)
    if (!c->side) {
        BFM_HIP(hipStreamCreateWithFlags(&c->side, hipStreamNonBlocking));
        BFM_HIP(hipEventCreateWithFlags(&c->ev_geom, hipEventDisableTiming));
        BFM_HIP(hipEventCreateWithFlags(&c->ev_coarse, hipEventDisableTiming));
    }
    BFM_HIP(hipEventRecord(c->ev_geom, c->stream));
    c->coarse_marked = true;
}

// The coarse build is 3 ceil(nb / 128) + 6 launches, most of them small (30 at
// 1000 bubbles). Queued by the solving thread they would hold it, and so the octree
// build that runs beside them on the main stream; a worker thread of the handle
// queues them instead. coarse_launch hands the build over and returns;
// coarse_join waits until the worker has queued the build and its completion
// event (not for the device), then orders the main stream after that event.
struct CoarseWorker {
    std::thread th;
    std::mutex mu;
    std::condition_variable cv;
    bfm_ctx *job = nullptr;  // pending build (taken by the worker)
    bool busy = false, stop = false;
    std::exception_ptr err;
};

static void coarse_worker_main(CoarseWorker *w, int device) {
    bool dev_set = false;
    for (;;) {
        bfm_ctx *c = nullptr;
        {
            std::unique_lock<std::mutex> lk(w->mu);
            w->cv.wait(lk, [&] { return w->job != nullptr || w->stop; });
            if (!w->job) return;  // stop, nothing pending
            c = w->job;
            w->job = nullptr;
        }
        try {
            if (!dev_set) {
                BFM_HIP(hipSetDevice(device));
                dev_set = true;
            }
            BFM_HIP(hipStreamWaitEvent(c->side, c->ev_geom, 0));
            coarse_build(c, c->side);
            BFM_HIP(hipEventRecord(c->ev_coarse, c->side));
        } catch (...) {
            std::lock_guard<std::mutex> lk(w->mu);
            w->err = std::current_exception();
        }
        {
            std::lock_guard<std::mutex> lk(w->mu);
            w->busy = false;
        }
        w->cv.notify_all();
    }
}

static void coarse_worker_wait(CoarseWorker *w) {
    std::unique_lock<std::mutex> lk(w->mu);
    w->cv.wait(lk, [&] { return !w->busy; });
    if (w->err) {
        std::exception_ptr e = w->err;
        w->err = nullptr;
        std::rethrow_exception(e);
    }
}

void coarse_worker_free(bfm_ctx *c) {
    CoarseWorker *w = c->coarse_worker;
    if (!w) return;
    {
        std::lock_guard<std::mutex> lk(w->mu);
        w->stop = true;
    }
    w->cv.notify_all();
    if (w->th.joinable()) w->th.join();
    delete w;
    c->coarse_worker = nullptr;
}

void coarse_launch(bfm_ctx *c) {
    if (!c->coarse_marked) coarse_mark(c);
    c->coarse_marked = false;
    if (!c->coarse_worker) {
        auto *w = new CoarseWorker();
        w->th = std::thread(coarse_worker_main, w, c->device);
        c->coarse_worker = w;
    }
    CoarseWorker *w = c->coarse_worker;
    {
        std::lock_guard<std::mutex> lk(w->mu);
        w->job = c;
        w->busy = true;
    }
    w->cv.notify_all();
    c->coarse_pending = true;
}

}  // namespace bfm
