// Direct (all-pairs) off-diagonal product of the discrete single- and
// double-layer operators on device arrays, without a handle (Section 3.2,
// ns1 with eq2_13):
//   out_k = 1/(4 pi) sum_{j != i} s_j [ f x_j / |r_i - r_j|
//                                       + g y_j n_j . (r_i - r_j) / |r_i - r_j|^3 ],
//   i = rows[k] (or k when rows is null).
// The sources are split into nsplit ranges so that a small receiver set
// still fills the device: one workgroup per (64 R receivers, source range)
// writes a partial sum per receiver, and a second kernel adds each receiver's
// partials in a fixed order (bitwise reproducible). The partial sums are the scratch
// buffer: bfm_direct_dev allocates it per call, stream-ordered;
// bfm_direct_dev_noalloc uses the file-scope device array `scratch` below.
#include <algorithm>
#include <cmath>
#include <mutex>

#include "direct.h"

namespace bfm {

constexpr int kDirThreads = 64;
constexpr int64_t kDirGroups = 1024;  // workgroups that fill the device
constexpr double kInv4PiD = 0.079577471545947667884441881686257;

// Scratch of the allocation-free entry point (kDirectScratch doubles,
// 32 MiB): every device the library runs on holds its own copy until the
// process ends, and every call on that device shares it.
__device__ __align__(256) double scratch[kDirectScratch];

// -2 / sqrt(x): the hardware estimate and one Newton step, written as
// y (x y^2 - 3); the powers of -2 are taken into the source weights.
__device__ inline double rsqrt_m2(double x) {
    const double y = __builtin_amdgcn_rsq(x);
    return y * fma(x * y, y, -3.0);
}

// One tile of 64 sources (records in LDS, read at wave-uniform addresses)
// against R receivers per lane. SELF: some receiver's own point is in the
// tile; own[k] is its slot (negative: not here).
template <bool MONO, bool DIP, int R, bool SELF>
__device__ inline void direct_tile(const double2 (*rec)[kDirThreads], int cnt, const double *rx, const double *ry,
                                   const double *rz, const int *own, double *acc) {
    for (int t = 0; t < cnt; ++t) {
        const double2 xy = rec[0][t], zq = rec[1][t];
        const double2 nxy = DIP ? rec[2][t] : make_double2(0.0, 0.0), nzw = DIP ? rec[3][t] : make_double2(0.0, 0.0);
#pragma unroll
        for (int k = 0; k < R; ++k) {
            const double dx = rx[k] - xy.x, dy = ry[k] - xy.y, dz = rz[k] - zq.x;
            double inv = rsqrt_m2(fma(dx, dx, fma(dy, dy, dz * dz)));
            if (SELF) inv = own[k] == t ? 0.0 : inv;  // j == i excluded by index
            if (MONO) acc[k] = fma(zq.y, inv, acc[k]);
            if (DIP) {
                const double nd = fma(nxy.x, dx, fma(nxy.y, dy, nzw.x * dz));
                acc[k] = fma(nzw.y * nd, inv * inv * inv, acc[k]);
            }
        }
    }
}

// part[sp * nr + k] = sum over sources [j0, j1) of split sp for receiver k
// (without the 1/(4 pi)); a receiver index outside [0, n) gives NaN. A
// workgroup of four waves owns 64 R receivers (R per lane); its sources pass
// in tiles of 4 x 64, one 64 per wave, staged in LDS as (x, y), (z, q),
// (n_x, n_y), (n_z, w) with the weights q = f s x and w = g s y formed once
// per source, and the four waves' sums are added at the end. Bound by FP64
// VALU: 17 operations and the 1/sqrt estimate a pair with both layers, each
// source read shared by R receivers. 2000 receivers, 256,200 sources, both
// layers: 1.04 ms with one receiver per lane, scalar source loads and the
// weights formed per pair; 0.36 ms so (26 TFLOP/s at 18 operations a pair, the
// rate of the pair step alone).
template <bool MONO, bool DIP, int R>
__global__ void __launch_bounds__(4 * kDirThreads) k_direct_part(int64_t n, const double *__restrict__ xyz,
                                                                 const double *__restrict__ s,
                                                                 const double *__restrict__ nrm, double f,
                                                                 const double *__restrict__ x, double g,
                                                                 const double *__restrict__ y, int64_t nr,
                                                                 const int64_t *__restrict__ rows, int nsplit,
                                                                 double *__restrict__ part) {
    constexpr int NREC = DIP ? 4 : 2;
    __shared__ double2 rec[4][NREC][kDirThreads];
    __shared__ double red[3][R][kDirThreads];
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const int sp = blockIdx.y;
    double rx[R], ry[R], rz[R], acc[R];
    int64_t ri[R];
    bool ok[R];
#pragma unroll
    for (int k = 0; k < R; ++k) {
        const int64_t e = ((int64_t)blockIdx.x * R + k) * kDirThreads + lane;
        ri[k] = e < nr ? (rows ? rows[e] : e) : -1;
        ok[k] = ri[k] >= 0 && ri[k] < n;
        // idle or invalid receivers sit far away; their sums are never stored
        rx[k] = ok[k] ? xyz[3 * ri[k]] : 1e100;
        ry[k] = ok[k] ? xyz[3 * ri[k] + 1] : 0.0;
        rz[k] = ok[k] ? xyz[3 * ri[k] + 2] : 0.0;
        acc[k] = 0.0;
    }
    const int64_t j0 = n * sp / nsplit, j1 = n * (sp + 1) / nsplit;
    for (int64_t base = j0; base < j1; base += 4 * kDirThreads) {
        const int64_t w0 = base + wave * kDirThreads, j = w0 + lane;
        __syncthreads();  // the previous tile has been read
        if (j < j1) {
            const double sj = s[j];
            rec[wave][0][lane] = make_double2(xyz[3 * j], xyz[3 * j + 1]);
            rec[wave][1][lane] = make_double2(xyz[3 * j + 2], MONO ? -0.5 * (f * sj * x[j]) : 0.0);
            if (DIP) {
                rec[wave][NREC - 2][lane] = make_double2(nrm[3 * j], nrm[3 * j + 1]);
                rec[wave][NREC - 1][lane] = make_double2(nrm[3 * j + 2], -0.125 * (g * sj * y[j]));
            }
        }
        __syncthreads();
        const int cnt = (int)(j1 - w0 < 0 ? 0 : (j1 - w0 < kDirThreads ? j1 - w0 : kDirThreads));
        int own[R];
        bool any = false;
#pragma unroll
        for (int k = 0; k < R; ++k) {
            const int64_t d = ri[k] - w0;
            own[k] = ok[k] && d >= 0 && d < cnt ? (int)d : -1;
            any |= own[k] >= 0;
        }
        if (__any(any))
            direct_tile<MONO, DIP, R, true>(rec[wave], cnt, rx, ry, rz, own, acc);
        else
            direct_tile<MONO, DIP, R, false>(rec[wave], cnt, rx, ry, rz, own, acc);
    }
#pragma unroll
    for (int k = 0; k < R; ++k)
        if (wave > 0) red[wave - 1][k][lane] = acc[k];
    __syncthreads();
    if (wave > 0) return;
#pragma unroll
    for (int k = 0; k < R; ++k) {
        const int64_t e = ((int64_t)blockIdx.x * R + k) * kDirThreads + lane;
        const double v = ((acc[k] + red[0][k][lane]) + red[1][k][lane]) + red[2][k][lane];
        if (e < nr) part[(int64_t)sp * nr + e] = ok[k] ? v : __builtin_nan("");
    }
}

// out[k] = 1/(4 pi) sum of receiver k's partials: 32 receivers x 8 groups of
// splits per workgroup, the groups added in a fixed order
__global__ void __launch_bounds__(256) k_direct_sum(const double *__restrict__ part, int64_t nr, int nsplit,
                                                    double *__restrict__ out) {
    __shared__ double red[8][32];
    const int c = threadIdx.x & 31, grp = threadIdx.x >> 5;
    const int64_t k = (int64_t)blockIdx.x * 32 + c;
    double v = 0.0;
    if (k < nr) {
#pragma unroll 4
        for (int sp = grp; sp < nsplit; sp += 8) v += part[(int64_t)sp * nr + k];
    }
    red[grp][c] = v;
    __syncthreads();
    if (grp != 0 || k >= nr) return;
    for (int q = 1; q < 8; ++q) v += red[q][c];
    out[k] = kInv4PiD * v;
}

// Receivers per lane: enough to share each source read, without idle lanes on
// short row lists, and fewer where the workgroups would not fill the device even
// with one tile of sources each: the call is then one chain of pair steps a wave,
// four times as long with four receivers (both layers, four and one, a call: 500
// points x 500 rows 51.6 and 35.3 us, of which the call's host side is 34; 2500 x
// 2500 52.4 and 44.5; 5000 x 5000 57.5 and 53.4; with one receiver and scalar source
// loads they took 42, 49 and 83).
int direct_recv(int64_t n, int64_t nr) {
    int r = nr <= kDirThreads ? 1 : (nr <= 2 * kDirThreads ? 2 : 4);
    const int64_t splits = std::max<int64_t>(1, n / (4 * kDirThreads));
    while (r > 1 && (nr + r * kDirThreads - 1) / (r * kDirThreads) * splits < kDirGroups) r /= 2;
    return r;
}

// Source splits: about kDirGroups workgroups (four waves each), at least one tile
// of sources a split, the partials within the fixed scratch array.
int direct_splits(int64_t n, int64_t nr) {
    const int64_t per = (int64_t)direct_recv(n, nr) * kDirThreads;
    const int64_t blocks = (nr + per - 1) / per;
    int64_t sp = (kDirGroups + blocks - 1) / blocks;
    sp = std::min<int64_t>(sp, n / (4 * kDirThreads));
    sp = std::min<int64_t>(sp, kDirectScratch / nr);
    return (int)std::max<int64_t>(sp, 1);
}

void direct_check(const DirectArgs &a) {
    BFM_CHECK(a.n >= 1, BFM_EINVAL, "n must be >= 1");
    BFM_CHECK(a.nr >= 0, BFM_EINVAL, "nr must be >= 0");
    BFM_CHECK(a.xyz && a.s && a.out, BFM_EINVAL, "null argument");
    BFM_CHECK(a.f == 0.0 || a.x, BFM_EINVAL, "x required when f != 0");
    BFM_CHECK(a.g == 0.0 || (a.y && a.nrm), BFM_EINVAL, "y and nrm required when g != 0");
    BFM_CHECK(a.rows || a.nr <= a.n, BFM_EINVAL, "nr > n without a row list");
}

template <bool MONO, bool DIP>
static void direct_part(const DirectArgs &a, double *part, int nsplit, hipStream_t st) {
    const int r = direct_recv(a.n, a.nr);
    const int64_t per = (int64_t)r * kDirThreads;
    const dim3 grid((unsigned)((a.nr + per - 1) / per), (unsigned)nsplit);
    auto kern = r == 1 ? k_direct_part<MONO, DIP, 1> : (r == 2 ? k_direct_part<MONO, DIP, 2> : k_direct_part<MONO, DIP, 4>);
    kern<<<grid, 4 * kDirThreads, 0, st>>>(a.n, a.xyz, a.s, a.nrm, a.f, a.x, a.g, a.y, a.nr, a.rows, nsplit, part);
    BFM_LAUNCHED();
}

void direct_launch(const DirectArgs &a, double *part, int nsplit, hipStream_t st) {
    if (a.nr == 0) return;
    const bool mono = a.f != 0.0, dip = a.g != 0.0;
    if (mono && dip)
        direct_part<true, true>(a, part, nsplit, st);
    else if (mono)
        direct_part<true, false>(a, part, nsplit, st);
    else if (dip)
        direct_part<false, true>(a, part, nsplit, st);
    else
        direct_part<false, false>(a, part, nsplit, st);
    k_direct_sum<<<(unsigned)((a.nr + 31) / 32), 256, 0, st>>>(part, a.nr, nsplit, a.out);
    BFM_LAUNCHED();
}

void direct_product(const DirectArgs &a, hipStream_t st) {
    direct_check(a);
    if (a.nr == 0) return;
    const int nsplit = direct_splits(a.n, a.nr);
    double *part = nullptr;
    BFM_HIP(hipMallocAsync((void **)&part, sizeof(double) * (size_t)nsplit * (size_t)a.nr, st));
    try {
        direct_launch(a, part, nsplit, st);
    } catch (...) {
        (void)hipFreeAsync(part, st);
        throw;
    }
    BFM_HIP(hipFreeAsync(part, st));
}

// Device address of the current device's copy of `scratch`, looked up once
// per device with that device current (in host code the array's name is a
// host-side stand-in, not a device address).
static double *scratch_ptr() {
    constexpr int kMaxDevices = 64;
    static std::mutex mu;
    static double *ptrs[kMaxDevices] = {nullptr};
    int dev = 0;
    BFM_HIP(hipGetDevice(&dev));
    BFM_CHECK(dev >= 0 && dev < kMaxDevices, BFM_EINVAL, "device ordinal beyond 63");
    std::lock_guard<std::mutex> lock(mu);
    if (!ptrs[dev]) {
        void *p = nullptr;
        BFM_HIP(hipGetSymbolAddress(&p, HIP_SYMBOL(scratch)));
        BFM_CHECK(p != nullptr, BFM_EDEVICE, "hipGetSymbolAddress returned no address for the scratch array");
        ptrs[dev] = static_cast<double *>(p);
    }
    return ptrs[dev];
}

void direct_product_noalloc(const DirectArgs &a, hipStream_t st) {
    direct_check(a);
    double *part = scratch_ptr();
    if (a.nr == 0) return;
    const int nsplit = direct_splits(a.n, a.nr);
    BFM_CHECK((int64_t)nsplit * a.nr <= kDirectScratch, BFM_EINVAL,
              "nr = " + std::to_string(a.nr) + " needs " + std::to_string((int64_t)nsplit * a.nr) +
                  " scratch doubles; the allocation-free entry point holds " + std::to_string(kDirectScratch));
    direct_launch(a, part, nsplit, st);
}

}  // namespace bfm
