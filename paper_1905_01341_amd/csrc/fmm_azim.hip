// FP64 translations (M2M, M2L, L2L of Section 3.9) with the azimuth taken
// out. A translation by d = (rho cos phi, rho sin phi, z) equals a rotation
// of the coordinates by phi about the z axis, a translation by (rho, 0, |z|)
// and the rotation back; z < 0 is a mirror image of z > 0. Both act on one
// (degree, order) pair of coefficients at a time:
//   (cos, sin) -> s (c cos - s' sin, s' cos + c sin),  c = cos(m phi),
//   s' = sin(m phi), s = (-1)^(n+m) when z < 0, else 1,
// and the remaining translation lies in the plane y = 0, where the cosine
// and the sine parts do not mix. A translated column therefore costs
// (p(p+1)/2)^2 + (p(p-1)/2)^2 products instead of p^4 (half), and the 316
// M2L offsets share 34 operators (the 8 octants of M2M and of L2L one each),
// a ninth of the operator bytes. The factored form is the same operator: it
// differs from the dense one by rounding (3e-16 of its largest entry).
//
// One kernel: a workgroup owns WAVES x 16 columns (task x channel) of one
// offset's group and a slab of PB pairs of 16-row blocks, rows i of the
// cosine block and the same rows of the sine block, so the pair (cos, sin)
// of a result sits in one lane. K runs in chunks of 16 pairs: each lane
// loads its column's (cos, sin) pairs with one 16-byte load per MFMA step
// and rotates them in registers into the two B operands; the operator
// chunk, stored in the order the A operand is read, passes through LDS and
// is shared by the waves (a single wave reads it straight into registers).
// The results are rotated back in registers and added to the targets.
//
// The M2L's products are bound by the FP64 matrix units on large lists (busy 66%
// of the cycles at order 20, five channels, 62% at order 16, one channel) and by the
// latency of the chunk loop on small ones; the stored results, written and read
// once, add a third to the time of the five-channel list. Measured alone, against
// the dense p^2 x p^2 kernel with atomic adds: 186,300 tasks, order 20, five
// channels, reduced distant orders 2.22 -> 1.84 ms; the same tasks, order 16, one
// channel 381 -> 278 us; 59,112 tasks, order 16 195 -> 134 us; 2504 tasks, order 16
// 53 -> 31 us.
#include <algorithm>
#include <cmath>
#include <cstring>
#include <map>
#include <mutex>
#include <type_traits>
#include <utility>
#include <vector>

#include "fmm_kernels.h"
#include "ops.h"

namespace bfm {

typedef double az_dbl4 __attribute__((ext_vector_type(4)));

constexpr int az_cdiv(int a, int b) { return (a + b - 1) / b; }
constexpr int kAzXcds = 8;                              // accelerator complex dies of an MI355X
constexpr int kAzPairs = kMaxP * (kMaxP - 1) / 2;       // (n, m >= 1) pairs, n < kMaxP
constexpr int kAzTab = kAzPairs + kMaxP;                // table entries per offset: the pairs, then order 0
// A (cos, sin) pair in memory: 8-byte aligned only.
struct __attribute__((packed, aligned(8))) AzPair {
    double x, y;
};

// Sizes at order P. Cosine rows: the pairs (n, m >= 1) by degree, then the
// order-0 values by degree; sine rows: the pairs. Operators are stored
// [chunk][row block][cosine 256, sine 256] with 256 = 16 k x 16 rows.
template <int P>
struct Az {
    static constexpr int NS = P * (P - 1) / 2, NC = P * (P + 1) / 2;
    static constexpr int CC = az_cdiv(NC, 16), CS = az_cdiv(NS, 16);
    static constexpr int OPW = CC * CC * 512;  // doubles per operator
};

template <int I>
using az_int = std::integral_constant<int, I>;
template <int I0, int I1, class F>
__device__ __forceinline__ void az_static_for(F &&f) {
    if constexpr (I0 < I1) {
        f(az_int<I0>{});
        az_static_for<I0 + 1, I1>(f);
    }
}

// Chunks in flight in the single-wave shape: with the tile records, one 12.5, two
// 10.7 us a between-level launch of 64,200 points, order 16 (four and six: the same,
// at twice the registers).
constexpr int kAzAhead = 2;

// The chunk loop and the result of one slab: NCB cosine and NSB sine row
// blocks starting at row block rb0.
template <int P, int PB, int WAVES, int NCB, int NSB, int KIND>
__device__ __forceinline__ void az_slab(int rb0, const double *__restrict__ Top, const double *__restrict__ bcol,
                               double (*As)[PB * 512], const double2 *Fs, const int *Os, int colbase, int ncols,
                               int t0, int nch, const int *tbox, int64_t ld, int task0,
                               double *__restrict__ out) {
    using S = Az<P>;
    constexpr bool DIRECT = WAVES == 1;  // operator straight to registers
    [[maybe_unused]] constexpr int NT = 64 * WAVES;
    [[maybe_unused]] constexpr int PER = az_cdiv(NCB * 256, NT);
    const int tid = threadIdx.x, lane = tid & 63;
    const int kq = lane >> 4, rl = lane & 15;
    az_dbl4 ac[NCB], as[NSB > 0 ? NSB : 1];
#pragma unroll
    for (int b = 0; b < NCB; ++b) ac[b] = az_dbl4{0, 0, 0, 0};
#pragma unroll
    for (int b = 0; b < NSB; ++b) as[b] = az_dbl4{0, 0, 0, 0};
    if constexpr (DIRECT) {
        // the operator and the expansions of kAzAhead chunks in flight, in
        // registers: a wave with one chunk ahead waited for memory at every
        // chunk
        constexpr int D = S::CC < kAzAhead ? S::CC : kAzAhead;
        AzPair raw[D][4];
        double dc[D][4 * NCB], ds[D][NSB > 0 ? 4 * NSB : 1];
        auto fetch = [&](int c, AzPair(&rw)[4], double(&oc)[4 * NCB], double(&os)[NSB > 0 ? 4 * NSB : 1]) {
            const double *src = Top + ((int64_t)c * S::CC + rb0) * 512 + lane;
#pragma unroll
            for (int kk = 0; kk < 4; ++kk) {
                rw[kk] = *reinterpret_cast<const AzPair *>(bcol + Os[16 * c + 4 * kk + kq]);
#pragma unroll
                for (int b = 0; b < NCB; ++b) oc[kk * NCB + b] = src[b * 512 + kk * 64];
#pragma unroll
                for (int b = 0; b < NSB; ++b) os[kk * NSB + b] = src[b * 512 + 256 + kk * 64];
            }
        };
        az_static_for<0, D>([&](auto ci) {
            constexpr int C = decltype(ci)::value;
            fetch(C, raw[C], dc[C], ds[C]);
        });
        az_static_for<0, S::CC>([&](auto ci) {
            constexpr int C = decltype(ci)::value, U = C % D;
            // MFMA steps of the chunk's cosine and sine part
            constexpr int KC = az_cdiv(S::NC - 16 * C, 4), KS = S::NS > 16 * C ? az_cdiv(S::NS - 16 * C, 4) : 0;
#pragma unroll
            for (int kk = 0; kk < 4; ++kk) {
                const double2 f = Fs[16 * C + 4 * kk + kq];
                const double bc = f.x * raw[U][kk].x - f.y * raw[U][kk].y;
                const double bs = f.y * raw[U][kk].x + f.x * raw[U][kk].y;
#pragma unroll
                for (int b = 0; b < NCB; ++b)
                    if (kk < KC) ac[b] = __builtin_amdgcn_mfma_f64_16x16x4f64(bc, dc[U][kk * NCB + b], ac[b], 0, 0, 0);
#pragma unroll
                for (int b = 0; b < NSB; ++b)
                    if (kk < KS) as[b] = __builtin_amdgcn_mfma_f64_16x16x4f64(bs, ds[U][kk * NSB + b], as[b], 0, 0, 0);
            }
            if constexpr (C + D < S::CC) {
                fetch(C + D, raw[U], dc[U], ds[U]);
                __builtin_amdgcn_sched_barrier(0);  // issued here, not where they are used
            }
        });
    } else {
        double2 pre[PER];
        AzPair raw[4];
        auto fetch = [&](int c) {
            const double2 *s2 = reinterpret_cast<const double2 *>(Top + ((int64_t)c * S::CC + rb0) * 512);
#pragma unroll
            for (int u = 0; u < PER; ++u) pre[u] = s2[min(tid + u * NT, NCB * 256 - 1)];
#pragma unroll
            for (int kk = 0; kk < 4; ++kk)
                raw[kk] = *reinterpret_cast<const AzPair *>(bcol + Os[16 * c + 4 * kk + kq]);
        };
        auto stash = [&](int buf) {
            double2 *d2 = reinterpret_cast<double2 *>(As[buf]);
#pragma unroll
            for (int u = 0; u < PER; ++u)
                if (PER * NT == NCB * 256 || tid + u * NT < NCB * 256) d2[tid + u * NT] = pre[u];
        };
        fetch(0);
        stash(0);
        __syncthreads();
        // chunk c: rotate its pairs into the two B operands, start the next
        // chunk's loads, multiply; NKC, NKS: MFMA steps of the cosine and the
        // sine part
        auto step = [&](int c, auto nkc, auto nks, auto last) {
            constexpr int NKC = decltype(nkc)::value, NKS = decltype(nks)::value;
            constexpr bool LAST = decltype(last)::value;
            double bc[4], bs[4];
#pragma unroll
            for (int kk = 0; kk < 4; ++kk) {
                const double2 f = Fs[16 * c + 4 * kk + kq];
                bc[kk] = f.x * raw[kk].x - f.y * raw[kk].y;
                bs[kk] = f.y * raw[kk].x + f.x * raw[kk].y;
            }
            if (!LAST) fetch(c + 1);
            const double *Ab = As[c & 1] + lane;
#pragma unroll
            for (int kk = 0; kk < 4; ++kk) {
#pragma unroll
                for (int b = 0; b < NCB; ++b)
                    if (kk < NKC)
                        ac[b] = __builtin_amdgcn_mfma_f64_16x16x4f64(bc[kk], Ab[b * 512 + kk * 64], ac[b], 0, 0, 0);
#pragma unroll
                for (int b = 0; b < NSB; ++b)
                    if (kk < NKS)
                        as[b] =
                            __builtin_amdgcn_mfma_f64_16x16x4f64(bs[kk], Ab[b * 512 + 256 + kk * 64], as[b], 0, 0, 0);
            }
            if (!LAST) {
                // the stores wait for the loads: keep them behind the products
                __builtin_amdgcn_sched_barrier(0);
                stash((c + 1) & 1);
                __syncthreads();
            }
        };
        // chunks full in both parts, then the tail's partial ones
        constexpr int CF = S::NS / 16;
        static_assert(CF < S::CC, "a tail chunk");
#pragma unroll 1
        for (int c = 0; c < CF; ++c) step(c, az_int<4>{}, az_int<4>{}, az_int<0>{});
        az_static_for<CF, S::CC>([&](auto ci) {
            constexpr int C = decltype(ci)::value;
            constexpr int KC = az_cdiv(S::NC - 16 * C, 4), KS = S::NS > 16 * C ? az_cdiv(S::NS - 16 * C, 4) : 0;
            step(C, az_int<(KC < 4 ? KC : 4)>{}, az_int<(KS < 4 ? KS : 4)>{}, az_int<(C + 1 == S::CC)>{});
        });
    }
    // lane l, element r: column l/16 + 4r, row l%16 of each block
#pragma unroll
    for (int r = 0; r < 4; ++r) {
        const int col = colbase + kq + 4 * r;
        if (col >= ncols) continue;
        // M2L: the column's row of results, cosine values then sine values
        double *dcol = KIND == 0 ? out + ((int64_t)(t0 - task0) * nch + col) * (P * P)
                             : out + ((int64_t)tbox[kq + 4 * r] * nch + col % nch) * ld;
#pragma unroll
        for (int b = 0; b < NCB; ++b) {
            const int i = (rb0 + b) * 16 + rl;
            if (i >= S::NC) continue;
            const double2 f = Fs[i];
            const double zc = ac[b][r], zs = b < NSB ? as[b < NSB ? b : 0][r] : 0.0;
            const double vc = f.x * zc + f.y * zs, vs = f.x * zs - f.y * zc;
            double *d = dcol + Os[i];
            if (KIND == 0) {
                dcol[i] = vc;
                if (i < S::NS) dcol[S::NC + i] = vs;
            } else if (KIND == 1) {  // a parent has up to eight children
                unsafeAtomicAdd(d, vc);
                if (i < S::NS) unsafeAtomicAdd(d + 1, vs);
            } else if (i < S::NS) {  // a child has one parent: nobody else adds to it
                AzPair v = *reinterpret_cast<AzPair *>(d);
                v.x += vc;
                v.y += vs;
                *reinterpret_cast<AzPair *>(d) = v;
            } else {
                *d += vc;
            }
        }
    }
}

// P: the order applied; LDP: the order the expansions are stored at (degrees
// P and above are left alone). tiles: records of the launch's ntiles tiles (one
// load instead of a search of the offsets, each step of which missed a cold L2:
// a small launch is a chain of such misses); canon[o] = operator of offset o in
// T, fac / off = rotation factors (per offset) and packed positions of the table
// entries. KIND: 0 M2L, 1 M2M (added to the parent atomically), 2
// L2L. The M2L results of task t go to row t - task0 of out ([nch][P^2],
// cosine values, then sine values) for k_az_reduce instead of being added to
// the target's expansion: FP64 atomic adds ran at 75 to 97 G adds/s whatever
// the kernel around them did (59,112 tasks at order 16: 190 us with half the
// products as with all of them, 137 us stored and summed).
template <int P, int LDP, int PB, int WAVES, int KIND>
__global__ void __launch_bounds__(64 * WAVES, WAVES == 1 ? 4 : (P == 12 ? 2 : (P == 20 ? 3 : 4))) k_translate_az(const int4 *__restrict__ tiles, int ntiles,
                                                             const int *__restrict__ tsrc,
                                                             const int *__restrict__ tdst, int nch,
                                                             const int *__restrict__ canon,
                                                             const double *__restrict__ T,
                                                             const double2 *__restrict__ fac,
                                                             const int *__restrict__ off, int task0,
                                                             const double *in, double *out) {
    using S = Az<P>;
    static_assert(P <= LDP, "applied order within the stored order");
    constexpr int FULL = S::CS / PB, NSLAB = az_cdiv(S::CC, PB);
    // slabs past the full ones: one (partial in either part), or single
    // cosine blocks
    static_assert(NSLAB - FULL <= 1 || PB == 1, "slab shape");
    constexpr int LCB = NSLAB > FULL ? (S::CC - FULL * PB < PB ? S::CC - FULL * PB : PB) : PB;
    constexpr int LSB = NSLAB > FULL ? S::CS - FULL * PB : PB;
    static_assert(LSB >= 0 && LSB <= LCB, "sine rows within the cosine rows");
    __shared__ __align__(16) double As[WAVES == 1 ? 1 : 2][PB * 512];
    __shared__ double2 Fs[S::CC * 16];
    __shared__ int Os[S::CC * 16];
    __shared__ int Bs[KIND == 0 ? 1 : 16 * WAVES];  // target boxes of the tile's columns
    // XCD-aware order: XCD x takes a contiguous run of logical blocks (the
    // tiles of a few offsets), whose operators then stay in its own L2
    const int nblock = gridDim.x, per = nblock / kAzXcds, rem = nblock % kAzXcds;
    const int xcd = blockIdx.x % kAzXcds, idx = blockIdx.x / kAzXcds;
    const int logical = xcd * per + (xcd < rem ? xcd : rem) + idx;
    if (logical / NSLAB >= ntiles) return;
    const int4 tile = tiles[logical / NSLAB];
    const int slab = logical % NSLAB;
    const int tid = threadIdx.x, wave = tid >> 6, lane = tid & 63;
    const int op = tile.x, t0 = tile.y, ncols = tile.z;
    const int colbase = tile.w + wave * 16;
    const int bcolid = colbase + (lane & 15);
    const bool bok = bcolid < ncols;
    // idle columns read the first one (valid memory) and are never stored
    const int bt = bok ? bcolid : 0;
    const int sbox = tsrc[t0 + bt / nch];
    const double *Top = T + (int64_t)canon[op] * S::OPW;
    if (KIND != 0 && tid < 16 * WAVES) Bs[tid] = tdst[t0 + min(tile.w + tid, ncols - 1) / nch];
    for (int e = tid; e < S::CC * 16; e += 64 * WAVES) {
        const int t = e < S::NS ? e : (e < S::NC ? kAzPairs + e - S::NS : -1);
        // rows past the order: zero factors and a valid position
        Fs[e] = t >= 0 ? fac[(int64_t)op * kAzTab + t] : make_double2(0.0, 0.0);
        Os[e] = t >= 0 ? off[t] : 0;
    }
    __syncthreads();
    const double *bcol = in + ((int64_t)sbox * nch + bt % nch) * (LDP * LDP);
    if (slab < FULL)
        az_slab<P, PB, WAVES, PB, PB, KIND>(slab * PB, Top, bcol, As, Fs, Os, colbase, ncols, t0, nch, Bs + 16 * wave, LDP * LDP,
                                               task0, out);
    else
        az_slab<P, PB, WAVES, LCB, LSB, KIND>(slab * PB, Top, bcol, As, Fs, Os, colbase, ncols, t0, nch, Bs + 16 * wave, LDP * LDP,
                                                 task0, out);
}

// L[b] (+)= the rows of target box b's tasks whose grouped positions lie in
// [lo, hi), in the order the tasks were generated (a fixed order: the sum is
// reproducible). One wave per (box, 128 of its nch x Q^2 values), 16 bytes per
// lane and task. FIRST: L is written (also where a box has no task).
template <int Q, bool FIRST>
__global__ void __launch_bounds__(256) k_az_reduce(const int *__restrict__ dst_off, const int *__restrict__ pos_of,
                                                   int64_t box0, int64_t nbox, int lo, int hi, int nch, int ld,
                                                   const double *__restrict__ part, const int *__restrict__ off,
                                                   double *__restrict__ L) {
    using S = Az<Q>;
    constexpr int Q2 = Q * Q;
    __shared__ int list[4][192];  // a box has at most 189 tasks
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const int row = nch * Q2, nchunk = (row + 127) / 128;
    const int64_t w = (int64_t)blockIdx.x * 4 + wave;
    const int64_t k = w / nchunk;
    if (k >= nbox) return;
    int n = 0;
    const int a = dst_off[k], e = dst_off[k + 1];
    for (int base = a; base < e; base += 64) {
        const int p = base + lane < e ? pos_of[base + lane] : -1;
        const bool ok = p >= lo && p < hi;
        const unsigned long long m = __ballot(ok);
        if (ok) list[wave][n + __popcll(m & ((1ull << lane) - 1))] = p - lo;
        n += __popcll(m);
    }
    // lanes read positions that other lanes of the wave wrote
    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
    __builtin_amdgcn_wave_barrier();
    if (!FIRST && n == 0) return;
    const int e0 = (int)(w % nchunk) * 128 + 2 * lane;
    if (e0 >= row) return;
    const double *src = part + e0;
    double sx = 0.0, sy = 0.0;
    int i = 0;
    for (; i + 8 <= n; i += 8) {
        double2 v[8];
#pragma unroll
        for (int u = 0; u < 8; ++u)
            v[u] = *reinterpret_cast<const double2 *>(src + (int64_t)list[wave][i + u] * row);
#pragma unroll
        for (int u = 0; u < 8; ++u) {
            sx += v[u].x;
            sy += v[u].y;
        }
    }
    for (; i < n; ++i) {
        const double2 v = *reinterpret_cast<const double2 *>(src + (int64_t)list[wave][i] * row);
        sx += v.x;
        sy += v.y;
    }
    double *lb = L + (box0 + k) * nch * ld;
#pragma unroll
    for (int u = 0; u < 2; ++u) {
        const int ch = (e0 + u) / Q2, r = (e0 + u) % Q2;
        const int at = r < S::NS ? off[r] : (r < S::NC ? off[kAzPairs + r - S::NS] : off[r - S::NC] + 1);
        const double v = u ? sy : sx;
        if (FIRST)
            lb[(int64_t)ch * ld + at] = v;
        else
            lb[(int64_t)ch * ld + at] += v;
    }
}

// Row-block pairs per workgroup of the wide shapes: an order-20 operator has
// 14 cosine and 12 sine blocks, order 16 has 9 and 8.
template <int P>
constexpr int az_pb() {
    return P <= 4 ? 1 : (P == 12 ? 5 : 3);
}

template <int P, int LDP, int KIND>
static void launch_az(int shape, const int4 *tiles, int ntiles, const TaskList &tl, bool swap,
                      int nch, const int *canon, const double *T, const double2 *fac, const int *off, int task0,
                      const double *in, double *out, hipStream_t st) {
    if (ntiles <= 0) return;
    constexpr int PB = az_pb<P>(), CC = Az<P>::CC;
    const int *src = swap ? tl.dst.get() : tl.src.get(), *dst = swap ? tl.src.get() : tl.dst.get();
    if (shape == 0)
        k_translate_az<P, LDP, PB, 8, KIND><<<(unsigned)(ntiles * az_cdiv(CC, PB)), 512, 0, st>>>(
            tiles, ntiles, src, dst, nch, canon, T, fac, off, task0, in, out);
    else if (shape == 1)
        k_translate_az<P, LDP, PB, 4, KIND><<<(unsigned)(ntiles * az_cdiv(CC, PB)), 256, 0, st>>>(
            tiles, ntiles, src, dst, nch, canon, T, fac, off, task0, in, out);
    else
        k_translate_az<P, LDP, 1, 1, KIND><<<(unsigned)(ntiles * CC), 64, 0, st>>>(
            tiles, ntiles, src, dst, nch, canon, T, fac, off, task0, in, out);
    BFM_LAUNCHED();
}

// ---------------------------------------------------------------------------
// Host side: operators and tables

// Rotation factors of offset (dx, dy, dz): (s cos m phi, s sin m phi) of the
// pairs (n, m >= 1) by degree, then (s, 0) of order 0.
static void az_factors(int dx, int dy, int dz, double2 *f) {
    const long double phi = (dx || dy) ? atan2l((long double)dy, (long double)dx) : 0.0L;
    int i = 0;
    for (int n = 0; n < kMaxP; ++n) {
        for (int m = 1; m <= n; ++m, ++i) {
            const double s = (dz < 0 && ((n + m) & 1)) ? -1.0 : 1.0;
            f[i] = make_double2(s * (double)cosl(m * phi), s * (double)sinl(m * phi));
        }
        f[kAzPairs + n] = make_double2((dz < 0 && (n & 1)) ? -1.0 : 1.0, 0.0);
    }
}

static int az_position(int t) {  // packed position of table entry t
    if (t >= kAzPairs) return (t - kAzPairs) * (t - kAzPairs);
    int n = 1;
    while (t >= n) t -= n++;
    return n * n + 2 * t + 1;
}

// The operator T (row-major, order p) of an offset with factors f in the
// rotated frame, at order q <= p, in the kernel's layout (zeros where rows
// or columns pass the order). The dropped cosine-sine blocks vanish up to
// rounding.
template <int Q>
static void az_pack(int p, const std::vector<double> &T, const double2 *f, double *dst) {
    using S = Az<Q>;
    const int P = p * p;
    auto entry = [&](int i) { return i < S::NS ? i : kAzPairs + i - S::NS; };
    // element (row part a, col part b) of R T R^T: rows and columns combined by
    // (s c, s s') of their pair
    auto at = [&](int ti, bool si, int tj, bool sj) {
        const int oi = az_position(ti), oj = az_position(tj);
        // (weight of the first, of the second) entry of the pair
        auto w = [&](int t, bool sine, double &a, double &b) {
            a = sine ? f[t].y : f[t].x;
            b = sine ? f[t].x : -f[t].y;
        };
        double ra, rb, ca, cb;
        w(ti, si, ra, rb);
        w(tj, sj, ca, cb);
        const bool pi = ti < kAzPairs, pj = tj < kAzPairs;
        double v = ra * ca * T[(size_t)oi * P + oj];
        if (pj) v += ra * cb * T[(size_t)oi * P + oj + 1];
        if (pi) v += rb * ca * T[(size_t)(oi + 1) * P + oj];
        if (pi && pj) v += rb * cb * T[(size_t)(oi + 1) * P + oj + 1];
        return v;
    };
    std::memset(dst, 0, sizeof(double) * S::OPW);
    for (int k = 0; k < S::NC; ++k)
        for (int i = 0; i < S::NC; ++i) {
            double *blk = dst + ((size_t)(k / 16) * S::CC + i / 16) * 512 + (k % 16) * 16 + i % 16;
            blk[0] = at(entry(i), false, entry(k), false);
            if (i < S::NS && k < S::NS) blk[256] = at(i, true, k, true);
        }
}

static void az_pack_at(int q, int p, const std::vector<double> &T, const double2 *f, double *dst) {
    switch (q) {
        case 4: return az_pack<4>(p, T, f, dst);
        case 8: return az_pack<8>(p, T, f, dst);
        case 12: return az_pack<12>(p, T, f, dst);
        case 16: return az_pack<16>(p, T, f, dst);
        default: return az_pack<20>(p, T, f, dst);
    }
}

static size_t az_opw(int q) {
    const int cc = az_cdiv(q * (q + 1) / 2, 16);
    return (size_t)cc * cc * 512;
}

namespace {
struct AzHost {
    std::vector<double> m2m, l2l, m2l;
    std::vector<int> canon;           // 316 offsets, then the 8 octants
    std::vector<double2> fac;         // likewise, kAzTab entries each
    std::vector<int> off;             // kAzTab packed positions
    size_t goff[kM2LClasses] = {0};   // first double of each order group in m2l
};
}  // namespace

static AzHost az_build(int p, int orders) {
    AzHost h;
    const int nt = kNumM2LOps + 8;
    h.canon.assign(nt, 0);
    h.fac.resize((size_t)nt * kAzTab);
    h.off.resize(kAzTab);
    for (int t = 0; t < kAzTab; ++t) h.off[t] = az_position(t);
    for (int o = 0; o < nt; ++o) {
        int d[3];
        if (o < kNumM2LOps) {
            m2l_op_offset(o, d);
        } else {
            const int c = o - kNumM2LOps;
            d[0] = ((c >> 2) & 1) ? 1 : -1;
            d[1] = ((c >> 1) & 1) ? 1 : -1;
            d[2] = (c & 1) ? 1 : -1;
        }
        az_factors(d[0], d[1], d[2], &h.fac[(size_t)o * kAzTab]);
    }
    int first[kM2LClasses + 1], order[kM2LClasses];
    const int ng = m2l_order_groups(p, orders, first, order);
    struct Job {
        int op, q;
        size_t at;
    };
    std::vector<Job> jobs;
    size_t total = 0;
    for (int g = 0; g < ng; ++g) {
        h.goff[g] = total;
        std::map<std::pair<int, int>, int> seen;  // (dx^2 + dy^2, |dz|) -> operator of the group
        for (int o = first[g]; o < first[g + 1]; ++o) {
            int d[3];
            m2l_op_offset(o, d);
            const auto key = std::make_pair(d[0] * d[0] + d[1] * d[1], std::abs(d[2]));
            auto it = seen.find(key);
            if (it == seen.end()) {
                it = seen.emplace(key, (int)seen.size()).first;
                jobs.push_back({o, order[g], total});
                total += az_opw(order[g]);
            }
            h.canon[o] = it->second;
        }
    }
    h.m2l.resize(total);
    h.m2m.resize(az_opw(p));
    h.l2l.resize(az_opw(p));
    const int nj = (int)jobs.size();
#pragma omp parallel for schedule(dynamic)
    for (int j = 0; j < nj + 2; ++j) {
        std::vector<double> T((size_t)p * p * p * p);
        if (j < nj) {
            // the leading block of the order-p operator is the order-q operator
            build_m2l(p, jobs[j].op, T.data());
            az_pack_at(jobs[j].q, p, T, &h.fac[(size_t)jobs[j].op * kAzTab], &h.m2l[jobs[j].at]);
        } else {
            const int oct = 7;
            if (j == nj)
                build_m2m(p, oct, T.data());
            else
                build_l2l(p, oct, T.data());
            az_pack_at(p, p, T, &h.fac[(size_t)(kNumM2LOps + oct) * kAzTab], j == nj ? h.m2m.data() : h.l2l.data());
        }
    }
    return h;
}

// Built once per process, order and order rule (at most 30 MB each).
static const AzHost &az_host(int p, int orders) {
    static std::mutex mu;
    static std::map<std::pair<int, int>, AzHost> cache;
    std::lock_guard<std::mutex> lock(mu);
    const auto key = std::make_pair(p, orders);
    auto it = cache.find(key);
    if (it == cache.end()) it = cache.emplace(key, az_build(p, orders)).first;
    return it->second;
}

void az_ops_upload(FmmWork &w, int p, hipStream_t st) {
    if (w.az_p == p && w.az_orders == w.m2l_orders) return;
    const AzHost &h = az_host(p, w.m2l_orders);
    auto up = [&](auto &buf, const auto &v) {
        buf.ensure(v.size());
        BFM_HIP(hipMemcpyAsync(buf.get(), v.data(), sizeof(v[0]) * v.size(), hipMemcpyHostToDevice, st));
    };
    up(w.az_m2m, h.m2m);
    up(w.az_l2l, h.l2l);
    up(w.az_m2l, h.m2l);
    up(w.az_canon, h.canon);
    up(w.az_fac, h.fac);
    up(w.az_off, h.off);
    for (int g = 0; g < kM2LClasses; ++g) w.az_goff[g] = h.goff[g];
    BFM_HIP(hipStreamSynchronize(st));
    w.az_p = p;
    w.az_orders = w.m2l_orders;
}

// Tiles of `width` columns (nch per task) before operator o of a task list.
static int az_tiles_before(const TaskList &tl, int nch, int width, int o) {
    int run = 0;
    for (int q = 0; q < o; ++q) run += ((tl.op_off_h[q + 1] - tl.op_off_h[q]) * nch + width - 1) / width;
    return run;
}

// Launch shape by size: 16-column single-wave tiles of one row-block pair
// where the groups are small (under 48 columns an offset a 64-column tile is
// mostly idle: 31 against 42 us for 2504 tasks, 8 an offset, order 16; 52 an
// offset 79 against 61 us) or the 64-column launch would leave half of the
// device without a workgroup pair, else 64-column tiles.
static int az_shape(const TaskList &tl, int nch, int nslab) {
    const int64_t cols = tl.ntasks * nch;
    if (cols < (int64_t)48 * tl.nops) return 2;
    return ((cols + 63) / 64) * nslab >= 512 ? 1 : 2;
}

// Tiles g0 .. g1 - 1 of the list; task0: the task whose results start `out` (M2L).
template <int P, int LDP, int KIND>
static void az_one(const AzLaunch &a, int shape, int g0, int g1, int task0, const double *T, const TaskList &tl,
                   double *out) {
    const int width = shape == 0 ? 128 : (shape == 1 ? 64 : 16);
    const int base = KIND ? kNumM2LOps : 0;
    launch_az<P, LDP, KIND>(shape, tl.tiles_for(a.nch, width) + g0, g1 - g0, tl, a.swap, a.nch,
                            a.w->az_canon.get() + base, T, a.w->az_fac.get() + (int64_t)base * kAzTab,
                            a.w->az_off.get(), task0, a.in, out, a.st);
}

// The batch of an M2L list that starts at task lo, a cut of offset op or its first
// task (op_off: first task of each offset, op_off[op1]: the end): the most
// tasks up to `most` that end at the end or at a cut. Cuts lie every `width` tasks
// of an offset, where one of its tiles of `width` columns (nch a task) ends.
// most >= width, so a batch is never empty. hop, htile: offset and tile of the
// end (tile 0: the offset's first).
void az_batch(const int *op_off, int op, int op1, int nch, int width, int64_t most, int lo, int *hi, int *hop,
              int *htile) {
    const int64_t want = lo + most;
    if (want >= op_off[op1]) {
        *hi = op_off[op1];
        *hop = op1;
        *htile = 0;
        return;
    }
    while (op_off[op + 1] <= want) ++op;
    const int cut = (int)((want - op_off[op]) / width);
    *hi = op_off[op] + cut * width;
    *hop = op;
    *htile = cut * nch;
}

// Doubles of per-task M2L results held at once (1 GiB, one workspace of the handle
// for both FP64 product groups, which run on one stream): longer lists run in
// batches, each summed into the targets before the next, which costs about 0.1 ms a
// batch on 3.2 M points (the targets read and written once more, short last waves;
// 11 batches in the diagonal pass). A solve of that size with up to 4 GiB / 1 GiB /
// 512 / 256 / 128 / 64 MiB: 44.8 / 45.8 / 47.1 / 49.7 / 53.0 / 58.1 ms; 642,000
// points 9.03 / 9.03 / 9.05 / 9.14 / 9.31 / 9.69.
constexpr int64_t kAzPart = (int64_t)1024 << 17;

// M2L of offsets op0 .. op1 - 1 at order P, added to (first: written over)
// the target expansions.
template <int P, int LDP>
static void az_m2l(const AzLaunch &a, int shape, int op0, int op1, const double *T, TaskList &tl, bool first) {
    const int width = shape == 0 ? 128 : (shape == 1 ? 64 : 16);
    const int64_t row = (int64_t)a.nch * P * P, most = std::max<int64_t>(kAzPart / row, width);
    const int *off = tl.op_off_h.data();
    const int64_t waves = tl.dst_nbox * ((row + 127) / 128);
    int op = op0, lo = off[op0], g0 = az_tiles_before(tl, a.nch, width, op0);
    do {  // (a list without tasks writes its targets all the same)
        int hi, hop, htile;
        az_batch(off, op, op1, a.nch, width, most, lo, &hi, &hop, &htile);
        const int g1 = az_tiles_before(tl, a.nch, width, hop) + htile;
        double *part = a.w->az_part->ensure((size_t)std::max<int64_t>((hi - lo) * row, 1));
        az_one<P, LDP, 0>(a, shape, g0, g1, lo, T, tl, part);
        auto kern = first ? k_az_reduce<P, true> : k_az_reduce<P, false>;
        kern<<<(unsigned)((waves + 3) / 4), 256, 0, a.st>>>(tl.dst_off.get(), tl.pos_of.get(), tl.dst_box0,
                                                            tl.dst_nbox, lo, hi, a.nch, LDP * LDP, part,
                                                            a.w->az_off.get(), a.out);
        BFM_LAUNCHED();
        first = false;
        op = hop;
        lo = hi;
        g0 = g1;
    } while (lo < off[op1]);
}

template <int P>
int launch_translate_az(const AzLaunch &a, TaskList &tl, bool m2l, int shape, double *flops) {
    constexpr int NSLAB = az_cdiv(Az<P>::CC, az_pb<P>());
    if (shape < 0) shape = az_shape(tl, a.nch, NSLAB);
    const int width = shape == 0 ? 128 : (shape == 1 ? 64 : 16);
    prepare_tiles(tl, a.nch, width, a.st);
    auto col_flops = [](int q) {  // products of the cosine and the sine block
        const double c = 0.5 * q * (q + 1), s = 0.5 * q * (q - 1);
        return 2.0 * (c * c + s * s);
    };
    *flops = 0.0;
    if (tl.ntasks <= 0) return shape;
    FmmWork &w = *a.w;
    if (!m2l) {
        *flops = col_flops(P) * (double)tl.ntasks * a.nch;
        const int nt = tl.ntiles_for(a.nch, width);
        if (a.swap)
            az_one<P, P, 2>(a, shape, 0, nt, 0, w.az_l2l.get(), tl, a.out);
        else
            az_one<P, P, 1>(a, shape, 0, nt, 0, w.az_m2m.get(), tl, a.out);
        return shape;
    }
    constexpr int P1 = m2l_class_order(P, 1), P2 = m2l_class_order(P, 2);
    int first[kM2LClasses + 1], order[kM2LClasses];
    const int ng = m2l_order_groups(P, w.m2l_orders, first, order);
    for (int g = 0; g < ng; ++g) {
        *flops += col_flops(order[g]) * (double)(tl.op_off_h[first[g + 1]] - tl.op_off_h[first[g]]) * a.nch;
        const double *T = w.az_m2l.get() + w.az_goff[g];
        if (order[g] == P)
            az_m2l<P, P>(a, shape, first[g], first[g + 1], T, tl, g == 0);
        else if (order[g] == P1)
            az_m2l<P1, P>(a, shape, first[g], first[g + 1], T, tl, false);
        else
            az_m2l<P2, P>(a, shape, first[g], first[g + 1], T, tl, false);
    }
    return shape;
}

template int launch_translate_az<4>(const AzLaunch &, TaskList &, bool, int, double *);
template int launch_translate_az<8>(const AzLaunch &, TaskList &, bool, int, double *);
template int launch_translate_az<12>(const AzLaunch &, TaskList &, bool, int, double *);
template int launch_translate_az<16>(const AzLaunch &, TaskList &, bool, int, double *);
template int launch_translate_az<20>(const AzLaunch &, TaskList &, bool, int, double *);

}  // namespace bfm
