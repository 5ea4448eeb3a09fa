// Leaf expansions of the fast multipole product (Section 3.9): P2M forms
// the multipole expansion of every leaf from its points' monopoles and
// dipoles, L2P evaluates every leaf's local expansion at its points. Both
// build the regular solid harmonics of a point by the three-term recurrences
// of the box-scaled normalised basis, in registers.
//
// Both kernels run one workgroup of SP x NW waves per leaf work item (a leaf and
// up to kLeafChunk of its points): SP groups of waves share out the points (up
// to four a lane), and the NW waves of a group the orders m. The recurrence
// over the degrees of one order is a serial chain, so splitting the orders
// makes the chains a quarter as long where the items are too few to fill the
// chip; with many items the split of the points repeats nothing. Several points
// a lane share each LDS read of a constant or coefficient and each reduction of
// the P2M. Against one wave per 128 points, alone: 642 points, order 16, P2M 27
// -> 11 us, L2P 22 -> 9 us; 642,000 points, five channels, order 20, P2M 547 ->
// 409 us, L2P 377 -> 185 us (VALU instructions alone are 59% of the P2M's time and
// 56% of the L2P's).
#include <cmath>
#include <type_traits>
#include <vector>

#include "fmm_kernels.h"

namespace bfm {

constexpr int kTri = kMaxP * (kMaxP + 1) / 2;  // (n, m >= 0) pairs, n < kMaxP
static_assert(kLeafChunk == 256, "up to four points per lane");

// Recurrence of the regular harmonics for degree n > m:
//   Rt_n^m = ae(n, m) z Rt_{n-1}^m - ab(n, m) r^2 Rt_{n-2}^m,
//   ae = (2n-1)/sqrt((n-m)(n+m)), ab = sqrt((n-m-1)(n+m-1))/sqrt((n-m)(n+m)),
// and for the sectoral ones Rt_m^m = f_m (x + i y) Rt_{m-1}^{m-1},
//   f_m = sqrt((2m-1)/(2m)).
__constant__ double2 c_rec[kTri];  // (ae, ab) at tri(n, m)
__constant__ double c_sect[kMaxP];  // f_m

__host__ __device__ constexpr int tri(int n, int m) { return n * (n + 1) / 2 + m; }

void leaf_tables_upload(int device) {
    static int done_mask = 0;  // one bit per device ordinal < 32
    if (device < 32 && (done_mask >> device) & 1) return;
    std::vector<double2> rec(kTri, make_double2(0.0, 0.0));
    std::vector<double> sect(kMaxP, 0.0);
    for (int n = 0; n < kMaxP; ++n)
        for (int m = 0; m < n; ++m) {
            const double a = 1.0 / std::sqrt((double)(n - m) * (n + m));
            const double b = n >= m + 2 ? std::sqrt((double)(n - m - 1) * (n + m - 1)) : 0.0;
            rec[tri(n, m)] = make_double2((2.0 * n - 1.0) * a, b * a);
        }
    for (int m = 1; m < kMaxP; ++m) sect[m] = std::sqrt((2.0 * m - 1.0) / (2.0 * m));
    BFM_HIP(hipMemcpyToSymbol(HIP_SYMBOL(c_rec), rec.data(), sizeof(double2) * kTri));
    BFM_HIP(hipMemcpyToSymbol(HIP_SYMBOL(c_sect), sect.data(), sizeof(double) * kMaxP));
    if (device < 32) done_mask |= 1 << device;
}

// Pair of recurrence constants in the arithmetic type R.
template <class R>
struct alignas(2 * sizeof(R)) Pair2 {
    R x, y;
};

// Copy the recurrence tables for order P into LDS (block-wide), rounded to R.
template <int P_, class R>
__device__ inline void stage_tables(Pair2<R> *rec, R *sect, int tid, int nthreads) {
    constexpr int NT = P_ * (P_ + 1) / 2;
    for (int t = tid; t < NT; t += nthreads) rec[t] = Pair2<R>{(R)c_rec[t].x, (R)c_rec[t].y};
    for (int t = tid; t < P_; t += nthreads) sect[t] = (R)c_sect[t];
}

// Order i of wave w of NW: blocks of 2 NW orders dealt back and forth (with four
// waves w, 7 - w, 8 + w, 15 - w, ...), so that the waves' degree counts sum to
// about the same (54, 53, 52, 51 of the 210 at order 20).
template <int NW>
__device__ inline int leaf_order(int w, int i) {
    return 2 * NW * (i >> 1) + ((i & 1) ? 2 * NW - 1 - w : w);
}

// ---------------------------------------------------------------------------
// Sum over the wave's lanes of several columns at a time. swap_add32(a, b):
// lanes 0-31 hold a's, lanes 32-63 b's sums of lanes l and l +- 32;
// swap_add16 continues with two such values, so four columns (a, b, c, d)
// become one value per lane whose 16-lane groups hold 16 partial sums of
// a, c, b, d.
template <bool W32, class R>
__device__ inline R swap_add(R a, R b) {
    auto sw = [](unsigned x, unsigned y) {
        if constexpr (W32)
            return __builtin_amdgcn_permlane32_swap(x, y, false, false);
        else
            return __builtin_amdgcn_permlane16_swap(x, y, false, false);
    };
    if constexpr (sizeof(R) == 8) {
        const unsigned long long ua = __builtin_bit_cast(unsigned long long, a);
        const unsigned long long ub = __builtin_bit_cast(unsigned long long, b);
        const auto lo = sw((unsigned)ua, (unsigned)ub);
        const auto hi = sw((unsigned)(ua >> 32), (unsigned)(ub >> 32));
        const unsigned long long pa = ((unsigned long long)hi[0] << 32) | lo[0];
        const unsigned long long pb = ((unsigned long long)hi[1] << 32) | lo[1];
        return __builtin_bit_cast(R, pa) + __builtin_bit_cast(R, pb);
    } else {
        const auto v = sw(__builtin_bit_cast(unsigned, a), __builtin_bit_cast(unsigned, b));
        return __builtin_bit_cast(R, (unsigned)v[0]) + __builtin_bit_cast(R, (unsigned)v[1]);
    }
}

// P2M. Lane l takes the item's points l, l + 64, ... (PPL of them), builds
// their regular harmonics for the wave's orders (loops over order and degree
// uniform across the wave, recurrence constants read from LDS at wave-uniform
// addresses) and sums its points' contributions for every coefficient and
// channel. Four such columns at a time are reduced to 16 partial sums each in
// registers; sixteen groups of four are buffered in LDS, then lane t adds up
// column t and adds it to the leaf's expansion (atomically where the leaf has
// several items).
//   Mt_n^m += q_j conj(Rt_n^m(v_j)) + (w_j / h) conj(n_j . grad_v Rt_n^m(v_j)),
// v_j = (r_j - c)/h. The directional derivative D = n_j . grad_v follows the
// same recurrence by forward differentiation:
//   D Rt_m^m = f_m [D Rt_{m-1}^{m-1} (x+iy) + Rt_{m-1}^{m-1} (n_x+i n_y)]
//   D Rt_n^m = ae (n_z Rt_{n-1} + z D Rt_{n-1}) - ab (2 v.n Rt_{n-2} + r^2 D Rt_{n-2})
//
// In FP32 the buffered columns are the lanes' own values, sixteen columns at a
// time, and four lanes add up each in a fixed order over groups of 128 points
// that does not depend on how the work is split: the order of an FP32 sum
// decides the bits that the split-BF16 translations round next, and a solve's
// answer at its tolerance moves with them. The groups of a leaf are added
// atomically: leaves of up to 256 points (two groups) come out the same on every
// run, larger ones up to the order in which their groups arrive.
constexpr int kP2MRows = 16;
template <class R>
constexpr int kP2MBuf = sizeof(R) == 4 ? 16 * 68 : kP2MRows * 64;  // values a wave; rows of 68: distinct banks
template <int P_, int NCH, bool MONO, bool DIP, class R, int NW, int PPL>
__device__ __forceinline__ void p2m_points(int j0, int re, double cx, double cy, double cz, double ih,
                                           const double *__restrict__ px, const double *__restrict__ py,
                                           const double *__restrict__ pz, const double *__restrict__ pnx,
                                           const double *__restrict__ pny, const double *__restrict__ pnz, int64_t n,
                                           const double *__restrict__ q, const double *__restrict__ w,
                                           const Pair2<R> *rec, const R *sect, R *buf, bool alone,
                                           R *__restrict__ mbox) {
    constexpr int PP = P_ * P_;
    // channels with monopoles (bit c): every channel, except in the five-channel
    // set of the diagonal pass, whose channels 0 and 4 are pure dipoles
    constexpr unsigned QMASK = !MONO ? 0u : (NCH == 5 ? 0x0Eu : (1u << NCH) - 1u);
    const int lane = threadIdx.x & 63, wave = (threadIdx.x >> 6) % NW;
    R x[PPL], y[PPL], z[PPL], r2[PPL], sq[PPL][NCH], sw[PPL][NCH];
    R ux[PPL], uy[PPL], uz[PPL], vu2[PPL];
#pragma unroll
    for (int u = 0; u < PPL; ++u) {
        const bool ok = j0 + 64 * u + lane < re;
        const int j = ok ? j0 + 64 * u + lane : j0;  // idle slots: the first point, zero strength
        // leaf-relative, box-scaled coordinates formed in FP64, then rounded to R
        x[u] = (R)((px[j] - cx) * ih);
        y[u] = (R)((py[j] - cy) * ih);
        z[u] = (R)((pz[j] - cz) * ih);
        r2[u] = x[u] * x[u] + y[u] * y[u] + z[u] * z[u];
#pragma unroll
        for (int c = 0; c < NCH; ++c) {
            sq[u][c] = ((QMASK >> c) & 1u) ? (R)(ok ? q[(int64_t)c * n + j] : 0.0) : R(0);
            sw[u][c] = DIP ? (R)(ok ? w[(int64_t)c * n + j] * ih : 0.0) : R(0);
        }
        ux[u] = DIP ? (R)pnx[j] : R(0);
        uy[u] = DIP ? (R)pny[j] : R(0);
        uz[u] = DIP ? (R)pnz[j] : R(0);
        vu2[u] = R(2) * (x[u] * ux[u] + y[u] * uy[u] + z[u] * uz[u]);
    }
    int row = 0;  // buffered groups of four columns (wave-uniform)
    // places of the buffered columns: lane r describes row r (bits 0-11 the
    // place of column a, 12-18 the step to b and d, 19-27 the step to c and d,
    // 28-31 which of a..d exist)
    unsigned desc = 0;
    // buffered columns -> the leaf's expansion; the wave's LDS rows are its own,
    // and a wave's LDS operations complete in order
    constexpr bool RAW = sizeof(R) == 4;
    auto flush = [&]() {
        __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
        __builtin_amdgcn_wave_barrier();
        const int cl = RAW ? lane >> 2 : lane;  // column of this lane
        const unsigned dd = (unsigned)__shfl((int)desc, cl >> 2);
        R s0 = 0, s1 = 0;
        if (cl < 4 * row) {
            const R *col = RAW ? buf + cl * 68 + (lane & 3) : buf + (cl >> 2) * 64 + (cl & 3) * 16;
#pragma unroll
            for (int t = 0; t < 16; t += 2) {  // reduced rows: rotated starts, distinct banks
                s0 += col[RAW ? 4 * t : (t + lane) & 15];
                s1 += col[RAW ? 4 * (t + 1) : (t + 1 + lane) & 15];
            }
        }
        R sum = s0 + s1;
        if constexpr (RAW) {
            sum += __shfl_xor(sum, 1);
            sum += __shfl_xor(sum, 2);
        }
        if (cl < 4 * row && (!RAW || (lane & 3) == 0)) {
            // reduced rows: the 16-lane groups hold a, c, b, d
            const int isb = RAW ? cl & 1 : (cl >> 1) & 1, isc = RAW ? (cl >> 1) & 1 : cl & 1;
            if ((dd >> (28 + isb + 2 * isc)) & 1) {
                R *o = mbox + (dd & 0xfff) + (isb ? (dd >> 12) & 0x7f : 0) + (isc ? (dd >> 19) & 0x1ff : 0);
                if (alone)
                    *o += sum;
                else
                    unsafeAtomicAdd(o, sum);
            }
        }
        __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
        __builtin_amdgcn_wave_barrier();
        row = 0;
    };
    static_assert(NCH * PP <= 4096 && 2 * P_ < 128 && PP < 512, "place description");
    // columns a..d at places p, p + sb, p + sc, p + sb + sc (mask: which exist)
    auto push4 = [&](R a, R b, R c, R dd, int place, int sb, int sc, unsigned mask) {
        if constexpr (RAW) {
            R *o = buf + 4 * row * 68 + lane;
            o[0] = a;
            o[68] = b;
            o[2 * 68] = c;
            o[3 * 68] = dd;
        } else {
            buf[row * 64 + lane] = swap_add<false>(swap_add<true>(a, b), swap_add<true>(c, dd));
        }
        const unsigned d = (unsigned)place | ((unsigned)sb << 12) | ((unsigned)sc << 19) | (mask << 28);
        desc = lane == row ? d : desc;
        if (++row == (RAW ? 4 : kP2MRows)) flush();
    };
    // a channel's sum over this lane's points (a term is left out where the
    // channel has no monopole, or no dipole)
    auto dot = [&](int c, const R(&v)[PPL], const R(&dv)[PPL]) -> R {
        const bool hq = (QMASK >> c) & 1u;
        R t = 0;
#pragma unroll
        for (int u = 0; u < PPL; ++u) {
            if (hq) t += sq[u][c] * v[u];
            if (DIP) t += sw[u][c] * dv[u];
        }
        return t;
    };
    R dr[PPL], di[PPL], Ddr[PPL], Ddi[PPL];  // Rt_m^m and its derivative
#pragma unroll
    for (int u = 0; u < PPL; ++u) {
        dr[u] = 1;
        di[u] = Ddr[u] = Ddi[u] = 0;
    }
    int ms = 0;  // order the sectoral values are at
#pragma unroll 1
    for (int i = 0; leaf_order<NW>(wave, i) < P_; ++i) {
        const int m = leaf_order<NW>(wave, i);
#pragma unroll 1
        for (; ms < m; ++ms) {
            const R f = sect[ms + 1];
#pragma unroll
            for (int u = 0; u < PPL; ++u) {
                const R nr = (dr[u] * x[u] - di[u] * y[u]) * f, ni = (dr[u] * y[u] + di[u] * x[u]) * f;
                if (DIP) {
                    const R nDr = (Ddr[u] * x[u] - Ddi[u] * y[u] + dr[u] * ux[u] - di[u] * uy[u]) * f;
                    const R nDi = (Ddr[u] * y[u] + Ddi[u] * x[u] + dr[u] * uy[u] + di[u] * ux[u]) * f;
                    Ddr[u] = nDr;
                    Ddi[u] = nDi;
                }
                dr[u] = nr;
                di[u] = ni;
            }
        }
        // degrees k = m, m + 1, ...: A holds degree k, B degree k + 1 (at first
        // degree m - 1, zero)
        R Ar[PPL], Ai[PPL], Br[PPL], Bi[PPL], DAr[PPL], DAi[PPL], DBr[PPL], DBi[PPL];
#pragma unroll
        for (int u = 0; u < PPL; ++u) {
            Ar[u] = dr[u];
            Ai[u] = di[u];
            DAr[u] = Ddr[u];
            DAi[u] = Ddi[u];
            Br[u] = Bi[u] = DBr[u] = DBi[u] = 0;
        }
        // P <- degree k from C (degree k-1) and P (degree k-2)
        auto advance = [&](int t, const R(&Cr)[PPL], const R(&Ci)[PPL], const R(&DCr)[PPL], const R(&DCi)[PPL],
                           R(&Pr)[PPL], R(&Pi)[PPL], R(&DPr)[PPL], R(&DPi)[PPL]) {
            const Pair2<R> ca = rec[t];
#pragma unroll
            for (int u = 0; u < PPL; ++u) {
                const R ez = ca.x * z[u], br = ca.y * r2[u];
                if (DIP) {
                    const R eu = ca.x * uz[u], bv = ca.y * vu2[u];
                    const R nDr = eu * Cr[u] + ez * DCr[u] - bv * Pr[u] - br * DPr[u];
                    const R nDi = eu * Ci[u] + ez * DCi[u] - bv * Pi[u] - br * DPi[u];
                    DPr[u] = nDr;
                    DPi[u] = nDi;
                }
                Pr[u] = ez * Cr[u] - br * Pr[u];
                Pi[u] = ez * Ci[u] - br * Pi[u];
            }
        };
        int k = m;
#pragma unroll 1
        for (; k + 1 < P_; k += 2) {
            advance(tri(k + 1, m), Ar, Ai, DAr, DAi, Br, Bi, DBr, DBi);
            if (m > 0) {  // the conjugated coefficients of degrees k and k + 1
#pragma unroll
                for (int c = 0; c < NCH; ++c)
                    push4(dot(c, Ar, DAr), -dot(c, Ai, DAi), dot(c, Br, DBr), -dot(c, Bi, DBi),
                          c * PP + k * k + 2 * m - 1, 1, 2 * k + 1, 15u);
            } else {
#pragma unroll
                for (int c = 0; c < NCH; c += 2) {
                    const bool two = c + 1 < NCH;
                    const int c1 = two ? c + 1 : c;
                    push4(dot(c, Ar, DAr), dot(c, Br, DBr), two ? dot(c1, Ar, DAr) : R(0),
                          two ? dot(c1, Br, DBr) : R(0), c * PP + k * k, 2 * k + 1, PP, two ? 15u : 3u);
                }
            }
            if (k + 2 < P_) advance(tri(k + 2, m), Br, Bi, DBr, DBi, Ar, Ai, DAr, DAi);
        }
        if (k < P_) {  // the last degree alone
            const int o0 = m > 0 ? k * k + 2 * m - 1 : k * k;
#pragma unroll
            for (int c = 0; c < NCH; c += 2) {
                const bool two = c + 1 < NCH;
                const int c1 = two ? c + 1 : c;
                push4(dot(c, Ar, DAr), -dot(c, Ai, DAi), two ? dot(c1, Ar, DAr) : R(0), two ? -dot(c1, Ai, DAi) : R(0),
                      c * PP + o0, 1, PP, (two ? 5u : 1u) * (m > 0 ? 3u : 1u));
            }
        }
    }
    if (row > 0) flush();
}

template <int P_, int NCH, bool MONO, bool DIP, class R, int SP, int NW>
__global__ void __launch_bounds__(64 * SP * NW, NCH == 5 ? 3 : 1) k_p2m(const int2 *__restrict__ items, int64_t leaf0,
                                                         const int *__restrict__ leaf_pt,
                                                         const double *__restrict__ centre, double h,
                                                         const double *__restrict__ px, const double *__restrict__ py,
                                                         const double *__restrict__ pz, const double *__restrict__ pnx,
                                                         const double *__restrict__ pny,
                                                         const double *__restrict__ pnz, int64_t n,
                                                         const double *__restrict__ q, const double *__restrict__ w,
                                                         R *__restrict__ mexp) {
    constexpr int NT = P_ * (P_ + 1) / 2;
    __shared__ R buf[SP * NW][kP2MBuf<R>];
    __shared__ Pair2<R> rec[NT];
    __shared__ R sect[P_];
    const int wave = threadIdx.x >> 6;
    const int2 it = items[blockIdx.x];
    const int leaf = it.x, l0 = leaf_pt[leaf], l1 = leaf_pt[leaf + 1];
    // the points of this wave's group of NW waves
    constexpr int SUB = kLeafChunk / SP;
    const int rb = it.y + SUB * (wave / NW), re = min(rb + SUB, l1);
    const int64_t box = leaf0 + leaf;
    stage_tables<P_, R>(rec, sect, threadIdx.x, 64 * SP * NW);
    __syncthreads();
    if (rb >= re) return;
    const double cx = centre[3 * box], cy = centre[3 * box + 1], cz = centre[3 * box + 2];
    const double ih = 1.0 / h;
    R *mbox = mexp + box * NCH * P_ * P_;
    const bool alone = rb == l0 && re == l1;  // nobody else adds to this expansion
    auto run = [&](auto ppl, int j0) {
        p2m_points<P_, NCH, MONO, DIP, R, NW, decltype(ppl)::value>(j0, re, cx, cy, cz, ih, px, py, pz, pnx, pny, pnz,
                                                                    n, q, w, rec, sect, buf[wave], alone, mbox);
    };
    // with the derivatives the registers hold two points a lane, else four
    constexpr int MOST = DIP ? 128 : SUB;
#pragma unroll 1
    for (int j0 = rb; j0 < re; j0 += MOST) {
        const int cnt = re - j0;
        if (cnt <= 64) {
            run(std::integral_constant<int, 1>{}, j0);
        } else if (MOST == 128 || cnt <= 128) {
            if constexpr (SUB > 64) run(std::integral_constant<int, 2>{}, j0);
        } else if constexpr (MOST == 256) {
            if (cnt <= 192)
                run(std::integral_constant<int, 3>{}, j0);
            else
                run(std::integral_constant<int, 4>{}, j0);
        }
    }
}

// L2P. Lane l takes the group's points l, l + 64, ... (PPL of them) and the
// wave's orders:
//   y_i += (1/h) sum_n [Lt_n^0 Rt_n^0 + 2 sum_{m>0} Re(Lt_n^m Rt_n^m)],
// the harmonics built in registers. The leaf's coefficients, as (real,
// imaginary) pairs with the factors 2 and -2 taken in, and the recurrence
// constants are first copied to LDS; every step reads them at a wave-uniform
// LDS address. The sums of a group's waves are added through LDS.
// FIN (one channel): the product's result fin.out = (y + ...) / (4 pi) [+ f lii x]
// [+ g mii yv] is written instead of the sum.
struct L2PFinal {
    double f, g;
    const double *x, *yv, *lii, *mii;
    double *out;
};
template <int P_, int NCH, class R, int NW, int PPL>
__device__ __forceinline__ void l2p_points(int rb, int re, double cx, double cy, double cz, double ih,
                                           const double *__restrict__ px, const double *__restrict__ py,
                                           const double *__restrict__ pz, const Pair2<R> (*Ls)[NCH],
                                           const Pair2<R> *rec, const R *sect, R (&acc)[4][NCH]) {
    const int lane = threadIdx.x & 63, wave = (threadIdx.x >> 6) % NW;
    R x[PPL], yy[PPL], z[PPL], r2[PPL];
#pragma unroll
    for (int u = 0; u < PPL; ++u) {
        const int j0 = rb + 64 * u + lane;
        const int j = j0 < re ? j0 : rb;
        x[u] = (R)((px[j] - cx) * ih);
        yy[u] = (R)((py[j] - cy) * ih);
        z[u] = (R)((pz[j] - cz) * ih);
        r2[u] = x[u] * x[u] + yy[u] * yy[u] + z[u] * z[u];
    }
    R dr[PPL], di[PPL];
#pragma unroll
    for (int u = 0; u < PPL; ++u) {
        dr[u] = 1;
        di[u] = 0;
    }
    int ms = 0;
#pragma unroll 1
    for (int i = 0; leaf_order<NW>(wave, i) < P_; ++i) {
        const int m = leaf_order<NW>(wave, i);
#pragma unroll 1
        for (; ms < m; ++ms) {
            const R f = sect[ms + 1];
#pragma unroll
            for (int u = 0; u < PPL; ++u) {
                const R nr = (dr[u] * x[u] - di[u] * yy[u]) * f, ni = (dr[u] * yy[u] + di[u] * x[u]) * f;
                dr[u] = nr;
                di[u] = ni;
            }
        }
        R Ar[PPL], Ai[PPL], Br[PPL], Bi[PPL];  // degree k, degree k + 1 (at first zero)
#pragma unroll
        for (int u = 0; u < PPL; ++u) {
            Ar[u] = dr[u];
            Ai[u] = di[u];
            Br[u] = Bi[u] = 0;
        }
        auto advance = [&](int t, const R(&Cr)[PPL], const R(&Ci)[PPL], R(&Pr)[PPL], R(&Pi)[PPL]) {
            const Pair2<R> ca = rec[t];
#pragma unroll
            for (int u = 0; u < PPL; ++u) {
                const R ez = ca.x * z[u], br = ca.y * r2[u];
                Pr[u] = ez * Cr[u] - br * Pr[u];
                Pi[u] = ez * Ci[u] - br * Pi[u];
            }
        };
        auto gather = [&](int t, const R(&Cr)[PPL], const R(&Ci)[PPL]) {
#pragma unroll
            for (int c = 0; c < NCH; ++c) {
                const Pair2<R> l = Ls[t][c];
#pragma unroll
                for (int u = 0; u < PPL; ++u) acc[u][c] += l.x * Cr[u] + l.y * Ci[u];
            }
        };
        int k = m, t = tri(m, m);
#pragma unroll 1
        for (; k + 1 < P_; k += 2) {
            gather(t, Ar, Ai);
            t += k + 1;
            advance(t, Ar, Ai, Br, Bi);
            gather(t, Br, Bi);
            t += k + 2;
            if (k + 2 < P_) advance(t, Br, Bi, Ar, Ai);
        }
        if (k < P_) gather(t, Ar, Ai);
    }
}

template <int P_, int NCH, class R, bool FIN, int SP, int NW>
__global__ void __launch_bounds__(64 * SP * NW) k_l2p(const int2 *__restrict__ items, int64_t leaf0,
                                                         const int *__restrict__ leaf_pt,
                                                         const double *__restrict__ centre, double h,
                                                         const double *__restrict__ px, const double *__restrict__ py,
                                                         const double *__restrict__ pz, int64_t n,
                                                         const R *__restrict__ lexp, double *__restrict__ y,
                                                         L2PFinal fin) {
    static_assert(!FIN || NCH == 1, "one channel");
    constexpr int PP = P_ * P_, NT = P_ * (P_ + 1) / 2;
    // the coefficients while the harmonics run, the waves' sums afterwards
    constexpr size_t LB = sizeof(Pair2<R>) * NT * NCH, SB = NW > 1 ? sizeof(R) * SP * NW * 4 * NCH * 64 : 0;
    __shared__ __align__(16) char mem[LB > SB ? LB : SB];
    __shared__ Pair2<R> rec[NT];
    __shared__ R sect[P_];
    Pair2<R>(*Ls)[NCH] = reinterpret_cast<Pair2<R>(*)[NCH]>(mem);
    R *sums = reinterpret_cast<R *>(mem);
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int2 it = items[blockIdx.x];
    constexpr int SUB = kLeafChunk / SP;  // points of a group of NW waves
    const int leaf = it.x, rb = it.y + SUB * (wave / NW);
    const int re = min(rb + SUB, leaf_pt[leaf + 1]);
    const int64_t box = leaf0 + leaf;
    const R *L = lexp + box * NCH * PP;
    for (int e = tid; e < NCH * PP; e += 64 * SP * NW) {
        const int c = e / PP, o = e - c * PP;
        int k = (int)sqrtf((float)o);  // degree: k^2 <= o < (k + 1)^2
        k -= k * k > o;
        k += (k + 1) * (k + 1) <= o;
        const int r = o - k * k, m = (r + 1) >> 1;
        Pair2<R> &d = Ls[tri(k, m)][c];
        const R v = L[e];
        if (m == 0)
            d = Pair2<R>{v, R(0)};
        else if (r & 1)
            d.x = R(2) * v;
        else
            d.y = R(-2) * v;
    }
    stage_tables<P_, R>(rec, sect, tid, 64 * SP * NW);
    const double ih = 1.0 / h;
    const double cx = centre[3 * box], cy = centre[3 * box + 1], cz = centre[3 * box + 2];
    R acc[4][NCH];
#pragma unroll
    for (int u = 0; u < 4; ++u)
#pragma unroll
        for (int c = 0; c < NCH; ++c) acc[u][c] = 0;
    __syncthreads();
    const int cnt = re - rb;
    auto run = [&](auto ppl) {
        l2p_points<P_, NCH, R, NW, decltype(ppl)::value>(rb, re, cx, cy, cz, ih, px, py, pz, Ls, rec, sect, acc);
    };
    if (cnt > 0 && cnt <= 64) {
        run(std::integral_constant<int, 1>{});
    } else if (cnt > 64 && cnt <= 128) {
        if constexpr (SUB >= 128) run(std::integral_constant<int, 2>{});
    } else if (cnt > 128) {
        if constexpr (SUB >= 256) {
            if (cnt <= 192)
                run(std::integral_constant<int, 3>{});
            else
                run(std::integral_constant<int, 4>{});
        }
    }
    auto finish = [&](int c, int j, R v) {
        if constexpr (FIN) {
            double o = kInv4Pi * (y[j] + (double)v * ih);
            if (fin.lii && fin.x) o += fin.f * fin.lii[j] * fin.x[j];
            if (fin.mii && fin.yv) o += fin.g * fin.mii[j] * fin.yv[j];
            fin.out[j] = o;
        } else {
            y[(int64_t)c * n + j] += (double)v * ih;
        }
    };
    if constexpr (NW == 1) {
#pragma unroll
        for (int u = 0; u < 4; ++u) {
            const int j = rb + 64 * u + lane;
            if (j >= re) break;
#pragma unroll
            for (int c = 0; c < NCH; ++c) finish(c, j, acc[u][c]);
        }
    } else {
        __syncthreads();  // the coefficients have been read
#pragma unroll
        for (int u = 0; u < 4; ++u)
#pragma unroll
            for (int c = 0; c < NCH; ++c) sums[((wave * 4 + u) * NCH + c) * 64 + lane] = acc[u][c];
        __syncthreads();
        const int wg = wave / NW * NW;  // the group's first wave
#pragma unroll 1
        for (int u = wave - wg; u < 4; u += NW) {  // wave u finishes points rb + 64 u + lane
            const int j = rb + 64 * u + lane;
            if (j >= re) break;
#pragma unroll
            for (int c = 0; c < NCH; ++c) {
                R v = 0;
#pragma unroll
                for (int q = 0; q < NW; ++q) v += sums[(((wg + q) * 4 + u) * NCH + c) * 64 + lane];
                finish(c, j, v);
            }
        }
    }
}

// Work items from which a launch fills the chip (six waves a CU) without
// splitting the orders of an item over waves: from there on the waves split
// its points, which repeats nothing. Measured alone, orders / points split, us:
// L2P five channels, order 20: 494 items 47 / 50, 2600 items 134 / 119, 4400
// items 225 / 185; one channel, order 16: 900 items 20 / 22, 2600 items 44 / 38.
// P2M five channels, order 20: 494 items 113 / 128, 2600 items 274 / 276, 4400
// items 468 / 409; FP32, order 8: 494 items 10.7 / 13.3, 4400 items 29.4 / 23.8.
// The FP64 P2M of monopoles alone stays with split orders (4400 items 75 / 82).
// The FP32 L2P splits points at every size (order 8, 494 items 9.0, 10.1 with
// 128 points a wave).
constexpr int64_t kLeafItemsMany = 1536;

template <int P_, int NCH, bool MONO, bool DIP, class R>
void launch_p2m(const Tree &t, const Sources &src, R *M, hipStream_t st) {
    if (t.n_leaf_items <= 0) return;
    const int64_t leaf0 = t.lvl_off[t.lmax];
    const double hleaf = t.side / (double)(1 << t.lmax);
    constexpr int S = sizeof(R) == 4 ? 2 : 1;  // FP32: groups of 128 points in either split
    const bool points = t.n_leaf_items >= kLeafItemsMany && (DIP || sizeof(R) == 4);
    auto kern = points ? k_p2m<P_, NCH, MONO, DIP, R, 2, 1> : k_p2m<P_, NCH, MONO, DIP, R, S, 4>;
    kern<<<(unsigned)t.n_leaf_items, points ? 128 : 256 * S, 0, st>>>(
        t.leaf_items.get(), leaf0, t.leaf_pt.get(), t.box_centre.get(), hleaf, t.px.get(), t.py.get(), t.pz.get(),
        t.pnx.get(), t.pny.get(), t.pnz.get(), t.n, src.q, src.w, M);
    BFM_LAUNCHED();
}

template <int P_, int NCH, class R>
void launch_l2p(const Tree &t, const Sources &src, const R *L, double *y, hipStream_t st) {
    if (t.n_leaf_items <= 0) return;
    const int64_t leaf0 = t.lvl_off[t.lmax];
    const double hleaf = t.side / (double)(1 << t.lmax);
    const L2PFinal fin{src.f, src.g, src.x, src.yv, src.lii, src.mii, src.out};
    const bool points = t.n_leaf_items >= kLeafItemsMany;
    constexpr int S = sizeof(R) == 4 ? 4 : 1, W = 4 / S;  // FP32: one wave adds up a point's orders
    auto kern = points ? k_l2p<P_, NCH, R, false, 4, 1> : k_l2p<P_, NCH, R, false, S, W>;
    if constexpr (NCH == 1)
        if (src.out) kern = points ? k_l2p<P_, NCH, R, true, 4, 1> : k_l2p<P_, NCH, R, true, S, W>;
    kern<<<(unsigned)t.n_leaf_items, 256, 0, st>>>(t.leaf_items.get(), leaf0, t.leaf_pt.get(),
                                                               t.box_centre.get(), hleaf, t.px.get(), t.py.get(),
                                                               t.pz.get(), t.n, L, y, fin);
    BFM_LAUNCHED();
}

#define BFM_LEAF_INST(P)                                                                   \
    template void launch_p2m<P, 1, true, false>(const Tree &, const Sources &, double *, hipStream_t); \
    template void launch_p2m<P, 1, false, true>(const Tree &, const Sources &, double *, hipStream_t); \
    template void launch_p2m<P, 1, true, true>(const Tree &, const Sources &, double *, hipStream_t);  \
    template void launch_p2m<P, 5, true, true>(const Tree &, const Sources &, double *, hipStream_t);  \
    template void launch_l2p<P, 1>(const Tree &, const Sources &, const double *, double *, hipStream_t); \
    template void launch_l2p<P, 5>(const Tree &, const Sources &, const double *, double *, hipStream_t); \
    template void launch_p2m<P, 1, true, false, float>(const Tree &, const Sources &, float *, hipStream_t); \
    template void launch_p2m<P, 1, false, true, float>(const Tree &, const Sources &, float *, hipStream_t); \
    template void launch_p2m<P, 1, true, true, float>(const Tree &, const Sources &, float *, hipStream_t);  \
    template void launch_l2p<P, 1, float>(const Tree &, const Sources &, const float *, double *, hipStream_t);
BFM_LEAF_INST(4)
BFM_LEAF_INST(8)
BFM_LEAF_INST(12)
BFM_LEAF_INST(16)
BFM_LEAF_INST(20)
#undef BFM_LEAF_INST

}  // namespace bfm
