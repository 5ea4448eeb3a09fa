// Geometry (ns1), the singular diagonals and right-hand side (s3, s5,
// eq3_1), the product with L (eq3_27) and restarted GMRES (Section 3.8),
// all on the handle's stream. Solve vectors live in the octree's sorted
// point order so that the fast multipole product needs no gather/scatter.
#include <algorithm>
#include <cmath>
#include <vector>

#include "ctx.h"
#include "xcd.h"

namespace bfm {

static unsigned nblk(int64_t n, int t) { return (unsigned)((n + t - 1) / t); }

// ---------------------------------------------------------------------------
// Geometry (Section 3.2, ns1): per triangle c = (r2 - r1) x (r3 - r1),
// A = |c|/2, N A = c/2; per vertex s = sum A/3, n = (sum N A)/|sum N A|.

// Per triangle: half the cross product (the area-weighted normal) and the
// area, one 32-byte record (x, y, z, area) so that a vertex gathers each of
// its triangles with one load
__global__ void k_tri_geom(const double *xyz, const int *tri, int64_t nt, int64_t nv, double4 *rec, int *flag) {
    const int64_t k = xcd_block() * blockDim.x + threadIdx.x;  // a bubble's vertices stay in one L2
    if (k >= nt) return;
    const int a = tri[3 * k], b = tri[3 * k + 1], c = tri[3 * k + 2];
    if (a < 0 || b < 0 || c < 0 || a >= nv || b >= nv || c >= nv) {
        atomicOr(flag, 2);
        rec[k] = make_double4(0.0, 0.0, 0.0, 0.0);
        return;
    }
    const double e1x = xyz[3 * b] - xyz[3 * a], e1y = xyz[3 * b + 1] - xyz[3 * a + 1],
                 e1z = xyz[3 * b + 2] - xyz[3 * a + 2];
    const double e2x = xyz[3 * c] - xyz[3 * a], e2y = xyz[3 * c + 1] - xyz[3 * a + 1],
                 e2z = xyz[3 * c + 2] - xyz[3 * a + 2];
    const double cx = e1y * e2z - e1z * e2y, cy = e1z * e2x - e1x * e2z, cz = e1x * e2y - e1y * e2x;
    const double len = sqrt(cx * cx + cy * cy + cz * cz);
    // zero area up to rounding: |e1 x e2| against |e1| |e2| (a repeated vertex
    // gives a cross product of rounding size, not exactly zero, under FMA)
    const double scale = sqrt((e1x * e1x + e1y * e1y + e1z * e1z) * (e2x * e2x + e2y * e2y + e2z * e2z));
    if (!(len > 1e-12 * scale)) atomicOr(flag, 1);
    rec[k] = make_double4(0.5 * cx, 0.5 * cy, 0.5 * cz, 0.5 * len);
}

__global__ void k_fill_flag(int *flag) { *flag = 0; }

__global__ void k_vertex_geom(const int *v2t_off, const int *v2t, const double4 *rec, int64_t nv, double *s,
                              double *nrm, int *flag) {
    const int64_t j = xcd_block() * blockDim.x + threadIdx.x;  // a bubble's triangles stay in one L2
    if (j >= nv) return;
    double sa = 0.0, mx = 0.0, my = 0.0, mz = 0.0;
    const int e0 = v2t_off[j], e1 = v2t_off[j + 1];
#pragma unroll 4
    for (int e = e0; e < e1; ++e) {  // ascending triangle index: a fixed summation order
        const double4 r = rec[v2t[e]];
        mx += r.x;
        my += r.y;
        mz += r.z;
        sa += r.w;
    }
    const double len = sqrt(mx * mx + my * my + mz * mz);
    if (!(len > 0.0)) atomicOr(flag, 4);
    const double il = (len > 0.0) ? 1.0 / len : 0.0;
    s[j] = sa / 3.0;
    nrm[j] = mx * il;
    nrm[nv + j] = my * il;
    nrm[2 * nv + j] = mz * il;
}

// The mesh checks of the geometry kernels land in a pinned flag; check_now
// waits for it, otherwise the first wait of the octree build that follows
// (geometry_check) brings it in with no extra round trip.
void ensure_geometry(bfm_ctx *c, bool check_now) {
    if (c->geom_valid) return;
    BFM_CHECK(c->nv > 0, BFM_EINVAL, "no mesh set");
    hipStream_t st = c->stream;
    c->s.ensure(c->nv);
    c->nrm.ensure(3 * c->nv);
    c->tri_rec.ensure(4 * c->nt);
    int *flag = c->flag.ensure(1);
    if (!c->host_flag) BFM_HIP(hipHostMalloc((void **)&c->host_flag, sizeof(int), 0));
    k_fill_flag<<<1, 1, 0, st>>>(flag);
    BFM_LAUNCHED();
    double4 *rec = reinterpret_cast<double4 *>(c->tri_rec.get());
    k_tri_geom<<<nblk(c->nt, 256), 256, 0, st>>>(c->xyz.get(), c->tri.get(), c->nt, c->nv, rec, flag);
    BFM_LAUNCHED();
    k_vertex_geom<<<nblk(c->nv, 256), 256, 0, st>>>(c->v2t_off.get(), c->v2t.get(), rec, c->nv, c->s.get(),
                                                    c->nrm.get(), flag);
    BFM_LAUNCHED();
    BFM_HIP(hipMemcpyAsync(c->host_flag, flag, sizeof(int), hipMemcpyDeviceToHost, st));
    corr_invalidate(c, false);
    c->geom_valid = true;
    c->geom_unchecked = true;
    if (check_now) geometry_check(c);
}

void geometry_check(bfm_ctx *c, bool synced) {
    if (!c->geom_unchecked) return;
    if (!synced) BFM_HIP(hipStreamSynchronize(c->stream));
    c->geom_unchecked = false;
    const int hf = *c->host_flag;
    if (hf) c->geom_valid = false;  // a later call rebuilds and fails the same way
    BFM_CHECK(!(hf & 2), BFM_EMESH, "triangle vertex index out of range");
    BFM_CHECK(!(hf & 1), BFM_EMESH, "degenerate (zero-area) triangle");
    BFM_CHECK(!(hf & 4), BFM_EMESH, "vertex with vanishing area-weighted normal");
}

void ensure_tree(bfm_ctx *c) {
    ensure_geometry(c, false);
    if (c->tree_valid) {
        geometry_check(c);
        return;
    }
    const int pi = c->prof.begin(KC_TREE, c->stream);
    build_tree(c->tree, c->xyz.get(), c->nv, c->opt.lmax, c->opt.leaf_target, c->opt.p2p_shape, c->stream);
    // the build has waited for the stream after the flag's copy (its bounding
    // box is read back first): no extra round trip
    geometry_check(c, true);
    sort_geometry(c->tree, c->s.get(), c->nrm.get(), c->stream);
    c->prof.end(pi, c->stream, 0.0, 0.0);
    c->tree_valid = true;
    c->diag_valid = false;
    corr_invalidate(c, false);  // the corrections are stored in the octree's order
    graph_invalidate(c);
}

int diag_order(const bfm_options &o) {
    if (o.p_diag > 0) return o.p_diag;
    return o.p + 4 <= kMaxP ? o.p + 4 : kMaxP;
}

void ensure_ops(bfm_ctx *c) {
    c->fmm.p = c->opt.p;
    c->fmm.m2l_shape = c->opt.m2l_shape;
    c->fmm.m2l_orders = c->opt.m2l_orders;
    fmm_prepare_ops(c->fmm, c->opt.p, c->stream);
    c->fmm_diag.p = diag_order(c->opt);
    c->fmm_diag.m2l_orders = c->opt.m2l_orders;
    c->fmm_diag.m2l_shape = c->opt.m2l_shape == 3 ? 3 : -1;  // the rotation-factored M2L follows the option
    fmm_prepare_ops(c->fmm_diag, c->fmm_diag.p, c->stream);
}

void ensure_ops_lo(bfm_ctx *c, int prec) {
    BFM_CHECK(prec == BFM_PREC_FP32 || prec == BFM_PREC_BF16X3, BFM_EINVAL, "not a low precision");
    const int p = c->opt.p_lo > 0 ? c->opt.p_lo : c->opt.p;
    if (c->fmm_lo.prec != prec || c->fmm_lo.p != p) graph_invalidate(c);
    c->fmm_lo.prec = prec;
    c->fmm_lo.p = p;
    c->fmm_lo.m2l_shape = c->opt.m2l_shape;
    c->fmm_lo.m2l_orders = c->opt.m2l_orders;
    fmm_prepare_ops(c->fmm_lo, p, c->stream);
}

// ---------------------------------------------------------------------------
// Permutations

__global__ void k_gather(const double *in, const int *perm, int64_t n, double *out) {
    int64_t i = blockIdx.x * (int64_t)blockDim.x + threadIdx.x;
    if (i < n) out[i] = in[perm[i]];
}

__global__ void k_scatter(const double *in, const int *perm, int64_t n, double *out) {
    int64_t i = blockIdx.x * (int64_t)blockDim.x + threadIdx.x;
    if (i < n) out[perm[i]] = in[i];
}

void to_sorted(bfm_ctx *c, const double *in, double *out) {
    k_gather<<<nblk(c->nv, 256), 256, 0, c->stream>>>(in, c->tree.idx_a.get(), c->nv, out);
    BFM_LAUNCHED();
}

void to_original(bfm_ctx *c, const double *in, double *out) {
    k_scatter<<<nblk(c->nv, 256), 256, 0, c->stream>>>(in, c->tree.idx_a.get(), c->nv, out);
    BFM_LAUNCHED();
}

// ---------------------------------------------------------------------------
// Diagonals + right-hand side: five channels over the same points,
// coordinates taken relative to the cube centre X; every dipole points along
// the vertex normal, so a channel stores its scalar weight w (moment w n_j):
//   ch0: w = s                          -> sum M_ij
//   ch1..3: q = -s n_a, w = s r_a       -> sum M_ij r_ja - sum L_ij n_ja
//   ch4: w = s phi                      -> sum M_ij phi_j
// (channels 0 and 4 carry no monopole: the five-channel P2M leaves their
// monopole terms out)

__global__ void k_diag_sources(const double *px, const double *py, const double *pz, const double *ps,
                               const double *pnx, const double *pny, const double *pnz,
                               const double *phi, int64_t n, double X, double Y, double Z, double *q,
                               double *w, double *pk) {
    int64_t i = blockIdx.x * (int64_t)blockDim.x + threadIdx.x;
    if (i >= n) return;
    const double s = ps[i];
    const double nn[3] = {pnx[i], pny[i], pnz[i]};
    const double r[3] = {px[i] - X, py[i] - Y, pz[i] - Z};
    const double w4 = s * (phi ? phi[i] : 0.0);
    q[i] = 0.0;
    q[4 * n + i] = 0.0;
    w[i] = s;
    w[4 * n + i] = w4;
    for (int a = 0; a < 3; ++a) {
        q[(1 + a) * n + i] = -s * nn[a];
        w[(1 + a) * n + i] = s * r[a];
    }
    // packed record for the near field (layout of Sources::packed)
    double *rec = pk + i * kDiagRec;
    rec[0] = px[i];
    rec[1] = py[i];
    rec[2] = pz[i];
    for (int a = 0; a < 3; ++a) {
        rec[3 + a] = nn[a];
        rec[6 + a] = -s * nn[a];
        rec[10 + a] = s * r[a];
    }
    rec[9] = s;
    rec[13] = w4;
    rec[14] = rec[15] = 0.0;
}

__global__ void k_diag_finalize(const double *y, const double *px, const double *py, const double *pz,
                                const double *pnx, const double *pny, const double *pnz,
                                const double *phi, int64_t n, double X, double Y, double Z,
                                double *mii, double *lii, double *b) {
    int64_t i = blockIdx.x * (int64_t)blockDim.x + threadIdx.x;
    if (i >= n) return;
    const double SM = kInv4Pi * y[i];
    const double r[3] = {px[i] - X, py[i] - Y, pz[i] - Z};
    const double nn[3] = {pnx[i], pny[i], pnz[i]};
    double L = 0.0;
    for (int a = 0; a < 3; ++a) L += nn[a] * (kInv4Pi * y[(1 + a) * n + i] - r[a] * SM);
    mii[i] = -0.5 - SM;
    lii[i] = L;
    if (phi) b[i] = -phi[i] * (1.0 + SM) + kInv4Pi * y[4 * n + i];
}

void diagonal_pass(bfm_ctx *c, const double *phi_dev) {
    ensure_tree(c);
    ensure_ops(c);
    hipStream_t st = c->stream;
    const int pi = c->prof.begin(KC_DIAG, st);
    Tree &t = c->tree;
    const int64_t n = c->nv;
    const double X = t.origin[0] + 0.5 * t.side, Y = t.origin[1] + 0.5 * t.side,
                 Z = t.origin[2] + 0.5 * t.side;
    double *phs = nullptr;
    if (phi_dev) {
        phs = c->phi_s.ensure(n);
        to_sorted(c, phi_dev, phs);
    }
    double *q = c->src_q.ensure(5 * n);
    double *wd = c->src_w.ensure(5 * n);
    double *y = c->ysum.ensure(5 * n);
    double *pk = c->src_pk.ensure((size_t)kDiagRec * n);
    k_diag_sources<<<nblk(n, 256), 256, 0, st>>>(t.px.get(), t.py.get(), t.pz.get(), t.ps.get(),
                                                 t.pnx.get(), t.pny.get(), t.pnz.get(), phs, n, X, Y, Z,
                                                 q, wd, pk);
    BFM_LAUNCHED();
    Sources src;
    src.nch = 5;
    src.mono = true;
    src.dip = true;
    src.q = q;
    src.w = wd;
    src.packed = pk;
    fmm_apply(c->fmm_diag, t, src, y, false, st);
    c->mii_s.ensure(n);
    c->lii_s.ensure(n);
    c->b_s.ensure(n);
    k_diag_finalize<<<nblk(n, 256), 256, 0, st>>>(y, t.px.get(), t.py.get(), t.pz.get(), t.pnx.get(),
                                                  t.pny.get(), t.pnz.get(), phs, n, X, Y, Z,
                                                  c->mii_s.get(), c->lii_s.get(), c->b_s.get());
    BFM_LAUNCHED();
    corr_diagonals(c, phs);
    c->prof.end(pi, st, 0.0, 0.0);
    c->diag_valid = true;
}

// ---------------------------------------------------------------------------
// Product with A = f L + g M (eq3_27), sorted order.

__global__ void k_sources_1ch(const double *ps, int64_t n, double f, const double *x, double g,
                              const double *yv, double *q, double *w) {
    int64_t i = blockIdx.x * (int64_t)blockDim.x + threadIdx.x;
    if (i >= n) return;
    const double s = ps[i];
    if (x) q[i] = f * s * x[i];
    if (yv) w[i] = g * s * yv[i];
}

__global__ void k_finalize_1ch(const double *y, int64_t n, double f, const double *x, double g,
                               const double *yv, const double *lii, const double *mii, double *out) {
    int64_t i = blockIdx.x * (int64_t)blockDim.x + threadIdx.x;
    if (i >= n) return;
    double v = kInv4Pi * y[i];
    if (lii && x) v += f * lii[i] * x[i];
    if (mii && yv) v += g * mii[i] * yv[i];
    out[i] = v;
}

void matvec_sorted(bfm_ctx *c, double f, const double *x_s, double g, const double *y_s, double *out_s,
                   bool add_diag, int precision, bool direct) {
    BFM_CHECK(precision == BFM_PREC_FP64 || precision == BFM_PREC_FP32 || precision == BFM_PREC_BF16X3,
              BFM_EINVAL, "unknown precision");
    ensure_tree(c);
    const bool lo = precision != BFM_PREC_FP64 && !direct;
    if (!direct) ensure_ops(c);
    if (lo) ensure_ops_lo(c, precision);
    if (add_diag && !c->diag_valid) diagonal_pass(c, nullptr);
    ensure_corr(c);
    hipStream_t st = c->stream;
    Tree &t = c->tree;
    const int64_t n = c->nv;
    const bool mono = (f != 0.0 && x_s), dip = (g != 0.0 && y_s);
    double *q = c->src_q.ensure(5 * n);
    double *wd = c->src_w.ensure(5 * n);
    double *y = c->ysum.ensure(5 * n);
    if (!mono && !dip) {
        BFM_HIP(hipMemsetAsync(out_s, 0, sizeof(double) * n, st));
        return;
    }
    Sources src;
    src.nch = 1;
    src.mono = mono;
    src.dip = dip;
    src.q = q;
    src.w = wd;
    src.f = f;
    src.g = g;
    src.x = mono ? x_s : nullptr;
    src.yv = dip ? y_s : nullptr;
    if (direct) {
        k_sources_1ch<<<nblk(n, 256), 256, 0, st>>>(t.ps.get(), n, f, src.x, g, src.yv, q, wd);
        BFM_LAUNCHED();
        fmm_apply(c->fmm, t, src, y, true, st);
        k_finalize_1ch<<<nblk(n, 256), 256, 0, st>>>(y, n, f, src.x, g, src.yv, add_diag ? c->lii_s.get() : nullptr,
                                                     add_diag ? c->mii_s.get() : nullptr, out_s);
        BFM_LAUNCHED();
    } else {  // the strengths and the result are formed by the product's own first and last kernel
        src.ps = t.ps.get();
        src.qout = q;
        src.wout = wd;
        src.out = out_s;
        src.lii = add_diag ? c->lii_s.get() : nullptr;
        src.mii = add_diag ? c->mii_s.get() : nullptr;
        fmm_apply(lo ? c->fmm_lo : c->fmm, t, src, y, false, st);
    }
    corr_apply(c, f, mono ? x_s : nullptr, g, dip ? y_s : nullptr, out_s);
}

// ---------------------------------------------------------------------------
// GMRES (restarted, classical Gram-Schmidt with one reorthogonalisation,
// Givens rotations on the device). Reductions are two-stage with a fixed
// block count for a given n, so sums are bitwise reproducible run to run.
//
// An Arnoldi step's orthogonalisation is a chain of short passes over the
// basis; with every dot product, reduction, update, norm, rotation and
// scaling in a launch of its own it was ten launches and a copy, 45 us of
// mostly launch latency (642 to 642,000 points). Each pass now starts by adding up the partial
// sums the pass before it left (every block does, which costs less than a
// launch) and ends with the partial sums of the next: dots of w; update and
// dots again (the basis is read once for both); update and norm; rotation
// and scaling. On small meshes one workgroup does the whole step (gs_in_one).
// Measured: see gs_step.

constexpr int kRedBlocks = 512;
constexpr int kRedThreads = 256;
constexpr int kGsFuse = 32;          // basis vectors a fused pass holds in registers
constexpr int64_t kSmallGs = 4096;   // points one workgroup holds
constexpr int kMaxRestart = 128;

// two points a thread at least: every block adds up all blocks' partials
static int red_blocks(int64_t n) { return (int)std::min<int64_t>(kRedBlocks, nblk(n, 2 * kRedThreads)); }

// Sums a wave's 64 lanes of KM values (a power of two up to 64): every
// exchange halves the values a lane keeps, so KM values cost about KM
// exchanges instead of 6 KM. On return lane l's v[0] is the sum of value
// wave_slot<KM>(l).
template <int KM>
__device__ inline int wave_slot(int lane) {
    int slot = 0;
#pragma unroll
    for (int w = KM / 2, mask = 32; w >= 1; w /= 2, mask /= 2) slot += (lane & mask) ? w : 0;
    return slot;
}
template <int W, int MASK, int KM>
__device__ __forceinline__ void wave_sum_step(double (&v)[KM], int lane) {
    if constexpr (W >= 1) {
        const bool up = (lane & MASK) != 0;
#pragma unroll
        for (int i = 0; i < W; ++i) {
            const double send = up ? v[i] : v[i + W];
            v[i] = (up ? v[i + W] : v[i]) + __shfl_xor(send, MASK);
        }
        wave_sum_step<W / 2, MASK / 2, KM>(v, lane);
    } else if constexpr (MASK >= 1) {
        v[0] += __shfl_xor(v[0], MASK);
        wave_sum_step<0, MASK / 2, KM>(v, lane);
    }
}
template <int KM>
__device__ __forceinline__ void wave_sum(double (&v)[KM], int lane) {
    wave_sum_step<KM / 2, 32, KM>(v, lane);
}

// part[k * kRedBlocks + block] = the block's sum of v[k], k < kn (256 threads)
template <int KM>
__device__ inline void block_part(double (&v)[KM], int kn, double *part, double (*red)[KM]) {
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    wave_sum<KM>(v, lane);
    red[wave][wave_slot<KM>(lane)] = v[0];  // lanes of one slot write the same value
    __syncthreads();
    if ((int)threadIdx.x < kn)
        part[threadIdx.x * kRedBlocks + blockIdx.x] =
            ((red[0][threadIdx.x] + red[1][threadIdx.x]) + red[2][threadIdx.x]) + red[3][threadIdx.x];
}

// h[k] = sum over the nblk partials of value k, k < nvec (a block of 256):
// eight lanes a value, so that 32 values' loads are in flight at once
__device__ inline void part_sum(const double *part, int nblk, int nvec, double *h) {
    const int l8 = threadIdx.x & 7;
    for (int k = threadIdx.x >> 3; k < nvec; k += kRedThreads / 8) {
        double a = 0.0;
#pragma unroll 8
        for (int b = l8; b < nblk; b += 8) a += part[k * kRedBlocks + b];
        for (int o = 4; o > 0; o >>= 1) a += __shfl_xor(a, o);
        if (l8 == 0) h[k] = a;
    }
    __syncthreads();
}

// partials of V_k . w for k in [k0, k0 + kn), kn <= KM
template <int KM>
__global__ void __launch_bounds__(kRedThreads) k_gs_dot(const double *__restrict__ V, int k0, int kn, int64_t ld,
                                                        const double *__restrict__ w, int64_t n,
                                                        double *__restrict__ part) {
    __shared__ double red[4][KM];
    double acc[KM];
#pragma unroll
    for (int k = 0; k < KM; ++k) acc[k] = 0.0;
    const double *Vk = V + k0 * ld;
    for (int64_t i = blockIdx.x * (int64_t)kRedThreads + threadIdx.x; i < n; i += (int64_t)gridDim.x * kRedThreads) {
        const double wi = w[i];
        double x[KM];
        // past the last vector: the last one again (all loads in flight at
        // once, no branch), its sum unused
#pragma unroll
        for (int k = 0; k < KM; ++k) x[k] = Vk[min(k, kn - 1) * ld + i];
#pragma unroll
        for (int k = 0; k < KM; ++k) acc[k] = fma(x[k], wi, acc[k]);
    }
    block_part<KM>(acc, kn, part + k0 * kRedBlocks, red);
}

// h = sums of part (stored to hout by block 0); w -= V h; then the partials of
// V_k . w (DOT, nvec <= KM: the basis values stay in registers) or of ||w||^2
// to part_out. KM == 0: any number of vectors, ||w||^2 only.
template <int KM, bool DOT>
__global__ void __launch_bounds__(kRedThreads) k_gs_update(const double *__restrict__ V, int nvec, int64_t ld,
                                                           const double *__restrict__ part, double *__restrict__ w,
                                                           int64_t n, double *__restrict__ hout,
                                                           double *__restrict__ part_out) {
    static_assert(KM > 0 || !DOT, "dots need the basis in registers");
    constexpr int KA = DOT ? KM : 1, KX = KM > 0 ? KM : 1;
    __shared__ double red[4][KA];
    __shared__ double h[kMaxRestart + 1];
    if (KM > 0 && (int)threadIdx.x >= nvec && (int)threadIdx.x < KM) h[threadIdx.x] = 0.0;
    part_sum(part, gridDim.x, nvec, h);
    if (blockIdx.x == 0)
        for (int k = threadIdx.x; k < nvec; k += kRedThreads) hout[k] = h[k];
    double acc[KA];
#pragma unroll
    for (int k = 0; k < KA; ++k) acc[k] = 0.0;
    for (int64_t i = blockIdx.x * (int64_t)kRedThreads + threadIdx.x; i < n; i += (int64_t)gridDim.x * kRedThreads) {
        double v = w[i];
        double x[KX];
        if constexpr (KM > 0) {
#pragma unroll
            for (int k = 0; k < KM; ++k) x[k] = V[min(k, nvec - 1) * ld + i];
#pragma unroll
            for (int k = 0; k < KM; ++k) v = fma(-x[k], h[k], v);
        } else {
#pragma unroll 8
            for (int k = 0; k < nvec; ++k) v = fma(-V[k * ld + i], h[k], v);
        }
        if constexpr (DOT) {
#pragma unroll
            for (int k = 0; k < KM; ++k) acc[k] = fma(x[k], v, acc[k]);
        } else {
            acc[0] = fma(v, v, acc[0]);
        }
        w[i] = v;
    }
    block_part<KA>(acc, DOT ? nvec : 1, part_out, red);
}

// r = b - r (sub) or b; partials of ||r||^2
__global__ void __launch_bounds__(kRedThreads) k_residual(const double *__restrict__ b, double *__restrict__ r,
                                                          int64_t n, int sub, double *__restrict__ part) {
    __shared__ double red[4][1];
    double acc[1] = {0.0};
    for (int64_t i = blockIdx.x * (int64_t)kRedThreads + threadIdx.x; i < n; i += (int64_t)gridDim.x * kRedThreads) {
        const double v = sub ? b[i] - r[i] : b[i];
        r[i] = v;
        acc[0] = fma(v, v, acc[0]);
    }
    block_part<1>(acc, 1, part, red);
}

__global__ void k_fill(double *v, int64_t n, double a) {
    int64_t i = blockIdx.x * (int64_t)blockDim.x + threadIdx.x;
    if (i < n) v[i] = a;
}

// x[i] = (add ? x[i] : 0) + sum_k V[k][i] y[k]
__global__ void k_combine(const double *__restrict__ V, int nvec, int64_t ld, const double *__restrict__ yv,
                          double *__restrict__ x, int64_t n, int add) {
    int64_t i = blockIdx.x * (int64_t)blockDim.x + threadIdx.x;
    if (i >= n) return;
    double v = add ? x[i] : 0.0;
#pragma unroll 8
    for (int k = 0; k < nvec; ++k) v = fma(V[k * ld + i], yv[k], v);
    x[i] = v;
}

// Small-state layout (doubles) for restart m:
//   H  [(m+1) * m] column-major, cs [m], sn [m], g [m+1], yv [m],
//   h1 [m+1], h2 [m+1]
struct SmallLayout {
    int m;
    int64_t H, cs, sn, g, yv, h1, h2, total;
    explicit SmallLayout(int m_) : m(m_) {
        H = 0;
        cs = H + (int64_t)(m + 1) * m;
        sn = cs + m;
        g = sn + m;
        yv = g + m + 1;
        h1 = yv + m;
        h2 = h1 + m + 1;
        total = h2 + m + 1;
    }
};

// Column j of H from the two Gram-Schmidt passes and beta = ||w||; apply the
// previous rotations, form rotation j, update g; *res = |g[j+1]|, the residual
// estimate. The rotations and the column are staged in LDS by the first wave
// (col [m + 1], rot [2 m]); one thread then runs the recurrence. Called by the
// first 64 threads of one workgroup.
__device__ inline void givens_column(double *sm, const SmallLayout &L, int j, double beta, double *col, double *rot,
                                     double *res) {
    double *H = sm + L.H + (int64_t)(L.m + 1) * j;
    double *cs = sm + L.cs, *sn = sm + L.sn, *g = sm + L.g;
    for (int i = threadIdx.x; i <= j; i += 64) {
        col[i] = sm[L.h1 + i] + sm[L.h2 + i];
        if (i < j) {
            rot[2 * i] = cs[i];
            rot[2 * i + 1] = sn[i];
        }
    }
    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
    __builtin_amdgcn_wave_barrier();
    if (threadIdx.x == 0) {
        double top = col[0];
        for (int i = 0; i < j; ++i) {  // (col[i], col[i+1]) through rotation i
            const double c = rot[2 * i], s = rot[2 * i + 1], below = col[i + 1];
            H[i] = c * top + s * below;
            top = -s * top + c * below;
        }
        const double den = hypot(top, beta);
        const double cj = (den > 0.0) ? top / den : 1.0;
        const double sj = (den > 0.0) ? beta / den : 0.0;
        cs[j] = cj;
        sn[j] = sj;
        H[j] = den;
        H[j + 1] = 0.0;
        const double gj = g[j], gn = -sj * gj;
        g[j + 1] = gn;
        g[j] = cj * gj;
        *res = fabs(gn);
    }
}

// End of Arnoldi step j: beta = ||w|| from its partials, v_{j+1} = w / beta (0
// on breakdown), column j of H by block 0, the residual estimate to res
// (pinned host memory)
__global__ void __launch_bounds__(kRedThreads) k_gs_finish(double *sm, SmallLayout L, int j,
                                                           const double *__restrict__ part, double *__restrict__ w,
                                                           int64_t n, double *res) {
    __shared__ double nrm[1], col[kMaxRestart + 1], rot[2 * kMaxRestart];
    part_sum(part, gridDim.x, 1, nrm);
    const double beta = sqrt(fmax(nrm[0], 0.0));
    const double inv = (beta > 0.0) ? 1.0 / beta : 0.0;
    for (int64_t i = blockIdx.x * (int64_t)kRedThreads + threadIdx.x; i < n; i += (int64_t)gridDim.x * kRedThreads)
        w[i] *= inv;
    if (blockIdx.x == 0 && threadIdx.x < 64) givens_column(sm, L, j, beta, col, rot, res);
}

// Start of a cycle: beta = ||r|| from its partials to res (pinned host memory),
// g = [beta, 0, ...], v_0 = r / beta. A residual that is not a number goes to res
// as one (fmax alone would make it 0, which the host takes for convergence).
__global__ void __launch_bounds__(kRedThreads) k_cycle_start(double *sm, SmallLayout L, const double *__restrict__ part,
                                                             double *__restrict__ r, int64_t n, double *res) {
    __shared__ double nrm[1];
    part_sum(part, gridDim.x, 1, nrm);
    const double beta = sqrt(fmax(nrm[0], 0.0));
    const double inv = (beta > 0.0) ? 1.0 / beta : 0.0;
    for (int64_t i = blockIdx.x * (int64_t)kRedThreads + threadIdx.x; i < n; i += (int64_t)gridDim.x * kRedThreads)
        r[i] *= inv;
    if (blockIdx.x == 0) {
        for (int i = threadIdx.x; i <= L.m; i += kRedThreads) sm[L.g + i] = i == 0 ? beta : 0.0;
        if (threadIdx.x == 0) *res = sqrt(nrm[0]);
    }
}

// ||v|| from its partials to res (pinned host memory)
__global__ void __launch_bounds__(kRedThreads) k_norm_out(const double *__restrict__ part, int nblk, double *res) {
    __shared__ double nrm[1];
    part_sum(part, nblk, 1, nrm);
    if (threadIdx.x == 0) *res = sqrt(fmax(nrm[0], 0.0));
}

// The whole orthogonalisation of Arnoldi step j (j < KM) for n <= kSmallGs
// points in one workgroup: w stays in LDS, the basis is read four times from
// L2.
constexpr int kSmallThreads = 512;
template <int KM>
__global__ void __launch_bounds__(kSmallThreads) k_gs_small(const double *__restrict__ V, int64_t ld,
                                                            double *__restrict__ w, int n, double *sm, SmallLayout L,
                                                            int j, double *res) {
    constexpr int NW = kSmallThreads / 64;
    __shared__ double wl[kSmallGs];
    __shared__ double red[NW][KM], h[KM], col[kMaxRestart + 1], rot[2 * kMaxRestart];
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int nvec = j + 1;
    double nr = 0.0;
    for (int i = tid; i < n; i += kSmallThreads) wl[i] = w[i];  // each thread reads its own entries only
    for (int pass = 0; pass < 2; ++pass) {
        double acc[KM];
#pragma unroll
        for (int k = 0; k < KM; ++k) acc[k] = 0.0;
        for (int i = tid; i < n; i += kSmallThreads) {
            const double wi = wl[i];
            double x[KM];
#pragma unroll
            for (int k = 0; k < KM; ++k) x[k] = V[min(k, nvec - 1) * ld + i];
#pragma unroll
            for (int k = 0; k < KM; ++k) acc[k] = fma(x[k], wi, acc[k]);
        }
        wave_sum<KM>(acc, lane);
        red[wave][wave_slot<KM>(lane)] = acc[0];
        __syncthreads();
        if (tid < KM) {
            double a = 0.0;
#pragma unroll
            for (int q = 0; q < NW; ++q) a += red[q][tid];
            h[tid] = tid < nvec ? a : 0.0;
            if (tid < nvec) sm[(pass ? L.h2 : L.h1) + tid] = a;
        }
        __syncthreads();
        for (int i = tid; i < n; i += kSmallThreads) {
            double v = wl[i], x[KM];
#pragma unroll
            for (int k = 0; k < KM; ++k) x[k] = V[min(k, nvec - 1) * ld + i];
#pragma unroll
            for (int k = 0; k < KM; ++k) v = fma(-x[k], h[k], v);
            wl[i] = v;
            if (pass) nr = fma(v, v, nr);
        }
    }
    for (int o = 32; o > 0; o >>= 1) nr += __shfl_xor(nr, o);
    if (lane == 0) red[wave][0] = nr;
    __syncthreads();
    double s = 0.0;
    for (int q = 0; q < NW; ++q) s += red[q][0];
    const double beta = sqrt(fmax(s, 0.0));
    const double inv = (beta > 0.0) ? 1.0 / beta : 0.0;
    for (int i = tid; i < n; i += kSmallThreads) w[i] = wl[i] * inv;
    if (tid < 64) givens_column(sm, L, j, beta, col, rot, res);
}

// Solve the k x k upper triangle H y = g: column by column, thread i holding
// row i (k <= kMaxRestart threads)
__global__ void __launch_bounds__(kMaxRestart) k_trisolve(double *sm, SmallLayout L, int k) {
    __shared__ double y;
    const int i = threadIdx.x;
    double v = i < k ? sm[L.g + i] : 0.0;
    double next = i < k ? sm[L.H + (int64_t)(L.m + 1) * (k - 1) + i] : 0.0;
    for (int c = k - 1; c >= 0; --c) {
        const double hc = next;  // H[i][c]; the column before it is loaded ahead
        if (c > 0 && i < c) next = sm[L.H + (int64_t)(L.m + 1) * (c - 1) + i];
        if (i == c) y = (hc != 0.0) ? v / hc : 0.0;
        __syncthreads();
        if (i == c) sm[L.yv + i] = y;
        if (i < c) v -= hc * y;
        __syncthreads();
    }
}

// Whether one workgroup takes the step (four launches else). Its time grows with
// the basis it reads, about 7 + 0.0007 n nvec us, that of the four launches is about
// 14.4 + 0.52 nvec whatever n <= kSmallGs: they meet at (n - 743) nvec = 10571.
// Means over a cycle of 30 / of 10, one and four launches: 642 points 14.2 and 20.4
// / 9.9 and 16.7 us, 1284 points 21.7 and 22.7 / 12.4 and 17.0, 2562 points 32.0
// and 22.7 / 17.5 and 17.4, 3852 points 44.9 and 22.8 / 22.9 and 17.7.
static bool gs_in_one(int64_t n, int nvec) {
    return n <= kSmallGs && nvec <= kGsFuse && (n - 743) * nvec <= 10571;
}

// Orthogonalisation of Arnoldi step j: w = V[j + 1] against V[0..j]: one launch
// where gs_in_one (642 points 45 -> 16 us a step,
// mean over a cycle of 30), else four (64,200 points 46 -> 30 us, 76,800 points
// 46 -> 27 us), or six past kGsFuse vectors.
static void gs_step(bfm_ctx *c, double *V, int j, int64_t n, double *part, double *sm, const SmallLayout &L,
                    double *res) {
    hipStream_t st = c->stream;
    double *w = V + (int64_t)(j + 1) * n;
    const int nvec = j + 1;
    if (gs_in_one(n, nvec)) {
        auto kern = nvec <= 4 ? k_gs_small<4> : (nvec <= 8 ? k_gs_small<8> : (nvec <= 16 ? k_gs_small<16> : k_gs_small<32>));
        kern<<<1, kSmallThreads, 0, st>>>(V, n, w, (int)n, sm, L, j, res);
        BFM_LAUNCHED();
        return;
    }
    const int G = red_blocks(n);
    double *part2 = part + (int64_t)(L.m + 1) * kRedBlocks;
    auto dots = [&](double *out) {
        for (int k0 = 0; k0 < nvec; k0 += kGsFuse) {
            const int kn = std::min(kGsFuse, nvec - k0);
            auto kern = kn <= 4 ? k_gs_dot<4> : (kn <= 8 ? k_gs_dot<8> : (kn <= 16 ? k_gs_dot<16> : k_gs_dot<32>));
            kern<<<G, kRedThreads, 0, st>>>(V, k0, kn, n, w, n, out);
            BFM_LAUNCHED();
        }
    };
    dots(part);
    auto update = [&](auto kern, const double *pin, int64_t hout, double *pout) {
        kern<<<G, kRedThreads, 0, st>>>(V, nvec, n, pin, w, n, sm + hout, pout);
        BFM_LAUNCHED();
    };
    if (nvec <= 4) {
        update(k_gs_update<4, true>, part, L.h1, part2);
        update(k_gs_update<4, false>, part2, L.h2, part);
    } else if (nvec <= 8) {
        update(k_gs_update<8, true>, part, L.h1, part2);
        update(k_gs_update<8, false>, part2, L.h2, part);
    } else if (nvec <= 16) {
        update(k_gs_update<16, true>, part, L.h1, part2);
        update(k_gs_update<16, false>, part2, L.h2, part);
    } else if (nvec <= kGsFuse) {
        update(k_gs_update<kGsFuse, true>, part, L.h1, part2);
        update(k_gs_update<kGsFuse, false>, part2, L.h2, part);
    } else {  // too many vectors for one pass: update, then the dots again
        update(k_gs_update<0, false>, part, L.h1, part2);
        dots(part2);
        update(k_gs_update<0, false>, part2, L.h2, part);
    }
    k_gs_finish<<<G, kRedThreads, 0, st>>>(sm, L, j, part, w, n, res);
    BFM_LAUNCHED();
}

void gmres_sorted(bfm_ctx *c, double *x, bool use_guess, bfm_solve_info *info) {
    hipStream_t st = c->stream;
    const int64_t n = c->nv;
    const int m = c->opt.gmres_restart;
    const int maxit = c->opt.gmres_maxit;
    const double tol = c->opt.gmres_tol;
    // mixed-precision iterative refinement: the Arnoldi products in low
    // precision, the residuals that start each cycle in FP64
    const int prec = c->opt.precision;
    const bool ir = prec != BFM_PREC_FP64;
    const double ir_tol = c->opt.ir_tol > 0.0 ? c->opt.ir_tol : 1e-4;
    SmallLayout L(m);
    double *V = c->V.ensure((size_t)(m + 1) * n);
    double *part = c->part.ensure((size_t)2 * (m + 1) * kRedBlocks);
    double *sm = c->small.ensure(L.total);
    if (!c->host_small) BFM_HIP(hipHostMalloc((void **)&c->host_small, 8 * sizeof(double), 0));
    // scalars the device writes straight to pinned host memory: [0] residual
    // estimate of the last step, [1] ||r|| of the cycle, [2] ||b||
    double *hs = c->host_small;
    const double *b = c->b_s.get();
    const int G = red_blocks(n);
    auto wait = [&] { BFM_HIP(hipStreamSynchronize(st)); };
    // V[0] = r / ||r|| with r = b - V[0] (sub) or b, ||r|| to hs[1], g reset
    auto cycle_start = [&](bool sub) {
        k_residual<<<G, kRedThreads, 0, st>>>(b, V, n, sub ? 1 : 0, part);
        BFM_LAUNCHED();
        k_cycle_start<<<G, kRedThreads, 0, st>>>(sm, L, part, V, n, hs + 1);
        BFM_LAUNCHED();
    };
    int matvecs = 0;
    const bool pc = c->opt.precond != BFM_PRECOND_NONE;
    // graphs replay recorded launches; kernel timing records its own events, so it runs eagerly
    const bool use_graph = c->opt.use_graph != 0 && !c->prof.on;
    double *Z = nullptr, *Tv = nullptr;
    if (pc) {
        BFM_CHECK(c->pre.nd > 0 && c->pre.genus == 0, BFM_EINVAL,
                  "the harmonic preconditioner needs a sphere template (bfm_set_sphere_template)");
        precond_build(c);
        precond_radii(c);
        if (c->opt.precond == BFM_PRECOND_SH_COARSE) {
            if (c->coarse_pending)  // built beside the diagonal pass
                coarse_join(c);
            else
                coarse_build(c, st);
        }
        Z = c->zbuf.ensure(n);
        Tv = c->tbuf.ensure(n);
    }
    info->iterations = 0;
    info->restarts = 0;
    // r0 and ||b||
    if (use_guess) {
        // ||b|| into the workspace of the first residual; V[0] is overwritten
        k_residual<<<G, kRedThreads, 0, st>>>(b, V, n, 0, part);
        BFM_LAUNCHED();
        k_norm_out<<<1, kRedThreads, 0, st>>>(part, G, hs + 2);
        BFM_LAUNCHED();
        wait();
        if (hs[2] > 0.0) {
            matvec_sorted(c, 1.0, x, 0.0, nullptr, V, true, BFM_PREC_FP64, false);
            ++matvecs;
            cycle_start(true);
            wait();
        }
    } else {
        k_fill<<<nblk(n, 256), 256, 0, st>>>(x, n, 0.0);
        BFM_LAUNCHED();
        cycle_start(false);
        wait();
        hs[2] = hs[1];
    }
    const double nb = hs[2];
    graph_release_stale(c);  // the stream has just been waited for
    if (!(nb > 0.0)) {
        k_fill<<<nblk(n, 256), 256, 0, st>>>(x, n, 0.0);
        BFM_LAUNCHED();
        info->rel_residual = 0.0;
        info->converged = 1;
        info->matvecs = 0;
        return;
    }
    double beta = hs[1];
    int it = 0;
    bool conv = beta <= tol * nb;
    while (!conv && it < maxit) {
        int k = 0;
        for (int j = 0; j < m && it < maxit; ++j) {
            double *vj = V + (int64_t)j * n;
            double *wj = V + (int64_t)(j + 1) * n;
            if (use_graph) {  // the same product, replayed from a captured graph
                graph_mvp(c, vj, wj, pc);
            } else if (pc) {  // right preconditioning: w = A P^{-1} v_j
                precond_apply(c, vj, Z);
                matvec_sorted(c, 1.0, Z, 0.0, nullptr, wj, true, prec, false);
            } else {
                matvec_sorted(c, 1.0, vj, 0.0, nullptr, wj, true, prec, false);
            }
            ++matvecs;
            const int pg = c->prof.begin(KC_GMRES, st);
            gs_step(c, V, j, n, part, sm, L, hs);
            c->prof.end(pg, st, 0.0, 0.0);
            ++it;
            k = j + 1;
            wait();
            const double res = hs[0];
            if (res <= tol * nb || (ir && res <= ir_tol * beta)) break;
        }
        k_trisolve<<<1, kMaxRestart, 0, st>>>(sm, L, k);
        BFM_LAUNCHED();
        if (pc) {  // x += P^{-1} V y
            k_combine<<<nblk(n, 256), 256, 0, st>>>(V, k, n, sm + L.yv, Tv, n, 0);
            BFM_LAUNCHED();
            precond_apply(c, Tv, x, true);
        } else {
            k_combine<<<nblk(n, 256), 256, 0, st>>>(V, k, n, sm + L.yv, x, n, 1);
            BFM_LAUNCHED();
        }
        // true residual (FP64)
        matvec_sorted(c, 1.0, x, 0.0, nullptr, V, true, BFM_PREC_FP64, false);
        ++matvecs;
        cycle_start(true);
        wait();
        beta = hs[1];
        info->restarts += 1;
        conv = beta <= tol * nb;
    }
    info->iterations = it;
    info->matvecs = matvecs;
    info->rel_residual = beta / nb;
    info->converged = conv ? 1 : 0;
}

}  // namespace bfm
