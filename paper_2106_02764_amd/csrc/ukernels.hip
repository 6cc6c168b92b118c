// gfx950 kernels of the unstructured-mesh path (paper: section Geometry
// module; Appendix A with general face vectors R_ij = A_ij n_ij / V_i;
// Appendix B, heat conduction with the non-orthogonal correction).
//
// Heat conduction (Eq. (final2)): the primary flux is implicit, the
// secondary flux explicit.  One workgroup runs the whole outer iteration of
// a mesh: least-squares cell gradients of the current T, the secondary flux
// of every face, then a conjugate-gradient solve of the volume-scaled
// primary-flux Laplacian (warm-started from the current T), until T stops
// changing.
//
// Transport: one wavefront owns one (m, l) system.  Within a direction the
// host puts the cells in rows of at most 64 that read only cells of earlier
// rows (the periodic faces cut), so a sweep is one pass over the rows, the
// values that later rows read in LDS.  The values entering through periodic
// faces form the system's wrap vector u; BiCGSTAB solves (I - G) e = r for its
// correction, G being one sweep with u as the only source, as on the
// structured grids.  All sums are in a fixed order: FP64 results are bitwise
// reproducible.
#include "device.h"
#include "umesh_internal.h"

namespace {

constexpr int UF_THREADS = 1024;

// Butterfly sum over the wave (partners 32, 16, 8, 4, 2, 1 lanes away), every
// lane the same value.  After a step the values repeat with its distance, so
// a rotation in a row of 16 lanes brings the same partner as the exchange
// would: moves within the vector unit, where LDS permutes take their latency
// six times in a row.
struct UPair {
    double x, y;          // of the even and of the odd half (or row pair), in both
};
template <bool HALF>
__device__ __forceinline__ UPair uswap(double a) {
    const unsigned lo = (unsigned)__double2loint(a), hi = (unsigned)__double2hiint(a);
    const auto l = HALF ? __builtin_amdgcn_permlane32_swap(lo, lo, false, false)
                        : __builtin_amdgcn_permlane16_swap(lo, lo, false, false);
    const auto h = HALF ? __builtin_amdgcn_permlane32_swap(hi, hi, false, false)
                        : __builtin_amdgcn_permlane16_swap(hi, hi, false, false);
    return {__hiloint2double((int)h[0], (int)l[0]), __hiloint2double((int)h[1], (int)l[1])};
}
// the steps after the first
__device__ __forceinline__ double ubutterfly_half(double v) {
    const UPair q = uswap<false>(v);
    v = q.x + q.y;
    v += dpp<0x128, 0xf>(v, 0.0);      // row_ror:8, 4, 2, 1
    v += dpp<0x124, 0xf>(v, 0.0);
    v += dpp<0x122, 0xf>(v, 0.0);
    v += dpp<0x121, 0xf>(v, 0.0);
    return v;
}
__device__ __forceinline__ double ubutterfly_sum(double v) {
    const UPair h = uswap<true>(v);
    return ubutterfly_half(h.x + h.y);
}

__device__ __forceinline__ double wave_max(double v) {
#pragma unroll
    for (int m = 32; m >= 1; m >>= 1) v = fmax(v, shfl_xor(v, m));
    return v;
}

// Block-wide sum (every thread gets the same value; waves combined in order).
__device__ double ublock_sum(double v, double* red) {
    v = ubutterfly_sum(v);
    const int w = threadIdx.x >> 6, nw = blockDim.x >> 6;
    __syncthreads();
    if ((threadIdx.x & 63) == 0) red[w] = v;
    __syncthreads();
    double s = 0.0;
    for (int k = 0; k < nw; ++k) s += red[k];
    return s;
}

// N block-wide sums in one exchange (each value summed as ublock_sum does;
// red: at least 16 N doubles)
template <int N>
__device__ void block_sum_n(double (&v)[N], double* red) {
#pragma unroll
    for (int n = 0; n < N; ++n) v[n] = ubutterfly_sum(v[n]);
    const int w = threadIdx.x >> 6, nw = blockDim.x >> 6;
    __syncthreads();
    if ((threadIdx.x & 63) == 0)
#pragma unroll
        for (int n = 0; n < N; ++n) red[n * 16 + w] = v[n];
    __syncthreads();
#pragma unroll
    for (int n = 0; n < N; ++n) {
        double s = 0.0;
        for (int k = 0; k < nw; ++k) s += red[n * 16 + k];
        v[n] = s;
    }
}

__device__ double block_max(double v, double* red) {
    v = wave_max(v);
    const int w = threadIdx.x >> 6, nw = blockDim.x >> 6;
    __syncthreads();
    if ((threadIdx.x & 63) == 0) red[w] = v;
    __syncthreads();
    double s = 0.0;
    for (int k = 0; k < nw; ++k) s = fmax(s, red[k]);
    return s;
}

// ---------------------------------------------------------------------------
// heat conduction with the explicit secondary flux
// ---------------------------------------------------------------------------
__device__ __forceinline__ void uface_gradient(const UFourierDev& f, int fc, double& gx, double& gy) {
    const int i = f.fi[fc], j = f.fj[fc];
    const double w = f.fw[fc];
    gx = (1.0 - w) * f.g[2 * i] + w * f.g[2 * j];
    gy = (1.0 - w) * f.g[2 * i + 1] + w * f.g[2 * j + 1];
}

// (A x)_i for A = minus the volume-scaled primary-flux Laplacian
__device__ __forceinline__ double uapply(const UFourierDev& f, const double* x, int i) {
    double y = 0.0;
    const double xi = x[i];
    for (int k = f.nb_ptr[i]; k < f.nb_ptr[i + 1]; ++k) y += f.nb_a[k] * (xi - x[f.nb_j[k]]);
    return y;
}

__device__ __forceinline__ double udiag(const UFourierDev& f, int i) {
    double d = 0.0;
    for (int k = f.nb_ptr[i]; k < f.nb_ptr[i + 1]; ++k) d += f.nb_a[k];
    return d > 0.0 ? d : 1.0;
}

// ---- the outer iteration over several blocks of UFB cells.  Every sum is
// taken as per-block partials that each consumer adds in block order, so
// every block takes the same decisions and FP64 results are reproducible.
constexpr int UFB = 256;
enum { UP_RR0, UP_RR1, UP_G0, UP_G1, UP_D0, UP_D1, UP_BB, UP_ST, UP_DM, UP_TM };
static_assert(UP_TM + 1 == UF_SLOTS, "partial slots of the heat-conduction kernels");

__host__ __device__ __forceinline__ int uf_blocks(int ns) { return (ns + UFB - 1) / UFB; }

// fixed-order sum (or max) of the B partials of a slot, in every thread
__device__ __forceinline__ double uf_sum(const UFourierDev& f, int slot, int B, double* red) {
    const double v = (int)threadIdx.x < B ? f.fpart[slot * UF_MAXB + threadIdx.x] : 0.0;
    return ublock_sum(v, red);
}
__device__ __forceinline__ double uf_max(const UFourierDev& f, int slot, int B, double* red) {
    const double v = (int)threadIdx.x < B ? f.fpart[slot * UF_MAXB + threadIdx.x] : 0.0;
    return block_max(v, red);
}

__device__ __forceinline__ void ucell_gradient(const UFourierDev& f, int i) {
    double gx = 0.0, gy = 0.0;
    const double Ti = f.T[i];
    for (int k = f.nb_ptr[i]; k < f.nb_ptr[i + 1]; ++k) {
        const double q = f.T[f.nb_j[k]] + f.nb_del[k] * f.dT - Ti;
        gx += f.nb_w[2 * k] * q;
        gy += f.nb_w[2 * k + 1] * q;
    }
    f.g[2 * i] = gx;
    f.g[2 * i + 1] = gy;
}

// cell gradients of the current T
__global__ void __launch_bounds__(UFB) k_uf_grad(const UFourierDev* __restrict__ fp) {
    const UFourierDev& f = *fp;
    const int i = blockIdx.x * UFB + threadIdx.x;
    if (i < f.ns) ucell_gradient(f, i);
}

// the secondary flux of every face from the interpolated face gradient
__global__ void __launch_bounds__(UFB) k_uf_face(const UFourierDev* __restrict__ fp) {
    const UFourierDev& f = *fp;
    const int fc = blockIdx.x * UFB + threadIdx.x;
    if (fc >= f.nfaces) return;
    double gx, gy;
    uface_gradient(f, fc, gx, gy);
    f.bf[fc] = gx * f.fc[2 * fc] + gy * f.fc[2 * fc + 1];
}

// b = -(P + B) (the right-hand side of A T = b, A = -Laplacian), the previous
// iterate, the diagonal and the first residual r = b - A T (warm start from
// T); partials of |b|^2 and r.r.  The CG's direction p and its image s of
// the iteration before the first are 0.
__global__ void __launch_bounds__(UFB) k_uf_init(const UFourierDev* __restrict__ fp) {
    __shared__ double red[UFB / 64];
    const UFourierDev& f = *fp;
    const int i = blockIdx.x * UFB + threadIdx.x;
    double bb = 0.0, rr = 0.0;
    if (i < f.ns) {
        double s = f.P[i];
        for (int k = f.nb_ptr[i]; k < f.nb_ptr[i + 1]; ++k) {
            const int code = f.nb_f[k];
            const double v = f.bf[code >> 1];
            s += (code & 1) ? -v : v;
        }
        const double ri = -s - uapply(f, f.T, i);
        f.tp[i] = f.T[i];
        f.dg[i] = udiag(f, i);
        f.r[i] = ri;
        f.p[i] = 0.0;
        f.s0[i] = 0.0;             // read as the previous s by the first iteration (parity 0)
        bb = s * s;
        rr = ri * ri;
    }
    bb = ublock_sum(bb, red);
    rr = ublock_sum(rr, red);
    if (threadIdx.x == 0) {
        f.fpart[UP_BB * UF_MAXB + blockIdx.x] = bb;
        f.fpart[UP_RR0 * UF_MAXB + blockIdx.x] = rr;
        if (blockIdx.x == 0) {
            f.fsc[0] = 0.0;            // this solve's CG runs
            f.fsc[10] = 0.0;           // iterations done before the next one of parity 0
        }
    }
}

// w = A u with u = M^-1 r (M the diagonal) for the first residual, and the
// partials of gamma = r.u and delta = w.u (parity 0)
__global__ void __launch_bounds__(UFB) k_uf_w0(const UFourierDev* __restrict__ fp) {
    __shared__ double red[UFB / 64];
    const UFourierDev& f = *fp;
    const int i = blockIdx.x * UFB + threadIdx.x;
    double gm = 0.0, dl = 0.0;
    if (i < f.ns) {
        const double ui = f.r[i] / f.dg[i];
        double w = 0.0;
        for (int k = f.nb_ptr[i]; k < f.nb_ptr[i + 1]; ++k) {
            const int j = f.nb_j[k];
            w += f.nb_a[k] * (ui - f.r[j] / f.dg[j]);
        }
        f.w0[i] = w;
        gm = f.r[i] * ui;
        dl = w * ui;
    }
    gm = ublock_sum(gm, red);
    dl = ublock_sum(dl, red);
    if (threadIdx.x == 0) {
        f.fpart[UP_G0 * UF_MAXB + blockIdx.x] = gm;
        f.fpart[UP_D0 * UF_MAXB + blockIdx.x] = dl;
    }
}

// One preconditioned CG iteration in the Chronopoulos-Gear arrangement (one
// kernel: both inner products of an iteration come from one pass).  With u =
// M^-1 r, w = A u and s = A p carried by recurrence, iteration k (parity q):
//   gamma = r.u, delta = w.u (partials of parity q), the stop test on r.r;
//   beta = gamma / gamma_prev, alpha = gamma / (delta - beta gamma /
//   alpha_prev)  (k = 0: beta = 0, alpha = gamma / delta);
//   p = u + beta p, s = w + beta s, T += alpha p, r' = r - alpha s,
//   u' = M^-1 r', w' = A u', and the partials of r'.u', w'.u', r'.r'.
// r, w and s are double buffered by parity (r0 = r, r1), and A u' at a cell
// needs u' at its neighbours, which every block forms from the unchanged
// parity-q buffers.  Scalars: fsc[6 + q] gamma, fsc[8 + q] alpha and
// fsc[10 + q] the iterations done before an iteration of parity q.
__global__ void __launch_bounds__(UFB) k_uf_cg(const UFourierDev* __restrict__ fp, int q, double cg_tol,
                                               int max_cg) {
    __shared__ double red[4 * 16];
    const UFourierDev& f = *fp;
    const int B = uf_blocks(f.ns);
    const auto r = gview(q ? f.r1 : f.r), w = gview(q ? f.w1 : f.w0);
    const auto so = gview(q ? f.s1 : f.s0);   // s of the previous iteration (parity q ^ 1 wrote it here)
    const auto rn = gmut(q ? f.r : f.r1), wn = gmut(q ? f.w0 : f.w1), sn = gmut(q ? f.s0 : f.s1);
    const auto dg = gview(f.dg), sc = gview(f.fsc), pt = gview(f.fpart);
    const auto p = gmut(f.p), T = gmut(f.T);
    const int i = blockIdx.x * UFB + threadIdx.x, ic = min(i, f.ns - 1);
    // everything that the iteration reads is asked for before the sums of the
    // partials, which the scalars wait for (a 5609-cell mesh: 6.8 -> 5.5 us)
    const double done = sc[0], g1 = sc[6 + (q ^ 1)], a1 = sc[8 + (q ^ 1)];
    const int it = (int)sc[10 + q];
    const double ri0 = r[ic], wi0 = w[ic], si0 = so[ic], dgi = dg[ic], pi0 = p[ic], Ti0 = T[ic];
    const auto nj = gview(f.nb4_j) + (size_t)ic * UFACES;
    const auto ak = gview(f.nb4_a) + (size_t)ic * UFACES;
    int jk[UFACES];
#pragma unroll
    for (int k = 0; k < UFACES; ++k) jk[k] = nj[k];
    double na[UFACES], nr[UFACES], nw[UFACES], ns[UFACES], nd[UFACES];
#pragma unroll
    for (int k = 0; k < UFACES; ++k) {
        const int j = jk[k] < 0 ? ic : jk[k];
        na[k] = ak[k];
        nr[k] = r[j];
        nw[k] = w[j];
        ns[k] = so[j];
        nd[k] = dg[j];
    }
    // the four sums of the partials in one exchange (block order, as uf_sum)
    double sm[4] = {0.0, 0.0, 0.0, 0.0};
    if ((int)threadIdx.x < B) {
        sm[0] = pt[(UP_RR0 + q) * UF_MAXB + threadIdx.x];
        sm[1] = pt[UP_BB * UF_MAXB + threadIdx.x];
        sm[2] = pt[(UP_G0 + q) * UF_MAXB + threadIdx.x];
        sm[3] = pt[(UP_D0 + q) * UF_MAXB + threadIdx.x];
    }
    if (done != 0.0) return;
    block_sum_n(sm, red);
    const double rr = sm[0], bb = sm[1], gam = sm[2], del = sm[3];
    double alpha = gam / del, beta = 0.0;
    if (it > 0) {
        beta = gam / g1;
        alpha = gam / (del - beta * gam / a1);
    }
    if (!(rr > cg_tol * cg_tol * bb) || it >= max_cg || !(alpha > 0.0) || !isfinite(alpha)) {
        if (blockIdx.x == 0 && threadIdx.x == 0) f.fsc[0] = 1.0;
        return;
    }
    double gm = 0.0, dl = 0.0, r2 = 0.0;
    if (i < f.ns) {
        const double pc = ri0 / dgi + beta * pi0;
        const double si = wi0 + beta * si0;
        p[i] = pc;
        T[i] = Ti0 + alpha * pc;
        const double ri = ri0 - alpha * si;
        const double ui = ri / dgi;
        double wv = 0.0;
#pragma unroll
        for (int k = 0; k < UFACES; ++k) {
            const double rj = nr[k] - alpha * (nw[k] + beta * ns[k]);
            const double t = wv + na[k] * (ui - rj / nd[k]);
            wv = jk[k] < 0 ? wv : t;
        }
        rn[i] = ri;
        wn[i] = wv;
        sn[i] = si;
        gm = ri * ui;
        dl = wv * ui;
        r2 = ri * ri;
    }
    double en[3] = {gm, dl, r2};
    block_sum_n(en, red);
    if (threadIdx.x == 0) {
        f.fpart[(UP_G0 + (q ^ 1)) * UF_MAXB + blockIdx.x] = en[0];
        f.fpart[(UP_D0 + (q ^ 1)) * UF_MAXB + blockIdx.x] = en[1];
        f.fpart[(UP_RR0 + (q ^ 1)) * UF_MAXB + blockIdx.x] = en[2];
        if (blockIdx.x == 0) {
            f.fsc[6 + q] = gam;
            f.fsc[8 + q] = alpha;
            f.fsc[10 + (q ^ 1)] = (double)(it + 1);
            f.fsc[2] += 1.0;
        }
    }
}

// end of an outer iteration: partials of the sum of T ...
__global__ void __launch_bounds__(UFB) k_uf_sum(const UFourierDev* __restrict__ fp) {
    __shared__ double red[UFB / 64];
    const UFourierDev& f = *fp;
    const int i = blockIdx.x * UFB + threadIdx.x;
    const double v = ublock_sum(i < f.ns ? f.T[i] : 0.0, red);
    if (threadIdx.x == 0) f.fpart[UP_ST * UF_MAXB + blockIdx.x] = v;
}

// ... the mean removed, and partials of max |T - T_prev| and max |T|
__global__ void __launch_bounds__(UFB) k_uf_center(const UFourierDev* __restrict__ fp) {
    __shared__ double red[UFB / 64];
    const UFourierDev& f = *fp;
    const double mean = uf_sum(f, UP_ST, uf_blocks(f.ns), red) / (double)f.ns;
    const int i = blockIdx.x * UFB + threadIdx.x;
    double dmax = 0.0, tmax = 0.0;
    if (i < f.ns) {
        const double v = f.T[i] - mean;
        f.T[i] = v;
        dmax = fabs(v - f.tp[i]);
        tmax = fabs(v);
    }
    dmax = block_max(dmax, red);
    tmax = block_max(tmax, red);
    if (threadIdx.x == 0) {
        f.fpart[UP_DM * UF_MAXB + blockIdx.x] = dmax;
        f.fpart[UP_TM * UF_MAXB + blockIdx.x] = tmax;
    }
}

// ... the change and the outer stop test (one block)
__global__ void __launch_bounds__(UFB) k_uf_change(const UFourierDev* __restrict__ fp, double tol) {
    __shared__ double red[UFB / 64];
    const UFourierDev& f = *fp;
    const int B = uf_blocks(f.ns);
    const double dmax = uf_max(f, UP_DM, B, red), tmax = uf_max(f, UP_TM, B, red);
    if (threadIdx.x == 0) {
        f.fsc[3] += 1.0;
        f.fsc[4] = tmax > 0.0 ? dmax / tmax : 0.0;
        f.fsc[5] = dmax <= tol * fmax(tmax, 1e-300) ? 1.0 : 0.0;
    }
}

// kappa_F: the total face flux (primary + secondary) across the periodic
// plane of the gradient axis, from the final T's gradients (one block; the
// gradients are taken by k_uf_grad before it); the statistics into out
__global__ void __launch_bounds__(UF_THREADS) k_uf_kappa(const UFourierDev* __restrict__ fp) {
    __shared__ double red[UF_THREADS / 64];
    const UFourierDev& f = *fp;
    double tot = 0.0;
    for (int c = threadIdx.x; c < f.ncut; c += blockDim.x) {
        const int fc = f.cut_f[c];
        double gx, gy;
        uface_gradient(f, fc, gx, gy);
        const int ip = f.cut_s[c] > 0 ? f.fi[fc] : f.fj[fc];
        const int jn = f.cut_s[c] > 0 ? f.fj[fc] : f.fi[fc];
        const double a = f.cut_K[3 * c], kx = f.cut_K[3 * c + 1], ky = f.cut_K[3 * c + 2];
        const double gd = gx * f.cut_d[2 * c] + gy * f.cut_d[2 * c + 1];
        // a = n.K n / (n.d); the secondary part g.K n - (n.K n)(g.d)/(n.d)
        tot += f.cut_A[c] * (a * (f.T[jn] + f.dT - f.T[ip]) + (gx * kx + gy * ky) - a * gd);
    }
    tot = ublock_sum(tot, red);
    if (threadIdx.x == 0) {
        f.out[0] = f.Lg / (f.dT * f.Aperp) * tot;
        f.out[1] = f.fsc[3];
        f.out[2] = f.fsc[2];
        f.out[3] = f.fsc[4];
    }
}

// ---------------------------------------------------------------------------
// transport: one pass for every system
// ---------------------------------------------------------------------------
struct USys {
    int sys, l, nrow, nw;
    double lam;
};

// A lane's cell of a row, as loaded.
template <int NIN>
struct UCell {
    double sg, d, c[NIN], b0, bw;
    uint32_t s0, s1, s2;          // URec2's offsets, or URec3's in pairs
    __device__ __forceinline__ uint32_t in(int q) const {
        return NIN == 2 ? (q ? s1 : s0) : (q == 0 ? s0 & 0xffffu : (q == 1 ? s0 >> 16 : s1 & 0xffffu));
    }
    __device__ __forceinline__ uint32_t out() const { return NIN == 2 ? s2 : s1 >> 16; }
};

// A direction's sweep tables as buffer resources: pointers that come out of
// memory are generic, and a flat load would count as an LDS access, whose
// waits then hold up the chain.  All tables have 16 bytes a position, so that
// a row costs one lane offset and one scalar offset.
struct UTab {
    rsrc_t rec, c01, pd, pb, rows;
};

__device__ __forceinline__ double udouble(unsigned lo, unsigned hi) { return __hiloint2double((int)hi, (int)lo); }

// Lanes past the row's end take its last cell, whose value they then write as
// well: no load sits in a branch, so the compiler counts the loads in flight
// exactly, and nothing is masked.
template <int NIN, bool SRC>
__device__ __forceinline__ void ufetch(const UTab& t, int base, int last, UCell<NIN>& e) {
    const int o = min((int)threadIdx.x * 16, last);
    const auto a = __builtin_amdgcn_raw_buffer_load_b128(t.rec, o, base, 0);
    const auto p = __builtin_amdgcn_raw_buffer_load_b128(t.pd, o, base, 0);
    const auto c = __builtin_amdgcn_raw_buffer_load_b128(t.c01, o, base, 0);
    if constexpr (NIN == 2) {
        e.s0 = a[0];
        e.s1 = a[1];
        e.s2 = a[2];
    } else {
        e.c[2] = udouble(a[0], a[1]);
        e.s0 = a[2];
        e.s1 = a[3];
    }
    e.sg = udouble(p[0], p[1]);
    e.d = udouble(p[2], p[3]);
    e.c[0] = udouble(c[0], c[1]);
    e.c[1] = udouble(c[2], c[3]);
    if constexpr (SRC) {
        const auto b = __builtin_amdgcn_raw_buffer_load_b128(t.pb, o, base, 0);
        e.b0 = udouble(b[0], b[1]);
        e.bw = udouble(b[2], b[3]);
    }
}

// The kappa sums of a pass (fixed order: each thread a contiguous chunk, then
// the block in order).
__device__ void ukappa(const UGeomDev& g) {
    __shared__ double red[4];
    double a = 0.0, b = 0.0, w = 0.0;
    const int kb = (g.ns + g.nwalls + UITEMS - 1) / UITEMS * USTRANDS;
    for (int i = threadIdx.x; i < kb; i += blockDim.x) a += g.kpart[i];
    const int per = (g.n_sys + blockDim.x - 1) / blockDim.x;
    const int i0 = threadIdx.x * per, i1 = min(g.n_sys, i0 + per);
    for (int i = i0; i < i1; ++i) {
        b += g.kfsys[i];
        w = fmax(w, g.wres[i]);
    }
    a = ublock_sum(a, red);
    b = ublock_sum(b, red);
    w = block_max(w, red);
    if (threadIdx.x == 0) {
        g.kap[0] = g.Lg / (g.dT * g.Vbox) * a;
        g.kap[1] = b;
        g.kap[2] = w;
    }
}

// The pass's sources in every direction's sweep order: sigma, sigma T_L and
// the inflow wall sum of the cell at each position (one thread per position);
// with_kappa: the last block takes the kappa sums of the pass before.
__global__ void __launch_bounds__(256) k_upack(const UGeomDev* __restrict__ gp, int with_kappa) {
    const UGeomDev& g = *gp;
    const int n = g.n_dir * (g.ns + 1), nb = (int)gridDim.x - with_kappa;
    if ((int)blockIdx.x == nb) {
        ukappa(g);
        return;
    }
    for (int o = blockIdx.x * blockDim.x + threadIdx.x; o < n; o += nb * blockDim.x) {
        const int i = g.ord[o];
        double wall = 0.0;
        {
#pragma clang fp contract(off)
            for (int k = g.wall_ptr[o]; k < g.wall_ptr[o + 1]; ++k) wall = wall + g.wall_c[k] * g.T_w[g.wall_id[k]];
        }
        const double sg = i < 0 ? 1.0 : g.sigma[i], T = i < 0 ? 0.0 : g.T_L[i];
        g.pd[o] = make_double2(sg, g.dout[o]);
        g.pb[o] = make_double2(sg * T, wall);
    }
}

// 1 / d to the last place, for normal numbers.
__device__ __forceinline__ double urecip(double d) {
    double r = __builtin_amdgcn_rcp(d);
    r = fma(fma(-d, r, 1.0), r, r);
    return fma(fma(-d, r, 1.0), r, r);
}

// a store at a lane offset and a scalar offset
__device__ __forceinline__ void ust(double v, rsrc_t r, uint32_t vo, uint32_t so) {
    u32x2_t w;
    w.x = (unsigned)__double2loint(v);
    w.y = (unsigned)__double2hiint(v);
    __builtin_amdgcn_raw_buffer_store_b64(w, r, (int)vo, (int)so, 0);
}

// One sweep of the system from the wrap inflow staged in LDS and, SRC, the
// sources; SRC also stores the solution, by position (whole lines, for
// k_ureduce to put in order).  The workgroup is one
// wavefront, whose LDS accesses are executed in program order, so a row reads
// what the rows before it wrote without a barrier.
//
// What bounds it is the chain from row to row: LDS read, the inflow sum, the
// quotient, LDS write.  So UROWS rows of table entries are in flight; the
// reciprocal 1 / (sigma + Lambda d) is taken before the row's inflow arrives,
// and the quotient from it in one product and a residual correction (the
// division's own result); a row is some 30 instructions; and LDS holds the
// live values alone, a few hundred slots, so that every system of a pass is
// resident at once.  5609 triangles in 165 rows: 22 us a sweep with 1440
// systems at once (130 ns a row); a pass of them with all cells in LDS (three
// systems a CU), levels for rows, entries two levels ahead and flat loads took
// 947 us, now 243 us.
template <int NIN, bool SRC, bool STORE>
__device__ __forceinline__ void usweep(const UTab& t, const USys& s, double* x, rsrc_t X) {
    const int lane = threadIdx.x, l8 = (lane & (UROWS - 1)) * 8;
    auto rows = [&](int r) { return __builtin_amdgcn_raw_buffer_load_b64(t.rows, l8, r * 8, 0); };
    auto at = [&](uint32_t o) -> double& { return *(double*)((char*)x + o); };
    auto den_of = [&](const UCell<NIN>& c) { return fma(s.lam, c.d, c.sg); };
    UCell<NIN> e[UROWS];
    auto rc = rows(0), rn = rows(UROWS);     // this iteration's rows and the next's
#pragma unroll
    for (int k = 0; k < UROWS - 1; ++k) {
        ufetch<NIN, SRC>(t, __builtin_amdgcn_readlane(rc[0], k), __builtin_amdgcn_readlane(rc[1], k), e[k]);
        __builtin_amdgcn_sched_barrier(0);   // in the order they are waited for
    }
    double den = den_of(e[0]), inv = urecip(den);
    __builtin_amdgcn_sched_barrier(0);
    for (int r = 0; r < s.nrow; r += UROWS) {
        const auto rn2 = rows(r + 2 * UROWS);
#pragma unroll
        for (int k = 0; k < UROWS; ++k) {
            // the row's inflow is read; while it is on its way the entries of
            // the row UROWS - 1 ahead are asked for, in the place of the row
            // before, and the next row's reciprocal is taken
            const UCell<NIN>& c = e[k];
            double v[NIN];
#pragma unroll
            for (int q = 0; q < NIN; ++q) v[q] = at(c.in(q));
            __builtin_amdgcn_sched_barrier(0);
            const auto& rf = k == 0 ? rc : rn;
            const int kf = (k + UROWS - 1) % UROWS;
            ufetch<NIN, SRC>(t, __builtin_amdgcn_readlane(rf[0], kf), __builtin_amdgcn_readlane(rf[1], kf), e[kf]);
            const double b = SRC ? fma(s.lam, c.bw, c.b0) : 0.0;
            const double den1 = den_of(e[(k + 1) % UROWS]), inv1 = urecip(den1);
            // (kept apart: the scheduler would move every reciprocal of an
            // iteration to its start, and wait there for the rows asked for last)
            __builtin_amdgcn_sched_barrier(0);
            double acc = c.c[0] * v[0];
            {
                // products and sum apart: the products start with their reads
#pragma clang fp contract(off)
#pragma unroll
                for (int q = 1; q < NIN; ++q) acc = acc + c.c[q] * v[q];
            }
            const double num = SRC ? fma(s.lam, acc, b) : s.lam * acc;
            const double q0 = num * inv;
            const double xv = fma(fma(-den, q0, num), inv, q0);
            at(c.out()) = xv;
            __builtin_amdgcn_sched_barrier(0);
            if constexpr (STORE) {
                const int base = __builtin_amdgcn_readlane(rc[0], k), last = __builtin_amdgcn_readlane(rc[1], k);
                ust(xv, X, (uint32_t)min(lane * 16, last) / 2u, (uint32_t)base / 2u);
            }
            den = den1;
            inv = inv1;
        }
        rc = rn;
        rn = rn2;
    }
    __builtin_amdgcn_wave_barrier();
}

template <int WPL>
__device__ __forceinline__ void ustage(const USys& s, const double (&v)[WPL], double* uin) {
#pragma unroll
    for (int k = 0; k < WPL; ++k) {
        const int q = k * WAVE + threadIdx.x;
        if (q < s.nw) uin[q] = v[k];
    }
    __builtin_amdgcn_wave_barrier();
}

// G v: the values a homogeneous sweep with inflow v carries back across the
// periodic faces (up: their slots)
template <int WPL>
__device__ __forceinline__ void ugather(const double* x, const int (&up)[WPL], double (&out)[WPL]) {
#pragma unroll
    for (int k = 0; k < WPL; ++k) out[k] = *(const double*)((const char*)x + up[k]);
}

template <int WPL>
__device__ __forceinline__ double udot(const double (&a)[WPL], const double (&b)[WPL]) {
    double v = 0.0;
#pragma unroll
    for (int k = 0; k < WPL; ++k) v += a[k] * b[k];
    return ubutterfly_sum(v);
}

// |a|^2.  With one value a lane its square goes into the first step's sum
// unrounded (an FMA, so each half of the wave has its own last bit): the wrap
// solves amplify it, so it is written out here and not left to the compiler's
// contraction, and decisions are taken for the whole wave (uyes).
template <int WPL>
__device__ __forceinline__ double unorm2(const double (&a)[WPL]) {
    if constexpr (WPL == 1) {
        const UPair h = uswap<true>(a[0] * a[0]);
        return ubutterfly_half(fma(a[0], a[0], threadIdx.x < 32 ? h.y : h.x));
    } else {
        return udot(a, a);
    }
}

// the first lane's answer
__device__ __forceinline__ bool uyes(bool b) { return __builtin_amdgcn_readfirstlane((int)b) != 0; }

template <int WPL, int NIN>
__global__ void __launch_bounds__(WAVE) k_upass(const UGeomDev* __restrict__ gp, double inner_tol, double inner_rtol,
                                                int max_inner) {
    extern __shared__ double lds[];
    const UGeomDev& g = *gp;
    const int lane = threadIdx.x;
    USys s;
    // longest MFPs first (they take the most wrap iterations); the direction
    // is the fast index, so with the workgroups dealt to the eight XCDs in
    // turn each XCD sweeps a fixed subset of the directions and their tables
    // stay in its L2
    s.l = (int)blockIdx.x % g.n_dir;
    const int m = g.n_mfp - 1 - (int)blockIdx.x / g.n_dir;
    s.sys = m * g.n_dir + s.l;
    s.lam = g.mfp[m];
    s.nrow = g.nrow[s.l];
    s.nw = g.nwrap[s.l];
    double* x = lds;
    double* uin = lds + USLOT_WRAP;
    if (lane == 0) x[USLOT_ZERO] = 0.0;
    const uint32_t np = (uint32_t)g.ns + 1u;
    const rsrc_t X = make_rsrc(g.X + (size_t)s.sys * np, np * 8u);
    const size_t p0 = (size_t)s.l * np;
    const UTab t = {make_rsrc((const URec2*)g.rec + p0, np * 16u), make_rsrc(g.c01 + p0, np * 16u),
                    make_rsrc(g.pd + p0, np * 16u), make_rsrc(g.pb + p0, np * 16u),
                    make_rsrc(g.rows + g.rbase[s.l], (uint32_t)(s.nrow + UROW_SLACK) * 8u)};
    const size_t w0 = (size_t)s.l * g.wmax;
    const auto U = gmut(g.U) + (size_t)s.sys * g.wmax;
    const auto wslot = gview(g.wslot) + w0;
    const auto wdel = gview(g.wdel) + w0;
    int up[WPL];
    double u[WPL], ez[WPL], r[WPL];
#pragma unroll
    for (int k = 0; k < WPL; ++k) {
        const int q = k * WAVE + lane;
        u[k] = q < s.nw ? U[q] : 0.0;
        up[k] = q < s.nw ? wslot[q] : 8 * USLOT_ZERO;
    }
    double scale = 0.0, rn = 0.0;
    long long its = 0;
    // the sweep with the sources and the wrap inflow of the last pass, and a
    // second time with the corrected inflow (one loop: one copy of the code)
    // (a system that corrected its inflow in the last pass will again, most
    // often: its first sweep then stores nothing)
    bool store = !gview(g.corrected)[s.sys], corrected = false, fixed = false;
    for (;;) {
        ustage(s, u, uin);
        if (store) {
            usweep<NIN, true, true>(t, s, x, X);
        } else {
            usweep<NIN, true, false>(t, s, x, X);
        }
        if (corrected) break;
        ugather(x, up, ez);
#pragma unroll
        for (int k = 0; k < WPL; ++k) {
            const int q = k * WAVE + lane;
            if (q < s.nw) ez[k] += wdel[q];
            r[k] = ez[k] - u[k];
        }
        scale = sqrt(unorm2(ez));
        rn = sqrt(unorm2(r));
        // this pass's target: inner_tol relative to the inflow, or (forcing
        // term) a cut by inner_rtol of the residual the pass started from; the
        // rest carries into the next pass through U
        const double thr = fmax(inner_tol * scale, inner_rtol * rn);
        if (!uyes(s.nw > 0 && scale > 0.0 && rn > thr)) {
            if (store) break;
            store = true;                   // the same sweep again, stored
            corrected = true;
            continue;
        }
        // ---- BiCGSTAB on (I - G) e = r, the best iterate kept
        double e[WPL], eb[WPL], rh[WPL], p[WPL], v[WPL], sv[WPL], tt[WPL], gx[WPL];
#pragma unroll
        for (int k = 0; k < WPL; ++k) {
            e[k] = 0.0; eb[k] = 0.0; rh[k] = r[k]; p[k] = 0.0; v[k] = 0.0;
        }
        double best = rn, rho_old = 1.0, alpha = 1.0, omega = 1.0;
        int restarts = 0;
        for (int it = 0; it < max_inner; ++it) {
            double rho = udot(rh, r);
            if (uyes(fabs(rho) <= 1e-30 * rn * rn || !(omega != 0.0))) {
#pragma unroll
                for (int k = 0; k < WPL; ++k) { rh[k] = r[k]; p[k] = 0.0; v[k] = 0.0; }
                rho = unorm2(r);
                rho_old = 1.0; alpha = 1.0; omega = 1.0;
            }
            const double beta = (rho / rho_old) * (alpha / omega);
#pragma unroll
            for (int k = 0; k < WPL; ++k) p[k] = r[k] + beta * (p[k] - omega * v[k]);
            ustage(s, p, uin);
            usweep<NIN, false, false>(t, s, x, X);
            ugather(x, up, gx);
#pragma unroll
            for (int k = 0; k < WPL; ++k) v[k] = p[k] - gx[k];
            const double rv = udot(rh, v);
            if (!uyes(isfinite(rv))) break;
            if (!uyes(fabs(rv) > 1e-30 * fabs(rho))) {
                if (restarts++ >= 4) break;
                omega = 0.0;
                continue;
            }
            alpha = rho / rv;
#pragma unroll
            for (int k = 0; k < WPL; ++k) sv[k] = r[k] - alpha * v[k];
            const double sn = sqrt(unorm2(sv));
            ++its;
            if (uyes(sn <= thr)) {
#pragma unroll
                for (int k = 0; k < WPL; ++k) e[k] += alpha * p[k];
                if (uyes(sn < best)) {
                    best = sn;
#pragma unroll
                    for (int k = 0; k < WPL; ++k) eb[k] = e[k];
                }
                break;
            }
            ustage(s, sv, uin);
            usweep<NIN, false, false>(t, s, x, X);
            ugather(x, up, gx);
#pragma unroll
            for (int k = 0; k < WPL; ++k) tt[k] = sv[k] - gx[k];
            const double t2 = unorm2(tt);
            const double ts = udot(tt, sv);
            omega = t2 > 0.0 ? ts / t2 : 0.0;
#pragma unroll
            for (int k = 0; k < WPL; ++k) {
                e[k] += alpha * p[k] + omega * sv[k];
                r[k] = sv[k] - omega * tt[k];
            }
            rn = sqrt(unorm2(r));
            rho_old = rho;
            if (!uyes(isfinite(rn))) break;
            if (uyes(rn < best)) {
                best = rn;
#pragma unroll
                for (int k = 0; k < WPL; ++k) eb[k] = e[k];
            }
            if (uyes(rn <= thr)) break;
        }
        rn = best;
        // ---- the corrected inflow
#pragma unroll
        for (int k = 0; k < WPL; ++k) {
            u[k] += eb[k];
            const int q = k * WAVE + lane;
            if (q < s.nw) U[q] = u[k];
        }
        fixed = store = corrected = true;
    }
    // ---- this system's kappa_face share: the flow across the cut, each of
    // whose faces is a wrap slot with its upwind cell's value
    const double Sx = g.S[2 * s.sys], Sy = g.S[2 * s.sys + 1];
    double kf = 0.0, xu[WPL];
    ugather(x, up, xu);
#pragma unroll
    for (int k = 0; k < WPL; ++k) {
        const int q = k * WAVE + lane;
        if (q < s.nw) {
            const auto c = gview(g.wcut) + 3 * (w0 + q);
            kf -= (Sx * c[0] + Sy * c[1]) * (xu[k] + c[2]);
        }
    }
    kf = ubutterfly_sum(kf);
    if (lane == 0) {
        g.kfsys[s.sys] = g.Lg / (g.dT * g.Aperp) * kf;
        g.iters[s.sys] += its;
        g.corrected[s.sys] = fixed;
        g.wres[s.sys] = scale > 0.0 ? rn / scale : 0.0;
    }
}

// T_L = sum D x per cell, T_w = sum of the outgoing weights times x at the
// wall's cell, and the cells' shares of kappa_cc.  The systems are taken in UQ
// chunks, each chunk's every fourth system by one strand of workgroups (what a
// chunk has past a multiple of eight goes to the first), one after the other:
// the system's solution goes through LDS from sweep order to the cells, the
// next two on their way meanwhile.  5609 cells, 1440 systems (65 MB): 40 us
// with two workgroups a strand, each reading the whole system; 51 us with one
// and one system on its way; 107 us with a block per 64 cells on an X by cell,
// whose scattered stores the sweeps had to make.
__global__ void __launch_bounds__(URED_THREADS) k_ureduce(const UGeomDev* __restrict__ gp) {
    extern __shared__ double lds[];
    const UGeomDev& g = *gp;
    const int tid = threadIdx.x, ns = g.ns, nw = g.nwalls, items = ns + nw;
    const int strand = (int)blockIdx.x % USTRANDS, q = strand >> 2, j = strand & 3;
    const int it0 = (int)blockIdx.x / USTRANDS * UITEMS + tid;
    const int per = (g.n_sys + UQ - 1) / UQ;
    const int i0 = q * per, i1 = min(g.n_sys, i0 + per), n8 = max(i1 - i0, 0) & ~7;
    const int n = n8 / 4 + (j == 0 ? max(i1 - i0, 0) - n8 : 0);
    auto sys = [&](int t) { return i0 + (t < n8 / 4 ? 4 * t + j : n8 + t - n8 / 4); };
    const auto gX = gview(g.X);
    const auto gI = gview(g.ipos);
    const auto gW = gview(g.wout);
    constexpr int ROWS = 8;                       // ns <= 8192
    // two systems on their way
    struct Next {
        double x[ROWS], w[UITEMS_PER];
        unsigned ip[UITEMS_PER];
    } nx[2];
    double a[UITEMS_PER], v[UITEMS_PER], z = 0.0;
    auto load = [&](int k, Next& e) {
#pragma unroll
        for (int u = 0; u < ROWS; ++u)
            if (tid + u * URED_THREADS < ns) e.x[u] = gX[(size_t)k * (ns + 1) + tid + u * URED_THREADS];
        const auto I = gI + (size_t)(k % g.n_dir) * items;
#pragma unroll
        for (int u = 0; u < UITEMS_PER; ++u) {
            const int it = it0 + u * URED_THREADS;
            e.ip[u] = I[min(it, items - 1)];
            e.w[u] = it >= ns && it < items ? gW[(size_t)k * nw + (it - ns)] : 0.0;
        }
    };
    auto take = [&](int t, Next& e) {
        const double D = g.Dw[sys(t)], S = g.S[2 * sys(t) + g.grad_axis];
        __syncthreads();
#pragma unroll
        for (int u = 0; u < ROWS; ++u)
            if (tid + u * URED_THREADS < ns) lds[tid + u * URED_THREADS] = e.x[u];
        double w[UITEMS_PER];
        unsigned ip[UITEMS_PER];
#pragma unroll
        for (int u = 0; u < UITEMS_PER; ++u) {
            w[u] = it0 + u * URED_THREADS < ns ? D : e.w[u];
            ip[u] = e.ip[u];
        }
        if (t + 2 < n) load(sys(t + 2), e);
        __syncthreads();
        double vx = 0.0;
#pragma unroll
        for (int u = 0; u < UITEMS_PER; ++u) {
            const double xv = lds[ip[u]];
            a[u] = fma(w[u], xv, a[u]);
            vx = fma(v[u], xv, vx);
        }
        z = fma(S, vx, z);
    };
#pragma unroll
    for (int u = 0; u < UITEMS_PER; ++u) {
        const int it = it0 + u * URED_THREADS;
        a[u] = 0.0;
        v[u] = it < ns ? g.V[it] : 0.0;
    }
    if (n > 0) load(sys(0), nx[0]);
    if (n > 1) load(sys(1), nx[1]);
    for (int t = 0; t < n; t += 2) {
        take(t, nx[0]);
        if (t + 1 < n) take(t + 1, nx[1]);
    }
#pragma unroll
    for (int u = 0; u < UITEMS_PER; ++u) {
        const int it = it0 + u * URED_THREADS;
        if (it < items) g.part[(size_t)strand * items + it] = a[u];
    }
    __syncthreads();
    z = ublock_sum(z, lds);
    if (tid == 0) g.kpart[blockIdx.x] = z;
}

// The strands' sums combined in order, one thread per cell or wall face.
__global__ void __launch_bounds__(256) k_ucombine(const UGeomDev* __restrict__ gp) {
    const UGeomDev& g = *gp;
    const int items = g.ns + g.nwalls, it = blockIdx.x * 256 + threadIdx.x;
    if (it >= items) return;
    const auto p = gview(g.part) + it;
    double s = 0.0;
#pragma unroll 4
    for (int q = 0; q < UQ; ++q) {
        const double a0 = p[(size_t)(4 * q) * items], a1 = p[(size_t)(4 * q + 1) * items];
        const double a2 = p[(size_t)(4 * q + 2) * items], a3 = p[(size_t)(4 * q + 3) * items];
        s += (a0 + a1) + (a2 + a3);
    }
    if (it < g.ns) g.T_L[it] = s;
    else g.T_w[it - g.ns] = s;
}

}  // namespace

hipError_t ulaunch_fourier_start(const UFourierDev* f_dev, int ns, int nfaces, hipStream_t st) {
    (void)hipGetLastError();
    const int B = uf_blocks(ns), BF = (nfaces + UFB - 1) / UFB;
    hipLaunchKernelGGL(k_uf_grad, dim3(B), dim3(UFB), 0, st, f_dev);
    if (BF > 0) hipLaunchKernelGGL(k_uf_face, dim3(BF), dim3(UFB), 0, st, f_dev);
    hipLaunchKernelGGL(k_uf_init, dim3(B), dim3(UFB), 0, st, f_dev);
    hipLaunchKernelGGL(k_uf_w0, dim3(B), dim3(UFB), 0, st, f_dev);
    return hipGetLastError();
}

hipError_t ulaunch_fourier_cg(const UFourierDev* f_dev, int ns, int iters, double cg_tol, int max_cg,
                              hipStream_t st) {
    (void)hipGetLastError();
    const int B = uf_blocks(ns);
    for (int k = 0; k < iters; ++k) {
        // the parity of an iteration is its count's, which is even at the
        // start of every chunk (chunks are even and a solve starts at 0)
        hipLaunchKernelGGL(k_uf_cg, dim3(B), dim3(UFB), 0, st, f_dev, k & 1, cg_tol, max_cg);
    }
    return hipGetLastError();
}

hipError_t ulaunch_fourier_end(const UFourierDev* f_dev, int ns, double tol, hipStream_t st) {
    (void)hipGetLastError();
    const int B = uf_blocks(ns);
    hipLaunchKernelGGL(k_uf_sum, dim3(B), dim3(UFB), 0, st, f_dev);
    hipLaunchKernelGGL(k_uf_center, dim3(B), dim3(UFB), 0, st, f_dev);
    hipLaunchKernelGGL(k_uf_change, dim3(1), dim3(UFB), 0, st, f_dev, tol);
    return hipGetLastError();
}

hipError_t ulaunch_fourier_kappa(const UFourierDev* f_dev, int ns, hipStream_t st) {
    (void)hipGetLastError();
    hipLaunchKernelGGL(k_uf_grad, dim3(uf_blocks(ns)), dim3(UFB), 0, st, f_dev);
    hipLaunchKernelGGL(k_uf_kappa, dim3(1), dim3(UF_THREADS), 0, st, f_dev);
    return hipGetLastError();
}

hipError_t ulaunch_pack(const UGeomDev* g_dev, int n_pos, bool with_kappa, hipStream_t st) {
    (void)hipGetLastError();
    int blocks = (n_pos + 255) / 256;
    blocks = blocks < 1 ? 1 : (blocks > 2048 ? 2048 : blocks);
    hipLaunchKernelGGL(k_upack, dim3(blocks + with_kappa), dim3(256), 0, st, g_dev, (int)with_kappa);
    return hipGetLastError();
}

hipError_t ulaunch_pass(const UGeomDev* g_dev, int n_sys, int nin, int wpl, int slots, double inner_tol,
                        double inner_rtol, int max_inner, hipStream_t st) {
    (void)hipGetLastError();
    auto go = [&](auto* k) {
        hipLaunchKernelGGL(k, dim3(n_sys), dim3(WAVE), (size_t)slots * sizeof(double), st, g_dev, inner_tol,
                           inner_rtol, max_inner);
        return hipGetLastError();
    };
    const bool tri = nin <= 2;
    switch (wpl) {
    case 1: return tri ? go(k_upass<1, 2>) : go(k_upass<1, 3>);
    case 2: return tri ? go(k_upass<2, 2>) : go(k_upass<2, 3>);
    case 4: return tri ? go(k_upass<4, 2>) : go(k_upass<4, 3>);
    case 8: return tri ? go(k_upass<8, 2>) : go(k_upass<8, 3>);
    default: return hipErrorInvalidValue;
    }
}

hipError_t ulaunch_reduce(const UGeomDev* g_dev, int ns, int nwalls, hipStream_t st) {
    (void)hipGetLastError();
    const int items = ns + nwalls;
    const size_t lds = sizeof(double) * (size_t)(ns < 64 ? 64 : ns);
    hipLaunchKernelGGL(k_ureduce, dim3(USTRANDS * ((items + UITEMS - 1) / UITEMS)), dim3(URED_THREADS), lds, st, g_dev);
    hipLaunchKernelGGL(k_ucombine, dim3((items + 255) / 256), dim3(256), 0, st, g_dev);
    return hipGetLastError();
}
