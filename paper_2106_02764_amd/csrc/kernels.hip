// gfx950 kernels of the aMFP-BTE hot path.
//
// One outer pass (paper: Eq. (iter), Algorithm 1) solves, for every
// direction l and MFP m,
//     (sigma + Lambda_m A_l) x = b,
//     b = sigma T_L + Lambda_m [wall inflow (T_w) + periodic-jump inflow]
// with the upwind finite-volume operator of Appendix A, Eq. (iter2), then
// reduces the solutions into T_L = sum D x, the diffuse-wall temperatures
// T_w and kappa.
//
// Inner solve (sweep2d.h, sweep3d.h, rows.h).  Ordering the cells of a
// structured grid in upwind order makes A_l lower triangular except for the
// periodic wrap couplings.  One wavefront owns one (m,l) system and sweeps the
// grid row by row in upwind order (and plane by plane in z-upwind order in
// 3D); 2D rows run along the axis that the direction crosses more often, 3D
// rows along x.  Inside a row the recurrence x_i = a_i + q_i x_{i-1}, cyclic
// when its axis is periodic, is solved exactly with a wavefront-wide scan of
// affine maps.  The sweep M^{-1} is therefore exact up to the wrap coupling E
// (first row <- last row).  BiCGSTAB right-preconditioned by the sweep works
// on A M^{-1} = I - E M^{-1}: its Krylov vectors are supported on the wrap row
// only (2D: held in the wavefront's registers; 3D: a plane per vector) and
// every dot product is a wavefront reduction.  Each matrix-vector product is
// one sweep whose only source is the wrap row.  A system stores its solution
// on the solid cells; b is formed on the fly from tables shared by all
// systems.
//
// Reductions.  One kernel sums the stored solutions per cell and wall in a
// fixed order, another reduces kappa, so FP64 results are bitwise reproducible
// (no floating-point atomics).
#include "device.h"
#include <climits>

namespace {

// ---------------------------------------------------------------------------
// Per-cell / per-wall sums over the systems' stored solutions (fixed order)
// and the next pass's inputs sigma T_L and T_w.  Forward: T_L = sum D x and
// T_w = sum ReLu(S.n)/sum ReLu(S.n) x at the wall cell.  Adjoint: Psi = sigma
// sum lambda and Phi_f = sum of c_a lambda over the directions entering
// through f (the transpose of the wall coupling).  A block owns a strip of RC
// solid cells (consecutive solid indices: one 128-byte segment of a system's
// FP32 values); each of its RQ waves holds the strip twice (lanes 0-31 and
// 32-63), and the 2 RQ half-waves split the systems in fixed chunks, so twice
// as many loads are in flight per strip as with one chunk per wave.  A
// half-wave stages the weights of RC systems at a time in LDS (D, or 1 in
// the adjoint, and the wall weights), zero beyond its chunk, so every
// half-wave runs the same trip count, in groups of RG in-range loads.  A wall face reads
// only its own cell's values, so the walls of the strip's cells are summed
// from the same loads.  Every sum is combined over the chunks in order.
// Pore entries of the outputs are never written: they are set to 0 once per
// solve (k_prep_sigma) and stay 0.
// ---------------------------------------------------------------------------
constexpr int RQ = 16;      // waves per reduction block
constexpr int RC = 32;      // solid cells per strip
constexpr int RH = 2 * RQ;  // system chunks per strip: one per half-wave
constexpr int RG = 16;      // loads in flight per lane: systems per group
static_assert(RC == 32 && RC % RG == 0 && RG % 4 == 0, "a strip is one half of a wave, read in groups of RG systems");

template <typename T>
__global__ void __launch_bounds__(64 * RQ) k_reduce_pass(const GeomDev* __restrict__ geoms, PassParams pp) {
    __shared__ double wt[RH][7][RC];       // per half-wave: row 0 D (or 1), rows 1..6 the wall weights
    __shared__ double part[RH][RC];
    const GeomDev& g = geoms[blockIdx.y];
    if (g.ctrl[CTRL_DONE] && pp.mode == 0) return;
    const int pass = g.ctrl[CTRL_PASS];
    const int out = (pass + 1) & 1;
    const int adj = pp.adjoint;
    const int nc = g.ncells, nf = g.nf, ns = g.n_sys, nd = g.n_dir, nsol = g.nsolid, xs = g.xs;
    if ((int)blockIdx.x * RC >= nsol) return;          // block-uniform
    const gptr_t<T> X = gview(reinterpret_cast<const T*>(g.X));
    const gptr_t<double> D = gview(g.Dw);
    const int q = threadIdx.x >> 6, cl = threadIdx.x & 63;
    const int h = cl >> 5, c = cl & (RC - 1);
    const int hq = 2 * q + h;                           // this half-wave's chunk
    const int j = blockIdx.x * RC + c;                  // solid index of this lane
    const bool in = j < nsol;
    const int js = in ? j : nsol - 1;                   // in-range loads, dropped below
    const int cell = in ? g.scell[j] : -1;
    const int per = (ns + RH - 1) / RH;                 // the same trip count in every chunk
    const int i0 = hq * per, i1 = min(ns, i0 + per);
    // wall faces of this lane's cell (bit f), and of the strip: the same in
    // every wave of the block
    int wm = 0;
    if (in) {
        const uint16_t w = g.fc[cell];
        for (int f = 0; f < nf; ++f) wm |= (fc_class(w, f) == FC_WALL ? 1 : 0) << f;
    }
    int wany = wm;
#pragma unroll
    for (int m = 1; m < 64; m <<= 1) wany |= shfl_xor(wany, m);
    double a0 = 0.0, a1 = 0.0, a2 = 0.0, a3 = 0.0;
    double aw[6] = {0.0, 0.0, 0.0, 0.0, 0.0, 0.0};
    for (int r = 0; r < per; r += RC) {
        // lane c of the half-wave: the weights of system i0 + r + c (forward
        // walls: ReLu(S.n) / sum; adjoint walls: c_a of the directions
        // entering through the face)
        const int is = i0 + r + c;
        const bool lv = is < i1;
        const int il = lv ? is : ns - 1;
        wt[hq][0][c] = lv ? (adj ? 1.0 : D[il]) : 0.0;
        if (wany) {
            double cf[6];
            if (!adj) {
#pragma unroll
                for (int f = 0; f < 6; ++f) cf[f] = g.wout[(size_t)min(f, nf - 1) * ns + il];
            } else {
                const int m = il / nd, l = il - m * nd;
                const double mf = g.mfp[m];
                const double sd3[3] = {g.dirs[l * 3], g.dirs[l * 3 + 1], g.dirs[l * 3 + 2]};
#pragma unroll
                for (int f = 0; f < 6; ++f) {
                    const int ax = f >> 1;
                    const double sd = sd3[ax];
                    const double nsgn = (f & 1) ? 1.0 : -1.0;
                    cf[f] = sd * nsgn < 0.0 ? mf * fabs(sd) / g.h[ax] : 0.0;
                }
            }
#pragma unroll
            for (int f = 0; f < 6; ++f)
                if (f < nf && ((wany >> f) & 1)) wt[hq][1 + f][c] = lv ? cf[f] : 0.0;
        }
        // the wave reads back its own rows (LDS ops of a wave complete in order)
        __builtin_amdgcn_wave_barrier();
        // groups of RG systems: past the chunk's end the weights are 0 and the
        // loads stay in range
        const int nb = min(RC, (per - r + RG - 1) & ~(RG - 1));
        const int ib = i0 + r;
        for (int u0 = 0; u0 < nb; u0 += RG) {
            double xv[RG];
#pragma unroll
            for (int u = 0; u < RG; ++u) xv[u] = (double)X[(size_t)min(ib + u0 + u, ns - 1) * xs + js];
#pragma unroll
            for (int u = 0; u < RG; u += 4) {
                a0 += wt[hq][0][u0 + u] * xv[u];
                a1 += wt[hq][0][u0 + u + 1] * xv[u + 1];
                a2 += wt[hq][0][u0 + u + 2] * xv[u + 2];
                a3 += wt[hq][0][u0 + u + 3] * xv[u + 3];
            }
            if (wany) {
#pragma unroll
                for (int f = 0; f < 6; ++f) {
                    if (f >= nf || !((wany >> f) & 1)) continue;
                    const double* cp = &wt[hq][1 + f][u0];
#pragma unroll
                    for (int u = 0; u < RG; ++u) aw[f] += cp[u] * xv[u];   // zero weight: + 0
                }
            }
        }
        // this round's weights are read before the next round writes them
        __builtin_amdgcn_wave_barrier();
    }
    part[hq][c] = in ? (a0 + a1) + (a2 + a3) : 0.0;
    __syncthreads();
    const bool head = q == 0 && h == 0;                 // lanes 0..RC-1 of wave 0 write
    if (head && in) {
        double tot = part[0][c];
#pragma unroll
        for (int u = 1; u < RH; ++u) tot += part[u][c];
        if (!adj) g.T_L[cell] = tot;
        if (g.aa_m > 0) {
            g.ag[cell] = tot;              // the mixing step writes the next inputs
        } else {
            g.ax[cell] = tot;
            if (adj) g.lam_psi[(size_t)out * nc + cell] = g.sigma[cell] * tot;
            else g.sT[(size_t)out * nc + cell] = g.sigma[cell] * tot;
        }
    }
    if (!wany) return;                     // block-uniform
    double* bnd_out = g.bnd + ((size_t)(adj ? 2 : 0) + out) * nf * nc;
#pragma unroll
    for (int f = 0; f < 6; ++f) {
        if (f >= nf || !((wany >> f) & 1)) continue;
        __syncthreads();                   // the previous sum's reads are done
        part[hq][c] = aw[f];
        __syncthreads();
        if (head && ((wm >> f) & 1)) {
            double a = part[0][c];
#pragma unroll
            for (int u = 1; u < RH; ++u) a += part[u][c];
            const int wi = g.wall_idx[cell * nf + f];
            if (g.aa_m > 0) {
                g.ag[nc + wi] = a;
            } else {
                g.ax[nc + wi] = a;
                if (adj) g.lam_phi[(size_t)out * g.nwalls + wi] = a;
                else g.Tw[(size_t)out * g.nwalls + wi] = a;
                bnd_out[(size_t)f * nc + cell] = a;
            }
        }
    }
}

// kappa, history and the convergence test of Algorithm 1 (one block per geometry).
__global__ void k_finalize(const GeomDev* __restrict__ geoms, PassParams pp) {
    __shared__ double red[56];
    const GeomDev& g = geoms[blockIdx.x];
    if (g.ctrl[CTRL_DONE]) return;
    double k = 0.0, kf = 0.0, wr = 0.0;
    const int ns = g.n_sys, bd = blockDim.x;
    // thread t takes t, t + bd, ... in that order, 8 loads of each in flight
    for (int i0 = threadIdx.x; i0 < ns; i0 += 8 * bd) {
        double a[8], b[8], c[8];
#pragma unroll
        for (int u = 0; u < 8; ++u) {
            const int i = min(i0 + u * bd, ns - 1);
            a[u] = g.ksys[i];
            b[u] = g.kfsys[i];
            c[u] = g.wres[i];
        }
#pragma unroll
        for (int u = 0; u < 8; ++u)
            if (i0 + u * bd < ns) {
                k += a[u];
                kf += b[u];
                wr = fmax(wr, c[u]);
            }
    }
    // fixed-order: every thread sums a fixed strided subset, then block_sum
    block_sum2(k, kf, red);
    // max of the wrap residuals (every value is >= 0: max via the sum of a
    // one-hot is not needed, a plain block max suffices)
    __syncthreads();
    {
        const int lane = threadIdx.x & 63, wid = threadIdx.x >> 6;
        for (int m2 = 32; m2 >= 1; m2 >>= 1) wr = fmax(wr, shfl_xor(wr, m2));
        if (lane == 0) red[36 + wid] = wr;
        __syncthreads();
        wr = 0.0;
        for (int i = 0; i < (int)(blockDim.x >> 6); ++i) wr = fmax(wr, red[36 + i]);
    }
    if (threadIdx.x == 0) {
        const int pass = g.ctrl[CTRL_PASS];
        if (pass >= pp.max_outer) {      // history is sized for max_outer passes
            g.ctrl[CTRL_DONE] = 1;
            return;
        }
        g.hist[pass] = k;
        g.hist_face[pass] = kf;
        g.wres_hist[pass] = wr;
        const int n = pass + 1;
        g.ctrl[CTRL_PASS] = n;
        // Algorithm 1's test on the relative change of kappa; with a bounded
        // number of inner iterations per pass the wrap rows must be solved too
        const bool wrap_ok = wr <= pp.wrap_tol;
        bool small = n >= 2 && fabs(k - g.hist[pass - 1]) <= pp.outer_tol * fabs(k);
        if (pp.stop_rule == 1) {
            // error estimate of a linear fixed-point iteration: the
            // contraction is the largest of the last two ratios of
            // successive changes and of the mean ratio over ten passes (the
            // window sees through a transient or noisy pair)
            small = false;
            if (n >= 12) {
                const double d0 = fabs(k - g.hist[pass - 1]);
                const double d1 = fabs(g.hist[pass - 1] - g.hist[pass - 2]);
                const double d2 = fabs(g.hist[pass - 2] - g.hist[pass - 3]);
                const double d10 = fabs(g.hist[pass - 10] - g.hist[pass - 11]);
                double rho = fmax(d1 > 0.0 ? d0 / d1 : 0.0, d2 > 0.0 ? d1 / d2 : 0.0);
                if (d10 > 0.0) rho = fmax(rho, pow(d0 / d10, 0.1));
                rho = fmin(rho, 0.995);
                small = d0 * rho / (1.0 - rho) <= pp.outer_tol * fabs(k);
            }
        }
        // with mixing, successive kappa can agree before the iterate has
        // settled: the error estimated from the fixed-point residual must
        // meet the tolerance too
        if (g.aa_m > 0) small = small && g.fscal[3] <= pp.outer_tol;
        if (!isfinite(k)) {
            g.ctrl[CTRL_NONFINITE] = 1;
            g.ctrl[CTRL_DONE] = 1;
        } else if (wrap_ok && small) {
            g.ctrl[CTRL_CONVERGED] = 1;
            g.ctrl[CTRL_DONE] = 1;
        } else if (n >= pp.max_outer) {
            g.ctrl[CTRL_DONE] = 1;
        }
    }
}

// ---------------------------------------------------------------------------
// Anderson mixing of the outer fixed point x -> G(x).  The pass computed
// G(x_k); with f_k = G(x_k) - x_k and the last aa_m differences dX, dF of
// iterates and residuals,
//   gamma = argmin |f_k - dF gamma|,   x_{k+1} = x_k + f_k - (dX + dF) gamma
// (gamma from the normal equations of the column-scaled dF, Cholesky in
// double; a failed factorisation drops the history and takes the plain step
// x_{k+1} = G(x_k)).  Two kernels over up to AAB_MAX blocks per geometry:
// the first stores the new difference column and the per-block partial dot
// products, the second sums them in a fixed order, solves the small system
// in every block (the same numbers everywhere), and writes the next pass's
// inputs: sigma T_L (or sigma sum lambda), the wall values and their inflow
// table entries.  The history counters are double buffered by pass parity.
// ---------------------------------------------------------------------------
constexpr int AAB_MAX = 256, AA_THREADS = 256, AA_NP = 2 * AA_MAX + 3;

struct AView {
    int n, B, c0, c1;
};
__device__ __forceinline__ AView aa_view(const GeomDev& g, int b) {
    AView v;
    v.n = g.n_aa;
    v.B = min(AAB_MAX, (v.n + AA_THREADS - 1) / AA_THREADS);
    const int chunk = (v.n + v.B - 1) / v.B;
    v.c0 = min(v.n, b * chunk);
    v.c1 = min(v.n, v.c0 + chunk);
    return v;
}

__global__ void __launch_bounds__(AA_THREADS) k_aa_partial(const GeomDev* __restrict__ geoms) {
    __shared__ double red[AA_NP][AA_THREADS / 64];
    const GeomDev& g = geoms[blockIdx.y];
    if (g.aa_m <= 0 || g.ctrl[CTRL_DONE]) return;
    const AView v = aa_view(g, blockIdx.x);
    if ((int)blockIdx.x >= v.B) return;
    const int n = v.n, M = g.aa_m;
    const int* ac = g.actl + 4 * (g.ctrl[CTRL_PASS] & 1);
    const int cnt = ac[0], head = ac[1], have = ac[2];
    const int slot = head;                            // the new column (when have)
    const int cnt1 = have ? min(cnt + 1, M) : cnt;    // valid columns: 0 .. cnt1-1
    double dA[AA_MAX], db[AA_MAX];
#pragma unroll
    for (int j = 0; j < AA_MAX; ++j) { dA[j] = 0.0; db[j] = 0.0; }
    double ff = 0.0, xx = 0.0, dxx = 0.0;
    for (int i = v.c0 + threadIdx.x; i < v.c1; i += blockDim.x) {
        // every load first (the stored columns from in-range slots, unused
        // ones dropped below), so they are in flight together
        const double x = g.ax[i], gi = g.ag[i], fp = g.afp[i], xp = g.axp[i];
        double hF[AA_MAX];
#pragma unroll
        for (int j = 0; j < AA_MAX; ++j) hF[j] = g.adF[(size_t)min(j, M - 1) * n + i];
        const double f = gi - x;
        xx += x * x;
        ff += f * f;
        double df = 0.0;
        if (have) {
            df = f - fp;
            const double dx = x - xp;
            dxx += dx * dx;
            g.adX[(size_t)slot * n + i] = dx;
            g.adF[(size_t)slot * n + i] = df;
        }
        g.axp[i] = x;
        g.afp[i] = f;
#pragma unroll
        for (int j = 0; j < AA_MAX; ++j) {
            if (j < cnt1) {
                const double Fj = (have && j == slot) ? df : hF[j];
                db[j] += Fj * f;
                if (have) dA[j] += df * Fj;
            }
        }
    }
    const int lane = threadIdx.x & 63, wid = threadIdx.x >> 6, nw = blockDim.x >> 6;
    double sums[AA_NP];
#pragma unroll
    for (int j = 0; j < AA_MAX; ++j) {
        sums[j] = dA[j];
        sums[AA_MAX + j] = db[j];
    }
    sums[2 * AA_MAX] = ff;
    sums[2 * AA_MAX + 1] = xx;
    sums[2 * AA_MAX + 2] = dxx;
    wave_sum_n(sums);
    if (lane == 0)
#pragma unroll
        for (int q = 0; q < AA_NP; ++q) red[q][wid] = sums[q];
    __syncthreads();
    if (threadIdx.x < AA_NP) {
        double t = 0.0;
        for (int w = 0; w < nw; ++w) t += red[threadIdx.x][w];
        g.apart[(size_t)blockIdx.x * AA_NP + threadIdx.x] = t;
    }
}

__global__ void __launch_bounds__(AA_THREADS) k_aa_apply(const GeomDev* __restrict__ geoms, PassParams pp) {
    __shared__ double tot[AA_NP];
    __shared__ double wred[AA_NP][AA_THREADS / 64];
    __shared__ double gam[AA_MAX];
    const GeomDev& g = geoms[blockIdx.y];
    if (g.aa_m <= 0 || g.ctrl[CTRL_DONE]) return;
    const AView v = aa_view(g, blockIdx.x);
    if ((int)blockIdx.x >= v.B) return;
    const int n = v.n, M = g.aa_m, nc = g.ncells;
    const int adj = pp.adjoint;
    const int par = g.ctrl[CTRL_PASS] & 1;
    const int out = par ^ 1;                           // pass input buffers of the next pass
    const int* ac = g.actl + 4 * par;
    const int cnt = ac[0], head = ac[1], have = ac[2];
    const int slot = head;
    const int cnt1 = have ? min(cnt + 1, M) : cnt;
    // fixed-order sums of the per-block partials: thread b holds block b's
    // row (B <= blockDim), a butterfly per wave, then the waves in order
    {
        const int lane = threadIdx.x & 63, wid = threadIdx.x >> 6, nw = blockDim.x >> 6;
        const bool mine = (int)threadIdx.x < v.B;
        const double* row = g.apart + (size_t)(mine ? threadIdx.x : 0) * AA_NP;
        double sums[AA_NP];
#pragma unroll
        for (int q = 0; q < AA_NP; ++q) sums[q] = row[q];
#pragma unroll
        for (int q = 0; q < AA_NP; ++q) sums[q] = mine ? sums[q] : 0.0;
        wave_sum_n(sums);
        if (lane == 0)
#pragma unroll
            for (int q = 0; q < AA_NP; ++q) wred[q][wid] = sums[q];
        __syncthreads();
        if ((int)threadIdx.x < AA_NP) {
            double t = 0.0;
            for (int w = 0; w < nw; ++w) t += wred[threadIdx.x][w];
            tot[threadIdx.x] = t;
        }
        __syncthreads();
    }
    // The small least-squares solve on the first wave, one lane per entry of
    // the AA_MAX x AA_MAX Gram matrix: lane t holds entry (r, k) = (t / 8,
    // t % 8) and the vectors' entry j = t % 8.  Every loop runs over the
    // fixed AA_MAX; rows and columns beyond cnt1 are identity rows.
    static_assert(AA_MAX * AA_MAX == WAVE, "one lane per Gram matrix entry");
    if (threadIdx.x < WAVE) {
        const int t = threadIdx.x, r = t / AA_MAX, k = t % AA_MAX, j = k;
        const double* dxg = g.agram + M * M;            // |dX_j|^2 of the stored columns
        // this pass's Gram matrix: the new column's row from the partials,
        // the rest from the stored matrix (block 0 stores the new row)
        double a = r == k ? 1.0 : 0.0;
        if (r < cnt1 && k < cnt1) {
            const bool fresh = have && (r == slot || k == slot);
            a = fresh ? tot[r == slot ? k : r] : g.agram[r * M + k];
        }
        const bool vj = j < cnt1;
        const double dxn = vj ? ((have && j == slot) ? tot[2 * AA_MAX + 2] : dxg[j]) : 0.0;
        const double bj = vj ? tot[AA_MAX + j] : 0.0;
        const double gjj = shfl_at(a, (AA_MAX + 1) * j);
        if (blockIdx.x == 0 && have && t < cnt1) {
            const double val = tot[t];                  // new column against column t
            g.agram[slot * M + t] = val;
            g.agram[t * M + slot] = val;
            if (t == 0) g.agram[M * M + slot] = tot[2 * AA_MAX + 2];
        }
        // error estimate for the stop test: with f = (G - I) e for a linear G,
        // |e| <= |f| / s_min(I - G); s_min is estimated by the smallest
        // |dF_j| / |dX_j| over the stored columns (no columns: |f| itself)
        double sm = (vj && dxn > 0.0) ? sqrt(gjj / dxn) : 1.0;
#pragma unroll
        for (int m = 1; m < AA_MAX; m <<= 1) sm = fmin(sm, shfl_xor(sm, m));
        const double smin = fmax(fmin(sm, 1.0), 1e-3);
        const double sf = tot[2 * AA_MAX], sx = tot[2 * AA_MAX + 1];
        const double res = sx > 0.0 ? sqrt(sf / sx) : (sf > 0.0 ? INFINITY : 0.0);
        if (blockIdx.x == 0 && t == 0) g.fscal[3] = res / smin;
        // scaled normal equations with a small ridge, Cholesky in place
        // (right-looking: step p finishes column p and updates the trailing
        // block), then the two triangular solves; ok is wave-uniform
        const double dj = vj ? sqrt(gjj) : 1.0;
        bool ok = cnt1 > 0 && __all(dj > 0.0 && isfinite(dj));
        double y = 0.0;
        if (ok) {
            const double dr = shfl_at(dj, r);
            a = a / (dr * dj) + ((r == k && r < cnt1) ? 1e-10 : 0.0);
#pragma unroll
            for (int p = 0; p < AA_MAX; ++p) {
                const double s2 = shfl_at(a, (AA_MAX + 1) * p);
                ok = ok && s2 > 1e-14;
                const double lpp = sqrt(fmax(s2, 1e-300));
                if (k == p) a = r == p ? lpp : (r > p ? a / lpp : a);
                const double lr = shfl_at(a, AA_MAX * r + p), lk = shfl_at(a, AA_MAX * k + p);
                if (r > p && k > p && k <= r) a -= lr * lk;
            }
            y = bj / dj;
#pragma unroll
            for (int p = 0; p < AA_MAX; ++p) {
                const double yp = shfl_at(y, p) / shfl_at(a, (AA_MAX + 1) * p);
                const double ljp = shfl_at(a, AA_MAX * j + p);
                y = j == p ? yp : (j > p ? y - ljp * yp : y);
            }
#pragma unroll
            for (int p = AA_MAX - 1; p >= 0; --p) {
                const double zp = shfl_at(y, p) / shfl_at(a, (AA_MAX + 1) * p);
                const double lpj = shfl_at(a, AA_MAX * p + j);
                y = j == p ? zp : (j < p ? y - lpj * zp : y);
            }
            y = vj ? y / dj : 0.0;
            ok = ok && __all(isfinite(y));
        }
        if (t < AA_MAX) gam[t] = ok ? y : 0.0;
        if (blockIdx.x == 0 && t == 0) {
            int* ao = g.actl + 4 * out;
            if (ok || cnt1 == 0) {
                ao[0] = cnt1;
                ao[1] = have ? (slot + 1) % M : head;
            } else {          // drop the history; the next pass starts a new one
                ao[0] = 0;
                ao[1] = 0;
            }
            ao[2] = 1;
        }
    }
    __syncthreads();
    double* bnd_out = g.bnd + ((size_t)(adj ? 2 : 0) + out) * g.nf * nc;
    for (int i = v.c0 + threadIdx.x; i < v.c1; i += blockDim.x) {
        double hX[AA_MAX], hF[AA_MAX];       // loaded together, unused slots dropped
#pragma unroll
        for (int j = 0; j < AA_MAX; ++j) {
            const size_t o = (size_t)min(j, M - 1) * n + i;
            hX[j] = g.adX[o];
            hF[j] = g.adF[o];
        }
        double xn = g.axp[i] + g.afp[i];
#pragma unroll
        for (int j = 0; j < AA_MAX; ++j)
            if (j < cnt1) xn -= gam[j] * (hX[j] + hF[j]);
        if (i < nc) {
            const bool sol = fc_solid(g.fc[i]);
            xn = sol ? xn : 0.0;
            const double sx = sol ? g.sigma[i] * xn : 0.0;
            if (adj) g.lam_psi[(size_t)out * nc + i] = sx;
            else g.sT[(size_t)out * nc + i] = sx;
        } else {
            const int wi = i - nc;
            if (adj) g.lam_phi[(size_t)out * g.nwalls + wi] = xn;
            else g.Tw[(size_t)out * g.nwalls + wi] = xn;
            bnd_out[(size_t)g.wall_face[wi] * nc + g.wall_cell[wi]] = xn;
        }
        g.ax[i] = xn;
    }
}

// ---------------------------------------------------------------------------
// Fourier first guess: CG on the negated 5/7-point finite-volume Laplacian
// with adiabatic pores and the periodic jump (Appendix B on the structured
// grid), spread over up to FB_MAX blocks per geometry.  One kernel per
// iteration (the Chronopoulos-Gear arrangement of CG, below); it sums the
// per-block partials of the previous one in a fixed order (no atomics), so
// every block of a geometry takes the same decisions, and a converged
// geometry's blocks exit at once.
// ---------------------------------------------------------------------------
__device__ __forceinline__ double fourier_rhs(const GeomDev& g, uint16_t w, const double (&kf)[3]) {
    double b = 0.0;
    if (fc_solid(w))
        for (int f = 0; f < g.nf; ++f) {
            const int cl = fc_class(w, f);
            if (cl == FC_JUMP_P) b += kf[f >> 1] * g.dT;
            else if (cl == FC_JUMP_M) b -= kf[f >> 1] * g.dT;
        }
    return b;
}

constexpr int FB_MAX = 256, FB_THREADS = 256;
// geometries of one iteration launch (powers of 8; the table of block counts
// is a kernel argument, 2 KB of the 4 there may be).  The larger table is
// searched a level more, so it is taken where the smaller would need more
// launches, each as long as an iteration's chain (200 geometries, 24 to 48
// cells a side: 17.9 ms with four launches an iteration, 13.9 with one)
constexpr int FGRID_MIN = 64, FGRID_MAX = 512;

// This geometry's CG storage (in the fx region) and block b's cell range.
// r, s = A r and q = A p are double buffered by iteration parity; gp / dp hold
// the per-block partials of (r, r) and (r, s) by parity.  sc: [0] |b|, [1]
// done, [4] iterations, [6 + q] iterations done before an iteration of
// parity q, [8 + q] its (r, r) and [10 + q] its alpha.
// (the buffers are selected by ternaries, never by a run-time array index,
// which would put the view in private memory)
struct FView {
    double *x, *p, *r0, *r1, *s0, *s1, *q0, *q1, *gp0, *gp1, *dp0, *dp1, *sc;
    int n, B, c0, c1;
    __device__ double* r(int k) const { return k ? r1 : r0; }
    __device__ double* s(int k) const { return k ? s1 : s0; }
    __device__ double* q(int k) const { return k ? q1 : q0; }
    __device__ double* gp(int k) const { return k ? gp1 : gp0; }
    __device__ double* dp(int k) const { return k ? dp1 : dp0; }
};
__device__ __forceinline__ FView fourier_view(const GeomDev& g, int b) {
    FView v;
    const int n = g.ncells;
    v.n = n;
    v.B = min(FB_MAX, (n + FB_THREADS - 1) / FB_THREADS);
    double* f = g.fx;
    v.x = f;
    v.p = f + n;
    v.r0 = f + 2 * (size_t)n;
    v.r1 = f + 3 * (size_t)n;
    v.s0 = f + 4 * (size_t)n;
    v.s1 = f + 5 * (size_t)n;
    v.q0 = f + 6 * (size_t)n;
    v.q1 = f + 7 * (size_t)n;
    double* pt = f + 8 * (size_t)n;
    v.gp0 = pt;
    v.gp1 = pt + FB_MAX;
    v.dp0 = pt + 2 * FB_MAX;
    v.dp1 = pt + 3 * FB_MAX;
    v.sc = pt + 4 * FB_MAX;
    const int chunk = (n + v.B - 1) / v.B;
    v.c0 = min(n, b * chunk);
    v.c1 = min(n, v.c0 + chunk);
    return v;
}

__device__ __forceinline__ double axis_pick(double k0, double k1, double k2, int a) {
    return a == 0 ? k0 : (a == 1 ? k1 : k2);
}

// fixed-order sum of the B per-block partials, returned to every thread
__device__ __forceinline__ double sum_partials(const double* part, int B, double* red) {
    double t = 0.0;
    for (int i = threadIdx.x; i < B; i += blockDim.x) t += part[i];
    return block_sum(t, red);
}

// two of them in one pass (red: at least 34 doubles)
__device__ __forceinline__ void sum_partials2(const double* p, const double* q, int B, double* red, double& sp,
                                              double& sq) {
    sp = 0.0;
    sq = 0.0;
    for (int i = threadIdx.x; i < B; i += blockDim.x) {
        sp += p[i];
        sq += q[i];
    }
    block_sum2(sp, sq, red);
}

__global__ void __launch_bounds__(FB_THREADS) k_fourier_init(const GeomDev* __restrict__ geoms) {
    __shared__ double red[40];
    const GeomDev& g = geoms[blockIdx.y];
    const FView v = fourier_view(g, blockIdx.x);
    if ((int)blockIdx.x >= v.B) return;
    double kf[3];
    for (int a = 0; a < 3; ++a) kf[a] = (a < g.ndim) ? g.kappa_axis[a] / (g.h[a] * g.h[a]) : 0.0;
    // start from the linear profile T = -dT (i + 1/2) / n along the gradient
    // axis: the exact solution without pores, so the first residual lives
    // only next to pore faces
    const int ga = g.grad_axis;
    const double ng = (double)(ga == 0 ? g.nx : g.ny);
    auto lin = [&](int c) {
        const int i = ga == 0 ? c % g.nx : (c / g.nx) % g.ny;
        return -g.dT * ((double)i + 0.5) / ng;
    };
    double s = 0.0, bb = 0.0;
    for (int c = v.c0 + threadIdx.x; c < v.c1; c += blockDim.x) {
        const uint16_t w = g.fc[c];
        const CellPos cp = cell_pos(g, c);
        const double b = fourier_rhs(g, w, kf);
        double x0 = 0.0, r0 = 0.0;
        if (fc_solid(w)) {
            x0 = lin(c);
            double y = 0.0;
            for (int f = 0; f < g.nf; ++f)
                if (fc_class(w, f) != FC_WALL) y += kf[f >> 1] * (x0 - lin(nbr_cell(g, c, cp, f)));
            r0 = b - y;
        }
        v.x[c] = x0;
        v.r(0)[c] = r0;
        v.p[c] = 0.0;
        v.q(0)[c] = 0.0;
        s += r0 * r0;
        bb += b * b;
    }
    block_sum2(s, bb, red);
    if (threadIdx.x == 0) {
        v.gp(0)[blockIdx.x] = s;
        v.dp(1)[blockIdx.x] = bb;            // |b|^2 partials, read by k_fourier_norm
        if (blockIdx.x == 0) {
            v.sc[1] = 0.0;
            v.sc[4] = 0.0;
            v.sc[6] = 0.0;
        }
    }
}

// |b| of every geometry (one block each); a zero first residual is converged
__global__ void __launch_bounds__(FB_THREADS) k_fourier_norm(const GeomDev* __restrict__ geoms) {
    __shared__ double red[40];
    const GeomDev& g = geoms[blockIdx.x];
    const FView v = fourier_view(g, 0);
    double bb, rr;
    sum_partials2(v.dp(1), v.gp(0), v.B, red, bb, rr);
    if (threadIdx.x == 0) {
        v.sc[0] = sqrt(bb);
        if (!(bb > 0.0) || !(rr > 0.0)) v.sc[1] = 1.0;
    }
}

__device__ __forceinline__ void fourier_k(const GeomDev& g, double& k0, double& k1, double& k2) {
    k0 = g.kappa_axis[0] / (g.h[0] * g.h[0]);
    k1 = g.ndim > 1 ? g.kappa_axis[1] / (g.h[1] * g.h[1]) : 0.0;
    k2 = g.ndim > 2 ? g.kappa_axis[2] / (g.h[2] * g.h[2]) : 0.0;
}

// s_0 = A r_0 and the partials of (r_0, s_0).
__global__ void __launch_bounds__(FB_THREADS) k_fourier_s0(const GeomDev* __restrict__ geoms) {
    __shared__ double red[40];
    const GeomDev& g = geoms[blockIdx.y];
    const FView v = fourier_view(g, blockIdx.x);
    if ((int)blockIdx.x >= v.B) return;
    double k0, k1, k2;
    fourier_k(g, k0, k1, k2);
    const double* r = v.r(0);
    double d = 0.0;
    for (int c = v.c0 + threadIdx.x; c < v.c1; c += blockDim.x) {
        const uint16_t w = g.fc[c];
        const CellPos cp = cell_pos(g, c);
        double y = 0.0;
        if (fc_solid(w))
            for (int f = 0; f < g.nf; ++f) {
                if (fc_class(w, f) == FC_WALL) continue;
                y += axis_pick(k0, k1, k2, f >> 1) * (r[c] - r[nbr_cell(g, c, cp, f)]);
            }
        v.s(0)[c] = y;
        d += r[c] * y;
    }
    d = block_sum(d, red);
    if (threadIdx.x == 0) v.dp(0)[blockIdx.x] = d;
}

// One CG iteration in the Chronopoulos-Gear arrangement: s = A r and q = A p
// are carried by recurrence, so both inner products of an iteration, gamma =
// (r, r) and delta = (r, A r), come from one pass over the cells:
//   beta_k = gamma_k / gamma_{k-1},  alpha_k = gamma_k / (delta_k - beta_k
//   gamma_k / alpha_{k-1})  (k = 0: beta = 0, alpha = gamma / delta),
//   p = r + beta p,  q = s + beta q,  x += alpha p,  r' = r - alpha q,
//   s' = A r'  and the partials of (r', r'), (r', s').
// Iteration k (parity qq) reads r_k, s_k, q_{k-1} from buffers qq and writes
// r_{k+1}, s_{k+1}, q_k into buffers qq ^ 1; A r' at a cell needs r' at its
// neighbours, which every block forms itself from the unchanged buffers qq.
// The stop test (every block computes the same sums) is the one of the plain
// CG: |r_k| <= tol |b|, or max_iter iterations.
//
// A block's chain is what it costs: the geometry, the partials and their sum,
// the cells, the new partials.  So a thread's first cell is loaded before the
// sums of the partials (its loads need none of the scalars; they are all of
// its work up to FB_MAX * FB_THREADS cells), a wall face reads the cell itself
// (its difference is 0) so that no load sits in a branch, and of a batch only
// the blocks that have cells are launched.  An iteration of the 128 x 128 cell:
// 6.1 -> 5.2 us; of 24 geometries (517 000 cells, a grid of 6144 blocks for
// 2017 with cells): 20 -> 16 us, where the 80 bytes a cell would take 8 us.
template <int NG>
struct FGrid {
    int n, first[NG + 1];         // blocks per XCD before each geometry (INT_MAX past the last)
};

template <int NF>
struct FCell {
    uint16_t w;
    double r, s, q, p, x, rj[NF], sj[NF], qj[NF];
};

template <int NF>
__device__ __forceinline__ void fourier_cells(const GeomDev& g, const FView& v, int qq, double tol, int max_iter,
                                              double* red, int blk) {
    const gptr_t<double> r = gview(v.r(qq)), s = gview(v.s(qq)), q = gview(v.q(qq));
    const gmut_t<double> p = gmut(v.p), x = gmut(v.x);
    const gmut_t<double> rn = gmut(v.r(qq ^ 1)), sn = gmut(v.s(qq ^ 1)), qn = gmut(v.q(qq ^ 1));
    const auto fc = gview(g.fc);
    auto load = [&](int c, FCell<NF>& e) {
        e.w = fc[c];
        const int row = c / g.nx;
        const CellPos cp = NF == 4 ? CellPos{c - row * g.nx, row, 0} : cell_pos(g, c);
        e.r = r[c];
        e.s = s[c];
        e.q = q[c];
        e.p = p[c];
        e.x = x[c];
#pragma unroll
        for (int f = 0; f < NF; ++f) {
            const int j = fc_class(e.w, f) == FC_WALL ? c : nbr_cell(g, c, cp, f);
            e.rj[f] = r[j];
            e.sj[f] = s[j];
            e.qj[f] = q[j];
        }
    };
    FCell<NF> e;
    int c = v.c0 + (int)threadIdx.x;
    load(min(c, v.n - 1), e);
    const auto sc = gview(v.sc);
    const double bn = sc[0], done = sc[1], g1 = sc[8 + (qq ^ 1)], a1 = sc[10 + (qq ^ 1)];
    const int it = (int)sc[6 + qq];
    if (done != 0.0) return;
    double gam, del;
    sum_partials2(v.gp(qq), v.dp(qq), v.B, red, gam, del);
    if (!(sqrt(gam) > tol * bn) || it >= max_iter) {
        if (blk == 0 && threadIdx.x == 0) v.sc[1] = 1.0;
        return;
    }
    double alpha = gam / del, beta = 0.0;
    if (it > 0) {
        beta = gam / g1;
        alpha = gam / (del - beta * gam / a1);
    }
    double k0, k1, k2;
    fourier_k(g, k0, k1, k2);
    double gs = 0.0, ds = 0.0;
    for (; c < v.c1;) {
        double rc = 0.0, sa = 0.0, qc = 0.0;
        if (fc_solid(e.w)) {
            const double pc = e.r + beta * e.p;
            qc = e.s + beta * e.q;
            p[c] = pc;
            x[c] = e.x + alpha * pc;
            rc = e.r - alpha * qc;
#pragma unroll
            for (int f = 0; f < NF; ++f) {
                const double rj = e.rj[f] - alpha * (e.sj[f] + beta * e.qj[f]);
                sa += axis_pick(k0, k1, k2, f >> 1) * (rc - rj);
            }
        }
        rn[c] = rc;
        sn[c] = sa;
        qn[c] = qc;
        gs += rc * rc;
        ds += rc * sa;
        c += blockDim.x;
        if (c < v.c1) load(c, e);
    }
    block_sum2(gs, ds, red);
    if (threadIdx.x == 0) {
        v.gp(qq ^ 1)[blk] = gs;
        v.dp(qq ^ 1)[blk] = ds;
        if (blk == 0) {
            v.sc[8 + qq] = gam;
            v.sc[10 + qq] = alpha;
            v.sc[6 + (qq ^ 1)] = (double)(it + 1);
            v.sc[4] = (double)(it + 1);
        }
    }
}

// NF: faces of a cell (a batch is all 2D or all 3D).  2D runs
// with all waves of 517 000 cells resident (64 registers and 5 spilled, 8 waves
// a SIMD).
template <int NF, int NG>
__global__ void __launch_bounds__(FB_THREADS, NF == 4 ? 8 : 4) k_fourier_cg(const GeomDev* __restrict__ geoms, FGrid<NG> fg, int qq,
                                                         double tol, int max_iter) {
    __shared__ double red[40];
    // workgroups go to the eight XCDs in turn: an XCD takes consecutive blocks
    // of each geometry, so the rows that neighbouring blocks share are in its
    // L2 (with the blocks dealt out one by one each row was fetched three times)
    const int b = (int)blockIdx.x / 8, xcd = (int)blockIdx.x % 8;
    int k = 0;
    if (fg.n > 1) {
#pragma unroll
        for (int st = NG / 8; st > 0; st /= 8) {
            int d = 0;
#pragma unroll
            for (int i = 1; i < 8; ++i) d += b >= fg.first[k + i * st] ? st : 0;
            k += d;
        }
    }
    const GeomDev& g = geoms[k];
    const int blk = xcd * (fg.first[k + 1] - fg.first[k]) + b - fg.first[k];
    const FView v = fourier_view(g, blk);
    if (blk >= v.B) return;
    // in a batch, most blocks are soon those of geometries that have ended
    if (fg.n > 1 && v.sc[1] != 0.0) return;
    fourier_cells<NF>(g, v, qq, tol, max_iter, red, blk);
}

// geometries still iterating -> *pending (one block)
__global__ void __launch_bounds__(256) k_fourier_pending(const GeomDev* __restrict__ geoms, int n_geoms,
                                                        int* pending) {
    __shared__ double red[32];
    double c = 0.0;
    for (int i = threadIdx.x; i < n_geoms; i += blockDim.x) c += fourier_view(geoms[i], 0).sc[1] == 0.0 ? 1.0 : 0.0;
    c = block_sum(c, red);
    if (threadIdx.x == 0) *pending = (int)c;
}

// End of the Fourier solve, in two kernels over the geometry's cell blocks.
// The first stores per-block partials of the solid-cell sum of x and count
// (the mean, which the gauge removes) and of the plane flux through the
// periodic plane of the gradient axis (kappa_F; differences of x, so the mean
// drops out) in the CG's direction buffers, free once it has ended.  The
// second sums them in a fixed order in every block and writes the mean-free
// T_F as T_L, sigma T_F, the wall temperatures, the first iterate of the
// outer fixed point and the inflow tables: periodic jumps +-dT (fixed), walls
// T_w (updated every pass), interior 0; forward buffers 0 and 1, adjoint
// buffers 2 and 3 (no jump source; walls updated per pass).  A wall's first
// temperature is its cell's, so buffer 0's wall entries take the cell value.
// Block 0 also stores kappa_F and the CG statistics and resets the pass
// control words.
__global__ void __launch_bounds__(FB_THREADS) k_fourier_part(const GeomDev* __restrict__ geoms) {
    __shared__ double red[32];
    const GeomDev& g = geoms[blockIdx.y];
    const FView v = fourier_view(g, blockIdx.x);
    if ((int)blockIdx.x >= v.B) return;
    const int ga = g.grad_axis;
    const double* x = g.fx;
    double sx = 0.0, ns = 0.0, fl = 0.0;
    for (int c = v.c0 + threadIdx.x; c < v.c1; c += blockDim.x) {
        const uint16_t w = g.fc[c];
        if (!fc_solid(w)) continue;
        sx += x[c];
        ns += 1.0;
        const int f = 2 * ga;   // '-' face of the cell at index 0
        if (fc_class(w, f) == FC_JUMP_P) {
            const int j = nbr_cell(g, c, cell_pos(g, c), f);
            fl += g.kappa_axis[ga] * (x[j] + g.dT - x[c]) / g.h[ga];
        }
    }
    sx = block_sum(sx, red);
    ns = block_sum(ns, red);
    fl = block_sum(fl, red);
    if (threadIdx.x == 0) {
        v.s(0)[blockIdx.x] = sx;
        v.s(1)[blockIdx.x] = ns;
        v.q(0)[blockIdx.x] = fl;
    }
}

__global__ void __launch_bounds__(FB_THREADS) k_fourier_fill(const GeomDev* __restrict__ geoms) {
    __shared__ double red[40];
    const GeomDev& g = geoms[blockIdx.y];
    const FView v = fourier_view(g, blockIdx.x);
    if ((int)blockIdx.x >= v.B) return;
    const int n = g.ncells, nf = g.nf;
    double sx, sn;
    sum_partials2(v.s(0), v.s(1), v.B, red, sx, sn);
    const double mean = sx / sn;
    if (blockIdx.x == 0) {
        const int it = (int)v.sc[4];
        const double rn = sqrt(sum_partials(v.gp(it & 1), v.B, red));
        const double fl = sum_partials(v.q(0), v.B, red);
        const double bn = v.sc[0];
        const int ga = g.grad_axis;
        if (g.aa_m > 0 && threadIdx.x < 8) g.actl[threadIdx.x] = 0;
        if (threadIdx.x == 0) {
            g.fscal[0] = g.L[ga] / (g.dT * (double)g.n_perp) * fl;
            g.fscal[1] = (double)it;
            g.fscal[2] = bn > 0.0 ? rn / bn : 0.0;
            for (int i = 0; i < CTRL_N; ++i) g.ctrl[i] = 0;
        }
    }
    const double* x = g.fx;
    const size_t nb = (size_t)nf * n;
    for (int c = v.c0 + threadIdx.x; c < v.c1; c += blockDim.x) {
        const uint16_t w = g.fc[c];
        const bool sol = fc_solid(w);
        const double t = sol ? x[c] - mean : 0.0;
        g.T_L[c] = t;
        g.sT[c] = sol ? g.sigma[c] * t : 0.0;   // buffer 0
        g.ax[c] = t;
        for (int f = 0; f < nf; ++f) {
            const int cl = sol ? fc_class(w, f) : FC_INTERIOR;
            const double jv = cl == FC_JUMP_P ? g.dT : (cl == FC_JUMP_M ? -g.dT : 0.0);
            const size_t e = (size_t)f * n + c;
            g.bnd[e] = cl == FC_WALL ? t : jv;
            g.bnd[nb + e] = jv;
            g.bnd[2 * nb + e] = 0.0;
            g.bnd[3 * nb + e] = 0.0;
        }
    }
    for (int wi = blockIdx.x * blockDim.x + threadIdx.x; wi < g.nwalls; wi += v.B * blockDim.x) {
        const double t = x[g.wall_cell[wi]] - mean;
        g.Tw[wi] = t;
        g.ax[n + wi] = t;
    }
}

// sigma per cell (1 where not given or in pores) and its float copy; the
// pore entries of the per-cell pass arrays, which the reduction and the
// mixing never write, are set to 0 (the solid entries are left as they are,
// so a resumed solve keeps its state).
__global__ void __launch_bounds__(256) k_prep_sigma(const GeomDev* __restrict__ gp, const double* __restrict__ sig_in) {
    __shared__ double red[4];
    const GeomDev& g = *gp;
    const int nc = g.ncells;
    double vmin = INFINITY;         // smallest sigma over this block's solid cells
    for (int c = blockIdx.x * blockDim.x + threadIdx.x; c < nc; c += gridDim.x * blockDim.x) {
        const bool sol = fc_solid(g.fc[c]);
        double v = 1.0;
        if (sig_in && sol) v = sig_in[c];
        if (sol) vmin = fmin(vmin, v);
        g.sigma[c] = v;
        g.sigma_f[c] = (float)v;
        if (!sol) {
            g.T_L[c] = 0.0;
            g.sT[c] = 0.0;
            g.sT[nc + c] = 0.0;
            g.lam_psi[c] = 0.0;
            g.lam_psi[nc + c] = 0.0;
            g.ax[c] = 0.0;
            if (g.aa_m > 0) {
                g.ag[c] = 0.0;
                g.axp[c] = 0.0;
                g.afp[c] = 0.0;
            }
        }
    }
    for (int m = 32; m >= 1; m >>= 1) vmin = fmin(vmin, shfl_xor(vmin, m));
    if ((threadIdx.x & 63) == 0) red[threadIdx.x >> 6] = vmin;
    __syncthreads();
    if (threadIdx.x == 0) g.fx[blockIdx.x] = fmin(fmin(red[0], red[1]), fmin(red[2], red[3]));
}

// Smallest sigma over the solid cells into fscal[5]: the minimum of the
// per-block minima k_prep_sigma left in fx (one block).  The pass kernels
// bound the gain of a system's wrap map with it (see wrap_gain_bound).
__global__ void __launch_bounds__(256) k_sigma_min(const GeomDev* __restrict__ gp, int nblocks) {
    __shared__ double red[4];
    const GeomDev& g = *gp;
    double v = INFINITY;
    for (int b = threadIdx.x; b < nblocks; b += blockDim.x) v = fmin(v, g.fx[b]);
    for (int m = 32; m >= 1; m >>= 1) v = fmin(v, shfl_xor(v, m));
    if ((threadIdx.x & 63) == 0) red[threadIdx.x >> 6] = v;
    __syncthreads();
    if (threadIdx.x == 0) g.fscal[5] = fmin(fmin(red[0], red[1]), fmin(red[2], red[3]));
}

// Flux map of one geometry from the stored solutions of the replayed last
// sweep: J_i = sum_ml S_ml x_iml.
// (the flux and the gradient: a block takes 64 cells, its FQ waves fixed chunks
// of the systems with eight loads of each in flight, combined in order; with a
// thread per cell for all systems a quarter of the CUs had a block, and one
// load each: 128 x 128 cells, 1440 systems, FP64: flux 389 -> 46 us, gradient
// 628 -> 64 us)
constexpr int FQ = 16;

template <typename T>
__global__ void __launch_bounds__(64 * FQ) k_flux(const GeomDev* __restrict__ gp, double* J_out) {
    __shared__ double part[3][FQ][64];
    const GeomDev& g = *gp;
    const int q = threadIdx.x >> 6, cl = threadIdx.x & 63, nd = g.ndim;
    const int c = blockIdx.x * 64 + cl;
    const bool in = c < g.ncells;
    const int i = in ? g.sidx[c] : -1;
    const gptr_t<T> X = gview(reinterpret_cast<const T*>(g.X)) + max(i, 0);
    const gptr_t<double> S = gview(g.S);
    const size_t xs = g.xs;
    const int per = (g.n_sys + FQ - 1) / FQ, s0 = q * per, s1 = min(g.n_sys, s0 + per);
    double j[3] = {0.0, 0.0, 0.0};
    for (int k = s0; k < s1; k += 8) {
        double x[8];
#pragma unroll
        for (int u = 0; u < 8; ++u) x[u] = (double)X[(size_t)min(k + u, s1 - 1) * xs];
#pragma unroll
        for (int u = 0; u < 8; ++u)
            if (k + u < s1)
#pragma unroll
                for (int a = 0; a < 3; ++a) j[a] += S[(k + u) * 3 + a] * x[u];
    }
#pragma unroll
    for (int a = 0; a < 3; ++a) part[a][q][cl] = j[a];
    __syncthreads();
    if (q >= nd || !in) return;            // wave a sums axis a
    double t = 0.0;
#pragma unroll
    for (int u = 0; u < FQ; ++u) t += part[q][u][cl];
    J_out[(size_t)c * nd + q] = i >= 0 ? t : 0.0;
}

// Adjoint gradient of one geometry: -sum_ml lambda_iml (T_iml - T_L,i) from
// the stored adjoint solutions and the stored forward state.
template <typename T>
__global__ void __launch_bounds__(64 * FQ) k_grad(const GeomDev* __restrict__ gp, double* grad_out) {
    __shared__ double part[FQ][64];
    const GeomDev& g = *gp;
    const int q = threadIdx.x >> 6, cl = threadIdx.x & 63;
    const int c = blockIdx.x * 64 + cl;
    const bool in = c < g.ncells;
    const int i = in ? g.sidx[c] : -1;
    const gptr_t<T> X = gview(reinterpret_cast<const T*>(g.X)) + max(i, 0);
    const gptr_t<double> F = gview(g.Tstore) + max(i, 0);
    const double tl = g.T_L[in ? c : 0];
    const size_t xs = g.xs;
    const int per = (g.n_sys + FQ - 1) / FQ, s0 = q * per, s1 = min(g.n_sys, s0 + per);
    double acc = 0.0;
    for (int k = s0; k < s1; k += 8) {
        double x[8], f[8];
#pragma unroll
        for (int u = 0; u < 8; ++u) {
            const size_t e = (size_t)min(k + u, s1 - 1) * xs;
            x[u] = (double)X[e];
            f[u] = F[e];
        }
#pragma unroll
        for (int u = 0; u < 8; ++u)
            if (k + u < s1) acc += x[u] * (f[u] - tl);
    }
    part[q][cl] = acc;
    __syncthreads();
    if (q != 0 || !in) return;
    double t = 0.0;
#pragma unroll
    for (int u = 0; u < FQ; ++u) t += part[u][cl];
    grad_out[c] = i >= 0 ? -t : 0.0;
}

// Energy balance of the last pass (paper, section Model: T_L is fixed by
// energy conservation, sum_ml alpha_ml sigma_i (T_iml - T_L,i) = 0 at the
// fixed point).  With alpha = D sum alpha the residual of cell i is
// sum alpha |sigma_i sum_ml D_ml T_iml - sigma_i T_L,i^in|, measured against
// the mean weighted magnitude sum alpha sum_i sum_ml D_ml |T_iml| / N_solid;
// sum alpha cancels.  One block per 64 solid cells writes its maximum and its
// sum; k_energy_finish combines them in a fixed order into fscal[4].
constexpr int EQ = 16;      // waves per energy block: system chunks of one 64-cell strip

template <typename T>
__global__ void __launch_bounds__(64 * EQ) k_energy(const GeomDev* __restrict__ gp) {
    __shared__ double pm[EQ][64], ps[EQ][64];
    const GeomDev& g = *gp;
    const int nsol = g.nsolid, ns = g.n_sys, xs = g.xs;
    const int q = threadIdx.x >> 6, cl = threadIdx.x & 63;
    const int j = blockIdx.x * 64 + cl;
    const bool in = j < nsol;
    const int js = in ? j : nsol - 1;           // in-range loads, dropped below
    const gptr_t<T> X = gview(reinterpret_cast<const T*>(g.X));
    const gptr_t<double> D = gview(g.Dw);
    const int per = (ns + EQ - 1) / EQ;
    const int i0 = q * per, i1 = min(ns, i0 + per);
    double t[4] = {0.0, 0.0, 0.0, 0.0}, a[4] = {0.0, 0.0, 0.0, 0.0};
    int i = i0;
    for (; i + 3 < i1; i += 4) {
        double x[4];
#pragma unroll
        for (int u = 0; u < 4; ++u) x[u] = (double)X[(size_t)(i + u) * xs + js];
#pragma unroll
        for (int u = 0; u < 4; ++u) {
            t[u] += D[i + u] * x[u];
            a[u] += D[i + u] * fabs(x[u]);
        }
    }
    for (; i < i1; ++i) {
        const double x = (double)X[(size_t)i * xs + js];
        t[0] += D[i] * x;
        a[0] += D[i] * fabs(x);
    }
    pm[q][cl] = (t[0] + t[1]) + (t[2] + t[3]);
    ps[q][cl] = (a[0] + a[1]) + (a[2] + a[3]);
    __syncthreads();
    if (q == 0) {
        double tl = 0.0, ab = 0.0, r = 0.0;
#pragma unroll
        for (int u = 0; u < EQ; ++u) {
            tl += pm[u][cl];
            ab += ps[u][cl];
        }
        if (in) {
            const int cell = g.scell[j];
            const int buf = (g.ctrl[CTRL_PASS] + 1) & 1;     // the last pass's input
            r = fabs(g.sigma[cell] * tl - g.sT[(size_t)buf * g.ncells + cell]);
        } else {
            ab = 0.0;
        }
        for (int m = 32; m >= 1; m >>= 1) {
            r = fmax(r, shfl_xor(r, m));
            ab += shfl_xor(ab, m);
        }
        if (cl == 0) {
            g.fx[2 * blockIdx.x] = r;
            g.fx[2 * blockIdx.x + 1] = ab;
        }
    }
}

__global__ void __launch_bounds__(256) k_energy_finish(const GeomDev* __restrict__ gp, int nblocks) {
    __shared__ double red[40];
    const GeomDev& g = *gp;
    double r = 0.0, ab = 0.0;
    for (int b = threadIdx.x; b < nblocks; b += blockDim.x) {
        r = fmax(r, g.fx[2 * b]);
        ab += g.fx[2 * b + 1];
    }
    for (int m = 32; m >= 1; m >>= 1) r = fmax(r, shfl_xor(r, m));
    const int lane = threadIdx.x & 63, wid = threadIdx.x >> 6;
    if (lane == 0) red[wid] = r;
    __syncthreads();
    double rm = 0.0;
    for (int w = 0; w < (int)(blockDim.x >> 6); ++w) rm = fmax(rm, red[w]);
    __syncthreads();
    ab = block_sum(ab, red);
    if (threadIdx.x == 0) {
        const double mean = g.nsolid > 0 ? ab / (double)g.nsolid : 0.0;
        g.fscal[4] = mean > 0.0 ? rm / mean : 0.0;
    }
}

// Lattice temperature of one geometry with the solid-cell mean removed.
__global__ void __launch_bounds__(1024) k_output(const GeomDev* __restrict__ gp, double* T_L_out) {
    __shared__ double red[32];
    const GeomDev& g = *gp;
    const int n = g.ncells;
    if (T_L_out) {
        double sx = 0.0, ns = 0.0;
        for (int c = threadIdx.x; c < n; c += blockDim.x)
            if (fc_solid(g.fc[c])) { sx += g.T_L[c]; ns += 1.0; }
        sx = block_sum(sx, red);
        ns = block_sum(ns, red);
        const double mean = ns > 0.0 ? sx / ns : 0.0;
        for (int c = threadIdx.x; c < n; c += blockDim.x)
            T_L_out[c] = fc_solid(g.fc[c]) ? g.T_L[c] - mean : 0.0;
    }
}

}  // namespace

// ---------------------------------------------------------------------------
// launchers
// ---------------------------------------------------------------------------
static_assert(fourier_scratch_doubles(0) == 4 * FB_MAX + 16 && fourier_scratch_doubles(1) == 4 * FB_MAX + 24,
              "Fourier scratch carve and kernels disagree");
static_assert(aa_partial_doubles() == (size_t)AAB_MAX * AA_NP, "mixing partials carve and kernels disagree");

int fourier_blocks(int max_cells) {
    const int b = (max_cells + FB_THREADS - 1) / FB_THREADS;
    return b < FB_MAX ? b : FB_MAX;
}

hipError_t launch_fourier_init(const GeomDev* geoms_dev, int n_geoms, int max_cells, hipStream_t st) {
    (void)hipGetLastError();
    hipLaunchKernelGGL(k_fourier_init, dim3(fourier_blocks(max_cells), n_geoms), dim3(FB_THREADS), 0, st, geoms_dev);
    hipLaunchKernelGGL(k_fourier_norm, dim3(n_geoms), dim3(FB_THREADS), 0, st, geoms_dev);
    hipLaunchKernelGGL(k_fourier_s0, dim3(fourier_blocks(max_cells), n_geoms), dim3(FB_THREADS), 0, st, geoms_dev);
    return hipGetLastError();
}

template <int NG>
static hipError_t launch_fourier_cg(const GeomDev* geoms_dev, const int* ncells, int n_geoms, int ndim, int parity, double tol,
                                    int max_iter, hipStream_t st) {
    (void)hipGetLastError();
    for (int g0 = 0; g0 < n_geoms; g0 += NG) {
        FGrid<NG> fg;
        fg.n = n_geoms - g0 < NG ? n_geoms - g0 : NG;
        int per = 0;
        for (int k = 0; k <= NG; ++k) {
            fg.first[k] = k <= fg.n ? per : INT_MAX;
            if (k < fg.n) per += (fourier_blocks(ncells[g0 + k]) + 7) / 8;
        }
        hipLaunchKernelGGL((ndim > 2 ? k_fourier_cg<6, NG> : k_fourier_cg<4, NG>), dim3(8 * per), dim3(FB_THREADS), 0, st,
                           geoms_dev + g0, fg, parity, tol, max_iter);
    }
    return hipGetLastError();
}

hipError_t launch_fourier_iter(const GeomDev* geoms_dev, const int* ncells, int n_geoms, int ndim, int parity, double tol,
                               int max_iter, hipStream_t st) {
    return n_geoms <= FGRID_MIN ? launch_fourier_cg<FGRID_MIN>(geoms_dev, ncells, n_geoms, ndim, parity, tol, max_iter, st)
                                : launch_fourier_cg<FGRID_MAX>(geoms_dev, ncells, n_geoms, ndim, parity, tol, max_iter, st);
}

hipError_t launch_fourier_pending(const GeomDev* geoms_dev, int n_geoms, int* pending_dev, hipStream_t st) {
    (void)hipGetLastError();
    hipLaunchKernelGGL(k_fourier_pending, dim3(1), dim3(256), 0, st, geoms_dev, n_geoms, pending_dev);
    return hipGetLastError();
}

hipError_t launch_fourier_finish(const GeomDev* geoms_dev, int n_geoms, int max_cells, hipStream_t st) {
    (void)hipGetLastError();
    const dim3 grid(fourier_blocks(max_cells), n_geoms);
    hipLaunchKernelGGL(k_fourier_part, grid, dim3(FB_THREADS), 0, st, geoms_dev);
    hipLaunchKernelGGL(k_fourier_fill, grid, dim3(FB_THREADS), 0, st, geoms_dev);
    return hipGetLastError();
}

// The pass kernels are compiled in one unit per precision and row width
// (sweep2d_*.hip, sweep3d_*.hip).
template <typename T, int CPL>
hipError_t launch_sweep2(const GeomDev*, const Item*, int, int, PassParams, size_t, hipStream_t, int);
template <typename T, int CPL>
hipError_t launch_sweep3(const GeomDev*, const Item*, int, int, PassParams, size_t, hipStream_t, int);
template <typename T>
hipError_t launch_queue2(const GeomDev*, const Item*, int, int, PassParams, size_t, hipStream_t, int*);

template <typename T>
static hipError_t launch_sweep_t(int cpl, int nz, const GeomDev* g, const Item* it, int n, int waves, PassParams pp,
                                 size_t lds, hipStream_t st, int full) {
    if (nz > 1) {
        switch (cpl) {
            case 1: return launch_sweep3<T, 1>(g, it, n, waves, pp, lds, st, full);
            case 2: return launch_sweep3<T, 2>(g, it, n, waves, pp, lds, st, full);
            case 3: return launch_sweep3<T, 3>(g, it, n, waves, pp, lds, st, full);
            default: return launch_sweep3<T, 4>(g, it, n, waves, pp, lds, st, full);
        }
    }
    switch (cpl) {
        case 1: return launch_sweep2<T, 1>(g, it, n, waves, pp, lds, st, full);
        case 2: return launch_sweep2<T, 2>(g, it, n, waves, pp, lds, st, full);
        case 3: return launch_sweep2<T, 3>(g, it, n, waves, pp, lds, st, full);
        default: return launch_sweep2<T, 4>(g, it, n, waves, pp, lds, st, full);
    }
}

hipError_t launch_sweep_pass(int precision, int cpl, int nz, const GeomDev* g, const Item* it, int n, int waves,
                             PassParams pp, size_t lds, hipStream_t st, int full) {
    return precision == 1 ? launch_sweep_t<float>(cpl, nz, g, it, n, waves, pp, lds, st, full)
                          : launch_sweep_t<double>(cpl, nz, g, it, n, waves, pp, lds, st, full);
}

hipError_t launch_sweep_queue(int precision, const GeomDev* g, const Item* it, int n, int waves, PassParams pp,
                              size_t lds, hipStream_t st, int* queue) {
    return precision == 1 ? launch_queue2<float>(g, it, n, waves, pp, lds, st, queue)
                          : launch_queue2<double>(g, it, n, waves, pp, lds, st, queue);
}

// 2D pass inputs in the order of the sweeps' rows (see sweep2d.h), per
// orientation o (0: rows along x, 1: along y) and row direction negr: sources,
// boundary values of the row's inflow face, of the two faces across the rows
// and (adjoint) of the row's outflow face.  Rows are padded in front with
// zeros to q_rs[o] records.
struct RowRec {
    int o, negr, cell;       // cell -1: padding
    size_t nrec, e;          // records of a table, record in it
};
__device__ __forceinline__ RowRec row_rec(const GeomDev& g, size_t i) {
    RowRec r;
    const size_t n0 = (size_t)g.ny * g.q_rs[0];
    r.o = i >= 2 * n0;
    if (r.o) i -= 2 * n0;
    r.nrec = r.o ? (size_t)g.nx * g.q_rs[1] : n0;
    r.negr = i >= r.nrec;
    r.e = r.negr ? i - r.nrec : i;
    const int rs = r.o ? g.q_rs[1] : g.q_rs[0], nr = r.o ? g.ny : g.nx;
    const int row = (int)(r.e / rs), p = (int)(r.e - (size_t)row * rs) - (rs - nr);
    const int pp = r.negr ? nr - 1 - p : p;
    r.cell = p < 0 ? -1 : (r.o ? pp * g.nx + row : row * g.nx + pp);
    return r;
}
__device__ __forceinline__ size_t row_recs(const GeomDev& g) {
    return 2 * ((size_t)g.ny * g.q_rs[0] + (g.q_tr ? (size_t)g.nx * g.q_rs[1] : 0));
}

template <typename T>
__global__ void __launch_bounds__(256) k_pack_rows(const GeomDev* __restrict__ geoms, PassParams pp,
                                                   int* __restrict__ queue) {
    // the pass's item queue (persistent launches) starts at the first item
    if (queue && blockIdx.x == 0 && blockIdx.y == 0 && threadIdx.x == 0) *queue = 0;
    const GeomDev& g = geoms[blockIdx.y];
    if (pp.mode == 0 && g.ctrl[CTRL_DONE]) return;
    // the buffers the pass's sweeps read
    const int pass = g.ctrl[CTRL_PASS];
    const int buf = (pp.mode == 1) ? ((pass + 1) & 1) : (pass & 1);
    const int nc = g.ncells;
    const double* src = (pp.adjoint ? g.lam_psi : g.sT) + (size_t)buf * nc;
    const double* bnd = g.bnd + ((size_t)(pp.adjoint ? 2 : 0) + buf) * g.nf * nc;
    const size_t n = row_recs(g);
    for (size_t i = blockIdx.x * blockDim.x + threadIdx.x; i < n; i += gridDim.x * blockDim.x) {
        const RowRec r = row_rec(g, i);
        T* t = static_cast<T*>(r.o ? g.qtab[1] : g.qtab[0]) + (size_t)r.negr * 6 * r.nrec + r.e;
        const bool sol = r.cell >= 0 && fc_solid(g.fc[r.cell < 0 ? 0 : r.cell]);
        const int c = sol ? r.cell : 0, fr = 2 * r.o, fw = 2 - fr;       // '-' faces along the row / across the rows
        t[0] = sol ? (T)src[c] : T(0);
        t[r.nrec] = sol ? (T)bnd[(size_t)(fr + r.negr) * nc + c] : T(0);
        t[2 * r.nrec] = sol ? (T)bnd[(size_t)fw * nc + c] : T(0);
        t[3 * r.nrec] = sol ? (T)bnd[(size_t)(fw + 1) * nc + c] : T(0);
        if (pp.adjoint) t[4 * r.nrec] = sol ? (T)bnd[(size_t)(fr + 1 - r.negr) * nc + c] : T(0);
    }
}

hipError_t launch_pack_rows(int precision, const GeomDev* geoms_dev, int n_geoms, int max_cells, PassParams pp,
                            hipStream_t st, int* queue) {
    // about four records per cell; at most 512 blocks per geometry (grid-stride)
    int blocks = (4 * max_cells + 255) / 256;
    blocks = blocks < 1 ? 1 : (blocks > 512 ? 512 : blocks);
    (void)hipGetLastError();
    if (precision == 1) hipLaunchKernelGGL(k_pack_rows<float>, dim3(blocks, n_geoms), dim3(256), 0, st, geoms_dev, pp, queue);
    else hipLaunchKernelGGL(k_pack_rows<double>, dim3(blocks, n_geoms), dim3(256), 0, st, geoms_dev, pp, queue);
    return hipGetLastError();
}

// What stays the same over a solve's passes: the sigma field in the rows'
// order and the store offsets (rows along x; rows along y take them by cell).
template <typename T>
__global__ void __launch_bounds__(256) k_pack_static(const GeomDev* __restrict__ gp) {
    const GeomDev& g = *gp;
    const T* sig = sigma_ptr<T>(g);
    const size_t n = row_recs(g);
    for (size_t i = blockIdx.x * blockDim.x + threadIdx.x; i < n; i += gridDim.x * blockDim.x) {
        const RowRec r = row_rec(g, i);
        T* t = static_cast<T*>(r.o ? g.qtab[1] : g.qtab[0]) + (size_t)r.negr * 6 * r.nrec + r.e;
        t[5 * r.nrec] = r.cell >= 0 ? sig[r.cell] : T(1);
        const int si = r.cell >= 0 ? g.sidx[r.cell] : -1;
        const uint32_t off = si >= 0 ? (uint32_t)si * (uint32_t)sizeof(T) : QOFF_NONE;
        if (!r.o) g.qoff[(size_t)r.negr * r.nrec + r.e] = off;
        if (!r.o && !r.negr && r.cell >= 0) g.qoffc[r.cell] = off;
    }
}

// Lane masks of every sweep row (one wave per sweep orientation and row; o:
// rows along y; 2D: orientations by the directions along and across the rows;
// 3D: by x, y and the order of the rows: y, z or y, reversed z, in which the
// sweep then runs forwards or backwards), per cell of a lane: inflow along the
// row open (set in the padding), inflow across the rows open, 3D: inflow
// through the z face open; solid; and (row_mask_scan) the scan's masks.
__global__ void __launch_bounds__(256) k_row_masks(const uint16_t* __restrict__ fc, int nx, int ny, int nz, int cpl, int o,
                                                   unsigned long long* __restrict__ out) {
    const bool d3 = nz > 1;
    const int nr = o ? ny : nx, nw = o ? nx : ny * nz, words = row_mask_words(cpl, d3);
    const int lane = threadIdx.x & 63, pad = WAVE * cpl - nr, fr = 2 * o, fw = 2 - fr;
    const size_t n = (size_t)(d3 ? 8 : 4) * nw;
    for (size_t r = (size_t)blockIdx.x * 4 + (threadIdx.x >> 6); r < n; r += (size_t)gridDim.x * 4) {
        const int tab = (int)(r / nw), row = (int)(r - (size_t)tab * nw);
        const int negr = d3 ? tab >> 2 : tab >> 1, negw = d3 ? (tab >> 1) & 1 : tab & 1, zrev = d3 ? tab & 1 : 0;
        const int iz = d3 ? (zrev ? nz - 1 - row % nz : row % nz) : 0;
        const int fz = 4 + (zrev ? 1 - negw : negw);       // '-' face of a sweep towards + z
        unsigned long long* w = out + r * words;
        unsigned long long good = ~0ull;
        for (int c = 0; c < cpl; ++c) {
            const int p = lane * cpl + c - pad;
            bool xo = true, yo = false, zo = false, sol = false;
            if (p >= 0) {
                const int pp = negr ? nr - 1 - p : p;
                const uint16_t v = fc[o ? pp * nx + row : (d3 ? row / nz + ny * iz : row) * nx + pp];
                sol = fc_solid(v);
                xo = sol && fc_class(v, fr + negr) != FC_WALL;
                yo = sol && fc_class(v, fw + negw) != FC_WALL;
                zo = sol && d3 && fc_class(v, fz) != FC_WALL;
            }
            const unsigned long long bx = __ballot(xo), by = __ballot(yo), bz = __ballot(zo), bs = __ballot(sol);
            good &= bx;
            if (lane == 0) {
                w[c] = bx;
                w[cpl + c] = by;
                if (d3) w[2 * cpl + c] = bz;
                w[(d3 ? 3 : 2) * cpl + c] = bs;
            }
        }
        if (row_mask_scan(cpl, d3)) {
            ScanMask m;
            scan_mask(good, m);
            if (lane == 0) {
                for (int k = 0; k < 6; ++k) w[4 * cpl + k] = m.brk[k];
                w[4 * cpl + 6] = m.om;
                w[4 * cpl + 7] = m.nb;
            }
        }
    }
}

hipError_t launch_row_masks(const uint16_t* fc, int nx, int ny, int nz, int cpl, int o, unsigned long long* out,
                            hipStream_t st) {
    (void)hipGetLastError();
    // four rows a block, at most 2^16 blocks (grid-stride)
    const size_t n = (size_t)(nz > 1 ? 8 : 4) * (o ? nx : (size_t)ny * nz), blocks = (n + 3) / 4;
    hipLaunchKernelGGL(k_row_masks, dim3((unsigned)(blocks < 65536 ? blocks : 65536)), dim3(256), 0, st, fc, nx, ny, nz, cpl, o,
                       out);
    return hipGetLastError();
}

// The adjoint's forward state: the replayed pass's solutions in double.
template <typename T>
__global__ void __launch_bounds__(256) k_keep(const GeomDev* __restrict__ gp) {
    const GeomDev& g = *gp;
    const size_t n = (size_t)g.n_sys * g.xs;
    const T* X = reinterpret_cast<const T*>(g.X);
    for (size_t i = (size_t)blockIdx.x * blockDim.x + threadIdx.x; i < n; i += (size_t)gridDim.x * blockDim.x)
        g.Tstore[i] = (double)X[i];
}

hipError_t launch_keep(int precision, const GeomDev* geom_dev, hipStream_t st) {
    (void)hipGetLastError();
    if (precision == 1) hipLaunchKernelGGL(k_keep<float>, dim3(4096), dim3(256), 0, st, geom_dev);
    else hipLaunchKernelGGL(k_keep<double>, dim3(4096), dim3(256), 0, st, geom_dev);
    return hipGetLastError();
}

// 3D: the pass's sources (sigma T_L, or sigma sum lambda in the adjoint) and
// inflow tables, read from the buffers the pass's sweeps consume (the rule of
// the pass kernel), in the compute type and in sweep order: rows by y, z and
// by y, reversed z; a row's block of q_row3 bytes holds nx each of the
// sources, the boundary values of faces 0 to 5 and sigma, then nx store
// offsets.
struct Rec3 {
    char* row;
    int cell, x;
};
__device__ __forceinline__ Rec3 rec3(const GeomDev& g, int i) {
    const int zrev = i >= g.ncells, e = zrev ? i - g.ncells : i;
    const int row = e / g.nx, iy = row / g.nz, k = row - iy * g.nz;
    Rec3 r;
    r.x = e - row * g.nx;
    r.cell = r.x + g.nx * (iy + g.ny * (zrev ? g.nz - 1 - k : k));
    r.row = static_cast<char*>(g.qtab[0]) + ((size_t)zrev * g.ny * g.nz + row) * g.q_row3;
    return r;
}

template <typename T>
__global__ void __launch_bounds__(256) k_pack3(const GeomDev* __restrict__ geoms, PassParams pp) {
    const GeomDev& g = geoms[blockIdx.y];
    if (pp.mode == 0 && g.ctrl[CTRL_DONE]) return;
    const int pass = g.ctrl[CTRL_PASS];
    const int buf = (pp.mode == 1) ? ((pass + 1) & 1) : (pass & 1);
    const int nc = g.ncells;
    const double* src = (pp.adjoint ? g.lam_psi : g.sT) + (size_t)buf * nc;
    const double* bnd = g.bnd + ((size_t)(pp.adjoint ? 2 : 0) + buf) * 6 * nc;
    for (int i = blockIdx.x * blockDim.x + threadIdx.x; i < 2 * nc; i += gridDim.x * blockDim.x) {
        const Rec3 r = rec3(g, i);
        T* t = reinterpret_cast<T*>(r.row) + r.x;
        t[0] = (T)src[r.cell];
#pragma unroll
        for (int f = 0; f < 6; ++f) t[(1 + f) * g.nx] = (T)bnd[(size_t)f * nc + r.cell];
    }
}

// What stays the same over a solve's passes: sigma and the store offsets.
template <typename T>
__global__ void __launch_bounds__(256) k_pack3_static(const GeomDev* __restrict__ gp) {
    const GeomDev& g = *gp;
    const T* sig = sigma_ptr<T>(g);
    for (int i = blockIdx.x * blockDim.x + threadIdx.x; i < 2 * g.ncells; i += gridDim.x * blockDim.x) {
        const Rec3 r = rec3(g, i);
        T* t = reinterpret_cast<T*>(r.row);
        t[7 * g.nx + r.x] = sig[r.cell];
        const int si = g.sidx[r.cell];
        reinterpret_cast<uint32_t*>(t + 8 * g.nx)[r.x] = si >= 0 ? (uint32_t)si * (uint32_t)sizeof(T) : QOFF_NONE;
    }
}

hipError_t launch_pack_static(int precision, int nz, const GeomDev* geom_dev, int ncells, hipStream_t st) {
    int blocks = (4 * ncells + 255) / 256;
    blocks = blocks < 1 ? 1 : (blocks > 1024 ? 1024 : blocks);
    (void)hipGetLastError();
    if (nz > 1) {
        if (precision == 1) hipLaunchKernelGGL(k_pack3_static<float>, dim3(blocks), dim3(256), 0, st, geom_dev);
        else hipLaunchKernelGGL(k_pack3_static<double>, dim3(blocks), dim3(256), 0, st, geom_dev);
    } else {
        if (precision == 1) hipLaunchKernelGGL(k_pack_static<float>, dim3(blocks), dim3(256), 0, st, geom_dev);
        else hipLaunchKernelGGL(k_pack_static<double>, dim3(blocks), dim3(256), 0, st, geom_dev);
    }
    return hipGetLastError();
}

hipError_t launch_pack3(int precision, const GeomDev* geoms_dev, int n_geoms, int max_cells, PassParams pp,
                        hipStream_t st) {
    int blocks = (2 * max_cells + 255) / 256;
    blocks = blocks < 1 ? 1 : (blocks > 1024 ? 1024 : blocks);
    (void)hipGetLastError();
    if (precision == 1) hipLaunchKernelGGL(k_pack3<float>, dim3(blocks, n_geoms), dim3(256), 0, st, geoms_dev, pp);
    else hipLaunchKernelGGL(k_pack3<double>, dim3(blocks, n_geoms), dim3(256), 0, st, geoms_dev, pp);
    return hipGetLastError();
}

hipError_t launch_reduce_pass(int precision, const GeomDev* geoms_dev, int n_geoms, int max_solid,
                              PassParams pp, hipStream_t st) {
    int blocks = (max_solid + RC - 1) / RC;
    if (blocks < 1) blocks = 1;
    (void)hipGetLastError();
    if (precision == 1) hipLaunchKernelGGL(k_reduce_pass<float>, dim3(blocks, n_geoms), dim3(64 * RQ), 0, st, geoms_dev, pp);
    else hipLaunchKernelGGL(k_reduce_pass<double>, dim3(blocks, n_geoms), dim3(64 * RQ), 0, st, geoms_dev, pp);
    return hipGetLastError();
}

// Gauge of the outer iteration with a mode table.  The interpolated weights
// do not conserve energy exactly (S_ml is not alpha_ml Lambda_m s_l), so the
// pass map has no fixed point: its iterates drift by a common constant each
// pass, which no conductivity sees.  Removing that drift (the mean lattice
// temperature over the solid cells is set back to 0 after every pass) leaves
// a map with a fixed point, which Anderson mixing and the lagged wrap need.
// The stored wrap inflows stay as they are: re-centred, the next inputs are
// close to this pass's, whose inflows they hold.  ax[n_aa] carries the shift
// from the first kernel to the second.
//
// One block of 1024 threads with eight cells of each in flight: it is its
// loads' latency that counts (96 x 96 cells: 20.5 -> 5 us from 256 threads
// with one).
__global__ void __launch_bounds__(1024) k_gauge_mean(const GeomDev* __restrict__ geoms) {
    __shared__ double red[40];
    const GeomDev& g = geoms[blockIdx.x];
    if (!g.gauge || g.ctrl[CTRL_DONE]) return;
    const auto T = gview(g.T_L);
    const auto fc = gview(g.fc);
    const int nc = g.ncells, bd = blockDim.x;
    double s = 0.0, ns = 0.0;
    for (int c0 = threadIdx.x; c0 < nc; c0 += 8 * bd) {
        double t[8];
        uint16_t w[8];
#pragma unroll
        for (int u = 0; u < 8; ++u) {
            const int c = min(c0 + u * bd, nc - 1);
            t[u] = T[c];
            w[u] = fc[c];
        }
#pragma unroll
        for (int u = 0; u < 8; ++u)
            if (c0 + u * bd < nc && fc_solid(w[u])) {
                s += t[u];
                ns += 1.0;
            }
    }
    block_sum2(s, ns, red);
    if (threadIdx.x == 0) g.ax[g.n_aa] = ns > 0.0 ? s / ns : 0.0;
}

__global__ void __launch_bounds__(256) k_gauge_apply(const GeomDev* __restrict__ geoms) {
    const GeomDev& g = geoms[blockIdx.y];
    if (!g.gauge || g.ctrl[CTRL_DONE]) return;
    const double d = g.ax[g.n_aa];
    const int out = (g.ctrl[CTRL_PASS] + 1) & 1;
    const int nc = g.ncells;
    const int i = blockIdx.x * blockDim.x + threadIdx.x;
    if (i < nc) {
        if (!fc_solid(g.fc[i])) return;
        if (g.aa_m > 0) {
            g.ag[i] -= d;
        } else {
            g.sT[(size_t)out * nc + i] -= g.sigma[i] * d;
            g.ax[i] -= d;
        }
    } else if (i < nc + g.nwalls) {
        const int wi = i - nc;
        if (g.aa_m > 0) {
            g.ag[i] -= d;
        } else {
            g.Tw[(size_t)out * g.nwalls + wi] -= d;
            g.ax[i] -= d;
            g.bnd[((size_t)out * g.nf + g.wall_face[wi]) * nc + g.wall_cell[wi]] -= d;
        }
    }
}

hipError_t launch_gauge(const GeomDev* geoms_dev, int n_geoms, int max_aa, hipStream_t st) {
    (void)hipGetLastError();
    hipLaunchKernelGGL(k_gauge_mean, dim3(n_geoms), dim3(1024), 0, st, geoms_dev);
    hipLaunchKernelGGL(k_gauge_apply, dim3((max_aa + 255) / 256, n_geoms), dim3(256), 0, st, geoms_dev);
    return hipGetLastError();
}

hipError_t launch_finalize(const GeomDev* geoms_dev, int n_geoms, PassParams pp, hipStream_t st) {
    (void)hipGetLastError();
    hipLaunchKernelGGL(k_finalize, dim3(n_geoms), dim3(256), 0, st, geoms_dev, pp);
    return hipGetLastError();
}

// Mode-resolved kappa (paper Eq. mode-resolved, cell-centred form): a gather
// of the per-system sums with each mode's interpolation weights, measured
// from the mean lattice temperature (sum_i T_L,i = sum_ml D_ml sum_i T_iml;
// the weights of a mode add up to 1).  One block: the D-weighted total in a
// fixed-order tree, then the modes strided over the threads.
__global__ void __launch_bounds__(256) k_kappa_modes(const int* __restrict__ sys, const double* __restrict__ w,
                                                     const double* __restrict__ Sg, int n_modes, int terms,
                                                     const double* __restrict__ D, int n_sys,
                                                     const double* __restrict__ kraw, double pref,
                                                     double* __restrict__ out) {
    __shared__ double red[256];
    const int t = threadIdx.x;
    double a = 0.0;
    for (int i = t; i < n_sys; i += 256) a += D[i] * kraw[i];
    red[t] = a;
    __syncthreads();
    for (int h = 128; h > 0; h >>= 1) {
        if (t < h) red[t] += red[t + h];
        __syncthreads();
    }
    const double tot_L = red[0];
    for (int mu = t; mu < n_modes; mu += 256) {
        double s = 0.0;
        for (int k = 0; k < terms; ++k) {
            const double c = w[(size_t)mu * terms + k];
            if (c != 0.0) s += c * kraw[sys[(size_t)mu * terms + k]];
        }
        out[mu] = pref * Sg[mu] * (s - tot_L);
    }
}

hipError_t launch_kappa_modes(const int* sys, const double* w, const double* Sg, int n_modes, int terms,
                              const double* D, int n_sys, const double* kraw, double pref, double* out,
                              hipStream_t st) {
    (void)hipGetLastError();
    hipLaunchKernelGGL(k_kappa_modes, dim3(1), dim3(256), 0, st, sys, w, Sg, n_modes, terms, D, n_sys, kraw,
                       pref, out);
    return hipGetLastError();
}

hipError_t launch_anderson(const GeomDev* geoms_dev, int n_geoms, int max_naa, PassParams pp, hipStream_t st) {
    (void)hipGetLastError();
    int b = (max_naa + AA_THREADS - 1) / AA_THREADS;
    if (b > AAB_MAX) b = AAB_MAX;
    const dim3 grid(b, n_geoms);
    hipLaunchKernelGGL(k_aa_partial, grid, dim3(AA_THREADS), 0, st, geoms_dev);
    hipLaunchKernelGGL(k_aa_apply, grid, dim3(AA_THREADS), 0, st, geoms_dev, pp);
    return hipGetLastError();
}

hipError_t launch_energy(const GeomDev* geom_dev, int precision, int nsolid, hipStream_t st) {
    const int blocks = nsolid > 0 ? (nsolid + 63) / 64 : 1;
    (void)hipGetLastError();
    if (precision == 1) hipLaunchKernelGGL(k_energy<float>, dim3(blocks), dim3(64 * EQ), 0, st, geom_dev);
    else hipLaunchKernelGGL(k_energy<double>, dim3(blocks), dim3(64 * EQ), 0, st, geom_dev);
    hipLaunchKernelGGL(k_energy_finish, dim3(1), dim3(256), 0, st, geom_dev, blocks);
    return hipGetLastError();
}

hipError_t launch_prep_sigma(const GeomDev* g_dev, int ncells, const double* sig, hipStream_t st) {
    int blocks = (ncells + 255) / 256;
    if (blocks > 1024) blocks = 1024;
    (void)hipGetLastError();
    hipLaunchKernelGGL(k_prep_sigma, dim3(blocks), dim3(256), 0, st, g_dev, sig);
    hipLaunchKernelGGL(k_sigma_min, dim3(1), dim3(256), 0, st, g_dev, blocks);
    return hipGetLastError();
}

hipError_t launch_output(const GeomDev* geom_dev, int precision, int ncells, double* T_L_out, double* J_out,
                         double* grad_out, hipStream_t st) {
    (void)hipGetLastError();
    const dim3 grid((ncells + 63) / 64), block(64 * FQ);
    if (T_L_out) hipLaunchKernelGGL(k_output, dim3(1), dim3(1024), 0, st, geom_dev, T_L_out);
    if (J_out) {
        if (precision == 1) hipLaunchKernelGGL(k_flux<float>, grid, block, 0, st, geom_dev, J_out);
        else hipLaunchKernelGGL(k_flux<double>, grid, block, 0, st, geom_dev, J_out);
    }
    if (grad_out) {
        if (precision == 1) hipLaunchKernelGGL(k_grad<float>, grid, block, 0, st, geom_dev, grad_out);
        else hipLaunchKernelGGL(k_grad<double>, grid, block, 0, st, geom_dev, grad_out);
    }
    return hipGetLastError();
}
