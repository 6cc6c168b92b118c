// The 3D pass (see kernels.hip for the method): one wavefront owns one (m, l)
// system and sweeps rows along x, the planes of a y row in z-upwind order.
// The previous y row of every plane is in the wave's LDS, which also brings
// the wrap inflow in (as the row before the first) and the last y row out;
// the row below in z is in registers.  The wrap plane of a system (nx nz
// values) is too large for registers, so its Krylov vectors live in a
// per-system slab of the workspace (KRY3_VECS planes), where every element is
// read and written only by the lane owning its column.
//
// Bound: instruction issue (5 waves per SIMD, about 1.1 instructions per four
// cycles) and, in the first sweep, the store.  With the row's face classes as
// lane masks and constant scan weights (rows.h) a row of 64 FP32 cells takes
// 32 vector instructions where decoding the face words per system and scanning
// Q along took 79.  The pass inputs are laid out in the order the rows are
// swept (two copies, one with the planes reversed: the eight octants walk one
// of them forwards or backwards; a row's values are one block behind one
// advancing resource), so a row takes 27 scalar instructions, 20 of them its
// scan masks (rows.h), where indexing it took 53.  Solutions are stored past
// the caches (non-temporal: the tables stay in the L2).
#pragma once
#include "rows.h"

namespace {

enum { KV_R, KV_E, KV_EB, KV_RH, KV_P, KV_V, KV_S, KV_T, KV_N };
static_assert(KV_N == KRY3_VECS, "workspace carve and kernel disagree on the 3D slab");

template <typename T>
struct Sys3 {
    int sys;
    int neg[3];              // the sweep runs towards - along the axis
    double cd[3];            // Lambda |s_a| / h_a
    T sk, sdm;               // adjoint: constant source and T_L weight
    T mb[3], mo[3];          // weights of the boundary values of the inflow / outflow faces
    double kw, Sg;
};

template <typename T>
__device__ __forceinline__ Sys3<T> make_sys3(const GeomDev& g, int m, int l, int adj) {
    Sys3<T> s;
    s.sys = uni(m * g.n_dir + l);
    const double lam = g.mfp[m];
#pragma unroll
    for (int a = 0; a < 3; ++a) {
        double sa = g.dirs[l * 3 + a];
        if (adj) sa = -sa;   // A_l^T = A_{-l} on a uniform grid
        s.neg[a] = uni(sa > 0.0 ? 0 : 1);
        s.cd[a] = uni(lam * fabs(sa) / g.h[a]);
        s.mb[a] = uni((T)s.cd[a]);
        s.mo[a] = T(0);
        if (adj) {
            // the outgoing wall weight of the face S leaves through (the
            // sweep's inflow face, or with a mode table possibly its outflow
            // face)
            const int f = 2 * a + (g.S[s.sys * 3 + a] > 0.0 ? 1 : 0);
            const T wv = (T)g.wout[(size_t)f * g.n_sys + s.sys];
            const bool in = f == 2 * a + s.neg[a];
            s.mb[a] = uni(in ? wv : T(0));
            s.mo[a] = uni(in ? T(0) : wv);
        }
    }
    s.Sg = g.S[s.sys * 3 + g.grad_axis];
    s.kw = g.L[g.grad_axis] / (g.dT * (double)g.ncells) * s.Sg;
    s.sk = uni((T)s.kw);
    s.sdm = uni((T)g.Dw[s.sys]);
    return s;
}

template <typename T, int CPL, bool ST, bool WITH_B, bool ADJ, bool S1, bool FULL>
struct Sweep3 {
    static constexpr bool ADJB = ADJ && WITH_B;
    static constexpr int ROW = WAVE * CPL;
    static constexpr bool SCAN = S1 && sizeof(T) == 4 && row_mask_scan(CPL, true);
    using Bits = RowBits<CPL, ADJB, true, SCAN>;
    const Sys3<T>& s;
    const QConst<T, CPL, FULL>& k;
    const int lane, nx, ny, nz;
    T* const zl;             // this lane's cells in the wave's LDS rows: plane p at zl + p * ROW
    const rsrc_t X;
    // byte offsets of this lane's cells in a row's block (OOB in the padding):
    // sources, inflow (and outflow) boundary values, sigma, store offset
    uint32_t vs[CPL], vb[3][CPL], vo[3][CPL], vg[CPL], vf[CPL];
    // next row to load (reads run up to two rows past either end of the
    // table, into the slack kept there), its masks
    const char* row;
    long rstep;
    uint32_t rbytes;
    mview_t mask;
    int mstep;
    double kt;
    T xz[CPL];               // the row below in z

    struct In {
        T sb[CPL], b[3][CPL], o[3][CPL], sg[CPL];
        uint32_t so[CPL];
    };

    __device__ __forceinline__ Sweep3(const GeomDev& g, const Sys3<T>& s_, const QConst<T, CPL, FULL>& k_, int lane_, T* zrows,
                                      rsrc_t X_)
        : s(s_), k(k_), lane(lane_), nx(uni(g.nx)), ny(uni(g.ny)), nz(uni(g.nz)), zl(zrows + lane_ * CPL), X(X_) {
        const int zrev = s.neg[1] != s.neg[2], nrows = ny * nz, first = s.neg[1] ? nrows - 1 : 0;
        rbytes = uni(g.q_row3);
#pragma unroll
        for (int c = 0; c < CPL; ++c) {
            const int p = lane * CPL + c - (WAVE * CPL - nx);
            const int cell = s.neg[0] ? nx - 1 - p : p;
            auto at = [&](int field) { return p >= 0 ? (uint32_t)(field * nx + cell) * (uint32_t)sizeof(T) : BUF_OOB; };
            vs[c] = at(0);
#pragma unroll
            for (int a = 0; a < 3; ++a) {
                vb[a][c] = at(1 + 2 * a + s.neg[a]);
                vo[a][c] = at(2 + 2 * a - s.neg[a]);
            }
            vg[c] = at(7);
            vf[c] = p >= 0 ? (uint32_t)(8 * nx) * (uint32_t)sizeof(T) + (uint32_t)cell * 4u : BUF_OOB;
        }
        row = uni(static_cast<const char*>(g.qtab[0]) + ((size_t)zrev * nrows + first) * rbytes);
        rstep = s.neg[1] ? -(long)rbytes : (long)rbytes;
        constexpr int ms = row_mask_words(CPL, true);
        mask = (mview_t)(uni(g.qmask[0]) + (size_t)((s.neg[0] * 4 + s.neg[1] * 2 + zrev) * nrows + first) * ms);
        mstep = s.neg[1] ? -ms : ms;
        kt = 0.0;
    }

    __device__ __forceinline__ void load(In& r) {
        const rsrc_t q = __builtin_amdgcn_make_buffer_rsrc(const_cast<char*>(row), 0, (int)rbytes, 0x00020000);
#pragma unroll
        for (int c = 0; c < CPL; ++c) {
            if (WITH_B) {
                r.sb[c] = bldT<T>(q, vs[c], 0u);
#pragma unroll
                for (int a = 0; a < 3; ++a) {
                    r.b[a][c] = bldT<T>(q, vb[a][c], 0u);
                    if (ADJB) r.o[a][c] = bldT<T>(q, vo[a][c], 0u);
                }
            }
            if (!S1) r.sg[c] = bldT<T>(q, vg[c], 0u);
            if (ST) {
                r.so[c] = bld32(q, vf[c], 0u);
                if (!FULL) r.so[c] |= vf[c] & BUF_OOB;
            }
        }
        row += rstep;
    }
    __device__ __forceinline__ void bits(Bits& m) {
        load_bits(mask, m);
        mask += mstep;
    }
    __device__ __forceinline__ T source(const In& r, const Bits& m, int c, T ksb, const T (&kb)[3], const T (&ko)[3], T kk) const {
        T a;
        if (ADJB) {
            a = kk + ksb * r.sb[c];
#pragma unroll
            for (int x = 0; x < 3; ++x) a += kb[x] * r.b[x][c] + ko[x] * r.o[x][c];
            a = sel0(m.sol[c], a);
        } else {
            a = ksb * r.sb[c];
#pragma unroll
            for (int x = 0; x < 3; ++x) a += kb[x] * r.b[x][c];
        }
        return a;
    }
    __device__ __forceinline__ void finish_row(const T (&a)[CPL], const T (&q)[CPL], T xp, const In& r, T* zr) {
#pragma unroll
        for (int c = 0; c < CPL; ++c) {
            xp = a[c] + q[c] * xp;
            xz[c] = xp;
            zr[c] = xp;
        }
        if (ST) {
            T t = FULL ? xz[0] : k.val[0] * xz[0];
#pragma unroll
            for (int c = 1; c < CPL; ++c) t = FULL ? t + xz[c] : t + k.val[c] * xz[c];
            kt += (double)t;
#pragma unroll
            for (int c = 0; c < CPL; ++c) bst_nt(xz[c], X, r.so[c]);
        }
    }

    // Rows are read two ahead in a rotation of three buffers and their masks
    // one ahead, with no load and no store inside a branch; the y neighbours
    // of the next row are read from LDS before this row's chain.
    __device__ __forceinline__ void run() {
#pragma unroll
        for (int c = 0; c < CPL; ++c) xz[c] = T(0);
        const int nrows = ny * nz;
        const char* const row0 = row;
        const mview_t mask0 = mask;
        In b0, b1, b2;
        load(b0);
        load(b1);
        T py[CPL];
#pragma unroll
        for (int c = 0; c < CPL; ++c) py[c] = zl[c];
        int r = 0, pc = 0;
        // LDS row of the next solved row, read ahead; this row's address
        auto advance = [&](T (&pn)[CPL]) -> T* {
            T* zr = zl + pc;
            pc = pc + ROW == nz * ROW ? 0 : pc + ROW;
            const T* zn = zl + pc;
#pragma unroll
            for (int c = 0; c < CPL; ++c) pn[c] = zn[c];
            return zr;
        };
        if constexpr (S1) {
            const T rdv = k.rdv;
            const T ky = (T)s.cd[1] * rdv, kz = (T)s.cd[2] * rdv, kk = s.sk * rdv, ksb = ADJ ? s.sdm * rdv : rdv;
            const T kb[3] = {s.mb[0] * rdv, s.mb[1] * rdv, s.mb[2] * rdv};
            const T ko[3] = {s.mo[0] * rdv, s.mo[1] * rdv, s.mo[2] * rdv};
            // the bits of this row and the next, this row's scan masks: the
            // next row's are formed while its chain runs
            Bits m, m1;
            ScanMask sm;
            bits(m);
            if constexpr (!SCAN) bits(m1);
            scan_mask(m, sm);
            auto one = [&](const In& in, In& fill) {
                Bits n;
                bits(n);
                ScanMask sn;
                scan_mask(SCAN ? n : m1, sn);
                load(fill);
                T pn[CPL];
                T* zr = advance(pn);
                T a[CPL], q[CPL];
                T Al;
#pragma unroll
                for (int c = 0; c < CPL; ++c) {
                    a[c] = ky * sel0(m.yo[c], py[c]) + kz * sel0(m.zo[c], xz[c]);
                    if (WITH_B) a[c] += source(in, m, c, ksb, kb, ko, kk);
                    q[c] = sel0(m.xo[c], FULL ? k.q : k.qc[FULL ? 0 : c]);
                    Al = c == 0 ? a[c] : a[c] + q[c] * Al;
                }
                T A = Al;
                const T om = ascan(A, k, sm);
                const T xin = readlane(A, WAVE - 1) * (lane_in(sm.nb) ? k.rpt : T(1));
                const T xe = A + om * xin;
                finish_row(a, q, dpp<0x138, 0xf>(xe, xin), in, zr);      // wave_shr:1
#pragma unroll
                for (int c = 0; c < CPL; ++c) py[c] = pn[c];
                m = SCAN ? n : m1;
                m1 = n;
                sm = sn;
            };
            if (nrows >= 3) {
                one(b0, b2);
                one(b1, b0);
                one(b2, b1);
                for (r = 3; r + 3 <= nrows; r += 3) {
                    one(b0, b2);
                    one(b1, b0);
                    one(b2, b1);
                }
            }
            if (r < nrows) one(b0, b2);
            if (r + 1 < nrows) one(b1, b0);
        } else {
            const T c0 = (T)s.cd[0], cr = (T)(s.cd[1] + s.cd[2]), cy = (T)s.cd[1], cz = (T)s.cd[2];
            Bits m0, m1;
            QPart<T, CPL> p0, p1;
            bits(m0);
            bits(m1);
            {
                T P = qpart_cells(c0, cr, k, m0, b0.sg, p0);
                pscan(P, p0.t);
                qpart_close<T, CPL>(P, p0);
            }
            auto one = [&](const In& in, const In& nxt, In& fill) {
                load(fill);
                Bits n;
                bits(n);
                T pn[CPL];
                T* zr = advance(pn);
                T Pn = qpart_cells(c0, cr, k, m1, nxt.sg, p1);
                T a[CPL];
                T Al;
#pragma unroll
                for (int c = 0; c < CPL; ++c) {
                    a[c] = cy * sel0(m0.yo[c], py[c]) + cz * sel0(m0.zo[c], xz[c]);
                    if (WITH_B) a[c] += source(in, m0, c, ADJ ? s.sdm : T(1), s.mb, s.mo, s.sk);
                    a[c] *= p0.rdv[c];
                    Al = c == 0 ? a[c] : a[c] + p0.q[c] * Al;
                }
                T A = Al;
                scan_pair(A, p0.t, Pn, p1.t);
                qpart_close<T, CPL>(Pn, p1);
                const T xin = readlane(A, WAVE - 1) * p0.rPt;
                const T xe = A + p0.omP * xin;
                finish_row(a, p0.q, dpp<0x138, 0xf>(xe, xin), in, zr);
#pragma unroll
                for (int c = 0; c < CPL; ++c) py[c] = pn[c];
                m0 = m1;
                m1 = n;
                p0 = p1;
            };
            if (nrows >= 3) {
                one(b0, b1, b2);
                one(b1, b2, b0);
                one(b2, b0, b1);
                for (r = 3; r + 3 <= nrows; r += 3) {
                    one(b0, b1, b2);
                    one(b1, b2, b0);
                    one(b2, b0, b1);
                }
            }
            if (r < nrows) one(b0, b1, b2);
            if (r + 1 < nrows) one(b1, b2, b0);
        }
        row = row0;              // the wrap solve runs its sweeps from one view
        mask = mask0;
    }
};

// every element of the wrap plane this lane owns: plane kp, cell c, index i,
// value z of the wave's LDS row
#define PLOOP(body)                                            \
    for (int kp = 0; kp < nz; ++kp)                            \
        _Pragma("unroll") for (int c = 0; c < CPL; ++c) {      \
            if (p0 + c >= 0) {                                 \
                const int i = kp * nx + p0 + c;                \
                [[maybe_unused]] T& z = zrows[kp * WAVE * CPL + lane * CPL + c]; \
                body;                                          \
            }                                                  \
        }

template <typename T, int CPL, int ADJ, int SIG1, bool FULL>
__global__ void __launch_bounds__(512) __attribute__((amdgpu_waves_per_eu(CPL == 1 ? (sizeof(T) == 4 ? 5 : 4) : 1))) k_sweep_pass3(const GeomDev* __restrict__ geoms,
                                                     const Item* __restrict__ items, int n_items,
                                                     PassParams pp) {
    extern __shared__ double lds[];
    const int it = blockIdx.x;
    if (it >= n_items) return;
    const Item item = items[it];
    const GeomDev& g = geoms[item.geom];
    if (pp.mode == 0 && g.ctrl[CTRL_DONE]) return;
    // the wave index is wave-uniform: read it into a scalar so that every
    // per-system quantity (and the buffer resources built from it) is too
    const int lane = threadIdx.x & 63, w = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int m = item.m0 + w;
    // inactive waves leave: the waves of a group never wait for each other
    if (!(w < item.nm && m < g.n_mfp)) return;
    constexpr int adj = ADJ;
    const Sys3<T> s = make_sys3<T>(g, m, item.l, adj);
    const int nx = g.nx, nz = g.nz, nw = g.nwrap;
    QConst<T, CPL, FULL> qk;
    make_qconst<T, CPL, SIG1 != 0, FULL>(s.cd[0], s.cd[1] + s.cd[2], nx, lane, qk);
    const size_t half = adj ? (size_t)g.n_sys : 0;
    const gmut_t<T> U = gmut(reinterpret_cast<T*>(g.U) + (half + s.sys) * (size_t)nw);
    const gmut_t<T> K = gmut(reinterpret_cast<T*>(g.kry) + (size_t)s.sys * KRY3_VECS * nw);
    T* zrows = reinterpret_cast<T*>(lds) + (size_t)w * nz * WAVE * CPL;
    const rsrc_t X = make_rsrc(reinterpret_cast<T*>(g.X) + (size_t)s.sys * g.xs, (uint32_t)g.nsolid * (uint32_t)sizeof(T));
    const int p0 = lane * CPL - (WAVE * CPL - nx);       // row position of this lane's first cell
    // pairs across the wrap: the first y row's inflow along y (its nz rows are
    // the first swept)
    const int mstep = s.neg[1] ? -row_mask_words(CPL, true) : row_mask_words(CPL, true);
    const mview_t mrow = (mview_t)(uni(g.qmask[0]) + (size_t)((s.neg[0] * 4 + s.neg[1] * 2 + (s.neg[1] != s.neg[2])) * g.ny * nz +
                                                              (s.neg[1] ? g.ny * nz - 1 : 0)) * row_mask_words(CPL, true));
    auto open = [&](int kp, int c) { return lane_in(mrow[(long)kp * mstep + CPL + c]); };
    const bool has_wrap = g.periodic[1] != 0;
    long long n_it = 0, n_sw = 0;
    int need = 0;
    double kt = 0.0;
    for (int round = 0;; ++round) {
        // ---- phase A
        PLOOP(z = U[i]);
        {
            Sweep3<T, CPL, true, true, ADJ != 0, SIG1 != 0, FULL> a(g, s, qk, lane, zrows, X);
            a.run();
            kt = a.kt;
        }
        ++n_sw;
        if (round > 0 || pp.mode != 0 || !has_wrap) break;
        // ---- phase B: the residual of the wrap system (in units of the
        // solution) and its correction
        const gmut_t<T> r = K + (size_t)KV_R * nw;
        const gmut_t<T> e = K + (size_t)KV_E * nw;
        const gmut_t<T> eb = K + (size_t)KV_EB * nw;
        const gmut_t<T> rh = K + (size_t)KV_RH * nw;
        const gmut_t<T> p = K + (size_t)KV_P * nw;
        const gmut_t<T> v = K + (size_t)KV_V * nw;
        const gmut_t<T> sv = K + (size_t)KV_S * nw;
        const gmut_t<T> t = K + (size_t)KV_T * nw;
        double ss = 0.0, rr = 0.0;
        PLOOP({
            const T ez = open(kp, c) ? z : T(0);
            const T rv = ez - U[i];
            r[i] = rv;
            ss += (double)ez * (double)ez;
            rr += (double)rv * (double)rv;
        });
        const double scale = sqrt(wave_sum(ss));
        rr = wave_sum(rr);
        double rn = sqrt(rr);
        const double thr = fmax(pp.inner_tol * scale, pp.inner_rtol * rn);
        const double thr_final = pp.inner_tol * scale;
        if (rn > thr_final && scale > 0.0) need = 1;
        const double rho_g = wrap_gain_bound(g.fscal[5], s.cd[1], g.ny);
        if (rn > thr && scale > 0.0 && rho_g * rn <= fmin(thr, fmax(thr_final, RICH_MAX * rn))) {
            // weakly coupled wrap: e = r, no sweep (as in 2D)
            PLOOP(U[i] += r[i]);
            rn = rho_g * rn;
        } else if (rn > thr && scale > 0.0) {
            // BiCGSTAB on (I - G) e = r with the best iterate kept (as in 2D).
            // Most systems are done after the first sweep (p = r, e = alpha
            // r): until then only r is in the slab, A p is taken from the
            // sweep's last row in LDS, and the other vectors are written
            // when the second half needs them.
            double best = rn;
            int restarts = 0;
            double rho_old = 1.0, alpha = 1.0, omega = 1.0;
            bool done = false;
            Sweep3<T, CPL, false, false, ADJ != 0, SIG1 != 0, FULL> h(g, s, qk, lane, zrows, X);
            for (int iter = 0; iter < pp.max_inner; ++iter) {
                const bool first = iter == 0;
                double acc = 0.0, rho = rr;
                if (first) {
                    PLOOP(z = r[i]);
                } else {
                    PLOOP(acc += (double)rh[i] * (double)r[i]);
                    rho = wave_sum(acc);
                    if (fabs(rho) <= 1e-30 * rn * rn || !(omega != 0.0)) {
                        acc = 0.0;
                        PLOOP({ rh[i] = r[i]; p[i] = T(0); v[i] = T(0); acc += (double)r[i] * (double)r[i]; });
                        rho = wave_sum(acc);
                        rho_old = 1.0; alpha = 1.0; omega = 1.0;
                    }
                    const double beta = (rho / rho_old) * (alpha / omega);
                    PLOOP({ z = r[i] + (T)beta * (p[i] - (T)omega * v[i]); p[i] = z; });
                }
                h.run();
                ++n_sw;
                acc = 0.0;
                if (first) {
                    PLOOP({
                        const T x = r[i];
                        acc += (double)x * (double)(x - (open(kp, c) ? z : T(0)));
                    });
                } else {
                    PLOOP({
                        const T vv = p[i] - (open(kp, c) ? z : T(0));
                        v[i] = vv;
                        acc += (double)rh[i] * (double)vv;
                    });
                }
                const double rv = wave_sum(acc);
                if (!isfinite(rv)) {
                    done = first;
                    break;
                }
                if (!(fabs(rv) > 1e-30 * fabs(rho))) {
                    if (restarts++ >= 4) break;
                    omega = 0.0;
                    if (first) PLOOP({ e[i] = T(0); eb[i] = T(0); rh[i] = r[i]; p[i] = T(0); v[i] = T(0); });
                    continue;
                }
                alpha = rho / rv;
                acc = 0.0;
                if (first) {
                    PLOOP({
                        const T x = r[i];
                        const T y = x - (T)alpha * (x - (open(kp, c) ? z : T(0)));
                        acc += (double)y * (double)y;
                    });
                } else {
                    PLOOP({
                        const T x = r[i] - (T)alpha * v[i];
                        sv[i] = x;
                        z = x;
                        acc += (double)x * (double)x;
                    });
                }
                const double sn = sqrt(wave_sum(acc));
                ++n_it;
                if (sn <= thr) {
                    if (sn < best) {
                        best = sn;
                        if (first) {
                            PLOOP(U[i] += (T)alpha * r[i]);
                        } else {
                            PLOOP(eb[i] = e[i] + (T)alpha * p[i]);
                        }
                    }
                    done = first;
                    break;
                }
                if (first) {
                    PLOOP({
                        const T x = r[i];
                        const T vv = x - (open(kp, c) ? z : T(0));
                        e[i] = T(0);
                        eb[i] = T(0);
                        rh[i] = x;
                        p[i] = x;
                        v[i] = vv;
                        const T y = x - (T)alpha * vv;
                        sv[i] = y;
                        z = y;
                    });
                }
                h.run();
                ++n_sw;
                double tt = 0.0, ts = 0.0;
                PLOOP({
                    const T x = sv[i] - (open(kp, c) ? z : T(0));
                    t[i] = x;
                    tt += (double)x * (double)x;
                    ts += (double)x * (double)sv[i];
                });
                tt = wave_sum(tt);
                ts = wave_sum(ts);
                omega = tt > 0.0 ? ts / tt : 0.0;
                acc = 0.0;
                PLOOP({
                    e[i] += (T)alpha * p[i] + (T)omega * sv[i];
                    const T x = sv[i] - (T)omega * t[i];
                    r[i] = x;
                    acc += (double)x * (double)x;
                });
                rn = sqrt(wave_sum(acc));
                rho_old = rho;
                if (!isfinite(rn)) break;
                if (rn < best) {
                    best = rn;
                    PLOOP(eb[i] = e[i]);
                }
                if (rn <= thr) break;
            }
            rn = best;
            if (!done && n_sw > 1) PLOOP(U[i] += eb[i]);
        }
        if (lane == 0) g.wres[s.sys] = scale > 0.0 ? rn / scale : 0.0;
        // ---- the solution for the corrected inflow (skipped when the
        // correction is lagged into the next pass)
        if (pp.lag_wrap || !need) break;
    }
    // kappa sums (see the 2D kernel)
    __builtin_amdgcn_fence(__ATOMIC_SEQ_CST, "workgroup");
    const bool ga0 = g.grad_axis == 0;
    const bool pos = !(ga0 ? s.neg[0] : s.neg[1]);
    const int np = g.n_plane[pos ? 1 : 0];
    const int* plane = pos ? g.plane[1] : g.plane[0];
    double kf = 0.0;
    for (int i = lane; i < np; i += WAVE) kf += (double)bldT<T>(X, (uint32_t)plane[i] * (uint32_t)sizeof(T), 0u);
    const double ks = wave_sum(kt);
    kf = wave_sum(kf);
    if (lane == 0) {
        if (adj) {
            g.ksys[s.sys] = kf * ((pos ? -1.0 : 1.0) * (ga0 ? s.cd[0] : s.cd[1]) * g.dT);
            g.kfsys[s.sys] = 0.0;
        } else {
            if (pos) kf += g.dT * (double)np;
            g.kraw[s.sys] = ks;
            g.ksys[s.sys] = g.L[g.grad_axis] / (g.dT * (double)g.ncells) * s.Sg * ks;
            g.kfsys[s.sys] = g.L[g.grad_axis] / (g.dT * (double)g.n_perp) * s.Sg * kf;
        }
        if (pp.mode == 0) {
            g.iters[s.sys] += n_it;
            g.sweeps[s.sys] += n_sw;
        }
    }
}
#undef PLOOP

}  // namespace

template <typename T, int CPL, bool FULL>
static hipError_t launch_sweep3_f(const GeomDev* g, const Item* it, int n, int waves, PassParams pp,
                                  size_t lds, hipStream_t st) {
    (void)hipGetLastError();
    const dim3 grid(n), block(64 * waves);
    if (pp.adjoint) {
        if (pp.sigma1) hipLaunchKernelGGL((k_sweep_pass3<T, CPL, 1, 1, FULL>), grid, block, lds, st, g, it, n, pp);
        else hipLaunchKernelGGL((k_sweep_pass3<T, CPL, 1, 0, FULL>), grid, block, lds, st, g, it, n, pp);
    } else {
        if (pp.sigma1) hipLaunchKernelGGL((k_sweep_pass3<T, CPL, 0, 1, FULL>), grid, block, lds, st, g, it, n, pp);
        else hipLaunchKernelGGL((k_sweep_pass3<T, CPL, 0, 0, FULL>), grid, block, lds, st, g, it, n, pp);
    }
    return hipGetLastError();
}

template <typename T, int CPL>
hipError_t launch_sweep3(const GeomDev* g, const Item* it, int n, int waves, PassParams pp, size_t lds, hipStream_t st,
                         int full) {
    return full ? launch_sweep3_f<T, CPL, true>(g, it, n, waves, pp, lds, st)
                : launch_sweep3_f<T, CPL, false>(g, it, n, waves, pp, lds, st);
}
