// The 2D pass (see kernels.hip for the method): one wavefront owns one (m, l)
// system, sweeps its rows in upwind order, corrects its periodic inflow and
// leaves its solution on the solid cells.
//
// Rows run along x, or along y ("transposed"), whichever axis the direction
// crosses more often (obte_internal.h, transposed()): a row's own periodic
// closure is exact, so the coupling left to the Krylov solve is the one
// across the rows.  With rows along x for every direction the ones near y
// crossed the wrap up to 15 times per pass of the other axis, their wrap map
// was close to a shift, and they took 8 to 14 sweeps per pass where the
// median system takes 2; a pass lasts as long as its longest system (128 x
// 128 cells, 48 directions x 30 MFPs, FP32, with the lane masks: 198 -> 72 us a
// launch, 69 us with the scan's masks formed from the open lanes).
//
// What every system of an orientation reads of a row is the same, so it is
// laid out once per pass in the row's order (k_pack_rows): a lane's cells are
// consecutive.  Rows are right-aligned on the lanes (the last cell is lane
// 63's last), padded in front to a multiple of the cells per lane; padding
// holds zeros.
#pragma once
#include "rows.h"

namespace {

// ---------------------------------------------------------------------------
// one system's view of the pass
// ---------------------------------------------------------------------------
template <typename T>
struct Sys2 {
    int sys, m, l, tr;
    int negr, negw;          // the sweep runs towards - along the rows / across them
    int nr, nw, rs;          // cells of a row, rows, records per row
    int nx;
    double c0, c1;           // Lambda |s_a| / h_a along the rows / across them
    T sk, sdm;               // adjoint: constant source and T_L weight
    T mb0, mb1, mo0, mo1;    // weights of the boundary values of the inflow / outflow faces
    double kw, Sg;
    int pos_ga;              // the sweep runs towards + along the gradient axis
    double cga;              // Lambda |s_g| / h_g
};

template <typename T>
__device__ __forceinline__ Sys2<T> make_sys2(const GeomDev& g, int m, int l, int tr, int adj) {
    Sys2<T> s;
    s.m = uni(m);
    s.l = uni(l);
    s.tr = uni(tr);
    s.sys = s.m * g.n_dir + s.l;
    const double lam = g.mfp[s.m];
    double sx = g.dirs[s.l * 3], sy = g.dirs[s.l * 3 + 1];
    if (adj) { sx = -sx; sy = -sy; }          // A_l^T = A_{-l} on a uniform grid
    const double cx = lam * fabs(sx) / g.h[0], cy = lam * fabs(sy) / g.h[1];
    const int nx_ = sx > 0.0 ? 0 : 1, ny_ = sy > 0.0 ? 0 : 1;
    s.negr = uni(s.tr ? ny_ : nx_);
    s.negw = uni(s.tr ? nx_ : ny_);
    s.c0 = uni(s.tr ? cy : cx);
    s.c1 = uni(s.tr ? cx : cy);
    s.nx = uni(g.nx);
    s.nr = uni(s.tr ? g.ny : g.nx);
    s.nw = uni(s.tr ? g.nx : g.ny);
    s.rs = uni(s.tr ? g.q_rs[1] : g.q_rs[0]);
    const double S0 = g.S[s.sys * 3], S1 = g.S[s.sys * 3 + 1];
    s.Sg = g.grad_axis == 0 ? S0 : S1;
    s.kw = g.L[g.grad_axis] / (g.dT * (double)g.ncells) * s.Sg;
    s.pos_ga = g.grad_axis == 0 ? !nx_ : !ny_;
    s.cga = g.grad_axis == 0 ? cx : cy;
    if (!adj) {
        s.mb0 = uni((T)s.c0);
        s.mb1 = uni((T)s.c1);
        s.mo0 = s.mo1 = s.sk = s.sdm = T(0);
    } else {
        // the outgoing wall weight of the face S leaves through (the sweep's
        // inflow face, or with a mode table possibly its outflow face)
        const int fx = S0 > 0.0 ? 1 : 0, fy = 2 + (S1 > 0.0 ? 1 : 0);
        const T wx = (T)g.wout[fx * g.n_sys + s.sys], wy = (T)g.wout[fy * g.n_sys + s.sys];
        const bool inx = fx == nx_, iny = fy == 2 + ny_;
        const T bx = inx ? wx : T(0), ox = inx ? T(0) : wx, by = iny ? wy : T(0), oy = iny ? T(0) : wy;
        s.mb0 = uni(s.tr ? by : bx);
        s.mb1 = uni(s.tr ? bx : by);
        s.mo0 = uni(s.tr ? oy : ox);
        s.mo1 = uni(s.tr ? ox : oy);
        s.sk = uni((T)s.kw);
        s.sdm = uni((T)g.Dw[s.sys]);
    }
    return s;
}

// buffer resources and lane offsets of a sweep
template <typename T, int CPL>
struct Views2 {
    rsrc_t sb, br, bw, bro, bwo, sg, off;
    uint32_t vT, v4;         // byte offsets of this lane's first record within a row
    // running scalars, advanced row by row (reads run up to three rows past
    // either end of a table, into the slack kept there): byte offsets of the
    // next row to load and their steps, the next row's masks
    uint32_t oT, sT, o4, s4;
    mview_t mask;
    int mstep;
    // transposed stores: this lane's place in a flush, the table offset of the
    // next flush step and its steps (bytes)
    int lv, lp, j;
    int fb, fstep, fbatch;
};

template <typename T, int CPL>
struct QIn {
    T sb[CPL], br[CPL], bw[CPL], bro[CPL], bwo[CPL], sg[CPL];
    uint32_t so[CPL];
};

// Transposed stores.  A lane holds cells of one column, whose solid indices
// lie a grid row apart, so the columns are staged in LDS and stored RB at a
// time: 64 / RB grid rows of RB neighbouring cells per store (32-byte runs;
// the L2 joins the runs of neighbouring batches).  Two batches alternate, and
// the stores of one are spread over the row steps of the next, so they add
// one LDS read and one table read per store to a direct store's cost.
template <typename T>
constexpr int tr_rb() { return 32 / (int)sizeof(T); }
// row of a staged column: 4 words (mod 32) apart for RB = 8, 4 doubles (mod
// 16) for RB = 4, so that a flush's reads of RB columns x 64/RB rows spread
// over the banks
template <int CPL>
constexpr int tr_ls() { return 64 * CPL + 4; }

template <typename T, int CPL, int ST, bool WITH_B, bool ADJ, bool S1, bool FULL>
struct Sweep2 {
    static constexpr int RB = tr_rb<T>(), PB = WAVE / RB, LS = tr_ls<CPL>();
    static constexpr bool ADJB = ADJ && WITH_B;
    using Bits = RowBits<CPL, ADJB>;
    const GeomDev& g;
    const Sys2<T>& s;
    const QConst<T, CPL, FULL>& k;
    const int lane;
    T* tile;
    rsrc_t X;
    Views2<T, CPL> v;
    T kt;
    T y[CPL];                // the row below (wrap inflow before the first row)

    __device__ __forceinline__ Sweep2(const GeomDev& g_, const Sys2<T>& s_, const QConst<T, CPL, FULL>& k_, int lane_,
                                      T* tile_, rsrc_t X_)
        : g(g_), s(s_), k(k_), lane(lane_), tile(tile_), X(X_) {
        const size_t nrec = (size_t)s.nw * s.rs, lead = (size_t)ROW_SLACK * s.rs;
        const uint32_t bytes = uni((uint32_t)((nrec + 2 * lead) * sizeof(T)));
        const T* base = static_cast<const T*>(s.tr ? g.qtab[1] : g.qtab[0]) + (size_t)s.negr * 6 * nrec - lead;
        v.sb = make_rsrc(base, bytes);
        v.br = make_rsrc(base + nrec, bytes);
        v.bw = make_rsrc(base + (2 + s.negw) * nrec, bytes);
        if (ADJB) {
            v.bwo = make_rsrc(base + (3 - s.negw) * nrec, bytes);
            v.bro = make_rsrc(base + 4 * nrec, bytes);
        }
        if (!S1) v.sg = make_rsrc(base + 5 * nrec, bytes);
        if (ST == 1) v.off = make_rsrc(g.qoff + (size_t)s.negr * nrec - lead, uni((uint32_t)((nrec + 2 * lead) * 4)));
        if (ST == 2) v.off = make_rsrc(g.qoffc - OFF_SLACK, uni((uint32_t)(g.ncells + 2 * OFF_SLACK) * 4u));
        const int rec = FULL ? lane * CPL : lane * CPL - (WAVE * CPL - s.rs);   // < 0 (out of range) ahead of the row
        v.vT = (uint32_t)rec * (uint32_t)sizeof(T);
        v.v4 = (uint32_t)rec * 4u;
        if (!FULL && rec < 0) { v.vT = BUF_OOB; v.v4 = BUF_OOB; }
        const int first = s.negw ? s.nw - 1 : 0;
        v.oT = uni((uint32_t)((first + ROW_SLACK) * s.rs) * (uint32_t)sizeof(T));
        v.o4 = uni((uint32_t)((first + ROW_SLACK) * s.rs) * 4u);
        v.sT = uni((uint32_t)(s.negw ? -s.rs : s.rs) * (uint32_t)sizeof(T));
        v.s4 = uni((uint32_t)(s.negw ? -s.rs : s.rs) * 4u);
        constexpr int ms = row_mask_words(CPL, false);
        v.mask = (mview_t)(uni(s.tr ? g.qmask[1] : g.qmask[0]) + (size_t)((2 * s.negr + s.negw) * s.nw + first) * ms);
        v.mstep = s.negw ? -ms : ms;
        if (ST == 2) {
            v.j = lane % RB;
            v.lp = lane / RB;
            v.lv = ((s.negw ? RB - 1 - v.j : v.j) + (s.negr ? PB - 1 - v.lp : v.lp) * s.nx) * 4;
            v.fb = uni(flush_base(-RB, 0) * 4);          // no batch during the first RB rows: nothing is stored
            v.fstep = uni((s.negr ? -PB : PB) * s.nx * 4);
            v.fbatch = uni((s.negw ? -RB : RB) * 4 - RB * CPL * v.fstep);
        }
        kt = T(0);
    }

    // table index (cells, from OFF_SLACK before the first) of lane 0's place
    // in flush step `it` of the batch whose first sweep row is j0
    __device__ __forceinline__ int flush_base(int j0, int it) const {
        const int pad = WAVE * CPL - s.nr;
        const int p = s.negr ? s.nr - 1 + pad - it * PB - (PB - 1) : it * PB - pad;
        return p * s.nx + (s.negw ? s.nw - RB - j0 : j0) + OFF_SLACK;
    }
    // store offsets of the flush steps of row jj (of the previous batch);
    // start: jj may be the first row of a batch.  As loaded: what depends on
    // the value waits for it, and is done by the store.
    __device__ __forceinline__ void load_flush(int jj, bool start, uint32_t (&so)[CPL]) {
        if (start) v.fb += (jj & (RB - 1)) == 0 ? v.fbatch : 0;
#pragma unroll
        for (int c = 0; c < CPL; ++c) {
            so[c] = FULL ? bld32(v.off, (uint32_t)v.lv, (uint32_t)v.fb) : bld32(v.off, (uint32_t)(v.lv + v.fb), 0u);
            v.fb += v.fstep;
        }
    }
    __device__ __forceinline__ void flush(int jj, int q, const uint32_t (&so)[CPL]) const {
        // jj: first row of the group of four, q: row within it
        const T* src = tile + (((jj / RB) & 1) ^ 1) * RB * LS + v.j * LS + v.lp + (jj & (RB - 1)) * CPL * PB;
#pragma unroll
        for (int c = 0; c < CPL; ++c) {
            const int p = (((jj & (RB - 1)) + q) * CPL + c) * PB + v.lp - (WAVE * CPL - s.nr);
            const uint32_t o = FULL || (p >= 0 && p < s.nr) ? so[c] : QOFF_NONE;
            bst(src[(q * CPL + c) * PB], X, o | (jj >= RB ? 0u : BUF_OOB));      // no batch before the first
        }
    }
    // after the last row: what is left of the last full batch, and the last one
    __device__ __forceinline__ void drain() const {
        const int nb = (s.nw + RB - 1) / RB;
        for (int jj = s.nw; jj < (nb + 1) * RB; ++jj) {
            const int b = jj / RB - 1, rib = jj & (RB - 1);
            if (b < 0) continue;
            const int row = b * RB + v.j;                    // sweep row of this lane's column
            const T* src = tile + (b & 1) * RB * LS + v.j * LS + v.lp + rib * CPL * PB;
            uint32_t so[CPL];
#pragma unroll
            for (int c = 0; c < CPL; ++c) {
                const int it = rib * CPL + c;
                const int p = it * PB + v.lp - (WAVE * CPL - s.nr);
                const bool in = row < s.nw && p >= 0 && p < s.nr;
                so[c] = bld32(v.off, in ? (uint32_t)(v.lv + flush_base(b * RB, it) * 4) : BUF_OOB, 0u);
                so[c] = in ? so[c] : QOFF_NONE;
            }
#pragma unroll
            for (int c = 0; c < CPL; ++c) bst(src[c * PB], X, so[c]);
        }
    }

    // inputs of the next row, sweep row j (past the last row: unused)
    __device__ __forceinline__ void load(int j, bool start, QIn<T, CPL>& b) {
        if (WITH_B) {
            bld_T<T, CPL>(b.sb, v.sb, v.vT, v.oT);
            bld_T<T, CPL>(b.br, v.br, v.vT, v.oT);
            bld_T<T, CPL>(b.bw, v.bw, v.vT, v.oT);
            if (ADJB) {
                bld_T<T, CPL>(b.bro, v.bro, v.vT, v.oT);
                bld_T<T, CPL>(b.bwo, v.bwo, v.vT, v.oT);
            }
        }
        if (!S1) bld_T<T, CPL>(b.sg, v.sg, v.vT, v.oT);
        v.oT += v.sT;
        if (ST == 1) {
            bld_dw<CPL>(b.so, v.off, v.v4, v.o4);
            v.o4 += v.s4;
        }
        if (ST == 2) load_flush(j, start, b.so);
    }
    __device__ __forceinline__ void bits(Bits& m) {
        load_bits(v.mask, m);
        v.mask += v.mstep;
    }

    // the part of the right-hand side that does not come from the row below
    __device__ __forceinline__ T source(const QIn<T, CPL>& b, const Bits& m, int c, T ksb, T k0, T k1, T o0, T o1,
                                        T kk) const {
        T a;
        if (ADJB) {
            a = kk + ksb * b.sb[c];
            a += k0 * b.br[c] + k1 * b.bw[c];
            a += o0 * b.bro[c] + o1 * b.bwo[c];
            a = sel0(m.sol[c], a);
        } else {
            a = ksb * b.sb[c];
            a += k0 * b.br[c];
            a += k1 * b.bw[c];
        }
        return a;
    }

    // x of one row from its affine parts; leaves the row in y
    __device__ __forceinline__ void finish_row(const T (&a)[CPL], const T (&q)[CPL], T xp, const QIn<T, CPL>& b, int jj,
                                               int qr) {
#pragma unroll
        for (int c = 0; c < CPL; ++c) {
            xp = a[c] + q[c] * xp;
            y[c] = xp;
        }
        if (ST) {
            T r = FULL ? y[0] : k.val[0] * y[0];
#pragma unroll
            for (int c = 1; c < CPL; ++c) r = FULL ? r + y[c] : r + k.val[c] * y[c];
            kt += r;
        }
        if (ST == 1) {
#pragma unroll
            for (int c = 0; c < CPL; ++c) bst(y[c], X, FULL ? b.so[c] : b.so[c] | (v.v4 & BUF_OOB));   // lanes ahead of the row
        }
        if (ST == 2) {
            T* dst = tile + ((jj / RB) & 1) * RB * LS + (jj & (RB - 1)) * LS + qr * LS + lane * CPL;
#pragma unroll
            for (int c = 0; c < CPL; ++c) dst[c] = y[c];
            flush(jj, qr, b.so);
        }
    }

    // sigma = 1: row jj + qr (jj: its group of four) with its masks
    __device__ __forceinline__ void step(const QIn<T, CPL>& b, const Bits& m, const ScanMask& sm, int jj, int qr, T kc1, T kb0, T kb1, T ko0,
                                         T ko1, T ksb, T kk) {
        T a[CPL], q[CPL];
        T Al;
#pragma unroll
        for (int c = 0; c < CPL; ++c) {
            a[c] = kc1 * sel0(m.yo[c], y[c]);
            if (WITH_B) a[c] += source(b, m, c, ksb, kb0, kb1, ko0, ko1, kk);
            q[c] = sel0(m.xo[c], FULL ? k.q : k.qc[FULL ? 0 : c]);
            Al = c == 0 ? a[c] : a[c] + q[c] * Al;
        }
        T A = Al;
        const T om = ascan(A, k, sm);
        const T xin = readlane(A, WAVE - 1) * (lane_in(sm.nb) ? k.rpt : T(1));
        const T xe = A + om * xin;
        finish_row(a, q, dpp<0x138, 0xf>(xe, xin), b, jj, qr);        // wave_shr:1
    }

    // a sigma field: row jj + qr with its source-free part, and the next row's
    __device__ __forceinline__ void step(const QIn<T, CPL>& b, const Bits& m, const QPart<T, CPL>& p, const QIn<T, CPL>& bn,
                                         const Bits& mn, QPart<T, CPL>& pn, int jj, int qr, T c0, T c1) {
        T Pn = qpart_cells(c0, c1, k, mn, bn.sg, pn);
        T a[CPL];
        T Al;
#pragma unroll
        for (int c = 0; c < CPL; ++c) {
            a[c] = c1 * sel0(m.yo[c], y[c]);
            if (WITH_B) a[c] += source(b, m, c, ADJ ? s.sdm : T(1), s.mb0, s.mb1, s.mo0, s.mo1, s.sk);
            a[c] *= p.rdv[c];
            Al = c == 0 ? a[c] : a[c] + p.q[c] * Al;
        }
        T A = Al;
        scan_pair(A, p.t, Pn, pn.t);
        qpart_close<T, CPL>(Pn, pn);
        const T xin = readlane(A, WAVE - 1) * p.rPt;
        const T xe = A + p.omP * xin;
        finish_row(a, p.q, dpp<0x138, 0xf>(xe, xin), b, jj, qr);
    }

    // The sweep, from the wrap inflow u (in units of the solution) to the
    // last row.  Rows are read three ahead in a rotation of four buffers,
    // with no load and no store inside a branch, and the loop is entered from
    // a copy of its own body, so that its waits cover only the row they need
    // (the compiler keeps, per register, the latest load of any path).
    __device__ __forceinline__ void run(const T (&u)[CPL], T (&xl)[CPL]) {
#pragma unroll
        for (int c = 0; c < CPL; ++c) y[c] = u[c];
        const int nw = s.nw;
        const uint32_t oT0 = v.oT;
        const mview_t mask0 = v.mask;
        QIn<T, CPL> b0, b1, b2, b3;
        load(0, false, b0);
        load(1, false, b1);
        load(2, false, b2);
        int r = 0;
        if constexpr (S1) {
            const T kc1 = (T)s.c1 * k.rdv, kb0 = s.mb0 * k.rdv, kb1 = s.mb1 * k.rdv, ko0 = s.mo0 * k.rdv,
                    ko1 = s.mo1 * k.rdv, kk = s.sk * k.rdv, ksb = ADJ ? s.sdm * k.rdv : k.rdv;
            // the bits of this row and the next; without sources also this
            // row's scan masks, the next row's being formed while its chain
            // runs (a storing sweep has no scalar registers left for them,
            // and its sources to take meanwhile)
            constexpr bool AHEAD = !WITH_B;
            Bits m, m1;
            ScanMask sm;
            bits(m);
            if constexpr (AHEAD) {
                bits(m1);
                scan_mask(m, sm);
            }
            auto one = [&](const QIn<T, CPL>& b, int jj, int q) {
                Bits n;
                need_bits(AHEAD ? m1 : m);
                bits(n);
                ScanMask sn;
                scan_mask(AHEAD ? m1 : m, sn);
                step(b, m, AHEAD ? sm : sn, jj, q, kc1, kb0, kb1, ko0, ko1, ksb, kk);
                if constexpr (AHEAD) {
                    m = m1;
                    m1 = n;
                    sm = sn;
                } else {
                    m = n;
                }
            };
            auto group = [&](int jj) {
                load(jj + 3, false, b3);
                one(b0, jj, 0);
                load(jj + 4, true, b0);
                one(b1, jj, 1);
                load(jj + 5, false, b1);
                one(b2, jj, 2);
                load(jj + 6, false, b2);
                one(b3, jj, 3);
            };
            if (nw >= 4) {
                group(0);
                for (r = 4; r + 4 <= nw; r += 4) group(r);
            }
            if (r < nw) one(b0, r, 0);
            if (r + 1 < nw) one(b1, r, 1);
            if (r + 2 < nw) one(b2, r, 2);
        } else {
            const T c0 = (T)s.c0, c1 = (T)s.c1;
            Bits m0, m1;
            QPart<T, CPL> p0, p1;
            bits(m0);
            bits(m1);
            {
                T P = qpart_cells(c0, c1, k, m0, b0.sg, p0);
                pscan(P, p0.t);
                qpart_close<T, CPL>(P, p0);
            }
            auto one = [&](const QIn<T, CPL>& b, const QIn<T, CPL>& bn, int jj, int q) {
                Bits n;
                need_bits(m1);
                bits(n);
                step(b, m0, p0, bn, m1, p1, jj, q, c0, c1);
                m0 = m1;
                m1 = n;
                p0 = p1;
            };
            auto group = [&](int jj) {
                load(jj + 3, false, b3);
                one(b0, b1, jj, 0);
                load(jj + 4, true, b0);
                one(b1, b2, jj, 1);
                load(jj + 5, false, b1);
                one(b2, b3, jj, 2);
                load(jj + 6, false, b2);
                one(b3, b0, jj, 3);
            };
            if (nw >= 4) {
                group(0);
                for (r = 4; r + 4 <= nw; r += 4) group(r);
            }
            if (r < nw) one(b0, b1, r, 0);
            if (r + 1 < nw) one(b1, b2, r, 1);
            if (r + 2 < nw) one(b2, b0, r, 2);
        }
        if (ST == 2) drain();
        v.oT = oT0;              // the wrap solve runs its sweeps from one view
        v.mask = mask0;
#pragma unroll
        for (int c = 0; c < CPL; ++c) xl[c] = y[c];
    }
};

template <typename T, int CPL>
__device__ __forceinline__ double vdot2(const T (&a)[CPL], const T (&b)[CPL]) {
    double acc = 0.0;
#pragma unroll
    for (int c = 0; c < CPL; ++c) acc += (double)a[c] * (double)b[c];
    return wave_sum(acc);
}

#define VLOOP(body) _Pragma("unroll") for (int c = 0; c < CPL; ++c) { body; }

// One system's pass (wave w of work item `item`; w is wave-uniform, so every
// per-system quantity and the buffer resources built from it are scalars).
// Phase A sweeps with the sources and the previous wrap inflow u and stores
// the solution; phase B corrects u (BiCGSTAB on the wrap row); without
// lag_wrap, phase A runs again with the corrected u.  The wrap inflow is held
// in units of the solution: u = (last row where the pair across the wrap is
// solid).
template <typename T, int CPL, int ADJ, int SIG1, bool FULL>
__device__ __forceinline__ void pass_system(const GeomDev* __restrict__ geoms, const Item& item, int w, int lane,
                                            const PassParams& pp, T* tile) {
    const GeomDev& g = geoms[item.geom];
    if (pp.mode == 0 && g.ctrl[CTRL_DONE]) return;
    const int m = item.m0 + w;
    // inactive waves leave: the waves of a group never wait for each other
    if (!(w < item.nm && m < g.n_mfp)) return;
    constexpr int adj = ADJ;
    const Sys2<T> s = make_sys2<T>(g, m, item.l, item.tr, adj);
    QConst<T, CPL, FULL> qk;
    make_qconst<T, CPL, SIG1 != 0, FULL>(s.c0, s.c1, s.nr, lane, qk);
    const size_t half = adj ? (size_t)g.n_sys : 0;
    T* U = reinterpret_cast<T*>(g.U) + (half + s.sys) * (size_t)g.nwrap;
    const rsrc_t X = make_rsrc(reinterpret_cast<T*>(g.X) + (size_t)s.sys * g.xs, (uint32_t)g.nsolid * (uint32_t)sizeof(T));
    const int p0 = lane * CPL - (WAVE * CPL - s.nr);     // row position of this lane's first cell
    T u[CPL], xl[CPL];
    VLOOP(u[c] = p0 + c >= 0 ? U[p0 + c] : T(0));
    // pairs across the wrap: the first row's inflow across the rows
    bool mk[CPL];
    {
        RowBits<CPL, false> m0;
        const mview_t row = (mview_t)(uni(s.tr ? g.qmask[1] : g.qmask[0]) +
                                      (size_t)((2 * s.negr + s.negw) * s.nw + (s.negw ? s.nw - 1 : 0)) * row_mask_words(CPL, false));
        load_bits(row, m0);
        VLOOP(mk[c] = lane_in(m0.yo[c]));
    }
    const bool has_wrap = g.periodic[s.tr ? 0 : 1] != 0;
    long long n_it = 0, n_sw = 0;
    int need = 0;
    T kt;
    for (int round = 0;; ++round) {
        // ---- phase A
        if (s.tr) {
            Sweep2<T, CPL, 2, true, ADJ != 0, SIG1 != 0, FULL> a(g, s, qk, lane, tile, X);
            a.run(u, xl);
            kt = a.kt;
        } else {
            Sweep2<T, CPL, 1, true, ADJ != 0, SIG1 != 0, FULL> a(g, s, qk, lane, tile, X);
            a.run(u, xl);
            kt = a.kt;
        }
        ++n_sw;
        if (round > 0 || pp.mode != 0 || !has_wrap) break;
        // ---- phase B: residual of the wrap system for the inflow just used
        T r[CPL], ez[CPL];
        VLOOP({ ez[c] = mk[c] ? xl[c] : T(0); r[c] = ez[c] - u[c]; });
        const double scale = sqrt(vdot2<T, CPL>(ez, ez));
        double rn = sqrt(vdot2<T, CPL>(r, r));
        // target of this pass: inner_tol relative to the inflow, or (forcing)
        // a reduction by inner_rtol of the residual the pass started from
        const double thr = fmax(pp.inner_tol * scale, pp.inner_rtol * rn);
        const double thr_final = pp.inner_tol * scale;
        if (rn > thr_final && scale > 0.0) need = 1;
        const double rho_g = wrap_gain_bound(g.fscal[5], s.c1, s.nw);
        if (rn > thr && scale > 0.0 && rho_g * rn <= fmin(thr, fmax(thr_final, RICH_MAX * rn))) {
            // a weakly coupled wrap (short MFP across the rows): e = r leaves
            // the residual G r, at most rho_g |r|, within this pass's target
            // and below RICH_MAX |r| (or the final tolerance), with no sweep
            VLOOP(u[c] += r[c]);
            rn = rho_g * rn;
        } else if (rn > thr && scale > 0.0) {
            // BiCGSTAB for the remaining correction: (I - G) e = r.  A capped
            // BiCGSTAB is not monotone, so the iterate with the smallest
            // residual is kept: a pass never increases the wrap residual.
            T e[CPL], eb[CPL], rh[CPL], p[CPL], v[CPL], sv[CPL], t[CPL];
            VLOOP({ e[c] = T(0); eb[c] = T(0); rh[c] = r[c]; p[c] = T(0); v[c] = T(0); });
            double best = rn;
            int restarts = 0;
            double rho_old = 1.0, alpha = 1.0, omega = 1.0;
            Sweep2<T, CPL, 0, false, ADJ != 0, SIG1 != 0, FULL> h(g, s, qk, lane, tile, X);
            for (int iter = 0; iter < pp.max_inner; ++iter) {
                double rho = vdot2<T, CPL>(rh, r);
                if (fabs(rho) <= 1e-30 * rn * rn || !(omega != 0.0)) {
                    VLOOP({ rh[c] = r[c]; p[c] = T(0); v[c] = T(0); });
                    rho = vdot2<T, CPL>(r, r);
                    rho_old = 1.0; alpha = 1.0; omega = 1.0;
                }
                const double beta = (rho / rho_old) * (alpha / omega);
                VLOOP(p[c] = r[c] + (T)beta * (p[c] - (T)omega * v[c]));
                h.run(p, xl);
                ++n_sw;
                VLOOP(v[c] = p[c] - (mk[c] ? xl[c] : T(0)));
                const double rv = vdot2<T, CPL>(rh, v);
                if (!isfinite(rv)) break;
                if (!(fabs(rv) > 1e-30 * fabs(rho))) {
                    // breakdown (shadow residual orthogonal to A p): restart
                    // from the current residual on the next iteration
                    if (restarts++ >= 4) break;
                    omega = 0.0;
                    continue;
                }
                alpha = rho / rv;
                VLOOP(sv[c] = r[c] - (T)alpha * v[c]);
                const double sn = sqrt(vdot2<T, CPL>(sv, sv));
                ++n_it;
                if (sn <= thr) {
                    VLOOP(e[c] += (T)alpha * p[c]);
                    if (sn < best) { best = sn; VLOOP(eb[c] = e[c]); }
                    break;
                }
                h.run(sv, xl);
                ++n_sw;
                VLOOP(t[c] = sv[c] - (mk[c] ? xl[c] : T(0)));
                const double tt = vdot2<T, CPL>(t, t);
                omega = tt > 0.0 ? vdot2<T, CPL>(t, sv) / tt : 0.0;
                VLOOP(e[c] += (T)alpha * p[c] + (T)omega * sv[c]);
                VLOOP(r[c] = sv[c] - (T)omega * t[c]);
                rn = sqrt(vdot2<T, CPL>(r, r));
                rho_old = rho;
                if (!isfinite(rn)) break;
                if (rn < best) { best = rn; VLOOP(eb[c] = e[c]); }
                if (rn <= thr) break;
            }
            rn = best;
            VLOOP(u[c] += eb[c]);
        }
        if (lane == 0) g.wres[s.sys] = scale > 0.0 ? rn / scale : 0.0;
        if (need) VLOOP(if (p0 + c >= 0) U[p0 + c] = u[c]);
        // ---- the solution for the corrected inflow (skipped when the
        // correction is lagged into the next pass)
        if (pp.lag_wrap || !need) break;
    }
    // kappa sums.  kappa_face sums x over the plane cells (solid, last along
    // the gradient axis in sweep order, outflow face open), read back from
    // the stored solution; the forward adds the jump dT once per plane cell
    // when it crosses the plane towards + (the image there is hotter); the
    // adjoint weighs its jump faces by Lambda |s_g| / h_g dT, with the sign of
    // the jump (the '+' face's image is colder)
    __builtin_amdgcn_fence(__ATOMIC_SEQ_CST, "workgroup");
    const int side = s.pos_ga ? 1 : 0, np = g.n_plane[side];
    double kf = 0.0;
    for (int i = lane; i < np; i += WAVE)
        kf += (double)bldT<T>(X, (uint32_t)(side ? g.plane[1] : g.plane[0])[i] * (uint32_t)sizeof(T), 0u);
    const double ks = wave_sum((double)kt);
    kf = wave_sum(kf);
    if (lane == 0) {
        if (adj) {
            g.ksys[s.sys] = kf * ((s.pos_ga ? -1.0 : 1.0) * s.cga * g.dT);   // this system's share of p^T lambda
            g.kfsys[s.sys] = 0.0;
        } else {
            if (s.pos_ga) kf += g.dT * (double)np;
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
#undef VLOOP

// The 2D pass: one workgroup per work item, one of its systems per wave.
template <typename T, int CPL, int ADJ, int SIG1, bool FULL>
__global__ void __launch_bounds__((pass_threads<T, CPL>())) k_sweep_pass(const GeomDev* __restrict__ geoms,
                                                    const Item* __restrict__ items, int n_items,
                                                    PassParams pp) {
    extern __shared__ double lds[];
    const int it = blockIdx.x;
    if (it >= n_items) return;
    const int w = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    pass_system<T, CPL, ADJ, SIG1, FULL>(geoms, items[it], w, threadIdx.x & 63, pp,
                                         reinterpret_cast<T*>(lds) + (size_t)w * tr_tile_bytes(CPL) / sizeof(T));
}

// The 2D pass over every work item of a batch in one persistent launch: a
// workgroup takes the next item from a device-side queue (an atomic counter,
// set to 0 by the pack kernel before every pass) until none is left and runs
// it with its geometry's cells-per-lane body, so the items of every launch
// class share one grid (ordered longest MFPs first over all geometries).
// The waves of a group never wait for each other inside an item; the two
// barriers only order the group's read of the slot against its next write.
template <typename T, int ADJ, int SIG1>
__global__ void __launch_bounds__((pass_threads<T, 4>())) k_sweep_queue(const GeomDev* __restrict__ geoms,
                                                     const Item* __restrict__ items, int n_items,
                                                     PassParams pp, int* __restrict__ queue) {
    extern __shared__ double lds[];
    __shared__ int slot;
    const int w = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), lane = threadIdx.x & 63;
    for (;;) {
        __syncthreads();
        if (threadIdx.x == 0) slot = atomicAdd(queue, 1);
        __syncthreads();
        const int it = slot;
        if (it >= n_items) return;                     // every wave of the group leaves together
        const Item item = items[it];
        const int cpl = geoms[item.geom].q_cpl;
        T* tile = reinterpret_cast<T*>(lds) + (size_t)w * tr_tile_bytes(cpl) / sizeof(T);
        switch (cpl) {
            case 1: pass_system<T, 1, ADJ, SIG1, false>(geoms, item, w, lane, pp, tile); break;
            case 2: pass_system<T, 2, ADJ, SIG1, false>(geoms, item, w, lane, pp, tile); break;
            case 3: pass_system<T, 3, ADJ, SIG1, false>(geoms, item, w, lane, pp, tile); break;
            default: pass_system<T, 4, ADJ, SIG1, false>(geoms, item, w, lane, pp, tile); break;
        }
    }
}

}  // namespace

// ---------------------------------------------------------------------------
// launchers, instantiated once per precision
// ---------------------------------------------------------------------------
template <typename T, int CPL, bool FULL>
static hipError_t launch_sweep2_f(const GeomDev* g, const Item* it, int n, int waves, PassParams pp, size_t lds,
                                  hipStream_t st) {
    (void)hipGetLastError();
    const dim3 grid(n), block(64 * waves);
    if (pp.adjoint) {
        if (pp.sigma1) hipLaunchKernelGGL((k_sweep_pass<T, CPL, 1, 1, FULL>), grid, block, lds, st, g, it, n, pp);
        else hipLaunchKernelGGL((k_sweep_pass<T, CPL, 1, 0, FULL>), grid, block, lds, st, g, it, n, pp);
    } else {
        if (pp.sigma1) hipLaunchKernelGGL((k_sweep_pass<T, CPL, 0, 1, FULL>), grid, block, lds, st, g, it, n, pp);
        else hipLaunchKernelGGL((k_sweep_pass<T, CPL, 0, 0, FULL>), grid, block, lds, st, g, it, n, pp);
    }
    return hipGetLastError();
}

template <typename T, int CPL>
hipError_t launch_sweep2(const GeomDev* g, const Item* it, int n, int waves, PassParams pp, size_t lds, hipStream_t st,
                         int full) {
    return full ? launch_sweep2_f<T, CPL, true>(g, it, n, waves, pp, lds, st)
                : launch_sweep2_f<T, CPL, false>(g, it, n, waves, pp, lds, st);
}

template <typename T>
hipError_t launch_queue2(const GeomDev* g, const Item* it, int n, int waves, PassParams pp, size_t lds, hipStream_t st,
                         int* queue) {
    // enough groups to fill every SIMD; a group that starts once the queue is
    // empty leaves at once
    const int cap = 8192 / (waves > 1 ? waves : 1);
    const int groups = n < cap ? (n > 1 ? n : 1) : cap;
    (void)hipGetLastError();
    const dim3 grid(groups), block(64 * waves);
    if (pp.adjoint) {
        if (pp.sigma1) hipLaunchKernelGGL((k_sweep_queue<T, 1, 1>), grid, block, lds, st, g, it, n, pp, queue);
        else hipLaunchKernelGGL((k_sweep_queue<T, 1, 0>), grid, block, lds, st, g, it, n, pp, queue);
    } else {
        if (pp.sigma1) hipLaunchKernelGGL((k_sweep_queue<T, 0, 1>), grid, block, lds, st, g, it, n, pp, queue);
        else hipLaunchKernelGGL((k_sweep_queue<T, 0, 0>), grid, block, lds, st, g, it, n, pp, queue);
    }
    return hipGetLastError();
}
