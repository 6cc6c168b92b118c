// The 3D pass: see kernels.hip for the method.
#pragma once
#include "device.h"

namespace {

// per-row inputs of one lane (prefetched ahead of use; the 3D-only fields
// have one dummy entry in 2D, so the rotation buffers stay in registers)
template <typename T, int CPL, bool D3>
struct RowIn {
    uint32_t w[CPL];
    T sg[CPL];
    T sb[CPL];          // base source (sigma T_L, or k + D Psi), compute type
    T bx[CPL], by[CPL];                 // inflow boundary values per axis
    T bz[D3 ? CPL : 1];
    int si[CPL];        // solid index of the cell (sweeps that store), -1 in pores
    T ui[D3 ? CPL : 1]; // 3D: the wrap-plane input of the row's plane (used on the first y-row)
};

// Row results of a storing sweep, kept in registers until a group of rows is
// stored together.  A wave's global loads and stores share one counter on
// gfx9, and with both kinds in flight every wait for a prefetched row must
// drain the whole counter; storing once per group keeps the row prefetch
// overlapped everywhere else.
template <typename T, int CPL>
struct RowOut {
    T x[CPL];
    int si[CPL];        // -1: nothing to store
};

// per-sweep constant views: buffer resources of the per-cell tables and of
// the 3D wrap-plane input, and this lane's byte offsets within a row
template <typename T, int CPL>
struct Views {
    rsrc_t fc, sidx, sg, u, src, bx, by, bz;
    uint32_t o2[CPL], o4[CPL], oT[CPL], ou[CPL];
    // geometry scalars read once per sweep: the row loop stores to global
    // memory, after which the compiler would reload them from the view
    int nx, ny, nz, ga;
    int lx, cx;                        // lane and register of a row's last cell (p = nx - 1)
    double dT;
};

template <typename T, int CPL, bool D3, bool WITH_B, bool S1, bool ST>
__device__ __forceinline__ void load_row(const GeomDev& g, const SysC<T>& s, const Views<T, CPL>& v, int lane,
                                         int jj, int kk, RowIn<T, CPL, D3>& r) {
    // every lane loads (beyond the row: the row's first cell, masked by the
    // row step), so no load sits in a branch or feeds a select here: the
    // compiler then counts the loads in flight exactly and waits only for
    // the row it is about to use
    const int iy = s.pos[1] ? jj : v.ny - 1 - jj;
    const int iz = D3 ? (s.pos[2] ? kk : v.nz - 1 - kk) : 0;
    const uint32_t rowbase = uni((uint32_t)(v.nx * (iy + v.ny * iz)));
#pragma unroll
    for (int c = 0; c < CPL; ++c) {
        r.w[c] = bld16(v.fc, v.o2[c], rowbase * 2u);
        if (ST) r.si[c] = (int)bld32(v.sidx, v.o4[c], rowbase * 4u);
        r.sg[c] = S1 ? T(1) : bldT<T>(v.sg, v.oT[c], rowbase * (uint32_t)sizeof(T));
        if (WITH_B) {
            const uint32_t rb = rowbase * (uint32_t)sizeof(T);
            r.sb[c] = bldT<T>(v.src, v.oT[c], rb);
            r.bx[c] = bldT<T>(v.bx, v.oT[c], rb);
            r.by[c] = bldT<T>(v.by, v.oT[c], rb);
            if (D3) r.bz[c] = bldT<T>(v.bz, v.oT[c], rb);
        }
        if (D3) r.ui[c] = bldT<T>(v.u, v.ou[c], uni((uint32_t)(kk * v.nx)) * (uint32_t)sizeof(T));
    }
}

// Row storage of the sweep.  2D: the previous row in registers.  3D: the
// previous y-row of every z-plane in this wave's LDS region (the plane index
// is a runtime value), and the row just below in z in registers.
template <typename T, int CPL, bool D3>
struct Rows {
    T xr[CPL];    // 2D: row jj-1; 3D: row (jj, kk-1)
    T* xz;        // 3D: nz * ROW values, plane kk holds row (jj-1, kk) until overwritten
    int ROW;
    __device__ __forceinline__ T prev_y(int kk, int c, int lane) const {
        return D3 ? xz[kk * ROW + lane * CPL + c] : xr[c];
    }
    __device__ __forceinline__ T prev_z(int c) const { return D3 ? xr[c] : T(0); }
    __device__ __forceinline__ void put(int kk, int c, int lane, T v) {
        if (D3) xz[kk * ROW + lane * CPL + c] = v;
        xr[c] = v;
    }
};

// Wrap-row input (inflow u of the first row) and output (the last row).
// 2D: register arrays of this lane.  3D: the system's nz x nx plane in
// global memory, element (kk, p) at kk * nx + p, always touched by the lane
// that owns column p, so no cross-lane ordering is needed.
template <typename T, int CPL>
struct RegIO {
    const T (&u)[CPL];
    T (&xl)[CPL];
    __device__ __forceinline__ T in(int, int c, int) const { return u[c]; }
    __device__ __forceinline__ const T* input() const { return nullptr; }
    __device__ __forceinline__ void out(int, int c, int, T v) { xl[c] = v; }
};
template <typename T, int CPL>
struct GlobIO {
    gptr_t<T> u;
    rsrc_t xl;           // size 0 when the last row is not needed (or the wave is inactive)
    int nx;
    __device__ __forceinline__ const T* input() const { return (const T*)u; }
    // the row loads prefetch the input (Views::u); nothing is read here
    __device__ __forceinline__ T in(int, int, int) const { return T(0); }
    // a buffer store in no per-lane branch (beyond the row: an offset past
    // the plane, dropped), so the compiler keeps counting the row prefetches
    // in flight exactly across it
    __device__ __forceinline__ void out(int kk, int c, int lane, T v) {
        const int p = lane * CPL + c;
        bst(v, xl, p < nx ? (uint32_t)(kk * nx + p) * (uint32_t)sizeof(T) : BUF_OOB);
    }
};
// out_plane: the nz x nx plane receiving the last row, or nullptr
template <typename T, int CPL>
__device__ __forceinline__ GlobIO<T, CPL> make_gio(gptr_t<T> u, gmut_t<T> out_plane, int nx, int nz, int active) {
    GlobIO<T, CPL> io;
    io.u = u;
    io.xl = make_rsrc((const T*)out_plane, (out_plane && active) ? (uint32_t)(nx * nz) * (uint32_t)sizeof(T) : 0u);
    io.nx = nx;
    return io;
}

// One row step of the sweep (cells of row (jj, kk) in upwind order).  FULL:
// the row fills every lane (nx = 64 CPL), so no lane holds cells beyond it.
template <typename T, int CPL, bool D3, bool WITH_B, bool RED, bool ADD, bool S1, int GA, bool FULL = false,
          class IO>
__device__ __forceinline__ void row_step(const GeomDev& g, const SysC<T>& s, const Views<T, CPL>& vw,
                                         int active, int lane, int adj, int jj, int kk,
                                         const RowIn<T, CPL, D3>& cur, Rows<T, CPL, D3>& rows, IO& io,
                                         const double (&mb)[3], Red<T>* rd, RowOut<T, CPL>& ro) {
    const int nx = vw.nx, ny = vw.ny;
    const T cz = D3 ? s.c[2] : T(0);
    // diagonal without sigma (2D: no z term, so no +0 is left in the chain)
    const T cdiag = D3 ? s.c[0] + s.c[1] + cz : s.c[0] + s.c[1];
    const T cyz = D3 ? s.c[1] + cz : s.c[1];
    // sigma = 1: the cell coefficients are this system's constants
    const T rdv1 = S1 ? recip(T(1) + cdiag) : T(0);
    const T q1 = s.c[0] * rdv1, pxs1 = (T(1) + cyz) * rdv1, pnx1 = (T(1) + cdiag) * rdv1;
    T a[CPL], q[CPL];
    T Al, Pl;
#pragma unroll
    for (int c = 0; c < CPL; ++c) {
        const int p = lane * CPL + c;
        const uint32_t w = (FULL || p < nx) ? cur.w[c] : 0u;     // beyond the row: not solid
        const bool sol = active && fc_solid(w);
        const int clx = fc_class(w, s.fin[0]);
        const int cly = fc_class(w, s.fin[1]);
        const int clz = D3 ? fc_class(w, s.fin[2]) : FC_WALL;
        // sigma = 1 everywhere (no multiplier given): rdv is this system's constant
        const T sg = S1 ? T(1) : cur.sg[c];
        const T rdv = S1 ? rdv1 : recip(sg + cdiag);
        // kk and jj are wave-uniform: the wrap input is used on the first row
        // only (3D: prefetched with every row, so its load is in no branch)
        const T uin = D3 ? ((FULL || p < nx) ? cur.ui[c] : T(0)) : io.in(kk, c, lane);
        // the row below in y is read unconditionally (no branch around the
        // LDS load) and selected
        const T py = rows.prev_y(kk, c, lane);
        const T yin = cly != FC_WALL ? ((jj == 0) ? uin : s.c[1] * py) : T(0);
        T rhs = yin;
        if (WITH_B) {
            // in the compute type (the sources were converted once per pass)
            T sd = adj ? (T)s.kw + (T)s.Dml * cur.sb[c] : cur.sb[c];
            sd += (T)mb[0] * cur.bx[c] + (T)mb[1] * cur.by[c];
            if (D3) sd += (T)mb[2] * cur.bz[c];
            rhs = sd + yin;
        }
        if (D3) rhs += (clz != FC_WALL && kk > 0) ? cz * rows.prev_z(c) : T(0);
        const bool xs = (clx != FC_WALL);
        T av = rhs * rdv;
        T qv = xs ? (S1 ? q1 : s.c[0] * rdv) : T(0);
        T pv = S1 ? (xs ? pxs1 : pnx1) : (sg + (xs ? cyz : cdiag)) * rdv;
        // pore: (0, 0, 1) breaks the chain; beyond the row (face word 0, so
        // not solid either): the identity (0, 1, 0)
        const bool beyond = !FULL && p >= nx;
        av = sol ? av : T(0);
        qv = sol ? qv : (beyond ? T(1) : T(0));
        pv = sol ? pv : (beyond ? T(0) : T(1));
        a[c] = av;
        q[c] = qv;
        if (c == 0) {
            Al = av;
            Pl = pv;
        } else {
            Al = av + qv * Al;
            Pl = pv + qv * Pl;
        }
    }
    T A = Al, P = Pl;
    wave_scan(A, P);
    const T At = readlane(A, WAVE - 1), Pt = readlane(P, WAVE - 1);
    const T xin = (Pt > T(0)) ? At * recip(Pt) : T(0);   // cyclic closure x_{-1} = x_{nx-1}
    const T Ae = dpp<0x138, 0xf>(A, T(0)), Pe = dpp<0x138, 0xf>(P, T(0));   // wave_shr:1
    T xp = Ae + (T(1) - Pe) * xin;
    T xrow[CPL];
#pragma unroll
    for (int c = 0; c < CPL; ++c) {
        const T xv = a[c] + q[c] * xp;
        const int p = lane * CPL + c;
        xrow[c] = (FULL || p < nx) ? xv : T(0);
        rows.put(kk, c, lane, xrow[c]);
        xp = xv;
    }
    if (jj == ny - 1) {
#pragma unroll
        for (int c = 0; c < CPL; ++c) io.out(kk, c, lane, xrow[c]);
    }
    if (RED) {
        // branch-free: cells that contribute nothing add an exact 0 (an
        // inactive wave's sums are dropped, its stores skipped)
        // the row's cells summed in the compute type, the rows in double
        T rsum = T(0);
#pragma unroll
        for (int c = 0; c < CPL; ++c) {
            const int p = lane * CPL + c;
            const uint32_t wv = (FULL || p < nx) ? cur.w[c] : 0u;
            const bool sol = fc_solid(wv);
            ro.x[c] = xrow[c];
            ro.si[c] = sol ? cur.si[c] : -1;
            rsum += sol ? xrow[c] : T(0);
        }
        rd->kacc += (double)rsum;
        // Flux through the periodic plane of the gradient axis (kappa_face;
        // the adjoint: p^T lambda of the jump inflow, on the forward's jump
        // faces = this sweep's outflow faces).  The jump term belongs to the
        // b sweep only.
        if (GA == 0) {
            // the plane's cell of a row is its last cell in sweep order
            // (p = nx - 1): one lane's value, read into a scalar, added on
            // lane 0 (the wave sum then equals the sum over the rows)
            // (each register is read into a scalar and the scalars are
            // selected: selecting the registers first would let the compiler
            // index the row buffers at run time, which puts them in memory)
            T xl = readlane(xrow[0], vw.lx);
            uint32_t wl = (uint32_t)__builtin_amdgcn_readlane((int)cur.w[0], vw.lx);
#pragma unroll
            for (int c = 1; c < CPL; ++c) {
                const T xc = readlane(xrow[c], vw.lx);
                const uint32_t wc = (uint32_t)__builtin_amdgcn_readlane((int)cur.w[c], vw.lx);
                xl = (c == vw.cx) ? xc : xl;
                wl = (c == vw.cx) ? wc : wl;
            }
            double add = 0.0;
            if (fc_solid(wl)) {
                const int cl = fc_class(wl, s.fout[0]);
                const double xd = (double)xl;
                if (adj) {
                    const double cj = s.cd[0] * vw.dT;
                    add = cl == FC_JUMP_P ? cj * xd : (cl == FC_JUMP_M ? -cj * xd : 0.0);
                } else {
                    add = cl != FC_WALL ? xd + ((!ADD && s.pos[0]) ? vw.dT : 0.0) : 0.0;
                }
            }
            rd->kface += lane == 0 ? add : 0.0;
        } else if (GA == 1 && jj == ny - 1) {
#pragma unroll
            for (int c = 0; c < CPL; ++c) {
                const int p = lane * CPL + c;
                const uint32_t wv = (FULL || p < nx) ? cur.w[c] : 0u;
                // selects, not per-lane branches: a divergent region in the
                // row loop makes the compiler wait for every row prefetch
                const double xv = (double)xrow[c];
                const int cl = fc_class(wv, s.fout[1]);
                double add;
                if (adj) {
                    const double cj = s.cd[1] * vw.dT;
                    add = cl == FC_JUMP_P ? cj * xv : (cl == FC_JUMP_M ? -cj * xv : 0.0);
                } else {
                    add = cl != FC_WALL ? xv + ((!ADD && s.pos[1]) ? vw.dT : 0.0) : 0.0;
                }
                rd->kface += fc_solid(wv) ? add : 0.0;
            }
        }
    }
}

// Store a group of rows of a storing sweep (ADD: add to the stored values);
// cells with nothing to store get an out-of-range offset, so every lane
// issues the same stores and the hardware drops those.
template <typename T, int CPL, int NR, bool ADD>
__device__ __forceinline__ void store_rows(Red<T>* rd, const RowOut<T, CPL> (&ro)[NR]) {
    // no branch on rd->on: an inactive wave's resources have size 0
#pragma unroll
    for (int r = 0; r < NR; ++r)
#pragma unroll
        for (int c = 0; c < CPL; ++c) {
            const int i = ro[r].si[c];
            const uint32_t vo = i >= 0 ? (uint32_t)i * (uint32_t)sizeof(T) : BUF_OOB;
            T v = ro[r].x[c];
            if (ADD) v += bldT<T>(rd->X, vo, 0);
            bst(v, rd->X, vo);
            if (rd->store_T) bst((double)ro[r].x[c], rd->Tstore, i >= 0 ? (uint32_t)i * 8u : BUF_OOB);
        }
}

// ---------------------------------------------------------------------------
// The upwind sweep x = M^{-1}(src + P u): rows in y-upwind order (planes in
// z-upwind order), each row's cyclic x-recurrence solved by a wavefront scan.
// WITH_B: the pass sources are included, otherwise the only source is the
// wrap inflow u.  RED: lockstep reductions (every wave of the block calls
// it); ADD: add to the partials written by an earlier RED sweep of the same
// block.  Returns the last row (jj = ny-1) in xl.  Row inputs are prefetched
// two rows ahead (2D) through a three-buffer rotation without copies.
// ---------------------------------------------------------------------------


template <typename T, int CPL, bool D3, bool WITH_B, bool RED, bool ADD, bool S1, int GA, bool FULL = false,
          class IO>
__device__ __forceinline__ void sweep(const GeomDev& g, const SysC<T>& s, int active, int lane, int adj,
                                      const T* __restrict__ srcbase, const T* __restrict__ bnd,
                                      IO& io, Red<T>* rd, T* zrows) {
    constexpr int ND = D3 ? 3 : 2;
    double mb[3];
    // boundary input face per axis: forward, the wall this direction enters
    // from; adjoint, the wall whose temperature takes this system, the one
    // that S leaves through (with kappa_m weights: the reversed inflow face)
    int fb[3];
#pragma unroll
    for (int ax = 0; ax < 3; ++ax) {
        fb[ax] = adj ? 2 * ax + (s.S[ax] > 0.0 ? 1 : 0) : s.fin[ax];
        mb[ax] = adj ? (ax < ND ? g.wout[fb[ax] * g.n_sys + s.sys] : 0.0) : s.cd[ax];
    }
    Views<T, CPL> vw;
    const uint32_t nc = (uint32_t)g.ncells;
    vw.fc = make_rsrc(g.fc, nc * 2u);
    vw.sidx = make_rsrc(g.sidx, nc * 4u);
    vw.sg = make_rsrc(sigma_ptr<T>(g), nc * (uint32_t)sizeof(T));
    vw.u = make_rsrc(io.input(), (uint32_t)(g.nx * g.nz) * (uint32_t)sizeof(T));
    const uint32_t tb = nc * (uint32_t)sizeof(T);
    vw.src = make_rsrc(srcbase, tb);
    vw.bx = make_rsrc(bnd + (size_t)fb[0] * g.ncells, tb);
    vw.by = make_rsrc(bnd + (size_t)fb[1] * g.ncells, tb);
    vw.bz = make_rsrc(bnd + (size_t)(D3 ? fb[2] : 0) * g.ncells, tb);
#pragma unroll
    for (int c = 0; c < CPL; ++c) {
        // cell of this lane within a row (beyond the row: the row's first cell)
        const int p = lane * CPL + c;
        const uint32_t lo = p < g.nx ? (uint32_t)(s.pos[0] ? p : g.nx - 1 - p) : 0u;
        vw.o2[c] = lo * 2u;
        vw.o4[c] = lo * 4u;
        vw.oT[c] = lo * (uint32_t)sizeof(T);
        vw.ou[c] = (uint32_t)min(p, g.nx - 1) * (uint32_t)sizeof(T);
    }
    vw.nx = uni(g.nx);
    vw.ny = uni(g.ny);
    vw.nz = uni(g.nz);
    vw.ga = uni(g.grad_axis);
    vw.lx = (vw.nx - 1) / CPL;
    vw.cx = (vw.nx - 1) % CPL;
    vw.dT = uni(g.dT);
    Rows<T, CPL, D3> rows;
#pragma unroll
    for (int c = 0; c < CPL; ++c) rows.xr[c] = T(0);
    rows.xz = zrows;
    rows.ROW = WAVE * CPL;
    const int ny = g.ny;
    // Rows (jj, kk) in order, kk inner (2D: kk = 0).  A three-buffer
    // rotation keeps the inputs two rows ahead; prefetches are never skipped
    // (past the last row they reload it): a load inside a branch would leave
    // the compiler unsure how many loads are in flight at the join, and it
    // would then wait for all.  A storing sweep stores each group of three
    // rows after the group's last row.
    const int nz = D3 ? g.nz : 1, nrows = ny * nz;
    // row r -> (r / nz, r % nz) by a multiply with mz = ceil(2^32 / nz), not a
    // division per row: r mz / 2^32 = r / nz + r e / (nz 2^32) with e = mz nz
    // - 2^32 < nz, so the floor is exact while r e < 2^32, i.e. for every
    // r < 2^25 (nz <= 128)
    const uint64_t mz = D3 ? ((1ull << 32) + (uint64_t)nz - 1) / (uint64_t)nz : 1ull;
    auto row_j = [&](int r) { return D3 ? (int)(((uint64_t)(uint32_t)r * mz) >> 32) : r; };
    auto pre = [&](int r, RowIn<T, CPL, D3>& b) {
        const int rr = min(r, nrows - 1);
        const int jr = row_j(rr);
        load_row<T, CPL, D3, WITH_B, S1, RED>(g, s, vw, lane, jr, D3 ? rr - jr * nz : 0, b);
    };
    auto step = [&](int r, const RowIn<T, CPL, D3>& b, RowOut<T, CPL>& ro) {
        const int jr = row_j(r);
        row_step<T, CPL, D3, WITH_B, RED, ADD, S1, GA, FULL>(g, s, vw, active, lane, adj, jr, D3 ? r - jr * nz : 0,
                                                       b, rows, io, mb, rd, ro);
    };
    RowIn<T, CPL, D3> b0, b1, b2;
    pre(0, b0);
    pre(1, b1);
    for (int r = 0; r < nrows; r += 3) {
        RowOut<T, CPL> ro[3];
#pragma unroll
        for (int q = 0; q < 3; ++q)
#pragma unroll
            for (int c = 0; c < CPL; ++c) ro[q].si[c] = -1;
        pre(r + 2, b2);
        step(r, b0, ro[0]);
        pre(r + 3, b0);
        if (r + 1 < nrows) step(r + 1, b1, ro[1]);
        pre(r + 4, b1);
        if (r + 2 < nrows) step(r + 2, b2, ro[2]);
        if (RED) store_rows<T, CPL, 3, ADD>(rd, ro);
    }
}

template <typename T>
__device__ __forceinline__ Red<T> make_red(const GeomDev& g, const SysC<T>& s, int active, const PassParams& pp) {
    Red<T> rd;
    rd.kacc = 0.0;
    rd.kface = 0.0;
    rd.on = active;
    // size 0 for an inactive wave: every store through it is dropped
    rd.X = make_rsrc(reinterpret_cast<T*>(g.X) + (size_t)s.sys * g.xs,
                     active ? (uint32_t)g.nsolid * (uint32_t)sizeof(T) : 0u);
    rd.Tstore = make_rsrc(g.Tstore ? g.Tstore + (size_t)s.sys * g.xs : nullptr,
                          (g.Tstore && active) ? (uint32_t)g.nsolid * 8u : 0u);
    rd.store_T = pp.store_T && g.Tstore != nullptr;
    return rd;
}

template <typename T>
__device__ __forceinline__ void finish_system(const GeomDev& g, const SysC<T>& s, int active, int lane,
                                              int adj, const PassParams& pp, const Red<T>& rd,
                                              long long n_it, long long n_sw) {
    const double ks = wave_sum(rd.kacc), kf = wave_sum(rd.kface);
    if (active && lane == 0) {
        if (adj) {
            g.ksys[s.sys] = kf;                 // this system's share of p^T lambda
            g.kfsys[s.sys] = 0.0;
        } else {
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

// ---------------------------------------------------------------------------
// The 3D pass.  Same phases as the 2D kernel; the wrap plane of a system
// (nx * nz values) is too large for registers, so its Krylov vectors live in
// a per-system slab of the workspace (KV_N planes).  Every element (k, p) is
// read and written only by the lane owning column p, as in the sweep.
// ---------------------------------------------------------------------------
enum { KV_XL, KV_MK, KV_DU, KV_R, KV_E, KV_EB, KV_RH, KV_P, KV_V, KV_S, KV_T, KV_N };
static_assert(KV_N == KRY3_VECS, "workspace carve and kernel disagree on the 3D slab");

#define PLOOP(body)                                     \
    for (int k = 0; k < nz; ++k)                        \
        _Pragma("unroll") for (int c = 0; c < CPL; ++c) { \
            const int p_ = lane * CPL + c;              \
            if (p_ < nx) {                              \
                const int i = k * nx + p_;              \
                body;                                   \
            }                                           \
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
    const int active = (w < item.nm) && (m < g.n_mfp);
    constexpr int adj = ADJ;
    const SysC<T> s = make_sys<T>(g, active ? m : item.m0, item.l, adj);
    // the pass's sources and inflow tables, converted to the compute type by
    // k_pack3 before the pass
    const T* srcbase = static_cast<const T*>(g.qrec);
    const T* bnd = srcbase + g.ncells;
    const int nx = g.nx, nz = g.nz, nw = g.nwrap;
    const size_t half = adj ? (size_t)g.n_sys : 0;
    const gmut_t<T> U = gmut(reinterpret_cast<T*>(g.U) + (half + s.sys) * (size_t)nw);
    const gmut_t<T> K = gmut(reinterpret_cast<T*>(g.kry) + (size_t)s.sys * KV_N * nw);
    const gmut_t<T> xl = K + (size_t)KV_XL * nw;
    const gmut_t<T> du = K + (size_t)KV_DU * nw;
    // per-wave LDS: nz rows of this wave
    T* zrows = reinterpret_cast<T*>(lds) + (size_t)w * nz * WAVE * CPL;
    Red<T> rd = make_red<T>(g, s, active, pp);
    // ---- phase A
    {
        GlobIO<T, CPL> io = make_gio<T, CPL>(U, xl, nx, nz, active);
        if (g.grad_axis == 0)
            sweep<T, CPL, true, true, true, false, SIG1 != 0, 0, FULL>(g, s, active, lane, adj, srcbase, bnd, io, &rd, zrows);
        else
            sweep<T, CPL, true, true, true, false, SIG1 != 0, 1, FULL>(g, s, active, lane, adj, srcbase, bnd, io, &rd, zrows);
    }
    long long n_it = 0, n_sw = 1;
    int need = 0;
    const bool has_wrap = g.periodic[1] != 0;
    if (pp.mode == 0 && active && has_wrap) {
        const gmut_t<T> mk = K + (size_t)KV_MK * nw;
        const gmut_t<T> r = K + (size_t)KV_R * nw;
        const gmut_t<T> e = K + (size_t)KV_E * nw;
        const gmut_t<T> eb = K + (size_t)KV_EB * nw;
        const gmut_t<T> rh = K + (size_t)KV_RH * nw;
        const gmut_t<T> p = K + (size_t)KV_P * nw;
        const gmut_t<T> v = K + (size_t)KV_V * nw;
        const gmut_t<T> sv = K + (size_t)KV_S * nw;
        const gmut_t<T> t = K + (size_t)KV_T * nw;
        // wrap mask E' (c_y where the pair across the y-wrap is solid), the
        // inflow produced by the sweep and the residual of the wrap system
        const int iy = s.pos[1] ? 0 : g.ny - 1;
        double ss = 0.0, rr = 0.0;
        PLOOP({
            const int ix = s.pos[0] ? p_ : nx - 1 - p_;
            const int iz = s.pos[2] ? k : nz - 1 - k;
            const uint32_t wv = g.fc[ix + nx * (iy + g.ny * iz)];
            const T mv = (fc_solid(wv) && fc_class(wv, s.fin[1]) != FC_WALL) ? s.c[1] : T(0);
            mk[i] = mv;
            const T ez = mv * xl[i];
            const T rv = ez - U[i];
            r[i] = rv;
            du[i] = T(0);
            ss += (double)ez * (double)ez;
            rr += (double)rv * (double)rv;
        });
        const double scale = sqrt(wave_sum(ss));
        double rn = sqrt(wave_sum(rr));
        const double thr = fmax(pp.inner_tol * scale, pp.inner_rtol * rn);
        const double thr_final = pp.inner_tol * scale;
        if (rn > thr_final && scale > 0.0) need = 1;
        const double rho_g = wrap_gain_bound(g.fscal[5], s.cd[1], g.ny);
        if (rn > thr && scale > 0.0 && rho_g * rn <= fmin(thr, fmax(thr_final, RICH_MAX * rn))) {
            // weakly coupled wrap: e = r, no sweep (as in 2D)
            PLOOP(du[i] = r[i]);
            rn = rho_g * rn;
        } else if (rn > thr && scale > 0.0) {
            // BiCGSTAB on (I - G) e = r with the best iterate kept (as in 2D)
            PLOOP({ e[i] = T(0); eb[i] = T(0); rh[i] = r[i]; p[i] = T(0); v[i] = T(0); });
            double best = rn;
            int restarts = 0;
            double rho_old = 1.0, alpha = 1.0, omega = 1.0;
            for (int iter = 0; iter < pp.max_inner; ++iter) {
                double acc = 0.0;
                PLOOP(acc += (double)rh[i] * (double)r[i]);
                double rho = wave_sum(acc);
                if (fabs(rho) <= 1e-30 * rn * rn || !(omega != 0.0)) {
                    acc = 0.0;
                    PLOOP({ rh[i] = r[i]; p[i] = T(0); v[i] = T(0); acc += (double)r[i] * (double)r[i]; });
                    rho = wave_sum(acc);
                    rho_old = 1.0; alpha = 1.0; omega = 1.0;
                }
                const double beta = (rho / rho_old) * (alpha / omega);
                PLOOP(p[i] = r[i] + (T)beta * (p[i] - (T)omega * v[i]));
                {
                    GlobIO<T, CPL> io = make_gio<T, CPL>(p, xl, nx, nz, 1);
                    sweep<T, CPL, true, false, false, false, SIG1 != 0, -1, FULL>(g, s, active, lane, adj, srcbase, bnd, io, nullptr, zrows);
                }
                ++n_sw;
                acc = 0.0;
                PLOOP({
                    const T vv = p[i] - mk[i] * xl[i];
                    v[i] = vv;
                    acc += (double)rh[i] * (double)vv;
                });
                const double rv = wave_sum(acc);
                if (!isfinite(rv)) break;
                if (!(fabs(rv) > 1e-30 * fabs(rho))) {
                    if (restarts++ >= 4) break;
                    omega = 0.0;
                    continue;
                }
                alpha = rho / rv;
                acc = 0.0;
                PLOOP({
                    const T x = r[i] - (T)alpha * v[i];
                    sv[i] = x;
                    acc += (double)x * (double)x;
                });
                const double sn = sqrt(wave_sum(acc));
                ++n_it;
                if (sn <= thr) {
                    PLOOP(e[i] += (T)alpha * p[i]);
                    if (sn < best) {
                        best = sn;
                        PLOOP(eb[i] = e[i]);
                    }
                    break;
                }
                {
                    GlobIO<T, CPL> io = make_gio<T, CPL>(sv, xl, nx, nz, 1);
                    sweep<T, CPL, true, false, false, false, SIG1 != 0, -1, FULL>(g, s, active, lane, adj, srcbase, bnd, io, nullptr, zrows);
                }
                ++n_sw;
                double tt = 0.0, ts = 0.0;
                PLOOP({
                    const T x = sv[i] - mk[i] * xl[i];
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
            PLOOP(du[i] += eb[i]);
        }
        if (lane == 0) g.wres[s.sys] = scale > 0.0 ? rn / scale : 0.0;
        if (need) PLOOP(U[i] += du[i]);
    }
    // ---- phase C (see the 2D kernel)
    if (!pp.lag_wrap && need) {
        GlobIO<T, CPL> io = make_gio<T, CPL>(du, nullptr, nx, nz, 0);
        if (g.grad_axis == 0)
            sweep<T, CPL, true, false, true, true, SIG1 != 0, 0, FULL>(g, s, active, lane, adj, srcbase, bnd, io, &rd, zrows);
        else
            sweep<T, CPL, true, false, true, true, SIG1 != 0, 1, FULL>(g, s, active, lane, adj, srcbase, bnd, io, &rd, zrows);
        ++n_sw;
    }
    finish_system(g, s, active, lane, adj, pp, rd, n_it, n_sw);
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
