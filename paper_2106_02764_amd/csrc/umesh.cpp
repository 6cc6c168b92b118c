// Host driver of the unstructured-mesh path: polygon geometry and face
// lists, material weights, the rows of each direction's sweep, the tables of
// the non-orthogonal heat-conduction solve, and Algorithm 1's outer loop.
//
// Geometry (plain definitions): polygon area by the shoelace formula, the
// area centroid, edge length and the outward unit normal (dy, -dx) / |e| of
// each counter-clockwise edge.  An interior face joins two solid cells; d
// runs from the first cell's centroid to the centroid of the second cell's
// periodic image, and that image carries T + delta dT with
// T(x + L_g) = T(x) - dT (delta = minus the image shift along the gradient
// axis).  Faces towards pore cells are diffuse walls.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <array>
#include <climits>
#include <cmath>
#include <cstdarg>
#include <cstdio>
#include <map>
#include <string>
#include <vector>

#include "../../include/obte.h"
#include "obte_internal.h"
#include "umesh_internal.h"

namespace {

obte_status ufail(obte_status st, const char* fmt, ...) {
    char buf[512];
    va_list ap;
    va_start(ap, fmt);
    vsnprintf(buf, sizeof buf, fmt, ap);
    va_end(ap);
    obte_set_error(buf);
    return st;
}

#define UHIP(call)                                                                        \
    do {                                                                                  \
        hipError_t e_ = (call);                                                           \
        if (e_ != hipSuccess)                                                             \
            return ufail(OBTE_ERR_HIP, "%s failed: %s", #call, hipGetErrorString(e_));   \
    } while (0)

constexpr int MAX_SOLID = 8192;     // a solution goes through one workgroup's 64 KiB of LDS
static_assert(MAX_SOLID <= 256 * UF_MAXB, "heat-conduction partials: one slot per block of 256 cells");

}  // namespace

struct obte_umesh {
    double L[2] = {0, 0}, dT = 1.0;
    int ga = 0;
    int n_cells = 0, ns = 0, nf = 0, nw = 0;
    std::vector<int> scell, sid;
    std::vector<double> V, xc;                 // ns, 2 ns
    std::vector<int> fi, fj, fper;             // interior faces; fper: 1 across a periodic boundary
    std::vector<double> fA, fn, fd, fdel, fw;  // fn, fd: 2 per face
    std::vector<int> wcell;
    std::vector<double> wA, wn;
    std::vector<std::vector<int>> cfaces;      // per solid cell: 2 f (+1 if second cell), or -(w + 1)
    // material
    bool has_material = false;
    int n_mfp = 0, n_dir = 0, n_sys = 0;
    std::vector<double> mfp, dirs, Dw, S;
    double kax[2] = {0, 0};
    std::vector<int> nlev;
    int wmax = 0, slots = 0;                   // wrap slots of a direction, LDS slots of a system
    // device
    std::vector<void*> dev;
    UGeomDev gh{};
    UGeomDev* gd = nullptr;
    UFourierDev fh{};
    UFourierDev* fdv = nullptr;
    double* sigma1 = nullptr;
    int* scell_d = nullptr;
    int* wcell_d = nullptr;
    double* h_fsc = nullptr;                   // pinned: the heat-conduction loop scalars read back
};

namespace {

void free_dev(obte_umesh* m) {
    for (void* p : m->dev) (void)hipFree(p);
    m->dev.clear();
    if (m->h_fsc) (void)hipHostFree(m->h_fsc);
    m->h_fsc = nullptr;
    m->gd = nullptr;
    m->fdv = nullptr;
    (void)hipGetLastError();
}

template <typename T>
obte_status upload(obte_umesh* m, T** dst, const std::vector<T>& v) {
    const size_t n = std::max<size_t>(v.size(), 1);
    void* p = nullptr;
    UHIP(hipMalloc(&p, n * sizeof(T)));
    m->dev.push_back(p);
    if (!v.empty()) UHIP(hipMemcpy(p, v.data(), v.size() * sizeof(T), hipMemcpyHostToDevice));
    *dst = (T*)p;
    return OBTE_OK;
}

template <typename T>
obte_status alloc(obte_umesh* m, T** dst, size_t n) {
    void* p = nullptr;
    UHIP(hipMalloc(&p, std::max<size_t>(n, 1) * sizeof(T)));
    m->dev.push_back(p);
    UHIP(hipMemset(p, 0, std::max<size_t>(n, 1) * sizeof(T)));
    *dst = (T*)p;
    return OBTE_OK;
}

__global__ void k_uscatter(int ns, const int* __restrict__ scell, const double* __restrict__ src,
                           double* __restrict__ dst, double shift) {
    const int i = blockIdx.x * blockDim.x + threadIdx.x;
    if (i < ns) dst[scell[i]] = src[i] - shift;
}

__global__ void k_ugather(int n, const int* __restrict__ idx, const double* __restrict__ src, double* __restrict__ dst) {
    const int i = blockIdx.x * blockDim.x + threadIdx.x;
    if (i < n) dst[i] = src[idx[i]];
}

}  // namespace

extern "C" {

obte_status obte_umesh_create(const double* nodes, int n_nodes, const int* cells, const int* shifts, int n_cells,
                              int nv, const unsigned char* solid, double Lx, double Ly, int grad_axis, double dT,
                              obte_umesh** out) {
    if (!out) return ufail(OBTE_ERR_ARG, "out is NULL");
    *out = nullptr;
    if (!nodes || !cells || !shifts || !solid) return ufail(OBTE_ERR_ARG, "NULL mesh array");
    if (n_nodes < 3 || n_cells < 1) return ufail(OBTE_ERR_ARG, "need at least 3 nodes and 1 cell");
    if (nv != 3 && nv != 4) return ufail(OBTE_ERR_ARG, "cells must be triangles or quadrilaterals (nv 3 or 4)");
    if (!(Lx > 0.0) || !(Ly > 0.0) || !std::isfinite(Lx) || !std::isfinite(Ly))
        return ufail(OBTE_ERR_ARG, "Lx and Ly must be > 0");
    if (grad_axis != 0 && grad_axis != 1) return ufail(OBTE_ERR_ARG, "grad_axis must be 0 or 1");
    if (!(dT > 0.0) || !std::isfinite(dT)) return ufail(OBTE_ERR_ARG, "dT must be > 0");
    for (long long q = 0; q < (long long)n_cells * nv; ++q)
        if (cells[q] < 0 || cells[q] >= n_nodes) return ufail(OBTE_ERR_ARG, "cell node id out of range");
    obte_umesh* m = new obte_umesh();
    m->L[0] = Lx;
    m->L[1] = Ly;
    m->dT = dT;
    m->ga = grad_axis;
    m->n_cells = n_cells;
    // corner positions in each cell's own frame, areas and centroids
    std::vector<double> P((size_t)n_cells * nv * 2), area(n_cells), cen(2 * (size_t)n_cells);
    for (int c = 0; c < n_cells; ++c) {
        for (int k = 0; k < nv; ++k) {
            const size_t q = (size_t)c * nv + k;
            P[2 * q] = nodes[2 * cells[q]] + shifts[2 * q] * Lx;
            P[2 * q + 1] = nodes[2 * cells[q] + 1] + shifts[2 * q + 1] * Ly;
        }
        double a = 0.0, cx = 0.0, cy = 0.0;
        for (int k = 0; k < nv; ++k) {
            const size_t q0 = (size_t)c * nv + k, q1 = (size_t)c * nv + (k + 1) % nv;
            const double x0 = P[2 * q0], y0 = P[2 * q0 + 1], x1 = P[2 * q1], y1 = P[2 * q1 + 1];
            const double cr = x0 * y1 - x1 * y0;
            a += cr;
            cx += (x0 + x1) * cr;
            cy += (y0 + y1) * cr;
        }
        a *= 0.5;
        if (!(a > 0.0)) {
            delete m;
            return ufail(OBTE_ERR_ARG, "cell %d is clockwise or degenerate", c);
        }
        area[c] = a;
        cen[2 * c] = cx / (6.0 * a);
        cen[2 * c + 1] = cy / (6.0 * a);
    }
    // edges keyed by their node ids and the relative image shift
    using Key = std::array<long long, 4>;
    auto key_of = [&](int c, int k) {
        const size_t q0 = (size_t)c * nv + k, q1 = (size_t)c * nv + (k + 1) % nv;
        const long long a = cells[q0], b = cells[q1];
        if (a < b) return Key{a, b, shifts[2 * q1] - shifts[2 * q0], shifts[2 * q1 + 1] - shifts[2 * q0 + 1]};
        return Key{b, a, shifts[2 * q0] - shifts[2 * q1], shifts[2 * q0 + 1] - shifts[2 * q1 + 1]};
    };
    std::map<Key, std::vector<std::pair<int, int>>> edges;
    for (int c = 0; c < n_cells; ++c)
        for (int k = 0; k < nv; ++k) {
            const Key kk = key_of(c, k);
            if (kk[0] == kk[1]) {
                delete m;
                return ufail(OBTE_ERR_ARG, "cell %d has an edge from a node to itself", c);
            }
            edges[kk].push_back({c, k});
        }
    for (const auto& e : edges)
        if (e.second.size() != 2) {
            delete m;
            return ufail(OBTE_ERR_ARG, "an edge of cell %d is shared by %zu cells (need 2)", e.second[0].first,
                         e.second.size());
        }
    m->sid.assign(n_cells, -1);
    for (int c = 0; c < n_cells; ++c)
        if (solid[c]) {
            m->sid[c] = m->ns++;
            m->scell.push_back(c);
        }
    if (m->ns == 0) {
        delete m;
        return ufail(OBTE_ERR_ARG, "the mesh has no solid cell");
    }
    if (m->ns > MAX_SOLID) {
        const int ns = m->ns;
        delete m;
        return ufail(OBTE_ERR_ARG, "%d solid cells: the unstructured path takes at most %d", ns, MAX_SOLID);
    }
    for (int i = 0; i < m->ns; ++i) {
        const int c = m->scell[i];
        m->V.push_back(area[c]);
        m->xc.push_back(cen[2 * c]);
        m->xc.push_back(cen[2 * c + 1]);
    }
    m->cfaces.assign(m->ns, {});
    std::map<Key, int> face_of;
    for (int i = 0; i < m->ns; ++i) {
        const int c = m->scell[i];
        for (int k = 0; k < nv; ++k) {
            const Key kk = key_of(c, k);
            const auto& occ = edges[kk];
            const std::pair<int, int> other = occ[0] == std::make_pair(c, k) ? occ[1] : occ[0];
            const int c2 = other.first;
            const size_t q0 = (size_t)c * nv + k, q1 = (size_t)c * nv + (k + 1) % nv;
            const double ex = P[2 * q1] - P[2 * q0], ey = P[2 * q1 + 1] - P[2 * q0 + 1];
            const double len = std::hypot(ex, ey);
            const double nx = ey / len, ny = -ex / len;
            if (!solid[c2]) {
                m->cfaces[i].push_back(-(m->nw + 1));
                m->wcell.push_back(i);
                m->wA.push_back(len);
                m->wn.push_back(nx);
                m->wn.push_back(ny);
                ++m->nw;
                continue;
            }
            const auto it = face_of.find(kk);
            if (it != face_of.end()) {
                m->cfaces[i].push_back(2 * it->second + 1);
                continue;
            }
            // image offset bringing c2 into c's frame, from the shared nodes
            const int a = cells[q0], b = cells[q1];
            bool found = false;
            long long ox = 0, oy = 0;
            for (int qa = 0; qa < nv && !found; ++qa) {
                if (cells[(size_t)c2 * nv + qa] != a) continue;
                const long long cx_ = shifts[2 * q0] - shifts[2 * ((size_t)c2 * nv + qa)];
                const long long cy_ = shifts[2 * q0 + 1] - shifts[2 * ((size_t)c2 * nv + qa) + 1];
                for (int qb = 0; qb < nv; ++qb) {
                    const size_t r = (size_t)c2 * nv + qb;
                    if (cells[r] == b && shifts[2 * q1] - shifts[2 * r] == cx_ && shifts[2 * q1 + 1] - shifts[2 * r + 1] == cy_) {
                        ox = cx_;
                        oy = cy_;
                        found = true;
                        break;
                    }
                }
            }
            if (!found) {
                delete m;
                return ufail(OBTE_ERR_ARG, "inconsistent periodic shifts on an edge of cell %d", c);
            }
            const int f = m->nf++;
            face_of[kk] = f;
            m->cfaces[i].push_back(2 * f);
            const double dx = cen[2 * c2] + ox * Lx - cen[2 * c], dy = cen[2 * c2 + 1] + oy * Ly - cen[2 * c + 1];
            m->fi.push_back(i);
            m->fj.push_back(m->sid[c2]);
            m->fper.push_back(ox != 0 || oy != 0);
            m->fA.push_back(len);
            m->fn.push_back(nx);
            m->fn.push_back(ny);
            m->fd.push_back(dx);
            m->fd.push_back(dy);
            m->fdel.push_back(-(double)(grad_axis == 0 ? ox : oy));
            // fraction of d at which the centroid line crosses the face
            const double nd = dx * nx + dy * ny;
            m->fw.push_back(((P[2 * q0] - cen[2 * c]) * nx + (P[2 * q0 + 1] - cen[2 * c + 1]) * ny) / nd);
        }
    }
    *out = m;
    return OBTE_OK;
}

obte_status obte_umesh_material_set(obte_umesh* m, const double* mfp, int n_mfp, const double* dirs,
                                    const double* dir_w, int n_dir, const double* kappa_m) {
    if (!m) return ufail(OBTE_ERR_ARG, "mesh is NULL");
    if (!mfp || !dirs || !dir_w || !kappa_m) return ufail(OBTE_ERR_ARG, "NULL material array");
    if (n_mfp < 1 || n_dir < 2) return ufail(OBTE_ERR_ARG, "need n_mfp >= 1 and n_dir >= 2");
    double wsum = 0.0, sx = 0.0, sy = 0.0;
    for (int l = 0; l < n_dir; ++l) {
        const double x = dirs[2 * l], y = dirs[2 * l + 1];
        if (std::fabs(x * x + y * y - 1.0) > 1e-9) return ufail(OBTE_ERR_ARG, "direction %d is not a unit vector", l);
        if (!(dir_w[l] > 0.0)) return ufail(OBTE_ERR_ARG, "direction weight %d must be > 0", l);
        wsum += dir_w[l];
        sx += x * dir_w[l];
        sy += y * dir_w[l];
    }
    if (std::fabs(wsum - 1.0) > 1e-9) return ufail(OBTE_ERR_ARG, "direction weights must sum to 1");
    if (std::fabs(sx) > 1e-9 || std::fabs(sy) > 1e-9)
        return ufail(OBTE_ERR_ARG, "direction set must be centrally symmetric");
    for (int k = 0; k < n_mfp; ++k) {
        if (!(mfp[k] > 0.0) || !std::isfinite(mfp[k])) return ufail(OBTE_ERR_ARG, "mfp[%d] must be > 0", k);
        if (!(kappa_m[k] >= 0.0) || !std::isfinite(kappa_m[k])) return ufail(OBTE_ERR_ARG, "kappa_m[%d] must be >= 0", k);
    }
    free_dev(m);
    m->has_material = false;
    const int ns = m->ns, nw = m->nw, nf = m->nf, ga = m->ga;
    m->n_mfp = n_mfp;
    m->n_dir = n_dir;
    m->n_sys = n_mfp * n_dir;
    m->mfp.assign(mfp, mfp + n_mfp);
    m->dirs.assign(dirs, dirs + 2 * n_dir);
    // alpha_ml = kappa_m w_l / (Lambda_m^2 mu_g), D = alpha / sum alpha,
    // S = alpha Lambda s (section Model, Appendix A)
    double mu = 0.0;
    for (int l = 0; l < n_dir; ++l) mu += dir_w[l] * dirs[2 * l + ga] * dirs[2 * l + ga];
    if (!(mu > 0.0)) return ufail(OBTE_ERR_ARG, "directions have no component along the gradient axis");
    std::vector<double> alpha(m->n_sys);
    double asum = 0.0;
    for (int k = 0; k < n_mfp; ++k)
        for (int l = 0; l < n_dir; ++l) {
            alpha[k * n_dir + l] = kappa_m[k] * dir_w[l] / (mfp[k] * mfp[k] * mu);
            asum += alpha[k * n_dir + l];
        }
    if (!(asum > 0.0)) return ufail(OBTE_ERR_ARG, "kappa_m is all zero");
    m->Dw.assign(m->n_sys, 0.0);
    m->S.assign(2 * (size_t)m->n_sys, 0.0);
    m->kax[0] = m->kax[1] = 0.0;
    for (int k = 0; k < n_mfp; ++k)
        for (int l = 0; l < n_dir; ++l) {
            const int sys = k * n_dir + l;
            m->Dw[sys] = alpha[sys] / asum;
            for (int a = 0; a < 2; ++a) {
                m->S[2 * sys + a] = alpha[sys] * mfp[k] * dirs[2 * l + a];
                m->kax[a] += alpha[sys] * mfp[k] * mfp[k] * dirs[2 * l + a] * dirs[2 * l + a];
            }
        }
    // outgoing weights of each wall face: ReLu(S . n) / sum ReLu(S . n)
    std::vector<double> wout((size_t)nw * m->n_sys, 0.0);
    for (int w = 0; w < nw; ++w) {
        auto out = [&](int sys) {
            return std::max(0.0, m->S[2 * sys] * m->wn[2 * w] + m->S[2 * sys + 1] * m->wn[2 * w + 1]);
        };
        double tot = 0.0;
        for (int sys = 0; sys < m->n_sys; ++sys) tot += out(sys);
        for (int sys = 0; sys < m->n_sys; ++sys) wout[(size_t)sys * nw + w] = tot > 0.0 ? out(sys) / tot : 0.0;
    }
    // ---- per direction: the upwind graph (periodic faces cut), the rows of
    // its sweep and the LDS slots of the values that later rows read
    const size_t npos = (size_t)n_dir * (ns + 1);
    std::vector<int> ord(npos, -1), rbase(n_dir), nrow(n_dir), nwrap(n_dir, 0), wall_ptr{0}, wall_id;
    std::vector<URow> rows;
    struct Pos { double c[UIN]; int in[UIN], out; };
    std::vector<Pos> rec(npos);
    std::vector<double> dout(npos, 1.0), wall_c;
    std::vector<uint16_t> ipos((size_t)n_dir * (ns + nw));
    std::vector<std::vector<int>> wslot_l(n_dir);
    std::vector<std::vector<double>> wdel_l(n_dir), wcut_l(n_dir);
    wall_ptr.reserve(npos + 1);
    m->nlev.assign(n_dir, 0);
    int nin_max = 2, slots_max = USLOT_WRAP;
    struct Face { int code; double c; };                  // >= 0: upwind cell; < 0: wrap slot -1 - code
    std::vector<double> dcell(ns);
    std::vector<std::array<Face, UIN>> in(ns);
    std::vector<int> nin(ns), indeg(ns), down((size_t)ns * UFACES), ndown(ns), height(ns), level(ns), last(ns), slot(ns),
        queue, wallw, walln(ns + 1), byh, hptr, free_slots;
    std::vector<double> wallc;
    for (int l = 0; l < n_dir; ++l) {
        const double s0 = dirs[2 * l], s1 = dirs[2 * l + 1];
        std::vector<int> wup;
        std::fill(dcell.begin(), dcell.end(), 0.0);
        std::fill(nin.begin(), nin.end(), 0);
        std::fill(indeg.begin(), indeg.end(), 0);
        std::fill(ndown.begin(), ndown.end(), 0);
        wallw.clear();
        wallc.clear();
        for (int i = 0; i < ns; ++i) {
            walln[i] = (int)wallw.size();
            for (int code : m->cfaces[i]) {
                double nx, ny, A;
                int j = -1, w = -1, f = -1;
                bool second = false;
                if (code < 0) {
                    w = -code - 1;
                    nx = m->wn[2 * w];
                    ny = m->wn[2 * w + 1];
                    A = m->wA[w];
                } else {
                    f = code >> 1;
                    second = code & 1;
                    const double sg = second ? -1.0 : 1.0;
                    nx = sg * m->fn[2 * f];
                    ny = sg * m->fn[2 * f + 1];
                    A = m->fA[f];
                    j = second ? m->fi[f] : m->fj[f];
                }
                const double sn = s0 * nx + s1 * ny;
                if (sn > 0.0) {
                    dcell[i] += sn * A / m->V[i];
                } else if (sn < 0.0) {
                    const double c = -sn * A / m->V[i];
                    if (w >= 0) {
                        wallw.push_back(w);
                        wallc.push_back(c);
                        continue;
                    }
                    // the face vectors of a cell add to zero, so one with four
                    // inflows has only faces along the direction: 0 to rounding
                    if (nin[i] == UIN) continue;
                    Face& fc = in[i][nin[i]++];
                    fc.c = c;
                    if (m->fper[f]) {
                        fc.code = -1 - (int)wup.size();
                        wup.push_back(j);
                        wdel_l[l].push_back((second ? -m->fdel[f] : m->fdel[f]) * m->dT);
                        // the face as kappa_face takes it: oriented from its + side
                        const double sg = m->fdel[f] > 0.0 ? 1.0 : (m->fdel[f] < 0.0 ? -1.0 : 0.0);
                        const bool up_plus = second == (sg > 0.0);
                        wcut_l[l].push_back(m->fA[f] * (sg * m->fn[2 * f]));
                        wcut_l[l].push_back(m->fA[f] * (sg * m->fn[2 * f + 1]));
                        wcut_l[l].push_back(sg != 0.0 && !up_plus ? m->dT : 0.0);
                    } else {
                        fc.code = j;
                        ++indeg[i];
                        down[(size_t)j * UFACES + ndown[j]++] = i;
                    }
                }
            }
            nin_max = std::max(nin_max, nin[i]);
        }
        walln[ns] = (int)wallw.size();
        // levels (a cell follows every upwind neighbour it reads) and heights
        // (the longest chain of cells that wait for it)
        std::fill(level.begin(), level.end(), 0);
        queue.clear();
        for (int i = 0; i < ns; ++i)
            if (indeg[i] == 0) queue.push_back(i);
        std::vector<int> wait(indeg);
        for (size_t h = 0; h < queue.size(); ++h) {
            const int u = queue[h];
            for (int k = 0; k < ndown[u]; ++k) {
                const int v = down[(size_t)u * UFACES + k];
                level[v] = std::max(level[v], level[u] + 1);
                if (--wait[v] == 0) queue.push_back(v);
            }
        }
        if ((int)queue.size() != ns)
            return ufail(OBTE_ERR_ARG, "the upwind graph of direction %d has a cycle (non-convex cells?)", l);
        int nl = 0;
        for (int h = ns - 1; h >= 0; --h) {
            const int u = queue[h];
            height[u] = 0;
            for (int k = 0; k < ndown[u]; ++k) height[u] = std::max(height[u], height[down[(size_t)u * UFACES + k]] + 1);
            nl = std::max(nl, level[u] + 1);
        }
        m->nlev[l] = nl;
        // rows: of the cells whose upwind neighbours are in earlier rows, the
        // 64 with the greatest heights (so a level wider than a wavefront
        // gives its less urgent cells to later, narrower rows)
        const size_t p0 = (size_t)l * (ns + 1);
        rbase[l] = (int)rows.size();
        std::vector<std::vector<int>> ready(nl);           // by height
        int top = 0, left = ns, p = 0, nslots = 0, r = 0;
        for (int i = 0; i < ns; ++i)
            if (indeg[i] == 0) {
                ready[height[i]].push_back(i);
                top = std::max(top, height[i]);
            }
        wait = indeg;
        std::vector<int> row_of(ns, 0), row_end;
        for (; left > 0; ++r) {
            const int b = p;
            while (p - b < 64 && top >= 0) {
                if (ready[top].empty()) {
                    --top;
                    continue;
                }
                const int i = ready[top].back();
                ready[top].pop_back();
                row_of[i] = r;
                ord[p0 + p++] = i;
            }
            std::sort(ord.begin() + p0 + b, ord.begin() + p0 + p);
            left -= p - b;
            top = std::max(top, 0);
            for (int q = b; q < p; ++q) {
                const int u = ord[p0 + q];
                for (int k = 0; k < ndown[u]; ++k) {
                    const int v = down[(size_t)u * UFACES + k];
                    if (--wait[v] == 0) {
                        ready[height[v]].push_back(v);
                        top = std::max(top, height[v]);
                    }
                }
            }
            rows.push_back({16 * b, 16 * (p - b - 1)});
            row_end.push_back(p);
        }
        nrow[l] = (r + UROWS - 1) / UROWS * UROWS;
        for (int q = r; q < nrow[l] + UROW_SLACK; ++q) rows.push_back({16 * ns, 0});
        // slots: a value is kept until the last row that reads it (which may
        // give the slot to a cell of its own: a row reads before it writes),
        // a wrap slot's upwind cell to the end
        std::fill(last.begin(), last.end(), -1);
        for (int i = 0; i < ns; ++i)
            for (int k = 0; k < ndown[i]; ++k) last[i] = std::max(last[i], row_of[down[(size_t)i * UFACES + k]]);
        for (int i : wup) last[i] = INT_MAX;
        const int nwl = (int)wup.size(), first = USLOT_WRAP + nwl;
        nwrap[l] = nwl;
        free_slots.clear();
        std::vector<std::vector<int>> ends(r);
        for (int i = 0; i < ns; ++i)
            if (last[i] >= 0 && last[i] < r) ends[last[i]].push_back(i);
        for (int q = 0, k = 0; k < r; ++k) {
            for (int i : ends[k]) free_slots.push_back(slot[i]);
            for (; q < row_end[k]; ++q) {
                const int i = ord[p0 + q];
                if (last[i] < 0) {
                    slot[i] = USLOT_TRASH;
                } else if (!free_slots.empty()) {
                    slot[i] = free_slots.back();
                    free_slots.pop_back();
                } else {
                    slot[i] = first + nslots++;
                }
                Pos& e = rec[p0 + q];
                dout[p0 + q] = dcell[i];
                for (int t = 0; t < UIN; ++t) {
                    const Face fc = t < nin[i] ? in[i][t] : Face{0, 0.0};
                    e.in[t] = t >= nin[i] ? USLOT_ZERO : (fc.code >= 0 ? slot[fc.code] : USLOT_WRAP - 1 - fc.code);
                    e.c[t] = fc.c;
                }
                e.out = slot[i];
                for (int t = walln[i]; t < walln[i + 1]; ++t) {
                    wall_id.push_back(wallw[t]);
                    wall_c.push_back(wallc[t]);
                }
                wall_ptr.push_back((int)wall_id.size());
            }
        }
        rec[p0 + ns] = {{0.0, 0.0, 0.0}, {USLOT_ZERO, USLOT_ZERO, USLOT_ZERO}, USLOT_TRASH};
        wall_ptr.push_back((int)wall_id.size());
        for (int i : wup) wslot_l[l].push_back(8 * slot[i]);
        uint16_t* pos = ipos.data() + (size_t)l * (ns + nw);
        for (int q = 0; q < ns; ++q) pos[ord[p0 + q]] = (uint16_t)q;
        for (int w = 0; w < nw; ++w) pos[ns + w] = pos[m->wcell[w]];
        slots_max = std::max(slots_max, first + nslots);
    }
    int wmax = 0;
    for (int l = 0; l < n_dir; ++l) wmax = std::max(wmax, nwrap[l]);
    if (wmax > UWPL_MAX * 64) return ufail(OBTE_ERR_ARG, "%d periodic faces in one direction (at most %d)", wmax, UWPL_MAX * 64);
    if ((size_t)(ns + wmax) * 8 > 65536)
        return ufail(OBTE_ERR_ARG, "%d solid cells and %d periodic faces exceed one workgroup's LDS", ns, wmax);
    m->wmax = std::max(wmax, 1);
    // a value that is kept has a reader (three inflows a cell at most) among
    // the cells to come, so at most 3/4 of the cells have slots at a time
    m->slots = slots_max;
    if (slots_max > 8192) return ufail(OBTE_ERR_STATE, "%d values in flight in a sweep", slots_max);
    std::vector<URec2> rec2(nin_max > 2 ? 0 : npos);
    std::vector<URec3> rec3(nin_max > 2 ? npos : 0);
    std::vector<double> c01(2 * npos);
    for (size_t q = 0; q < npos; ++q) {
        const Pos& e = rec[q];
        c01[2 * q] = e.c[0];
        c01[2 * q + 1] = e.c[1];
        if (nin_max > 2)
            rec3[q] = {e.c[2], {(uint16_t)(8 * e.in[0]), (uint16_t)(8 * e.in[1]), (uint16_t)(8 * e.in[2])},
                       (uint16_t)(8 * e.out)};
        else
            rec2[q] = {{8u * e.in[0], 8u * e.in[1]}, 8u * e.out, 0u};
    }
    std::vector<int> wslot((size_t)n_dir * m->wmax, 8 * USLOT_ZERO);
    std::vector<double> wdel((size_t)n_dir * m->wmax, 0.0), wcut(3 * (size_t)n_dir * m->wmax, 0.0);
    for (int l = 0; l < n_dir; ++l) {
        const size_t q0 = (size_t)l * m->wmax;
        std::copy(wslot_l[l].begin(), wslot_l[l].end(), wslot.begin() + q0);
        std::copy(wdel_l[l].begin(), wdel_l[l].end(), wdel.begin() + q0);
        std::copy(wcut_l[l].begin(), wcut_l[l].end(), wcut.begin() + 3 * q0);
    }
    // ---- heat conduction tables (Appendix B, volume-scaled): per cell its
    // neighbour entries with the primary coefficient a = A n.K n / (n.d),
    // the jump of the neighbour's image and the least-squares weights
    const double Kx = m->kax[0], Ky = m->kax[1];
    std::vector<int> nb_ptr(ns + 1, 0), nb_j, nb_f;
    std::vector<double> nb_a, nb_del, nb_w, P(ns, 0.0);
    std::vector<double> fa(nf), fc(2 * (size_t)nf);
    for (int f = 0; f < nf; ++f) {
        const double nx = m->fn[2 * f], ny = m->fn[2 * f + 1], dx = m->fd[2 * f], dy = m->fd[2 * f + 1];
        const double nKn = nx * nx * Kx + ny * ny * Ky, nd = nx * dx + ny * dy;
        fa[f] = m->fA[f] * nKn / nd;
        fc[2 * f] = m->fA[f] * (dx * nKn / nd - Kx * nx);
        fc[2 * f + 1] = m->fA[f] * (dy * nKn / nd - Ky * ny);
    }
    for (int i = 0; i < ns; ++i) {
        std::vector<std::array<double, 2>> dl;
        const size_t k0 = nb_j.size();
        for (int code : m->cfaces[i]) {
            if (code < 0) continue;
            const int f = code >> 1;
            const bool second = code & 1;
            const double sg = second ? -1.0 : 1.0;
            nb_j.push_back(second ? m->fi[f] : m->fj[f]);
            nb_a.push_back(fa[f]);
            const double del = sg * m->fdel[f];
            nb_del.push_back(del);
            nb_f.push_back(code);
            dl.push_back({sg * m->fd[2 * f], sg * m->fd[2 * f + 1]});
            P[i] -= fa[f] * del * m->dT;
        }
        nb_ptr[i + 1] = (int)nb_j.size();
        // least squares: g = (M^T M)^+ M^T q, M's rows the d's
        double a11 = 0.0, a12 = 0.0, a22 = 0.0;
        for (const auto& d : dl) {
            a11 += d[0] * d[0];
            a12 += d[0] * d[1];
            a22 += d[1] * d[1];
        }
        const double tr = a11 + a22, det = a11 * a22 - a12 * a12;
        double i11, i12, i22;
        if (dl.empty()) {
            i11 = i12 = i22 = 0.0;
        } else if (det > 1e-12 * tr * tr) {
            i11 = a22 / det;
            i12 = -a12 / det;
            i22 = a11 / det;
        } else {
            // rank one: the pseudo-inverse keeps the dominant eigenpair
            const double lam = 0.5 * tr + std::sqrt(std::max(0.0, 0.25 * (a11 - a22) * (a11 - a22) + a12 * a12));
            double vx = a12, vy = lam - a11;
            if (std::fabs(vx) + std::fabs(vy) == 0.0) {
                vx = lam - a22;
                vy = a12;
            }
            if (std::fabs(vx) + std::fabs(vy) == 0.0) {
                vx = 1.0;
                vy = 0.0;
            }
            const double nn = vx * vx + vy * vy;
            i11 = vx * vx / (nn * lam);
            i12 = vx * vy / (nn * lam);
            i22 = vy * vy / (nn * lam);
        }
        for (size_t k = 0; k < dl.size(); ++k) {
            nb_w.push_back(i11 * dl[k][0] + i12 * dl[k][1]);
            nb_w.push_back(i12 * dl[k][0] + i22 * dl[k][1]);
        }
        (void)k0;
    }
    // cut faces (across the periodic plane of the gradient axis), oriented
    // from the cell on the + side
    std::vector<int> cut_f, cut_s;
    std::vector<double> cut_K, cut_d, cut_A;
    for (int f = 0; f < nf; ++f) {
        if (m->fdel[f] == 0.0) continue;
        const double sg = m->fdel[f] > 0.0 ? 1.0 : -1.0;
        const double nx = sg * m->fn[2 * f], ny = sg * m->fn[2 * f + 1];
        const double dx = sg * m->fd[2 * f], dy = sg * m->fd[2 * f + 1];
        cut_f.push_back(f);
        cut_s.push_back(sg > 0 ? 1 : -1);
        cut_K.push_back((nx * nx * Kx + ny * ny * Ky) / (nx * dx + ny * dy));
        cut_K.push_back(Kx * nx);
        cut_K.push_back(Ky * ny);
        cut_d.push_back(dx);
        cut_d.push_back(dy);
        cut_A.push_back(m->fA[f]);
    }
    // ---- device tables and buffers
    obte_status s = OBTE_OK;
    UGeomDev g{};
    g.ns = ns;
    g.nwalls = nw;
    g.n_sys = m->n_sys;
    g.n_dir = n_dir;
    g.n_mfp = n_mfp;
    g.grad_axis = ga;
    g.wmax = m->wmax;
    g.nin = nin_max;
    g.dT = m->dT;
    g.Lg = m->L[ga];
    g.Vbox = m->L[0] * m->L[1];
    g.Aperp = m->L[1 - ga];
    std::vector<double> ones(ns, 1.0);
#define UP(dst, v) \
    if ((s = upload(m, dst, v)) != OBTE_OK) { free_dev(m); return s; }
#define AL(dst, n) \
    if ((s = alloc(m, dst, n)) != OBTE_OK) { free_dev(m); return s; }
    UP((double**)&g.V, m->V);
    UP((double**)&g.mfp, m->mfp);
    UP((double**)&g.Dw, m->Dw);
    UP((double**)&g.S, m->S);
    UP((double**)&g.wout, wout);
    UP(&m->wcell_d, m->wcell);
    UP((uint16_t**)&g.ipos, ipos);
    UP((int**)&g.ord, ord);
    UP((int**)&g.rbase, rbase);
    UP((int**)&g.nrow, nrow);
    UP((URow**)&g.rows, rows);
    if (nin_max > 2) {
        UP((URec3**)&g.rec, rec3);
    } else {
        UP((URec2**)&g.rec, rec2);
    }
    UP((double**)&g.c01, c01);
    UP((double**)&g.dout, dout);
    UP((int**)&g.nwrap, nwrap);
    UP((int**)&g.wslot, wslot);
    UP((double**)&g.wdel, wdel);
    UP((double**)&g.wcut, wcut);
    UP((int**)&g.wall_ptr, wall_ptr);
    UP((int**)&g.wall_id, wall_id);
    UP((double**)&g.wall_c, wall_c);
    UP(&m->sigma1, ones);
    UP(&m->scell_d, m->scell);
    AL((double**)&g.sigma, ns);
    AL(&g.T_L, ns);
    AL(&g.T_w, nw);
    AL(&g.U, (size_t)m->n_sys * m->wmax);
    AL(&g.X, (size_t)m->n_sys * (ns + 1));
    AL(&g.part, (size_t)USTRANDS * (ns + nw));
    AL(&g.kpart, (size_t)USTRANDS * ((ns + nw + UITEMS - 1) / UITEMS));
    AL(&g.kfsys, m->n_sys);
    AL(&g.iters, m->n_sys);
    AL(&g.corrected, m->n_sys);
    AL(&g.kap, 4);
    AL(&g.wres, m->n_sys);
    AL((double**)&g.pd, 2 * npos);
    AL((double**)&g.pb, 2 * npos);
    UFourierDev fdv{};
    fdv.ns = ns;
    fdv.nfaces = nf;
    fdv.grad_axis = ga;
    fdv.ncut = (int)cut_f.size();
    fdv.dT = m->dT;
    fdv.Lg = m->L[ga];
    fdv.Aperp = m->L[1 - ga];
    UP((int**)&fdv.nb_ptr, nb_ptr);
    UP((int**)&fdv.nb_j, nb_j);
    UP((double**)&fdv.nb_a, nb_a);
    std::vector<int> nb4_j((size_t)ns * UFACES, -1);
    std::vector<double> nb4_a((size_t)ns * UFACES, 0.0);
    for (int i = 0; i < ns; ++i)
        for (int k = nb_ptr[i]; k < nb_ptr[i + 1]; ++k) {
            nb4_j[(size_t)i * UFACES + k - nb_ptr[i]] = nb_j[k];
            nb4_a[(size_t)i * UFACES + k - nb_ptr[i]] = nb_a[k];
        }
    UP((int**)&fdv.nb4_j, nb4_j);
    UP((double**)&fdv.nb4_a, nb4_a);
    UP((double**)&fdv.nb_del, nb_del);
    UP((double**)&fdv.nb_w, nb_w);
    UP((int**)&fdv.nb_f, nb_f);
    UP((int**)&fdv.fi, m->fi);
    UP((int**)&fdv.fj, m->fj);
    UP((double**)&fdv.fw, m->fw);
    UP((double**)&fdv.fc, fc);
    UP((double**)&fdv.P, P);
    UP((int**)&fdv.cut_f, cut_f);
    UP((int**)&fdv.cut_s, cut_s);
    UP((double**)&fdv.cut_K, cut_K);
    UP((double**)&fdv.cut_d, cut_d);
    UP((double**)&fdv.cut_A, cut_A);
    AL(&fdv.T, ns);
    AL(&fdv.r, ns);
    AL(&fdv.p, ns);
    AL(&fdv.q, ns);
    AL(&fdv.b, ns);
    AL(&fdv.g, 2 * (size_t)ns);
    AL(&fdv.bf, nf);
    AL(&fdv.out, 4);
    AL(&fdv.r1, ns);
    AL(&fdv.w0, ns);
    AL(&fdv.w1, ns);
    AL(&fdv.s0, ns);
    AL(&fdv.s1, ns);
    AL(&fdv.tp, ns);
    AL(&fdv.dg, ns);
    AL(&fdv.fpart, (size_t)UF_SLOTS * UF_MAXB);
    AL(&fdv.fsc, UF_SCALARS);
    if (hipHostMalloc((void**)&m->h_fsc, UF_SCALARS * sizeof(double), hipHostMallocDefault) != hipSuccess) {
        m->h_fsc = nullptr;
        free_dev(m);
        return ufail(OBTE_ERR_HIP, "hipHostMalloc failed");
    }
    std::vector<UGeomDev> gv{g};
    std::vector<UFourierDev> fv{fdv};
    UP(&m->gd, gv);
    UP(&m->fdv, fv);
#undef UP
#undef AL
    m->gh = g;
    m->fh = fdv;
    m->has_material = true;
    return OBTE_OK;
}

obte_status obte_umesh_fourier(obte_umesh* m, double tol, int max_outer, double cg_tol, void* stream,
                               double* T_dev, double* kappa_F, int* outer_iters) {
    if (!m) return ufail(OBTE_ERR_ARG, "mesh is NULL");
    if (!m->has_material) return ufail(OBTE_ERR_STATE, "material not set");
    if (!(tol >= 0.0) || !(cg_tol > 0.0) || max_outer < 1) return ufail(OBTE_ERR_ARG, "need tol >= 0, cg_tol > 0, max_outer >= 1");
    hipStream_t st = (hipStream_t)stream;
    UHIP(hipMemsetAsync(m->fh.T, 0, sizeof(double) * m->ns, st));
    UHIP(hipMemsetAsync(m->fh.fsc, 0, sizeof(double) * UF_SCALARS, st));
    // conjugate gradients end in at most n steps in exact arithmetic; twice
    // that caps a solve whose tolerance sits below the rounding floor
    const int max_cg = 2 * m->ns + 50;
    // CG iterations queued per read of the stop flag (even): a read costs some
    // 20 us, an iteration past the stop 3 us
    constexpr int CG_CHUNK = 32;
    double* h = m->h_fsc;               // pinned: the loop scalars read back
    for (int outer = 1; outer <= max_outer; ++outer) {
        UHIP(ulaunch_fourier_start(m->fdv, m->ns, m->nf, st));
        for (int done = 0; !done;) {
            UHIP(ulaunch_fourier_cg(m->fdv, m->ns, CG_CHUNK, cg_tol, max_cg, st));
            UHIP(hipMemcpyAsync(h, m->fh.fsc, sizeof(double) * UF_SCALARS, hipMemcpyDeviceToHost, st));
            UHIP(hipStreamSynchronize(st));
            done = h[0] != 0.0;
        }
        UHIP(ulaunch_fourier_end(m->fdv, m->ns, tol, st));
        UHIP(hipMemcpyAsync(h, m->fh.fsc, sizeof(double) * UF_SCALARS, hipMemcpyDeviceToHost, st));
        UHIP(hipStreamSynchronize(st));
        if (h[5] != 0.0 || !std::isfinite(h[4])) break;
    }
    UHIP(ulaunch_fourier_kappa(m->fdv, m->ns, st));
    double out[4];
    UHIP(hipMemcpyAsync(out, m->fh.out, sizeof out, hipMemcpyDeviceToHost, st));
    if (T_dev) {
        UHIP(hipMemsetAsync(T_dev, 0, sizeof(double) * m->n_cells, st));
        hipLaunchKernelGGL(k_uscatter, dim3((m->ns + 255) / 256), dim3(256), 0, st, m->ns, m->scell_d, m->fh.T, T_dev, 0.0);
        UHIP(hipGetLastError());
    }
    UHIP(hipStreamSynchronize(st));
    if (kappa_F) *kappa_F = out[0];
    if (outer_iters) *outer_iters = (int)out[1];
    if (!std::isfinite(out[0])) return ufail(OBTE_ERR_NUMERIC, "non-finite heat-conduction solution");
    if ((int)out[1] >= max_outer && out[3] > tol)
        return ufail(OBTE_ERR_NOT_CONVERGED, "heat conduction: no convergence in %d outer iterations", max_outer);
    return OBTE_OK;
}

obte_status obte_umesh_solve(obte_umesh* m, const obte_solve_opts* o, const double* sigma_dev, void* stream,
                             double* T_L_dev, obte_stats* stats) {
    if (!m || !o) return ufail(OBTE_ERR_ARG, "NULL argument");
    if (!m->has_material) return ufail(OBTE_ERR_STATE, "material not set");
    if (o->precision != OBTE_FP64) return ufail(OBTE_ERR_ARG, "the unstructured path runs in FP64 (precision 0)");
    if (o->init != 0) return ufail(OBTE_ERR_ARG, "the unstructured path starts from the Fourier guess (init 0)");
    if (o->accel != 0) return ufail(OBTE_ERR_ARG, "the unstructured path runs Algorithm 1 (accel 0)");
    if (o->max_outer < 1 || !(o->outer_tol >= 0.0) || !(o->inner_tol > 0.0) || o->max_inner < 1 ||
        !(o->inner_rtol >= 0.0 && o->inner_rtol < 1.0) ||
        !(o->fourier_tol >= 0.0) || o->max_fourier < 1)
        return ufail(OBTE_ERR_ARG, "invalid tolerances or iteration caps");
    hipStream_t st = (hipStream_t)stream;
    const int ns = m->ns, nw = m->nw;
    UGeomDev& g = m->gh;
    // sigma over the solid cells
    if (sigma_dev) {
        hipLaunchKernelGGL(k_ugather, dim3((ns + 255) / 256), dim3(256), 0, st, ns, m->scell_d, sigma_dev, (double*)g.sigma);
        UHIP(hipGetLastError());
    } else {
        UHIP(hipMemcpyAsync((double*)g.sigma, m->sigma1, sizeof(double) * ns, hipMemcpyDeviceToDevice, st));
    }
    // first guess: T_L = T_F, T_w = T_F of the wall's cell
    double kF = 0.0;
    int fit = 0;
    // each conjugate-gradient solve to a hundredth of the outer tolerance
    const double cg_tol = std::max(1e-14, 1e-2 * o->fourier_tol);
    obte_status sf = obte_umesh_fourier(m, o->fourier_tol, o->max_fourier, cg_tol, stream, nullptr, &kF, &fit);
    if (sf != OBTE_OK && sf != OBTE_ERR_NOT_CONVERGED) return sf;
    UHIP(hipMemcpyAsync(g.T_L, m->fh.T, sizeof(double) * ns, hipMemcpyDeviceToDevice, st));
    if (nw > 0) {
        hipLaunchKernelGGL(k_ugather, dim3((nw + 255) / 256), dim3(256), 0, st, nw, m->wcell_d, m->fh.T, g.T_w);
        UHIP(hipGetLastError());
    }
    UHIP(hipMemsetAsync(g.U, 0, sizeof(double) * (size_t)m->n_sys * m->wmax, st));
    UHIP(hipMemsetAsync(g.iters, 0, sizeof(long long) * m->n_sys, st));
    UHIP(hipMemsetAsync(g.corrected, 0, sizeof(int) * m->n_sys, st));
    int wpl = 1;
    while (wpl * 64 < m->wmax) wpl *= 2;
    std::vector<double> hist;
    double kap[4] = {0, 0, 0, 0};
    const double wrap_tol = o->wrap_tol > 0.0 ? o->wrap_tol : std::max(o->inner_tol, 0.2 * o->outer_tol);
    bool converged = false;
    int passes = 0;
    UHIP(ulaunch_pack(m->gd, m->n_dir * (ns + 1), false, st));
    for (passes = 1; passes <= o->max_outer; ++passes) {
        UHIP(ulaunch_pass(m->gd, m->n_sys, g.nin, wpl, m->slots, o->inner_tol, o->inner_rtol, o->max_inner, st));
        UHIP(ulaunch_reduce(m->gd, ns, nw, st));
        UHIP(ulaunch_pack(m->gd, m->n_dir * (ns + 1), true, st));
        UHIP(hipMemcpyAsync(kap, g.kap, sizeof kap, hipMemcpyDeviceToHost, st));
        UHIP(hipStreamSynchronize(st));
        if (!std::isfinite(kap[0])) return ufail(OBTE_ERR_NUMERIC, "non-finite kappa in pass %d", passes);
        hist.push_back(kap[0]);
        // Algorithm 1's test, and every wrap solved to wrap_tol (a forcing
        // term leaves part of the periodic coupling to later passes)
        if (hist.size() >= 2 && std::fabs(kap[0] - hist[hist.size() - 2]) <= o->outer_tol * std::fabs(kap[0]) &&
            kap[2] <= wrap_tol) {
            converged = true;
            break;
        }
    }
    if (passes > o->max_outer) passes = o->max_outer;
    if (T_L_dev) {
        std::vector<double> tl(ns);
        UHIP(hipMemcpy(tl.data(), g.T_L, sizeof(double) * ns, hipMemcpyDeviceToHost));
        double mean = 0.0;
        for (double v : tl) mean += v;
        mean /= ns;
        UHIP(hipMemsetAsync(T_L_dev, 0, sizeof(double) * m->n_cells, st));
        hipLaunchKernelGGL(k_uscatter, dim3((ns + 255) / 256), dim3(256), 0, st, ns, m->scell_d, g.T_L, T_L_dev, mean);
        UHIP(hipGetLastError());
        UHIP(hipStreamSynchronize(st));
    }
    if (stats) {
        std::vector<long long> its(m->n_sys);
        UHIP(hipMemcpy(its.data(), g.iters, sizeof(long long) * m->n_sys, hipMemcpyDeviceToHost));
        obte_stats S{};
        S.outer_iters = passes;
        for (long long v : its) S.inner_iters += v;
        S.fourier_iters = fit;
        S.kappa = kap[0];
        S.kappa_face = kap[1];
        S.kappa_fourier = kF;
        S.wrap_residual = kap[2];
        S.last_rel_change = hist.size() >= 2 ? std::fabs(hist.back() - hist[hist.size() - 2]) / std::fabs(hist.back()) : 0.0;
        S.status = converged ? OBTE_OK : OBTE_ERR_NOT_CONVERGED;
        *stats = S;
    }
    if (!converged) return ufail(OBTE_ERR_NOT_CONVERGED, "no convergence in %d passes", o->max_outer);
    return OBTE_OK;
}

void obte_umesh_destroy(obte_umesh* m) {
    if (!m) return;
    free_dev(m);
    delete m;
}

int obte_umesh_n_solid(const obte_umesh* m) { return m ? m->ns : -1; }
int obte_umesh_n_faces(const obte_umesh* m) { return m ? m->nf : -1; }
int obte_umesh_n_walls(const obte_umesh* m) { return m ? m->nw : -1; }
int obte_umesh_n_levels(const obte_umesh* m, int l) {
    if (!m || !m->has_material || l < 0 || l >= m->n_dir) return -1;
    return m->nlev[l];
}

}  // extern "C"
