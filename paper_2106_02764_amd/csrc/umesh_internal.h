// Internal types of the unstructured-mesh path, shared by its host driver
// (umesh.cpp) and its gfx950 kernels (ukernels.hip).
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

// At most four faces per cell (triangles and quadrilaterals).
constexpr int UFACES = 4;
// Inflow faces of a cell that read a solution value (walls are part of the
// source): two in a triangle, three in a quadrilateral.
constexpr int UIN = 3;
// Rows of a sweep in flight (row counts are multiples of it), and the row
// descriptors that may be read past a direction's last row.
constexpr int UROWS = 8;
constexpr int UROW_SLACK = 2 * UROWS;
// LDS slots of a system's sweep: one that holds 0 (read by unused inflows),
// one that is only written, the wrap inflow, then the values of the cells
// that a later row still reads.
constexpr int USLOT_ZERO = 0, USLOT_TRASH = 1, USLOT_WRAP = 2;
// Wrap slots per wave lane the pass kernel keeps in registers.
constexpr int UWPL_MAX = 8;

// What a sweep reads of a cell besides its first two inflow coefficients and
// sigma: the LDS byte offsets of its inflows' values and of its own, and the
// third inflow's coefficient.
struct alignas(16) URec2 {
    uint32_t in[2], out, pad;
};
struct alignas(16) URec3 {
    double c2;
    uint16_t in[3], out;
};
static_assert(sizeof(URec2) == 16 && sizeof(URec3) == 16, "one 16-byte load");
// A row: the byte offsets (16 a cell) of its first position, and of its last
// cell from there.
struct alignas(8) URow {
    int base, last;
};

// The sums over the systems: their systems in UQ chunks of four strands each
// (one workgroup a strand), UITEMS cells and wall faces a workgroup.
constexpr int UQ = 16, USTRANDS = 4 * UQ, URED_THREADS = 1024, UITEMS_PER = 3, UITEMS = URED_THREADS * UITEMS_PER;

struct UGeomDev {
    int ns, nwalls, n_sys, n_dir, n_mfp, grad_axis;
    int wmax;                 // wrap slots of the direction with the most
    int nin;                  // 2 or 3: inflows of the cell with the most
    double dT, Lg, Vbox, Aperp;
    // ---- static tables
    const double* V;          // ns: cell areas
    const double* mfp;        // n_mfp
    const double* Dw;         // n_sys: T_L weights
    const double* S;          // 2 * n_sys: flux weights
    const double* wout;       // n_sys * nwalls: outgoing weights of each wall face
    const uint16_t* ipos;     // n_dir * (ns + nwalls): sweep position of each cell and of each wall face's cell
    // sweep tables per direction l: the cells in rows of at most 64 that read
    // only cells of earlier rows
    // (n_pos = n_dir * (ns + 1): each direction's last position is a cell of
    // no effect, which rows past the direction's end sweep)
    const int* ord;           // n_pos: cell at each sweep position, -1 at the last
    const int* rbase;         // n_dir: start of direction l's rows
    const int* nrow;          // n_dir: rows (a multiple of UROWS)
    const URow* rows;
    const void* rec;          // n_pos: URec2 (nin 2) or URec3
    const double2* c01;       // n_pos: |s.n| A / V of the first two inflows
    const double* dout;       // n_pos: sum of the outflow |s.n| A / V
    const int* nwrap;         // n_dir: wrap slots of direction l
    const int* wslot;         // n_dir * wmax: LDS byte offset of each wrap slot's upwind cell
    const double* wdel;       // n_dir * wmax: jump of the value crossing (delta dT)
    const double* wcut;       // 3 * n_dir * wmax: A_f n_f of a face across the periodic plane of the
                              // gradient axis (n_f from its + side; 0 elsewhere), and the jump there
    const int* wall_ptr;      // n_pos + 1: the inflow walls of each position
    const int* wall_id;       // their wall faces
    const double* wall_c;     // their |s.n| A / V
    // ---- solve state (library-owned buffers)
    const double* sigma;      // ns
    double* T_L;              // ns
    double* T_w;              // nwalls
    double* U;                // n_sys * wmax: wrap inflow values
    double* X;                // n_sys * (ns + 1): each system's solution of the pass, by sweep position
    double* part;             // USTRANDS * (ns + nwalls): the strands' sums
    double* kpart;            // USTRANDS per UITEMS items: their share of kappa_cc
    double* kfsys;            // n_sys: kappa_face share
    long long* iters;         // n_sys: accumulated BiCGSTAB iterations
    double* kap;              // 4: kappa_cc, kappa_face of the pass, max relative wrap residual
    int* corrected;           // n_sys: whether the last pass corrected the system's wrap inflow
    double* wres;             // n_sys: relative wrap residual after the pass
    // ---- per pass, in every direction's sweep order (k_upack): sigma of the
    // cell at each position and its outflow sum; sigma T_L and the sum over its
    // inflow wall faces of |s.n| A / V T_w (the wall part of the source before
    // the factor Lambda)
    double2* pd;              // n_pos
    double2* pb;              // n_pos
};

struct UFourierDev {
    int ns, nfaces, grad_axis, ncut;
    double dT, Lg, Aperp;
    const int* nb_ptr;        // ns + 1: neighbour lists (both sides of every interior face)
    const int* nb_j;          // neighbour cell
    const double* nb_a;       // primary coefficient A_f n.K n / (n.d)
    const int* nb4_j;         // UFACES * ns: the neighbours again, -1 past a cell's last
    const double* nb4_a;      // their coefficients
    const double* nb_del;     // jump of the neighbour's image seen from the cell
    const double* nb_w;       // 2 per entry: least-squares weight column of the entry
    const int* nb_f;          // face index * 2 + (1 if the cell is the face's second cell)
    const int* fi;            // nfaces
    const int* fj;
    const double* fw;         // interpolation weight of the second cell's gradient
    const double* fc;         // 2 * nfaces: the secondary-flux vector c_f (first cell's side)
    const double* P;          // ns: perturbation (volume-scaled)
    const int* cut_f;         // ncut: face index of each cut face
    const int* cut_s;         // ncut: +1 if the face's first cell is on the + side, else -1
    const double* cut_K;      // 3 * ncut: n.K n / (n.d), (K n)_x, (K n)_y of the + side orientation
    const double* cut_d;      // 2 * ncut: d from the + side cell
    const double* cut_A;      // ncut
    // scratch (ns each) and outputs
    double* T;                // ns: the solution (mean zero)
    double* r;
    double* p;
    double* q;
    double* b;
    double* g;                // 2 * ns: cell gradients
    double* bf;               // nfaces: secondary flux per face
    double* out;              // 4: kappa_F, outer iterations, CG iterations, last relative change
    // multi-block solve: the second direction buffer, the previous outer
    // iterate, the diagonal, per-block partial sums and loop scalars
    double* r1;               // ns: r, A M^-1 r (w) and A p (s) by CG iteration parity
    double* w0;
    double* w1;
    double* s0;
    double* s1;
    double* tp;               // ns
    double* dg;               // ns
    double* fpart;            // UF_SLOTS * UF_MAXB
    double* fsc;              // UF_SCALARS
};
constexpr int UF_MAXB = 64;   // blocks of the multi-block heat-conduction kernels (256 cells each)
constexpr int UF_SLOTS = 10;
constexpr int UF_SCALARS = 16;

// Heat conduction, Eq. (final2), over several blocks: the start of an outer
// iteration (gradients, secondary fluxes, right-hand side, first residual),
// `iters` CG iterations (one kernel each; they return at once once the CG
// has stopped, which fsc[0] says), and the end of an outer iteration (mean
// removed, the change against the previous iterate in fsc[4], fsc[5] = 1 when
// it is within tol); then kappa_F and the statistics into out.
hipError_t ulaunch_fourier_start(const UFourierDev* f_dev, int ns, int nfaces, hipStream_t st);
hipError_t ulaunch_fourier_cg(const UFourierDev* f_dev, int ns, int iters, double cg_tol, int max_cg,
                              hipStream_t st);
hipError_t ulaunch_fourier_end(const UFourierDev* f_dev, int ns, double tol, hipStream_t st);
hipError_t ulaunch_fourier_kappa(const UFourierDev* f_dev, int ns, hipStream_t st);
// The sources of the next pass packed in sweep order (n_pos =
// n_dir * (n_solid + 1) positions) and, with_kappa, the sums of the pass before.
hipError_t ulaunch_pack(const UGeomDev* g_dev, int n_pos, bool with_kappa, hipStream_t st);
// every system's pass; slots: LDS slots of a system
hipError_t ulaunch_pass(const UGeomDev* g_dev, int n_sys, int nin, int wpl, int slots, double inner_tol,
                        double inner_rtol, int max_inner, hipStream_t st);
// T_L, T_w and the parts of kappa from the systems' solutions
hipError_t ulaunch_reduce(const UGeomDev* g_dev, int ns, int nwalls, hipStream_t st);
