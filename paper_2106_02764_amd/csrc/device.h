// Device helpers shared by the gfx950 kernels: wavefront sums and scans,
// wave-uniform values, buffer resources, per-system constants.
#pragma once
#include "obte_internal.h"
#include <type_traits>

namespace {

constexpr int WAVE = 64;

template <typename T>
__device__ __forceinline__ T shfl_at(T v, int l) { return __shfl(v, l, WAVE); }
template <typename T>
__device__ __forceinline__ T shfl_xor(T v, int m) { return __shfl_xor(v, m, WAVE); }

// ---------------------------------------------------------------------------
// cross-lane primitives: DPP row shifts / row broadcasts / wave shift and
// v_readlane.  `old` is what a lane receives when it has no source lane.
// ---------------------------------------------------------------------------
template <int CTRL, int RM>
__device__ __forceinline__ float dpp(float v, float old) {
    return __int_as_float(__builtin_amdgcn_update_dpp(__float_as_int(old), __float_as_int(v), CTRL, RM, 0xf, false));
}
template <int CTRL, int RM>
__device__ __forceinline__ double dpp(double v, double old) {
    const long long b = __double_as_longlong(v), o = __double_as_longlong(old);
    const int lo = __builtin_amdgcn_update_dpp((int)o, (int)b, CTRL, RM, 0xf, false);
    const int hi = __builtin_amdgcn_update_dpp((int)(o >> 32), (int)(b >> 32), CTRL, RM, 0xf, false);
    return __longlong_as_double(((long long)hi << 32) | (unsigned int)lo);
}
// the same over all lanes, 0 to a lane without a source (no register is set to
// 0 before)
template <int CTRL>
__device__ __forceinline__ float dpp0(float v) {
    return __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(v), CTRL, 0xf, 0xf, true));
}
template <int CTRL>
__device__ __forceinline__ double dpp0(double v) {
    const long long b = __double_as_longlong(v);
    const int lo = __builtin_amdgcn_update_dpp(0, (int)b, CTRL, 0xf, 0xf, true);
    const int hi = __builtin_amdgcn_update_dpp(0, (int)(b >> 32), CTRL, 0xf, 0xf, true);
    return __longlong_as_double(((long long)hi << 32) | (unsigned int)lo);
}
__device__ __forceinline__ float readlane(float v, int l) {
    return __int_as_float(__builtin_amdgcn_readlane(__float_as_int(v), l));
}
__device__ __forceinline__ double readlane(double v, int l) {
    const long long b = __double_as_longlong(v);
    const int lo = __builtin_amdgcn_readlane((int)b, l), hi = __builtin_amdgcn_readlane((int)(b >> 32), l);
    return __longlong_as_double(((long long)hi << 32) | (unsigned int)lo);
}

// The masks of a row's scan (sigma = 1), from the lanes g whose cells' inflow
// along the row is open: brk[k], the lanes whose segment before scan step k has
// no closed inflow (right in the lanes that the step writes); om, the lanes
// reached from the row's start without one; nb, all ones when the row has none.
// A run of 2^k lanes by doubling; a run from a segment's start is the ones
// below the carry of + 1.
struct ScanMask {
    unsigned long long brk[6], om, nb;
};
__device__ __forceinline__ uint32_t run_up(uint32_t g) { return g & ~(g + 1u); }
__device__ __forceinline__ void scan_mask(unsigned long long g, ScanMask& m) {
    m.brk[0] = g;
    m.brk[1] = g & (g << 1);
    m.brk[2] = m.brk[1] & (m.brk[1] << 2);
    m.brk[3] = m.brk[2] & (m.brk[2] << 4);
    const uint32_t lo = (uint32_t)g, hi = (uint32_t)(g >> 32);
    m.brk[4] = ((unsigned long long)run_up(hi | 0xffffu) << 32) | run_up(lo | 0xffffu);   // read in rows 1, 3
    m.brk[5] = (unsigned long long)run_up(hi) << 32;                                      // read in rows 2, 3
    m.om = g & ~(g + 1);
    m.nb = (unsigned long long)((long long)m.om >> 63);
}

// Sum over the wave, the same value in every lane.  The lanes are combined by
// DPP row shifts and broadcasts (a step is two moves and an add, where the
// LDS permutes of a butterfly cost their latency each: the pass of a 32 x 32
// FP64 cell, whose sweeps are short, 54 -> 46.8 us), in a fixed order.
template <int CTRL, int RM, typename T>
__device__ __forceinline__ void sum_step(T& v) {
    if constexpr (RM == 0xf) v += dpp0<CTRL>(v);
    else v += dpp<CTRL, RM>(v, T(0));
}
template <typename T>
__device__ __forceinline__ T wave_sum(T v) {
    sum_step<0x111, 0xf>(v);   // row_shr:1
    sum_step<0x112, 0xf>(v);   // row_shr:2
    sum_step<0x114, 0xf>(v);   // row_shr:4
    sum_step<0x118, 0xf>(v);   // row_shr:8
    sum_step<0x142, 0xa>(v);   // row_bcast:15 into rows 1, 3
    sum_step<0x143, 0xc>(v);   // row_bcast:31 into rows 2, 3
    return readlane(v, WAVE - 1);
}

// N sums at once, step by step, so that their chains interleave; each value
// is summed exactly as wave_sum does.
template <int CTRL, int RM, int N>
__device__ __forceinline__ void sum_step_n(double (&v)[N]) {
#pragma unroll
    for (int q = 0; q < N; ++q) sum_step<CTRL, RM>(v[q]);
}
template <int N>
__device__ __forceinline__ void wave_sum_n(double (&v)[N]) {
    sum_step_n<0x111, 0xf>(v);
    sum_step_n<0x112, 0xf>(v);
    sum_step_n<0x114, 0xf>(v);
    sum_step_n<0x118, 0xf>(v);
    sum_step_n<0x142, 0xa>(v);
    sum_step_n<0x143, 0xc>(v);
#pragma unroll
    for (int q = 0; q < N; ++q) v[q] = readlane(v[q], WAVE - 1);
}

// Deterministic block sum (blockDim.x multiple of 64, <= 1024).
[[maybe_unused]] __device__ double block_sum(double v, double* red) {
    const int lane = threadIdx.x & 63, wid = threadIdx.x >> 6, nw = blockDim.x >> 6;
    v = wave_sum(v);
    __syncthreads();
    if (lane == 0) red[wid] = v;
    __syncthreads();
    double t = 0.0;
    if (wid == 0) {
        t = lane < nw ? red[lane] : 0.0;
        t = wave_sum(t);
        if (lane == 0) red[16] = t;
    }
    __syncthreads();
    return red[16];
}

// Two block sums in one pass (red: at least 34 doubles); each value is summed
// exactly as block_sum sums it.
[[maybe_unused]] __device__ void block_sum2(double& a, double& b, double* red) {
    const int lane = threadIdx.x & 63, wid = threadIdx.x >> 6, nw = blockDim.x >> 6;
    double v[2] = {a, b};
    wave_sum_n(v);
    __syncthreads();
    if (lane == 0) {
        red[wid] = v[0];
        red[16 + wid] = v[1];
    }
    __syncthreads();
    if (wid == 0) {
        double t[2] = {lane < nw ? red[lane] : 0.0, lane < nw ? red[16 + lane] : 0.0};
        wave_sum_n(t);
        if (lane == 0) {
            red[32] = t[0];
            red[33] = t[1];
        }
    }
    __syncthreads();
    a = red[32];
    b = red[33];
}

// A cell's grid coordinates (one division chain per cell), and its
// neighbour across face f (2a: '-' side of axis a, 2a + 1: '+' side) with the
// periodic wrap taken by comparison, so the per-face lookups divide nothing.
struct CellPos {
    int ix, iy, iz;
};
__device__ __forceinline__ CellPos cell_pos(const GeomDev& g, int cell) {
    const int q = cell / g.nx, r = q / g.ny;
    return {cell - q * g.nx, q - r * g.ny, r};
}
__device__ __forceinline__ int nbr_cell(const GeomDev& g, int cell, const CellPos& cp, int f) {
    const int a = f >> 1;
    const bool up = f & 1;
    const int n = a == 0 ? g.nx : (a == 1 ? g.ny : g.nz);
    const int i = a == 0 ? cp.ix : (a == 1 ? cp.iy : cp.iz);
    const int st = a == 0 ? 1 : (a == 1 ? g.nx : g.nx * g.ny);
    if (up) return i == n - 1 ? cell - (n - 1) * st : cell + st;
    return i == 0 ? cell + (n - 1) * st : cell - st;
}

using rsrc_t = __amdgpu_buffer_rsrc_t;

// Wave-uniform copies of values the compiler cannot prove uniform (loaded
// after the kernel's first store, or derived from the wave index): scalar
// registers, so the buffer resources and row offsets built from them are too.
__device__ __forceinline__ int uni(int v) { return __builtin_amdgcn_readfirstlane(v); }
__device__ __forceinline__ uint32_t uni(uint32_t v) { return (uint32_t)__builtin_amdgcn_readfirstlane((int)v); }
__device__ __forceinline__ double uni(double v) {
    const long long b = __double_as_longlong(v);
    const int lo = __builtin_amdgcn_readfirstlane((int)b), hi = __builtin_amdgcn_readfirstlane((int)(b >> 32));
    return __longlong_as_double(((long long)hi << 32) | (unsigned int)lo);
}
__device__ __forceinline__ float uni(float v) { return __int_as_float(__builtin_amdgcn_readfirstlane(__float_as_int(v))); }
template <typename P>
__device__ __forceinline__ P* uni(P* p) {
    const unsigned long long a = (unsigned long long)p;
    const unsigned lo = (unsigned)__builtin_amdgcn_readfirstlane((int)(unsigned)a);
    const unsigned hi = (unsigned)__builtin_amdgcn_readfirstlane((int)(unsigned)(a >> 32));
    return (P*)(((unsigned long long)hi << 32) | lo);
}

__device__ __forceinline__ rsrc_t make_rsrc(const void* p, uint32_t bytes) {
    return __builtin_amdgcn_make_buffer_rsrc(const_cast<void*>(uni(p)), 0, (int)uni(bytes), 0x00020000);
}

// Upper bound of the gain of a system's wrap map G (inflow of the first row
// -> mask * c_y * outflow of the last row, sources zero).  One row of the
// sweep solves (D - C_in) x = c_y y, where D = sigma + sum c and C_in holds
// the in-row (x, and z in 3D) upwind couplings: an M-matrix whose rows and
// columns both exceed their off-diagonal sums by at least sigma_min + c_y.
// So every row transfer has max- and 1-norm (hence 2-norm) at most
// q = c_y / (sigma_min + c_y), walls and pores only lower it, and
// |G r| <= q^ny |r| for the BiCGSTAB's 2-norm.  1 when sigma_min <= 0.
// The sweep-free step is taken only where it cuts the wrap residual at least
// tenfold: with a weaker cut (up to the forcing term 0.3) the mixed outer
// iteration needed more passes (22 -> 26 on the 128x128 cell), which cost
// more than the sweeps saved.
constexpr double RICH_MAX = 0.1;

__device__ __forceinline__ double wrap_gain_bound(double smin, double cy, int ny) {
    if (!(smin > 0.0)) return 1.0;
    return pow(cy / (smin + cy), (double)ny);
}

template <typename T>
__device__ __forceinline__ const T* sigma_ptr(const GeomDev& g);
template <>
__device__ __forceinline__ const double* sigma_ptr<double>(const GeomDev& g) { return g.sigma; }
template <>
__device__ __forceinline__ const float* sigma_ptr<float>(const GeomDev& g) { return g.sigma_f; }


// Loads through these views compile to global (not flat) loads, which keep
// only the vector-memory counter pending while the row computes.
template <typename T>
using gptr_t = const __attribute__((address_space(1))) T*;
template <typename T>
__device__ __forceinline__ gptr_t<T> gview(const T* p) { return (gptr_t<T>)p; }
// Writable global views: stores through them are global (not flat) stores,
// which a barrier's wait on the LDS counter does not include.
template <typename T>
using gmut_t = __attribute__((address_space(1))) T*;
template <typename T>
__device__ __forceinline__ gmut_t<T> gmut(T* p) { return (gmut_t<T>)p; }

// Raw buffer access (gfx9 descriptors): a resource for the whole array, a
// per-lane byte offset fixed for the sweep and a scalar offset per row, so a
// row's loads need no per-lane address arithmetic.  A raw buffer access is
// range-checked on its per-lane offset: a store whose offset is at or past
// the array's size is dropped (used for pores and beyond-row lanes).
constexpr uint32_t BUF_OOB = 0x80000000u;
typedef unsigned int u32x2_t __attribute__((ext_vector_type(2)));
__device__ __forceinline__ uint32_t bld32(rsrc_t r, uint32_t vo, uint32_t so) {
    return __builtin_amdgcn_raw_buffer_load_b32(r, (int)vo, (int)so, 0);
}
__device__ __forceinline__ double bld64(rsrc_t r, uint32_t vo, uint32_t so) {
    const u32x2_t v = __builtin_amdgcn_raw_buffer_load_b64(r, (int)vo, (int)so, 0);
    return __longlong_as_double(((long long)v.y << 32) | (unsigned long long)v.x);
}
template <typename T>
__device__ __forceinline__ T bldT(rsrc_t r, uint32_t vo, uint32_t so);
template <>
__device__ __forceinline__ float bldT<float>(rsrc_t r, uint32_t vo, uint32_t so) {
    return __uint_as_float(bld32(r, vo, so));
}
template <>
__device__ __forceinline__ double bldT<double>(rsrc_t r, uint32_t vo, uint32_t so) {
    return bld64(r, vo, so);
}
// the same past the caches
__device__ __forceinline__ void bst_nt(float v, rsrc_t r, uint32_t vo) {
    __builtin_amdgcn_raw_buffer_store_b32(__float_as_uint(v), r, (int)vo, 0, 2);
}
__device__ __forceinline__ void bst_nt(double v, rsrc_t r, uint32_t vo) {
    const unsigned long long b = (unsigned long long)__double_as_longlong(v);
    u32x2_t w;
    w.x = (unsigned int)b;
    w.y = (unsigned int)(b >> 32);
    __builtin_amdgcn_raw_buffer_store_b64(w, r, (int)vo, 0, 2);
}
__device__ __forceinline__ void bst(float v, rsrc_t r, uint32_t vo) {
    __builtin_amdgcn_raw_buffer_store_b32(__float_as_uint(v), r, (int)vo, 0, 0);
}
__device__ __forceinline__ void bst(double v, rsrc_t r, uint32_t vo) {
    const unsigned long long b = (unsigned long long)__double_as_longlong(v);
    u32x2_t w;
    w.x = (unsigned int)b;
    w.y = (unsigned int)(b >> 32);
    __builtin_amdgcn_raw_buffer_store_b64(w, r, (int)vo, 0, 0);
}

// 1/d: hardware reciprocal (float), refined by two Newton steps (double).
__device__ __forceinline__ float recip(float d) { return __builtin_amdgcn_rcpf(d); }
__device__ __forceinline__ double recip(double d) {
    double r = __builtin_amdgcn_rcp(d);
    r = r * (2.0 - d * r);
    return r * (2.0 - d * r);
}

}  // namespace
