// Row inputs, lane masks and the row recurrence shared by the 2D and 3D pass
// kernels.
#pragma once
#include "device.h"

namespace {

typedef unsigned int u32x3_t __attribute__((ext_vector_type(3)));
typedef unsigned int u32x4_t __attribute__((ext_vector_type(4)));
// N consecutive dwords at one lane offset, in loads of at most four dwords
template <int N>
__device__ __forceinline__ void bld_dw(uint32_t (&d)[N], rsrc_t r, uint32_t vo, uint32_t so) {
#pragma unroll
    for (int i = 0; i < N; i += 4) {
        const int n = N - i < 4 ? N - i : 4;
        const uint32_t o = vo + 4u * (uint32_t)i;
        if (n == 4) {
            const u32x4_t v = __builtin_amdgcn_raw_buffer_load_b128(r, (int)o, (int)so, 0);
            d[i] = v.x; d[i + 1] = v.y; d[i + 2] = v.z; d[i + 3] = v.w;
        } else if (n == 3) {
            const u32x3_t v = __builtin_amdgcn_raw_buffer_load_b96(r, (int)o, (int)so, 0);
            d[i] = v.x; d[i + 1] = v.y; d[i + 2] = v.z;
        } else if (n == 2) {
            const u32x2_t v = __builtin_amdgcn_raw_buffer_load_b64(r, (int)o, (int)so, 0);
            d[i] = v.x; d[i + 1] = v.y;
        } else {
            d[i] = __builtin_amdgcn_raw_buffer_load_b32(r, (int)o, (int)so, 0);
        }
    }
}
template <typename T>
__device__ __forceinline__ T from_dw(const uint32_t* d);
template <>
__device__ __forceinline__ float from_dw<float>(const uint32_t* d) { return __uint_as_float(d[0]); }
template <>
__device__ __forceinline__ double from_dw<double>(const uint32_t* d) {
    return __longlong_as_double(((long long)d[1] << 32) | (unsigned long long)d[0]);
}
template <typename T, int CPL>
__device__ __forceinline__ void bld_T(T (&v)[CPL], rsrc_t r, uint32_t vo, uint32_t so) {
    uint32_t d[CPL * sizeof(T) / 4];
    bld_dw<CPL * (int)sizeof(T) / 4>(d, r, vo, so);
#pragma unroll
    for (int c = 0; c < CPL; ++c) v[c] = from_dw<T>(d + c * sizeof(T) / 4);
}

// ---------------------------------------------------------------------------
// lane masks of a row (tables of k_row_masks, read through the scalar cache)
// ---------------------------------------------------------------------------
using mask_t = unsigned long long;
using mview_t = const __attribute__((address_space(4))) mask_t*;
__device__ __forceinline__ bool lane_in(mask_t m) { return __builtin_amdgcn_inverse_ballot_w64(m); }
template <typename T>
__device__ __forceinline__ T sel0(mask_t m, T v) { return lane_in(m) ? v : T(0); }
// zero, or so small that it only scales terms it makes negligible (the low
// word stays: below 1e-300)
__device__ __forceinline__ float selw(mask_t m, float v) { return lane_in(m) ? v : 0.0f; }
__device__ __forceinline__ double selw(mask_t m, double v) {
    const long long b = __double_as_longlong(v);
    const int hi = lane_in(m) ? (int)(b >> 32) : 0;
    return __longlong_as_double(((long long)hi << 32) | (unsigned int)(int)b);
}

// What a sweep reads of a row's masks (k_row_masks).  xo / yo / zo: cells whose
// inflow along the row / across the rows / through the planes (3D) is open; sol
// (adjoint): solid cells; SCAN: the scan's masks.
//
// With sigma = 1 the scan's eight masks are formed from the open lanes in some
// 20 scalar instructions.  Loading them was cheaper to issue, but a row's line
// then came from the L2 (64 x 256 cells: 22 KB an orientation, and two CUs
// share 16 KB of scalar cache), and as the loads sat next to their use its
// latency was in the chain of every row.  With the few words left, asked for at
// the start of a row: 64 x 256, 48 x 30 systems, FP32: 97 -> 66 us a launch;
// 150 x 109 with a sigma field, 36 x 22 systems, FP32: 149 -> 99 us.
// Rows of 3 and 4 cells per lane in 3D FP32 keep the scan's masks loaded: two
// waves a SIMD do not hide the scalar instructions (256 x 16 x 6, 72 x 12
// systems: 3.47 against 3.65 ms for 6 passes; in FP64, with twice the vector
// instructions, 4.16 against 4.18).
template <int CPL, bool ADJB, bool D3 = false, bool SCAN = false>
struct RowBits {
    mask_t xo[CPL], yo[CPL], zo[D3 ? CPL : 1], sol[ADJB ? CPL : 1];
    mask_t sc[SCAN ? 8 : 1];
};
template <int CPL, bool ADJB, bool D3, bool SCAN>
__device__ __forceinline__ void load_bits(mview_t row, RowBits<CPL, ADJB, D3, SCAN>& m) {
#pragma unroll
    for (int c = 0; c < CPL; ++c) {
        m.xo[c] = row[c];
        m.yo[c] = row[CPL + c];
        if (D3) m.zo[c] = row[2 * CPL + c];
        if (ADJB) m.sol[c] = row[(D3 ? 3 : 2) * CPL + c];
    }
    if (SCAN)
#pragma unroll
        for (int k = 0; k < 8; ++k) m.sc[k] = row[4 * CPL + k];
    // the loads stay here, ahead of their use (to save registers the scheduler
    // would move them next to it, and their latency would be in the chain).
    // 3D: vector instructions may cross, its other waves fill the wait
    if constexpr (D3)
        __builtin_amdgcn_sched_barrier(0x2 | 0x4 | 0x10 | 0x20 | 0x40 | 0x80 | 0x100 | 0x200);
    else
        __builtin_amdgcn_sched_barrier(0);
}
// The wait for a row's bits (2D): before the next row's are asked for, as
// scalar loads come back in any order and a wait is for all of them.
template <int CPL, bool ADJB>
__device__ __forceinline__ void need_bits(const RowBits<CPL, ADJB>& m) {
    asm volatile("" ::"s"(m.xo[0]));
    __builtin_amdgcn_sched_barrier(0);
}
template <int CPL, bool ADJB, bool D3, bool SCAN>
__device__ __forceinline__ void scan_mask(const RowBits<CPL, ADJB, D3, SCAN>& b, ScanMask& m) {
    if constexpr (SCAN) {
#pragma unroll
        for (int k = 0; k < 6; ++k) m.brk[k] = b.sc[k];
        m.om = b.sc[6];
        m.nb = b.sc[7];
    } else {
        mask_t g = b.xo[0];
#pragma unroll
        for (int c = 1; c < CPL; ++c) g &= b.xo[c];
        scan_mask(g, m);
    }
}

// ---------------------------------------------------------------------------
// The row recurrence x_i = a_i + q_i x_{i-1} (cyclic).
//
// sigma = 1: q is this system's constant wherever the inflow is open, so the
// scan's weights (Q of the segment a lane holds before each step) are powers
// of q, zero where the segment holds a closed face: constants selected by the
// row's masks.  Only the affine part is scanned: 35 vector instructions per
// FP32 row of 2 cells per lane, against 57 when Q is scanned along.  The powers
// are formed in double from P = 1 - Q by P_{a+b} = P_a + (1 - P_a) P_b, which keeps P's
// relative accuracy where it is small (the closure divides by it).
// ---------------------------------------------------------------------------
template <typename T, int CPL, bool FULL>
struct QConst {
    T q, rdv;               // Q and 1 / diagonal of an open cell
    T tk[6];                // Q of a lane's segment before each scan step
    T om;                   // Q from the row's start through this lane
    T rpt;                  // 1 / (1 - Q of the whole row)
    T qc[FULL ? 1 : CPL];   // Q of this lane's cells (1 in the padding, which only passes the closure on)
    T val[FULL ? 1 : CPL];  // 1 for the row's cells, 0 for the padding
};

__device__ __forceinline__ double p_power(const double (&pb)[9], int n) {
    double p = 0.0;
#pragma unroll
    for (int b = 0; b < 9; ++b) p = ((n >> b) & 1) ? p + (1.0 - p) * pb[b] : p;
    return p;
}

// c0: Lambda |s_a| / h_a along the row, c1: the sum over the other axes
template <typename T, int CPL, bool S1, bool FULL>
__device__ __forceinline__ void make_qconst(double c0, double c1, int nr, int lane, QConst<T, CPL, FULL>& k) {
    if (S1) {
        const double rd = 1.0 / (1.0 + c0 + c1);
        double pb[9];
        pb[0] = (1.0 + c1) * rd;
#pragma unroll
        for (int b = 1; b < 9; ++b) pb[b] = pb[b - 1] * (2.0 - pb[b - 1]);
        k.q = (T)(c0 * rd);
        k.rdv = (T)rd;
#pragma unroll
        for (int b = 0; b < 4; ++b) k.tk[b] = (T)(1.0 - p_power(pb, CPL << b));
        k.tk[4] = (T)(1.0 - p_power(pb, CPL * ((lane & 15) + 1)));
        k.tk[5] = (T)(1.0 - p_power(pb, CPL * ((lane & 31) + 1)));
        const int upto = (lane + 1) * CPL - (WAVE * CPL - nr);
        k.om = (T)(1.0 - p_power(pb, upto > 0 ? upto : 0));
        k.rpt = (T)(1.0 / p_power(pb, nr));
    }
    if (!FULL) {
#pragma unroll
        for (int c = 0; c < CPL; ++c) {
            const bool in = lane * CPL + c >= WAVE * CPL - nr;
            k.val[c] = in ? T(1) : T(0);
            if (S1) k.qc[c] = in ? k.q : T(1);
        }
    }
}

// sigma = 1: scan of the affine parts A with the weights selected by the
// masks; returns Q from the row's start (for the closure).
template <int CPL, bool FULL>
__device__ __forceinline__ double ascan(double& A, const QConst<double, CPL, FULL>& k, const ScanMask& m) {
    A = A + selw(m.brk[0], k.tk[0]) * dpp0<0x111>(A);   // row_shr:1
    A = A + selw(m.brk[1], k.tk[1]) * dpp0<0x112>(A);   // row_shr:2
    A = A + selw(m.brk[2], k.tk[2]) * dpp0<0x114>(A);   // row_shr:4
    A = A + selw(m.brk[3], k.tk[3]) * dpp0<0x118>(A);   // row_shr:8
    A = A + selw(m.brk[4], k.tk[4]) * dpp<0x142, 0xa>(A, 0.0);   // row_bcast:15 into rows 1, 3
    A = A + selw(m.brk[5], k.tk[5]) * dpp<0x143, 0xc>(A, 0.0);   // row_bcast:31 into rows 2, 3
    return selw(m.om, k.om);
}
// FP32: the DPP read folded into v_fmac (the compiler does not fold its own
// moves); a DPP read needs two wait states after the write of its register,
// filled with the next weights' selects where there are any.  So does a select
// after a vector instruction that wrote its mask (one that the compiler reloads
// by v_readlane, which it may put right before the block: hence the first s_nop).
template <int CPL, bool FULL>
__device__ __forceinline__ float ascan(float& A, const QConst<float, CPL, FULL>& k, const ScanMask& m) {
    float t0, t1, om;
    asm("s_nop 1\n\t"
        "v_cndmask_b32_e64 %1, 0, %4, %11\n\t"
        "v_cndmask_b32_e64 %2, 0, %5, %12\n\t"
        "v_fmac_f32_dpp %0, %0, %1 row_shr:1 row_mask:0xf bank_mask:0xf bound_ctrl:1\n\t"
        "v_cndmask_b32_e64 %1, 0, %6, %13\n\t"
        "s_nop 0\n\t"
        "v_fmac_f32_dpp %0, %0, %2 row_shr:2 row_mask:0xf bank_mask:0xf bound_ctrl:1\n\t"
        "v_cndmask_b32_e64 %2, 0, %7, %14\n\t"
        "s_nop 0\n\t"
        "v_fmac_f32_dpp %0, %0, %1 row_shr:4 row_mask:0xf bank_mask:0xf bound_ctrl:1\n\t"
        "v_cndmask_b32_e64 %1, 0, %8, %15\n\t"
        "s_nop 0\n\t"
        "v_fmac_f32_dpp %0, %0, %2 row_shr:8 row_mask:0xf bank_mask:0xf bound_ctrl:1\n\t"
        "v_cndmask_b32_e64 %2, 0, %9, %16\n\t"
        "v_cndmask_b32_e64 %3, 0, %10, %17\n\t"
        "v_fmac_f32_dpp %0, %0, %1 row_bcast:15 row_mask:0xa bank_mask:0xf\n\t"
        "s_nop 1\n\t"
        "v_fmac_f32_dpp %0, %0, %2 row_bcast:31 row_mask:0xc bank_mask:0xf"
        : "+v"(A), "=&v"(t0), "=&v"(t1), "=&v"(om)
        : "v"(k.tk[0]), "v"(k.tk[1]), "v"(k.tk[2]), "v"(k.tk[3]), "v"(k.tk[4]), "v"(k.tk[5]), "v"(k.om),
          "s"(m.brk[0]), "s"(m.brk[1]), "s"(m.brk[2]), "s"(m.brk[3]), "s"(m.brk[4]), "s"(m.brk[5]), "s"(m.om));
    return om;
}

// A sigma field: the part of a row's maps that depends neither on the sources
// nor on the row below (Q and 1 / diagonal of each cell, the scan weights
// t_k = 1 - P before step k, 1 - P of the inclusive map, 1 / P of the row),
// taken one row ahead so that the chain from one row's solution to the next
// holds only the A half of the scan.
template <typename T, int CPL>
struct QPart {
    T q[CPL];
    T rdv[CPL];
    T t[6];
    T omP;
    T rPt;
};
template <typename T, int CPL, bool FULL, bool ADJB, bool D3>
__device__ __forceinline__ T qpart_cells(T c0, T c1, const QConst<T, CPL, FULL>& k, const RowBits<CPL, ADJB, D3>& m,
                                         const T (&sg)[CPL], QPart<T, CPL>& o) {
    const T cdiag = c0 + c1;
    T Pl;
#pragma unroll
    for (int c = 0; c < CPL; ++c) {
        const T rdv = recip(sg[c] + cdiag);
        const bool open = lane_in(m.xo[c]);
        T qv = open ? c0 * rdv : T(0);           // x inflow closed (wall, pore): Q = 0, P = 1
        T pv = open ? (sg[c] + c1) * rdv : T(1);
        if (!FULL) {
            // padding in front of the row: the identity (Q, P) = (1, 0)
            qv = k.val[c] != T(0) ? qv : T(1);
            pv = k.val[c] != T(0) ? pv : T(0);
        }
        o.q[c] = qv;
        o.rdv[c] = rdv;
        Pl = c == 0 ? pv : pv + qv * Pl;
    }
    return Pl;
}
template <typename T, int CPL>
__device__ __forceinline__ void qpart_close(T P, QPart<T, CPL>& o) {
    const T Pt = readlane(P, WAVE - 1);
    o.rPt = Pt > T(0) ? recip(Pt) : T(0);
    o.omP = T(1) - P;
}
// The P half of the scan alone (the first row of a sweep), recording t_k.
template <typename T>
__device__ __forceinline__ void pscan(T& P, T (&t)[6]) {
    t[0] = T(1) - P; P = P + t[0] * dpp0<0x111>(P);   // row_shr:1
    t[1] = T(1) - P; P = P + t[1] * dpp0<0x112>(P);   // row_shr:2
    t[2] = T(1) - P; P = P + t[2] * dpp0<0x114>(P);   // row_shr:4
    t[3] = T(1) - P; P = P + t[3] * dpp0<0x118>(P);   // row_shr:8
    t[4] = T(1) - P; P = P + t[4] * dpp<0x142, 0xa>(P, T(0));   // row_bcast:15 into rows 1, 3
    t[5] = T(1) - P; P = P + t[5] * dpp<0x143, 0xc>(P, T(0));   // row_bcast:31 into rows 2, 3
}
// This row's A scan with its recorded weights t, and the next row's P scan
// recording tn (the two chains interleave).
template <typename T>
__device__ __forceinline__ void scan_pair(T& A, const T (&t)[6], T& P, T (&tn)[6]) {
    tn[0] = T(1) - P; A = A + t[0] * dpp0<0x111>(A); P = P + tn[0] * dpp0<0x111>(P);
    tn[1] = T(1) - P; A = A + t[1] * dpp0<0x112>(A); P = P + tn[1] * dpp0<0x112>(P);
    tn[2] = T(1) - P; A = A + t[2] * dpp0<0x114>(A); P = P + tn[2] * dpp0<0x114>(P);
    tn[3] = T(1) - P; A = A + t[3] * dpp0<0x118>(A); P = P + tn[3] * dpp0<0x118>(P);
    tn[4] = T(1) - P; A = A + t[4] * dpp<0x142, 0xa>(A, T(0)); P = P + tn[4] * dpp<0x142, 0xa>(P, T(0));
    tn[5] = T(1) - P; A = A + t[5] * dpp<0x143, 0xc>(A, T(0)); P = P + tn[5] * dpp<0x143, 0xc>(P, T(0));
}
// FP32: the same with the DPP read folded into v_fmac (as in
// ascan); each accumulator's DPP read comes two instructions after its last write.
__device__ __forceinline__ void scan_pair(float& A, const float (&t)[6], float& P, float (&tn)[6]) {
    asm volatile(
        "s_nop 1\n\t"
        "v_sub_f32 %2, 1.0, %1\n\t"
        "v_fmac_f32_dpp %0, %0, %8 row_shr:1 row_mask:0xf bank_mask:0xf bound_ctrl:1\n\t"
        "v_fmac_f32_dpp %1, %1, %2 row_shr:1 row_mask:0xf bank_mask:0xf bound_ctrl:1\n\t"
        "v_sub_f32 %3, 1.0, %1\n\t"
        "v_fmac_f32_dpp %0, %0, %9 row_shr:2 row_mask:0xf bank_mask:0xf bound_ctrl:1\n\t"
        "v_fmac_f32_dpp %1, %1, %3 row_shr:2 row_mask:0xf bank_mask:0xf bound_ctrl:1\n\t"
        "v_sub_f32 %4, 1.0, %1\n\t"
        "v_fmac_f32_dpp %0, %0, %10 row_shr:4 row_mask:0xf bank_mask:0xf bound_ctrl:1\n\t"
        "v_fmac_f32_dpp %1, %1, %4 row_shr:4 row_mask:0xf bank_mask:0xf bound_ctrl:1\n\t"
        "v_sub_f32 %5, 1.0, %1\n\t"
        "v_fmac_f32_dpp %0, %0, %11 row_shr:8 row_mask:0xf bank_mask:0xf bound_ctrl:1\n\t"
        "v_fmac_f32_dpp %1, %1, %5 row_shr:8 row_mask:0xf bank_mask:0xf bound_ctrl:1\n\t"
        "v_sub_f32 %6, 1.0, %1\n\t"
        "v_fmac_f32_dpp %0, %0, %12 row_bcast:15 row_mask:0xa bank_mask:0xf\n\t"
        "v_fmac_f32_dpp %1, %1, %6 row_bcast:15 row_mask:0xa bank_mask:0xf\n\t"
        "v_sub_f32 %7, 1.0, %1\n\t"
        "v_fmac_f32_dpp %0, %0, %13 row_bcast:31 row_mask:0xc bank_mask:0xf\n\t"
        "v_fmac_f32_dpp %1, %1, %7 row_bcast:31 row_mask:0xc bank_mask:0xf"
        : "+v"(A), "+v"(P), "=&v"(tn[0]), "=&v"(tn[1]), "=&v"(tn[2]), "=&v"(tn[3]), "=&v"(tn[4]), "=&v"(tn[5])
        : "v"(t[0]), "v"(t[1]), "v"(t[2]), "v"(t[3]), "v"(t[4]), "v"(t[5]));
}

}  // namespace
