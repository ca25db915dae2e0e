// lanes.hpp -- device helpers of the matrix-core kernels.
//
// v_mfma_f64_4x4x4_4b multiplies four independent 4x4 blocks.  One partial
// of the likelihood is, per pattern, a 4-vector for each rate category, and
// an update multiplies it by that category's 4x4 transition matrix, so the
// four blocks are the categories and the four columns are patterns:
//   A (matrix)   lane 16 s + 4 b + i : P_b[i][s]
//   B (vectors)  lane 16 s + 4 b + j : entry s of column j
//   D (result)   lane 16 i + 4 b + j : entry i of column j
// D has B's layout, so a result is the next update's operand with no lane
// exchange, and a matrix costs one register for all categories.  The sum over
// s is a chain of fused multiply-adds in the order s = 0..3 from zero (checked
// bit for bit on the device over 262144 random results).
//
// With fewer than four padded categories the blocks also hold further columns
// (block b: category b % CB, column group b / CB); with eight, two registers
// hold categories 0-3 and 4-7.
#pragma once
#include <hip/hip_runtime.h>

#include "pt_device.hpp"

namespace pt {

template <int KP>
struct Lanes {
    static constexpr int CB = KP < 4 ? KP : 4;   // categories in a register's four blocks
    static constexpr int NQ = KP > 4 ? KP / 4 : 1;  // registers of one item
    static constexpr int PG = 4 / CB;            // column groups in the blocks
    static constexpr int kCols = 4 * PG;         // patterns of one item
    static constexpr int kMat = CB * 16;         // doubles of one register's matrices
};

// Where lane `lane` finds its entry of a register's matrices (kMat doubles,
// laid out [s][category][i]).
template <int KP>
__device__ inline int mat_index(int lane) {
    constexpr int CB = Lanes<KP>::CB;
    return (lane >> 4) * (CB * 4) + ((lane >> 2) & 3) % CB * 4 + (lane & 3);
}

// A tree's matrices in lane order, read through a buffer descriptor: the
// lane's place is a 32-bit offset and the edge a scalar one, so a load needs
// no address arithmetic.
template <int KP>
struct MatRows {
    __amdgpu_buffer_rsrc_t rows;
    uint32_t at;
    __device__ inline MatRows(const double *pmat, int n_edges, int lane)
        : rows(__builtin_amdgcn_make_buffer_rsrc(const_cast<double *>(pmat), 0, n_edges * KP * 128, 0x00020000)),
          at(8u * mat_index<KP>(lane)) {}
    __device__ inline void load(int e, double *m) const {
        typedef uint32_t u2 __attribute__((ext_vector_type(2)));
#pragma unroll
        for (int q = 0; q < Lanes<KP>::NQ; ++q) {
            const u2 v = __builtin_amdgcn_raw_buffer_load_b64(rows, at, (e * Lanes<KP>::NQ + q) * Lanes<KP>::kMat * 8, 0);
            m[q] = __hiloint2double((int)v.y, (int)v.x);
        }
    }
};

__device__ inline double mfma4(double a, double b) { return __builtin_amdgcn_mfma_f64_4x4x4f64(a, b, 0.0, 0, 0, 0); }

// Orders one wave's LDS accesses for the compiler (the hardware runs them in
// order): what other lanes of the wave wrote before it is read after it.
__device__ inline void wave_lds_fence() {
    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
    __builtin_amdgcn_wave_barrier();
}

// One op of a program.  Programs are never written during a launch, so they
// are read through the constant address space: scalar loads into SGPRs.
// (A kernel that stores partials would otherwise read its ops by vector
// loads, the global memory not being known constant, and wait on the vector
// memory counter before every branch on the opcode.)
__device__ inline Op load_op(const Op *ops, int64_t i) {
    static_assert(sizeof(Op) == 8 * sizeof(int32_t), "an op is eight words");
    const __attribute__((address_space(4))) int32_t *q = (const __attribute__((address_space(4))) int32_t *)(ops + i);
    Op op;
    op.code = q[0];
    op.dst = q[1];
    op.a = q[2];
    op.ea = q[3];
    op.b = q[4];
    op.eb = q[5];
    op.tip_a = q[6];
    op.tip_b = q[7];
    return op;
}

// A tree's descriptor, the same way.
__device__ inline TreeDev load_tree(const TreeDev *trees, int b) {
    static_assert(sizeof(TreeDev) % sizeof(int32_t) == 0, "whole words");
    const __attribute__((address_space(4))) int32_t *q = (const __attribute__((address_space(4))) int32_t *)(trees + b);
    int32_t w[sizeof(TreeDev) / sizeof(int32_t)];
#pragma unroll
    for (size_t i = 0; i < sizeof(TreeDev) / sizeof(int32_t); ++i) w[i] = q[i];
    TreeDev td;
    __builtin_memcpy(&td, w, sizeof(td));
    return td;
}

// Moves a double across lanes with a DPP row shift; lanes whose source lies
// outside their row of 16 receive 0.
template <int CTRL>
__device__ inline double dpp_shr(double v) {
    const int lo = __builtin_amdgcn_update_dpp(0, __double2loint(v), CTRL, 0xf, 0xf, false);
    const int hi = __builtin_amdgcn_update_dpp(0, __double2hiint(v), CTRL, 0xf, 0xf, false);
    return __hiloint2double(hi, lo);
}

// A double from the lane N further on in its row of 16, cyclically.
template <int N>
__device__ inline double row_ror(double v) {
    const int lo = __builtin_amdgcn_update_dpp(0, __double2loint(v), 0x120 + N, 0xf, 0xf, true);
    const int hi = __builtin_amdgcn_update_dpp(0, __double2hiint(v), 0x120 + N, 0xf, 0xf, true);
    return __hiloint2double(hi, lo);
}

// A double from another lane of the row by a DPP permutation.
template <int CTRL>
__device__ inline double dpp_add(double v) {
    const int lo = __builtin_amdgcn_update_dpp(0, __double2loint(v), CTRL, 0xf, 0xf, true);
    const int hi = __builtin_amdgcn_update_dpp(0, __double2hiint(v), CTRL, 0xf, 0xf, true);
    return __hiloint2double(hi, lo);
}

// Row 0 of a value (its first 16 lanes) in every row, and row 1 in row 2 (and
// row 0): halves and rows of a wave are exchanged between two copies.
__device__ inline double row0(double v) {
    typedef uint32_t u2 __attribute__((ext_vector_type(2)));
    uint32_t w[2] = {(uint32_t)__double2loint(v), (uint32_t)__double2hiint(v)};
#pragma unroll
    for (int x = 0; x < 2; ++x) {
        u2 r = __builtin_amdgcn_permlane32_swap(w[x], w[x], false, false);
        r = __builtin_amdgcn_permlane16_swap(r.x, r.x, false, false);
        w[x] = r.x;
    }
    return __hiloint2double((int)w[1], (int)w[0]);
}

__device__ inline double row1(double v) {
    typedef uint32_t u2 __attribute__((ext_vector_type(2)));
    uint32_t w[2] = {(uint32_t)__double2loint(v), (uint32_t)__double2hiint(v)};
#pragma unroll
    for (int x = 0; x < 2; ++x) {
        // rows 0 and 1 in both halves, then the odd rows in both rows of a half
        u2 r = __builtin_amdgcn_permlane32_swap(w[x], w[x], false, false);
        r = __builtin_amdgcn_permlane16_swap(r.x, r.x, false, false);
        w[x] = r.y;
    }
    return __hiloint2double((int)w[1], (int)w[0]);
}

// Rows 0 and 2 in both rows of their half.
__device__ inline double even_rows(double v) {
    typedef uint32_t u2 __attribute__((ext_vector_type(2)));
    uint32_t w[2] = {(uint32_t)__double2loint(v), (uint32_t)__double2hiint(v)};
#pragma unroll
    for (int x = 0; x < 2; ++x) {
        const u2 r = __builtin_amdgcn_permlane16_swap(w[x], w[x], false, false);
        w[x] = r.x;
    }
    return __hiloint2double((int)w[1], (int)w[0]);
}

__device__ inline double lane_value(double v, int lane) {
    return __hiloint2double(__builtin_amdgcn_readlane(__double2hiint(v), lane),
                            __builtin_amdgcn_readlane(__double2loint(v), lane));
}

// Wavefront sum in a fixed order: a prefix sum inside each row of 16 lanes
// (DPP row shifts by 1, 2, 4, 8), then the four row totals in row order.
// Every lane receives the total.
__device__ inline double wave_sum(double v) {
    v += dpp_shr<0x111>(v);
    v += dpp_shr<0x112>(v);
    v += dpp_shr<0x114>(v);
    v += dpp_shr<0x118>(v);
    return (lane_value(v, 15) + lane_value(v, 31)) + (lane_value(v, 47) + lane_value(v, 63));
}

// 1 / x from the hardware estimate plus two Newton-Raphson steps.
__device__ inline double recip(double x) {
    double r = __builtin_amdgcn_rcp(x);
    r = fma(r, fma(-x, r, 1.0), r);
    r = fma(r, fma(-x, r, 1.0), r);
    return r;
}

}  // namespace pt
