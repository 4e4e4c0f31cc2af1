// Internal declarations of the two-level hierarchical far field (Sec. 5.2):
// the fine level's table of singular harmonics and its local M2L.  Not part
// of the public ABI.
#pragma once

#include "pmmm_internal.h"

namespace pmmm {

// S_n^k (real storage, orders n <= 2p, cell units) at every fine offset d
// with |d_a| <= D, zero on the near cube max|d_a| <= cutoff; layout
// [((dz + D) W + dy + D) W + dx + D][Q], W = 2D + 1 (FP64 sums, FP32 values).
hipError_t build_hier_table_f32(int p, int cutoff, int D, float *out, hipStream_t s);

struct HierArgs {
    int p, nf, r, cutoff, D;   // fine mesh nf^3 = (coarse n r)^3, margin D = (c + 1) r - 1
    const float *M;            // fine moments [P(+1)][nf^3], cell units (mat: in hier_moment_order)
    float *L;                  // fine local expansions [P][nf^3], written in full
    const float *table;        // build_hier_table_f32
    const float *mat;          // build_hier_matrices_f32, NULL: the table serves
};
// Order of the moments that the matrix form reads (moment_place).
inline int hier_moment_order(int nf, int r) { return __builtin_ctz(nf) | __builtin_ctz(r) << 8; }

// The matrices of eq. realmatrix at the table's displacements in the register
// order of the fine-level kernel; hier_matrix_floats is their size, 0 where
// the table serves instead.
int64_t hier_matrix_floats(int p, int nf, int r, int D);
hipError_t build_hier_matrices_f32(int p, int D, const float *table, float *mat, hipStream_t s);
hipError_t launch_hier_m2l_f32(const HierArgs &a, hipStream_t s);

// The fine-level kernel of one order (pmmm_hier_cell.h; instantiated for
// 0 <= PO <= PMMM_PMAX by pmmm_hier_inst.hip).
template <int PO>
hipError_t hier_cell_launch(const HierArgs &a, hipStream_t s);
template <int PO>
int64_t hier_mat_floats(int nf, int r, int D);
template <int PO>
hipError_t hier_mat_build(int D, const float *table, float *mat, hipStream_t s);

}  // namespace pmmm
