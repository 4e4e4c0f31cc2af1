// Fine level of the two-level hierarchical far field (Sec. 5.2): dispatch
// to the kernels of the plan's order (pmmm_hier_cell.h, one compile unit per
// order).
#include "pmmm_hier.h"

namespace pmmm {

int64_t hier_matrix_floats(int p, int nf, int r, int D) {
    switch (p) {
        case 0: return hier_mat_floats<0>(nf, r, D);
        case 1: return hier_mat_floats<1>(nf, r, D);
        case 2: return hier_mat_floats<2>(nf, r, D);
        case 3: return hier_mat_floats<3>(nf, r, D);
        case 4: return hier_mat_floats<4>(nf, r, D);
        case 5: return hier_mat_floats<5>(nf, r, D);
        case 6: return hier_mat_floats<6>(nf, r, D);
        case 7: return hier_mat_floats<7>(nf, r, D);
        case 8: return hier_mat_floats<8>(nf, r, D);
        case 9: return hier_mat_floats<9>(nf, r, D);
        case 10: return hier_mat_floats<10>(nf, r, D);
        default: return 0;
    }
}

hipError_t build_hier_matrices_f32(int p, int D, const float *table, float *mat, hipStream_t s) {
    switch (p) {
        case 0: return hier_mat_build<0>(D, table, mat, s);
        case 1: return hier_mat_build<1>(D, table, mat, s);
        case 2: return hier_mat_build<2>(D, table, mat, s);
        case 3: return hier_mat_build<3>(D, table, mat, s);
        case 4: return hier_mat_build<4>(D, table, mat, s);
        case 5: return hier_mat_build<5>(D, table, mat, s);
        case 6: return hier_mat_build<6>(D, table, mat, s);
        case 7: return hier_mat_build<7>(D, table, mat, s);
        case 8: return hier_mat_build<8>(D, table, mat, s);
        case 9: return hier_mat_build<9>(D, table, mat, s);
        case 10: return hier_mat_build<10>(D, table, mat, s);
        default: return hipErrorInvalidValue;
    }
}

hipError_t launch_hier_m2l_f32(const HierArgs &a, hipStream_t s) {
    switch (a.p) {
        case 0: return hier_cell_launch<0>(a, s);
        case 1: return hier_cell_launch<1>(a, s);
        case 2: return hier_cell_launch<2>(a, s);
        case 3: return hier_cell_launch<3>(a, s);
        case 4: return hier_cell_launch<4>(a, s);
        case 5: return hier_cell_launch<5>(a, s);
        case 6: return hier_cell_launch<6>(a, s);
        case 7: return hier_cell_launch<7>(a, s);
        case 8: return hier_cell_launch<8>(a, s);
        case 9: return hier_cell_launch<9>(a, s);
        case 10: return hier_cell_launch<10>(a, s);
        default: return hipErrorInvalidValue;
    }
}

}  // namespace pmmm
