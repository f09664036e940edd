// 2D families with the multiple-relaxation-time collision: D2Q5 or the paper's D2Q9
// for g, h^A, h^B, with or without the D2Q9 fluid; all four storage precisions.  The D2Q9
// families are compiled in a translation unit of their own (lbm_mrt_2d_q9.hip).
#include "family.hpp"

namespace lbm {

const KernelSet* mrt2d_q9(int fluid, int prec);

const KernelSet* kernels_mrt_2d(int scalar, int fluid, int prec) {
    if (scalar == 5) {
        if (fluid == 0) return family_all_prec_noadj<D2Q5K, NoLattice, 256, COLL_MRT>(prec);
        if (fluid == 9) return family_all_prec_noadj<D2Q5K, D2Q9K, 256, COLL_MRT>(prec);
    } else if (scalar == 9) {
        return mrt2d_q9(fluid, prec);
    }
    return nullptr;
}

}  // namespace lbm
