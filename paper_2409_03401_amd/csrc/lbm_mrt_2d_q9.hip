// MRT, D2Q9 scalars, with or without the D2Q9 fluid: all four storage precisions.
#include "family.hpp"

namespace lbm {

const KernelSet* mrt2d_q9(int fluid, int prec) {
    if (fluid == 0) return family_all_prec_noadj<D2Q9K, NoLattice, 256, COLL_MRT>(prec);
    if (fluid == 9) return family_all_prec_noadj<D2Q9K, D2Q9K, 256, COLL_MRT>(prec);
    return nullptr;
}

}  // namespace lbm
