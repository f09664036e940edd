// Instantiation helper: the launchers of one (scalar lattice, fluid lattice,
// collision / model variant, number of independent compositions) family for the four
// storage precisions.
#pragma once

#include <algorithm>

#include "block2d.hpp"
#include "dispatch.hpp"
#include "kernels.hpp"

namespace lbm {

template <class SL, class FL, int PREC, int NT, bool ADJ = true, int COLL = COLL_BGK, int NC = 2>
struct Family {
    // the adjoint covers the ternary fluid (two compositions) at FP64 / FP32
    static constexpr bool kAdj = ADJ && NC == 2 && (PREC == P32 || PREC == P64);
    // gen: any grid, else rows of whole lines in 64 x 4 tiles (MODE_STEP; MODE_STEP_PHI of
    // the families with an adjoint, whose recompute it serves)
    static void fused(int mode, bool gen, unsigned grid, const KParams& kp, hipStream_t s) {
        constexpr int CM = COLL & (COLL_VD | COLL_GK);  // what the moments depend on
        const dim3 g(grid), block(NT);
        switch (mode) {
            case MODE_STEP:
                if (gen) hipLaunchKernelGGL((k_lbm<SL, FL, MODE_STEP, PREC, NT, true, COLL, NC>), g, block, 0, s, kp);
                else hipLaunchKernelGGL((k_lbm<SL, FL, MODE_STEP, PREC, NT, false, COLL, NC>), g, block, 0, s, kp);
                break;
            case MODE_STEP_PHI:
                if constexpr (kAdj)
                    if (!gen) {
                        hipLaunchKernelGGL((k_lbm<SL, FL, MODE_STEP_PHI, PREC, NT, false, COLL>), g, block, 0, s, kp);
                        break;
                    }
                if constexpr (NC == 2)  // lbm_step_external asks it of two compositions only
                    hipLaunchKernelGGL((k_lbm<SL, FL, MODE_STEP_PHI, PREC, NT, true, COLL>), g, block, 0, s, kp);
                break;
            case MODE_SCALARS:
                if constexpr (FL::Q > 0) {
                    hipLaunchKernelGGL((k_lbm<SL, FL, MODE_SCALARS, PREC, NT, false, (COLL & COLL_GK), NC>), g, block, 0, s, kp);
                    break;
                }
                [[fallthrough]];
            case MODE_MOMENTS:
                hipLaunchKernelGGL((k_lbm<SL, FL, MODE_MOMENTS, PREC, NT, false, CM, NC>), g, block, 0, s, kp);
                break;
            default:
                hipLaunchKernelGGL((k_lbm<SL, FL, MODE_DIAG, PREC, NT, false, CM, NC>), g, block, 0, s, kp);
                break;
        }
    }
    static void init(const KParams& kp, const double* phi0, const double* muA0, const double* muB0,
                     const double* muC0, hipStream_t s) {
        const dim3 grid((kp.nx + 255) / 256, kp.ny, kp.nz);
        hipLaunchKernelGGL((k_init<SL, FL, PREC, NC>), grid, dim3(256), 0, s, kp, phi0, muA0, muB0, muC0);
    }
    static void get_pops(const KParams& kp, int, long long nodes, double* out, hipStream_t s) {
        const dim3 grid(unsigned((nodes + 255) / 256));
        hipLaunchKernelGGL((k_pops<SL, FL, PREC, false, NC>), grid, dim3(256), 0, s, kp, nodes, out);
    }
    static void set_pops(const KParams& kp, int, long long nodes, const double* in, hipStream_t s) {
        const dim3 grid(unsigned((nodes + 255) / 256));
        hipLaunchKernelGGL((k_pops<SL, FL, PREC, true, NC>), grid, dim3(256), 0, s, kp, nodes,
                           const_cast<double*>(in));
    }
    static void walls(const KParams& kp, int axis, hipStream_t s) {
        const long long n[3] = {kp.nx, kp.ny, kp.nz};
        const long long face = n[axis == 0 ? 1 : 0] * n[axis == 2 ? 1 : 2];
        const dim3 grid(unsigned((2 * face + 255) / 256));
        hipLaunchKernelGGL((k_walls<SL, FL, PREC, NC>), grid, dim3(256), 0, s, kp, axis);
    }
    static void adj_step(const KParams& kp, long long nodes, const void* phi, hipStream_t s) {
        if constexpr (kAdj)
            hipLaunchKernelGGL((k_adj_node<SL, FL, PREC>), dim3(unsigned((nodes + 255) / 256)), dim3(256), 0, s, kp,
                               nodes, static_cast<const typename Stor<PREC>::C*>(phi));
    }
    static void adj_seed(const KParams& kp, long long nodes, const double* dL_dphi, hipStream_t s) {
        if constexpr (kAdj)
            hipLaunchKernelGGL((k_adj_seed<SL, FL, PREC>), dim3(unsigned((nodes + 255) / 256)), dim3(256), 0, s,
                               kp, nodes, dL_dphi);
    }
    static void adj_gather(const KParams& kp, long long nodes, int mode, double* grad_phi0, hipStream_t s) {
        if constexpr (kAdj) {
            using T = GatherTile<SL::DIM>;
            const long long tiles = ((kp.nx + T::X - 1LL) / T::X) * ((kp.ny + T::Y - 1LL) / T::Y) * ((kp.nz + T::Z - 1LL) / T::Z);
            const dim3 grid(unsigned(std::min(tiles, (nodes + 255) / 256)));
            if (mode == 0) hipLaunchKernelGGL((k_adj_gather<SL, FL, 0>), grid, dim3(256), 0, s, kp, int(tiles), grad_phi0);
            else hipLaunchKernelGGL((k_adj_gather<SL, FL, 1>), grid, dim3(256), 0, s, kp, int(tiles), grad_phi0);
        }
    }
    static void adj_init_local(const KParams& kp, long long nodes, const double* phi0, const double* muA0,
                               const double* muB0, hipStream_t s) {
        if constexpr (kAdj)
            hipLaunchKernelGGL((k_adj_init_local<SL, FL>), dim3(unsigned((nodes + 255) / 256)), dim3(256), 0, s,
                               kp, nodes, phi0, muA0, muB0);
    }
    static void adj_copy(const KParams& kp, int nslots, long long nodes, double* buf, bool set_, hipStream_t s) {
        const dim3 grid(unsigned((nodes + 255) / 256), nslots);
        if constexpr (kAdj) {
            if (set_) hipLaunchKernelGGL((k_adj_copy<SL, FL, true>), grid, dim3(256), 0, s, kp, nodes, buf);
            else hipLaunchKernelGGL((k_adj_copy<SL, FL, false>), grid, dim3(256), 0, s, kp, nodes, buf);
        }
    }
    // the narrow row segments (LBM_TILE) march one step per launch
    static constexpr bool kBlock = SL::DIM == 2 && NT == 256;
    static constexpr int kSmall = kSmallWindow, kLarge = kBlock ? large_window(FL::Q, SL::Q, PREC, COLL, NC) : 0;
    static void block(int nt, unsigned grid, const KParams& kp, const BlockGeom& g, hipStream_t s) {
        if constexpr (kBlock) {
            if (nt == kSmall) hipLaunchKernelGGL((k_block<SL, FL, PREC, kSmall, COLL, NC>), dim3(grid), dim3(kSmall), 0, s, kp, g);
            else hipLaunchKernelGGL((k_block<SL, FL, PREC, kLarge, COLL, NC>), dim3(grid), dim3(kLarge), 0, s, kp, g);
        }
    }
    static constexpr KernelSet set{&fused, &init, &get_pops, &set_pops, &walls,
                                   kAdj ? &adj_step : nullptr, kAdj ? &adj_seed : nullptr,
                                   kAdj ? &adj_gather : nullptr, kAdj ? &adj_init_local : nullptr,
                                   kAdj ? &adj_copy : nullptr, NT,
                                   kBlock ? &block : nullptr, {kBlock ? kSmall : 0, kLarge}};
};

template <class SL, class FL, int NT>
const KernelSet* family_for_prec(int prec) {
    switch (prec) {
        case P64: return &Family<SL, FL, P64, NT>::set;
        case P32: return &Family<SL, FL, P32, NT>::set;
        case P16: return &Family<SL, FL, P16, NT>::set;
        case PB16: return &Family<SL, FL, PB16, NT>::set;
        default: return nullptr;
    }
}

// the TRT / MRT collisions, the variable-density model and general curvatures: all
// four storage precisions, no adjoint
template <class SL, class FL, int NT, int COLL = COLL_BGK>
const KernelSet* family_all_prec_noadj(int prec) {
    switch (prec) {
        case P64: return &Family<SL, FL, P64, NT, false, COLL>::set;
        case P32: return &Family<SL, FL, P32, NT, false, COLL>::set;
        case P16: return &Family<SL, FL, P16, NT, false, COLL>::set;
        case PB16: return &Family<SL, FL, PB16, NT, false, COLL>::set;
        default: return nullptr;
    }
}

// a third independent composition (N components): BGK Boussinesq step, all four
// storage precisions, no adjoint
template <class SL, class FL, int NT>
const KernelSet* family_nc3(int prec) {
    switch (prec) {
        case P64: return &Family<SL, FL, P64, NT, false, COLL_BGK, 3>::set;
        case P32: return &Family<SL, FL, P32, NT, false, COLL_BGK, 3>::set;
        case P16: return &Family<SL, FL, P16, NT, false, COLL_BGK, 3>::set;
        case PB16: return &Family<SL, FL, PB16, NT, false, COLL_BGK, 3>::set;
        default: return nullptr;
    }
}

// one precision of a family without adjoint (for splitting large families over
// translation units)
template <class SL, class FL, int NT, int COLL, int PREC>
const KernelSet* family_one_prec() {
    return &Family<SL, FL, PREC, NT, false, COLL>::set;
}

}  // namespace lbm
