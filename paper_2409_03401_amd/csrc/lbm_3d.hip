// 3D lattice families (D3Q7 scalars, optional D3Q19 fluid), 256-node columns per
// work-group.
#include "family.hpp"

namespace lbm {

const KernelSet* kernels_3d(int fluid, int prec) {
    if (fluid == 0) return family_for_prec<D3Q7K, NoLattice, kTileNodes>(prec);
    if (fluid == 19) return family_for_prec<D3Q7K, D3Q19K, kTileNodes>(prec);
    return nullptr;
}

void launch_sum_partials(const double* v, long long n, double* partials, int nblocks, hipStream_t s) {
    hipLaunchKernelGGL((k_sum_partials<256>), dim3(nblocks), dim3(256), 0, s, v, n, partials);
}

void launch_finalize(const double* partials, int nparts, int width, int maxslot, double scale0,
                     double* out, hipStream_t s) {
    if (width == 1)
        hipLaunchKernelGGL((k_finalize<1>), dim3(1), dim3(256), 0, s, partials, nparts, maxslot, scale0, out);
    else if (width == 9)
        hipLaunchKernelGGL((k_finalize<9, false, 10>), dim3(1), dim3(256), 0, s, partials, nparts, maxslot, scale0,
                           out);
    else
        hipLaunchKernelGGL((k_finalize<8>), dim3(1), dim3(256), 0, s, partials, nparts, maxslot, scale0, out);
}

void launch_sum6(const double* partials, int nparts, double* out, bool accumulate, hipStream_t s) {
    if (accumulate)
        hipLaunchKernelGGL((k_finalize<6, true>), dim3(1), dim3(256), 0, s, partials, nparts, -1, 1.0, out);
    else
        hipLaunchKernelGGL((k_finalize<6, false>), dim3(1), dim3(256), 0, s, partials, nparts, -1, 1.0, out);
}

void launch_euler(const unsigned char* mask, const EulerGeom& g, double* partials, int nblocks, hipStream_t s) {
    using Long = unsigned long long;
    const dim3 grid(nblocks), block(256);
    if (g.d == 2) hipLaunchKernelGGL((k_euler<2, unsigned>), grid, block, 0, s, mask, g, partials);  // at most 2^31 anchors
    else if (!g.wide(256LL * nblocks)) hipLaunchKernelGGL((k_euler<3, unsigned>), grid, block, 0, s, mask, g, partials);
    else hipLaunchKernelGGL((k_euler<3, Long>), grid, block, 0, s, mask, g, partials);
}

void launch_zero(double* p, long long n, hipStream_t s) {
    if (n > 0) hipLaunchKernelGGL((k_zero_f64<256>), dim3(unsigned((n + 255) / 256)), dim3(256), 0, s, p, n);
}

void launch_zero_padding(const KParams& kp, int qf, int qs, int nslots, unsigned long long used_m,
                         unsigned long long used_r, hipStream_t s) {
    hipLaunchKernelGGL((k_zero_padding<256>), dim3(unsigned(nslots), 2), dim3(256), 0, s, kp, qf, qs, used_m, used_r);
}

}  // namespace lbm
