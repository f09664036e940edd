// Geometry of the droplet count (no HIP types: host programs include it as well).
#pragma once

namespace lbm {

// Euler characteristic of the closed cells of a node mask (droplet count of
// Section 4.2.2).  Only the d active axes of the run are listed: axis i has n[i]
// cells, mask stride stride[i], wall[i] != 0 when it ends at walls.  An anchor
// j_i in [0, n[i] + wall[i]) stands for the vertex position between cells j_i - 1
// and j_i and for cell j_i (when j_i < n[i]); nanchors = prod(n[i] + wall[i]).
struct EulerGeom {
    int d;
    int n[3], wall[3];
    long long stride[3];
    long long nanchors;
    // A grid has fewer than 2^30 nodes, but a closed one up to four times as many anchors
    // (4 (nz + 1) of 1 x 1 x nz).  True where an unsigned index, advanced by `step` from below
    // nanchors, could wrap: there the count takes 64-bit indices
    constexpr bool wide(long long step) const { return nanchors + step > 0xFFFFFFFFLL; }
};

}  // namespace lbm
