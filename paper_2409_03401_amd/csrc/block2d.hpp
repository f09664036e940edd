// Several time steps of 2D runs in one launch.
//
// A step of a 2D run reads and writes every population, and a launch costs about as much
// as a small grid's whole step.  Here a work-group keeps a window of bw x bh nodes on
// chip (one node per thread) and takes `nsub` steps before it writes anything back: it
// pulls the arriving populations of its window from memory once, collides, exchanges
// post-collision populations (and phi, for the stencil of the capillary force) with its
// neighbours in LDS, and stores the state after the last step.  A window overlaps its
// neighbours by a halo that each step eats into: after the first step (whose pulls come
// from memory) a node's update is exact where the stencil of phi lies inside the window,
// one ring less with flow; every further step loses one ring to the streaming and, with
// flow, one to the stencil.  An axis that fits into the window whole needs no halo: its
// periodic neighbours wrap inside the window.  Overlapped nodes are computed by every
// window that holds them and stored by the one that owns them.
//
// The exchange is in the storage format (the 16 bits of a moving population), so that a
// node sees the rounding that it would see through memory, and the update is the one of
// the marching kernel (node.hpp): the state is the same bit for bit, however the steps are
// cut into launches.
//
// What bounds it: on small grids the barriers and the collision's latency (a 256-node
// window takes about 0.5 us a step without flow, 1 us with), on large ones the memory
// traffic, 1 / nsub of the marching kernel's times the share of the windows that overlaps.
// Measured, us per step, marching kernel -> windows:
//   512 x 1   D2Q5 FP64, walls in x       8.3 -> 0.65 (nine windows, 100 steps per launch)
//   150 x 93  D2Q9 + 3 x D2Q5 FP32, walls 14.9 -> 2.7 (16 x 16 windows)
//   512^2     D2Q9 + 3 x D2Q5 FP32        14.9 -> 9.0
//   1024^2    3 x D2Q5 FP32               26.3 -> 10.8
//   4096^2    3 x D2Q9 BF16                430 -> 266
// Which windows run, how many steps each and whether any do is the plan's choice (plan.hpp).
#pragma once

#include "node.hpp"

namespace lbm {

template <class SL, class FL, int PREC, int NT, int COLL = COLL_BGK, int NC = 2>
__global__ void __launch_bounds__(NT) k_block(const KParams P, const BlockGeom B) {
    using NODE = Node<SL, FL, PREC, COLL, NC>;
    using C = typename NODE::C;
    using SLOTS = typename NODE::SLOTS;
    using SLT = std::common_type<SL>;
    using FLT = std::common_type<FL>;
    constexpr int QS = SL::Q, QF = FL::Q, QFN = NODE::QFN, QC = NODE::QC, N = SLOTS::N;
    constexpr int G0 = SLOTS::G0, A0 = SLOTS::A0, B0 = SLOTS::B0, HC0 = SLOTS::C0;
    constexpr bool FLOW = NODE::FLOW, NC3 = NODE::NC3, S16 = NODE::S16;
    static_assert(SL::DIM == 2, "2D windows");
    using LW = typename std::conditional<S16, unsigned short, C>::type;  // stored form of a moving population
    constexpr int NM = N - ((FLOW ? 1 : 0) + 1 + NC);                    // moving populations
    static_assert(window_lds(FL::Q, SL::Q, PREC, NC, NT) <= 160 * 1024, "window too large for LDS");

    __shared__ LW spop[NM * NT];
    __shared__ C sphi[FLOW ? NT : 1];

    // ---- the node of this thread
    const int tid = threadIdx.x;
    const int bw = 1 << B.lw, bh = NT >> B.lw;
    const int lx = tid & (bw - 1), lz = tid >> B.lw;
    const int tile = xcd_tile(blockIdx.x, B.tiles_x * B.tiles_z);
    const int bx = tile % B.tiles_x, bz = tile / B.tiles_x;
    const int ux = bx * B.ix - B.hx + lx, uz = bz * B.iz - B.hz + lz;  // not wrapped
    const bool owned = lx >= B.hx && lx < B.hx + B.ix && ux < P.nx && lz >= B.hz && lz < B.hz + B.iz && uz < P.nz;
    // the node in memory: wrapped once on a periodic axis, then any node of the grid for the
    // lanes beyond (their values reach no owned node)
    auto in_grid = [](int c, int n, int wall) __attribute__((always_inline)) -> int {
        if (!wall) c = c < 0 ? c + n : (c >= n ? c - n : c);
        return min(max(c, 0), n - 1);
    };
    const int x = in_grid(ux, P.nx, P.wall_x), z = in_grid(uz, P.nz, P.wall_z);
    const unsigned idx = unsigned(z * P.nx + x);
    const bool xlo = P.wall_x && ux == 0, xhi = P.wall_x && ux == P.nx - 1;
    const bool zlo = P.wall_z && uz == 0, zhi = P.wall_z && uz == P.nz - 1;

    // ---- neighbours in the window: an axis that fits whole wraps inside it, else a lane at
    // the window's edge takes itself (a ring that the halo covers)
    auto step_in = [](int l, int d, int n, int full, int m) __attribute__((always_inline)) -> int {
        int t = l + d;
        if (full) t = t < 0 ? n - 1 : (t >= n ? 0 : t);
        return min(max(t, 0), m - 1);
    };
    const int xm = step_in(lx, -1, P.nx, B.full_x, bw), xp = step_in(lx, 1, P.nx, B.full_x, bw);
    const int zm = step_in(lz, -1, P.nz, B.full_z, bh), zp = step_in(lz, 1, P.nz, B.full_z, bh);
    // where X_k(x) arrives from, in words relative to slot k of the window: slot k of the
    // lane at x - e_k, or slot opp(k) of this lane where that lies beyond a wall.  The
    // directions 1-4 are the same in D2Q5 and D2Q9, so one table serves every field
    constexpr int ND = FLOW ? 9 : QS;
    using DL = typename std::conditional<ND == 9, D2Q9K, D2Q5K>::type;
    int from[ND];
    static_for<1, ND>([&](auto kc) __attribute__((always_inline)) {
        constexpr int k = decltype(kc)::value, ex = DL::ex(k), ez = DL::ez(k);
        const bool cross = (ex > 0 && xlo) || (ex < 0 && xhi) || (ez > 0 && zlo) || (ez < 0 && zhi);
        const int sx = ex > 0 ? xm : ex < 0 ? xp : lx, sz = ez > 0 ? zm : ez < 0 ? zp : lz;
        from[k] = cross ? (DL::opp(k) - k) * NT + tid : (sz << B.lw) + sx;
    });
    // the phi stencil: mirror ghosts at walls
    const int px = xhi ? lx : xp, mx = xlo ? lx : xm, pz = zhi ? lz : zp, mz = zlo ? lz : zm;

    // ---- arriving populations of the first step, from memory
    using gconst = __attribute__((address_space(1))) const char;
    using gmut = __attribute__((address_space(1))) char;
    auto src = [&](auto s_) __attribute__((always_inline)) -> const char* {
        return (const char*)(gconst*)(unsigned long long)P.src_slot[decltype(s_)::value];
    };
    auto dst = [&](auto s_) __attribute__((always_inline)) -> char* {
        return (char*)(gmut*)(unsigned long long)P.dst_slot[decltype(s_)::value];
    };
    using RW = typename std::conditional<S16, unsigned, C>::type;
    RW raw[N];
    auto fetch = [&](auto to_, auto s_, unsigned t) __attribute__((always_inline)) {
        constexpr int S = decltype(s_)::value;
        RW& r = raw[decltype(to_)::value];
        if constexpr (!S16) r = *reinterpret_cast<const C*>(src(s_) + t * unsigned(sizeof(C)));
        else if constexpr (SLOTS::rest(S)) r = __builtin_bit_cast(unsigned, *reinterpret_cast<const float*>(src(s_) + t * 4u));
        else r = *reinterpret_cast<const unsigned short*>(src(s_) + t * 2u);
    };
    // every field's populations: fn(slot, direction, lattice tag)
    auto each = [&](auto&& fn) __attribute__((always_inline)) {
        static_for<0, QF>([&](auto kc) __attribute__((always_inline)) { fn(kc, kc, FLT{}); });
        static_for<0, QS>([&](auto kc) __attribute__((always_inline)) {
            constexpr int k = decltype(kc)::value;
            fn(IC<G0 + k>{}, kc, SLT{});
            fn(IC<A0 + k>{}, kc, SLT{});
            fn(IC<B0 + k>{}, kc, SLT{});
            if constexpr (NC3) fn(IC<HC0 + k>{}, kc, SLT{});
        });
    };
    const Nbr nb = neighbours(x, 0, z, P);
    each([&](auto s_, auto k_, auto lat_) __attribute__((always_inline)) {
        using L = typename decltype(lat_)::type;
        constexpr int k = decltype(k_)::value;
        fetch(s_, s_, unsigned(int(idx) + pull_offset<L::ex(k), 0, L::ez(k)>(nb)));
    });
    // walls: the node's own slot of opp(k) (x walls only while the source copy holds raw
    // post-collision populations there; after k_walls the wrapped pull is right)
    const bool rxlo = xlo && B.raw_x, rxhi = xhi && B.raw_x;
    if (rxlo || rxhi || zlo || zhi) {
        each([&](auto s_, auto k_, auto lat_) __attribute__((always_inline)) {
            using L = typename decltype(lat_)::type;
            constexpr int k = decltype(k_)::value, ex = L::ex(k), ez = L::ez(k);
            if constexpr (ex != 0 || ez != 0) {
                if ((ex > 0 && rxlo) || (ex < 0 && rxhi) || (ez > 0 && zlo) || (ez < 0 && zhi))
                    fetch(s_, IC<decltype(s_)::value - k + L::opp(k)>{}, idx);
            }
        });
    }
    C f[QFN], g[QS], a[QS], b[QS], cq[QC];
    auto slot_ref = [&](auto s_, auto k_) __attribute__((always_inline)) -> C& {
        constexpr int S = decltype(s_)::value, k = decltype(k_)::value;
        if constexpr (S < G0) return f[k];
        else if constexpr (S < A0) return g[k];
        else if constexpr (S < B0) return a[k];
        else if constexpr (S < HC0) return b[k];
        else return cq[k];
    };
    auto decode = [&](auto s_, auto k_, auto lat_, unsigned bits) __attribute__((always_inline)) -> C {
        return dec_lo<PREC>(bits, NODE::wref_dec(P, s_, k_, lat_), P.finv[SLOTS::field(decltype(s_)::value)]);
    };
    each([&](auto s_, auto k_, auto lat_) __attribute__((always_inline)) {
        constexpr int S = decltype(s_)::value;
        if constexpr (!S16) slot_ref(s_, k_) = raw[S];
        else if constexpr (SLOTS::rest(S)) slot_ref(s_, k_) = __builtin_bit_cast(float, raw[S]);
        else slot_ref(s_, k_) = decode(s_, k_, lat_, raw[S]);
    });

    // one step of this thread's node; the post-collision populations go to sink
    auto update = [&](auto&& sink) __attribute__((always_inline)) {
        double ps, sA, sB, sC, muC;
        NODE::pop_sums(g, a, b, cq, ps, sA, sB, sC);
        if constexpr (FLOW) {
            double unused;
            sphi[tid] = C(NODE::scalars(ps, sA, sB, sC, P, unused).phi);
            __syncthreads();
        }
        const Scalars m = NODE::scalars(ps, sA, sB, sC, P, muC);
        const C phi = C(m.phi);
        C grad[3] = {C(0), C(0), C(0)}, F[3] = {C(0), C(0), C(0)}, u[3] = {C(0), C(0), C(0)};
        C lap = C(0), p_h = C(0), irho = C(1);
        if constexpr (FLOW) {
            NODE::stencil(
                [&](auto ex_, auto, auto ez_) __attribute__((always_inline)) -> C {
                    constexpr int ex = decltype(ex_)::value, ez = decltype(ez_)::value;
                    const int sx = ex > 0 ? px : ex < 0 ? mx : lx, sz = ez > 0 ? pz : ez < 0 ? mz : lz;
                    return sphi[(sz << B.lw) + sx];
                },
                sphi[tid], grad, lap);
            NODE::flow(P, f, m.phi, phi, 0.0, grad, lap, F, u, p_h, irho);
        }
        NODE::collide(P, f, g, a, b, cq, ps, sA, sB, sC, m, muC, phi, F, u, p_h, irho, sink);
    };
    // slot of a moving population among the moving ones
    auto at = [](int s) constexpr { return (s - SLOTS::rest_before(s)) * NT; };

    C rest[5];
    for (int left = B.nsub;;) {
        update([&](auto s_, auto v) __attribute__((always_inline)) {
            constexpr int S = decltype(s_)::value;
            if constexpr (SLOTS::rest(S)) rest[SLOTS::field(S)] = v;
            else spop[at(S) + tid] = v;
        });
        if (--left == 0) break;
        __syncthreads();
        each([&](auto s_, auto k_, auto lat_) __attribute__((always_inline)) {
            constexpr int S = decltype(s_)::value, k = decltype(k_)::value;
            if constexpr (k == 0) slot_ref(s_, k_) = rest[SLOTS::field(S)];
            else if constexpr (S16) slot_ref(s_, k_) = decode(s_, k_, lat_, spop[at(S) + from[k]]);
            else slot_ref(s_, k_) = spop[at(S) + from[k]];
        });
        // the next collision writes spop: with flow the barrier after phi stands between
        if constexpr (!FLOW) __syncthreads();
    }
    // the state after the last step, from this thread's own words (plain stores: the rows of a
    // window end inside lines that its neighbours complete)
    if (owned) {
        each([&](auto s_, auto k_, auto) __attribute__((always_inline)) {
            constexpr int S = decltype(s_)::value;
            if constexpr (decltype(k_)::value == 0) st_raw<false>(dst(s_), idx, rest[SLOTS::field(S)]);
            else st_raw<false>(dst(s_), idx, spop[at(S) + tid]);
        });
    }
}

}  // namespace lbm
