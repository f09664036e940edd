// HIP kernels of the coupled lattice-Boltzmann step for gfx950.
//
// One fused kernel per (lattice family, mode, storage precision, tile).  A
// work-group owns a column of nodes (3D: tile_x x tile_y, 2D: a row segment) and marches
// along z over `zc` planes.
// When the capillary force (or the free-energy diagnostic) needs grad phi and
// lap phi, phi of three consecutive planes, each with a one-node ring, is staged
// in LDS: the work-group computes phi of plane z+1 (its own nodes from registers
// kept for the next iteration, ring nodes from L2-resident neighbour
// populations), then updates plane z.  Populations live in two copies (read one,
// write the other), so ring reads never race with writes.  Streaming is a pull:
// a copy holds post-collision populations; each node gathers X_k from x - e_k
// (periodic wrap), collides, and writes its post-collision populations to its
// own slots, so every store is aligned.  Half-way bounce-back at the z walls (the
// kernel frame's marching axis; the user's y axis in 2D) is taken when pulling: after
// a step a copy holds each node's raw post-collision populations, and a population
// X_k(x) whose source x - e_k lies beyond a z wall is read from the node's own slot
// opp(k) instead (zbounce).  Every reader of a state (step, moments, initialisation,
// population access, adjoint) follows this rule.  Walls on x and y are a small fix-up
// kernel after the step (k_walls).  2D runs of several steps go through k_block
// (block2d.hpp); the update of a node itself is in node.hpp.
//
// Memory layout of one copy: a sequence of slots, one [node] array per
// (field, direction) in the canonical order f_0.., g_0.., hA_0.., hB_0...  Every
// slot base is wave-uniform (SGPR) and every access uses a 32-bit per-lane
// offset, so each load / store is one `global_* voffset, saddr` instruction.
#pragma once

#include "node.hpp"

namespace lbm {

// ---------------------------------------------------------------------------
// block reduction of N doubles (entry `maxslot` takes a max, the others a sum),
// fixed order, one result per work-group

// ACC: add to out (each work-group owns its out entries, so repeated launches
// accumulate deterministically)
template <int N, int NT, bool ACC = false>
__device__ __forceinline__ void block_reduce_store(double (&v)[N], int maxslot, double* out) {
    static_assert(NT % 64 == 0, "work-group must be whole waves");
    __shared__ double red[NT / 64][N];
#pragma unroll
    for (int off = 32; off > 0; off >>= 1) {
#pragma unroll
        for (int i = 0; i < N; ++i) {
            const double o = __shfl_down(v[i], off, 64);
            v[i] = (i == maxslot) ? fmax(v[i], o) : v[i] + o;
        }
    }
    const int tid = threadIdx.y * blockDim.x + threadIdx.x;
    if ((tid & 63) == 0) {
#pragma unroll
        for (int i = 0; i < N; ++i) red[tid >> 6][i] = v[i];
    }
    __syncthreads();
    if (tid == 0) {
#pragma unroll
        for (int i = 0; i < N; ++i) {
            double a = red[0][i];
            for (int w = 1; w < NT / 64; ++w) a = (i == maxslot) ? fmax(a, red[w][i]) : a + red[w][i];
            if constexpr (ACC) out[i] += a;
            else out[i] = a;
        }
    }
}

// ---------------------------------------------------------------------------
// the fused step / moments / diagnostics kernel

#ifndef LBM_WAVES_PER_EU
#define LBM_WAVES_PER_EU 1
#endif
// occupancy target of the adjoint node kernel (register budget 512 / waves): the
// largest at which it does not spill (2D: 165 VGPRs, 3D: 234 VGPRs in FP32)
#ifndef LBM_ADJ_WAVES_2D
#define LBM_ADJ_WAVES_2D 3
#endif
#ifndef LBM_ADJ_WAVES_3D
#define LBM_ADJ_WAVES_3D 2
#endif
#ifndef LBM_EARLY_F
#define LBM_EARLY_F 1
#endif
#ifndef LBM_LDS_POPS
#define LBM_LDS_POPS 1
#endif
#ifndef LBM_NT_FLUID
#define LBM_NT_FLUID 1
#endif
#ifndef LBM_FRAW
#define LBM_FRAW 1
#endif

// occupancy floor of the fused kernel: one wave per SIMD (the compiler may use every
// register), except where a higher floor measured faster at 256^3:
// - the D3Q19 scalar lattices with 16-bit storage (the paper's 3D discretisation) and
//   the BGK, TRT or variable-density collisions, or MRT with BF16: with the packed LDS
//   ring they need about 260 registers; two waves per SIMD (256, at most 64 bytes of
//   spill) are 6-15 % faster than one;
// - D3Q7 with 16-bit storage, whose 3D launch puts three work-groups on a compute unit:
//   where the kernel needs more than 168 registers only two fit, and the 768 work-groups
//   of the 256^3 box run as one and a half rounds.  Three waves per SIMD (168 registers,
//   8-20 bytes of spill): general curvatures +27 % (BF16) and +8 % (FP16); a third
//   composition with BF16 (175 registers) +8 %.
// - 2D with 16-bit storage and flow, kernels of 129-146 registers (three waves): four
//   waves per SIMD measured at 2048^2 +9-13 % with a third composition, +13-14 % for the
//   variable-density model on D2Q9 scalars, +14 % for the paper's D2Q9 lattices with
//   FP16, +8 % for MRT on D2Q5 with BF16; general curvatures on D2Q5 need 127-135 registers:
//   2048^2 FP16 126 us a step against 147, 1500 x 700 BF16 in single steps 42.7 against 44.4;
// - the D3Q19 scalar lattices with flow in FP32, whose one-plane LDS ring lets two
//   work-groups share a compute unit (128^3: 294 us a step; 310 at one wave with the next
//   plane in registers).
// Measured slower with the higher floor: MRT on D3Q7 (-16 %, 200 registers) and on D3Q19
// with FP16, the third composition on D3Q7 with FP16, the general-curvature D3Q19 and
// D2Q9 (FP16) kernels, the variable-density model on D2Q5 (BF16), and every other kernel
// in FP32 / FP64
template <class SL, int PREC, int COLL, int NC = 2, int QF = 0>
constexpr int lbm_waves() {
    constexpr bool s16 = PREC == P16 || PREC == PB16;
    constexpr bool coll = (COLL & COLL_GK) == 0 && ((COLL & COLL_MRT) == 0 || PREC == PB16);
    if constexpr (s16 && SL::Q == 19 && coll) return 2;
    if constexpr (PREC == P32 && SL::Q == 19 && QF > 0) return 2;
    if constexpr (s16 && SL::Q == 7 && (COLL & COLL_GK) != 0) return 3;
    if constexpr (PREC == PB16 && SL::Q == 7 && NC == 3) return 3;
    if constexpr (s16 && SL::DIM == 2 && QF > 0) {
        if constexpr (NC == 3) return 4;
        if constexpr (SL::Q == 9 && COLL == COLL_VD) return 4;
        if constexpr (SL::Q == 9 && COLL == COLL_BGK && PREC == P16) return 4;
        if constexpr (SL::Q == 5 && COLL == COLL_MRT && PREC == PB16) return 4;
        if constexpr (SL::Q == 5 && COLL == COLL_GK) return 4;
    }
    return LBM_WAVES_PER_EU;
}

// GEN: any grid.  3D: the tile is P.tile_x x P.tile_y nodes, and a source copy with raw
// populations at the x and y walls (P.raw_xy) bounces back there; stores are plain.
// Otherwise 64 x 4 tiles (3D), exchanged copies, and non-temporal stores: the grids whose
// rows are whole 128-byte lines.  The general kernel spills more scalar registers: on D3Q7 with
// flow 83 against 31 in FP32 and 98 against 39 in FP64, to vector lanes (2-6 % on such a grid);
// on D3Q19 scalars 370 against 56 and 422 against 70, with 72 and 68 bytes of scratch memory,
// most of them for the x and y walls of raw copies (224 x 128 x 128 FP32, which has none, 647 us a
// step against 530).  Which grids take it: general_tiles, pull_walls (plan.hpp).
template <class SL, class FL, int MODE, int PREC, int NT, bool GEN, int COLL = COLL_BGK, int NC = 2>
__global__ void __launch_bounds__(NT) __attribute__((amdgpu_waves_per_eu(lbm_waves<SL, PREC, COLL, NC, FL::Q>())))
k_lbm(const KParams P) {
    using C = typename Stor<PREC>::C;
    using SLOTS = Slots<FL::Q, SL::Q, NC>;
    constexpr int QS = SL::Q;
    constexpr int QF = FL::Q;
    constexpr bool FLOW = QF > 0 && MODE != MODE_SCALARS;
    constexpr bool STENCIL = FLOW || MODE == MODE_DIAG;
    constexpr bool HAS_Y = SL::DIM == 3;
    using NODE = Node<SL, FL, PREC, COLL, NC>;
    using STL = typename NODE::STL;
    // 3D: a tile of up to NT nodes (GEN: P.tile_x x P.tile_y, lbm_api.hip); 2D: a row
    // segment of NT nodes
    constexpr int NSLOT = STENCIL ? 3 : 1;
    constexpr int CELLS = HAS_Y ? (GEN ? kTileCells : (kTileX + 2) * (kTileY + 2)) : NT + 2;  // phi of a tile and its ring
    constexpr int G0 = SLOTS::G0, A0 = SLOTS::A0, B0 = SLOTS::B0, HC0 = SLOTS::C0;
    // NC = 3: a third independent composition C (N components), BGK Boussinesq step
    constexpr bool NC3 = NC == 3;
    constexpr int QC = NC3 ? QS : 1;
    static_assert(NC == 2 || (NC == 3 && COLL == COLL_BGK), "a third composition runs with the BGK Boussinesq step");
    static_assert(SLOTS::N <= kMaxSlots, "slot table too small for this lattice family");
    constexpr bool VD = NODE::VD;
    constexpr bool GK = NODE::GK;
    // the private LDS ring of scalar populations: two planes where they leave room for a
    // second work-group per compute unit.  One plane, exchanged in place (INPLACE: the next
    // plane's populations go in as the current plane's come out), for FP64 on D3Q7 and FP32
    // on D3Q19 scalars: half the LDS, two work-groups per compute unit instead of one.  The
    // D3Q19 kernels with 16-bit storage take the packed ring (30 words per node and plane,
    // 61 KB) and two waves per SIMD (lbm_waves).  FP64 on D3Q19 keeps the next plane in
    // registers (117 KB a plane)
    constexpr int PLANE = (1 + NC) * QS * NT * int(sizeof(C));
    constexpr bool S16 = PREC == P16 || PREC == PB16;
    // wall planes replace their bounced populations after the common loads instead of taking a
    // copy of the whole fill: in the general kernel, and where the copy crowds the registers
    // (128^3 D3Q19 scalars BF16 210 us a step against 230).  The variable-density model in FP16
    // keeps the copy (256^3 D3Q19 scalars 1720 us a step, 1770 with the replacement)
    constexpr bool REPL = GEN || (S16 && QS == 19 && !(VD && PREC == P16));
    constexpr bool INPLACE = HAS_Y && STENCIL && !S16 && 2 * PLANE > 64 * 1024 && PLANE <= 64 * 1024;
    constexpr bool LDS_POPS = LBM_LDS_POPS && (INPLACE || lbm_waves<SL, PREC, COLL, NC, FL::Q>() == 2 ||
                                               2 * PLANE <= 96 * 1024);
    static_assert((QS - 1) % 2 == 0, "moving directions come in opposite pairs");

    __shared__ C sphi[NSLOT][CELLS];
    // this thread's own scalar populations of the current and the next plane
    // (thread-private ring of two planes, [plane][word][thread], no barriers needed).
    // FP32 / FP64: one word per population.  16-bit storage (PACKED): per field, the
    // FP32 rest population and the raw 16-bit moving populations of k and opp(k) packed
    // in one 32-bit word: 12 LDS words per node and plane instead of 21 (29 KB per
    // work-group instead of 48 KB; registers then bound the occupancy at three waves per
    // SIMD)
    constexpr bool PACKED = LDS_POPS && (PREC == P16 || PREC == PB16);
    constexpr int NPAIR = (QS - 1) / 2;
    constexpr int NWORD = PACKED ? (1 + NC) * (1 + NPAIR) : (1 + NC) * QS;
    using W = typename std::conditional<PACKED, unsigned, C>::type;
    __shared__ W spop[(STENCIL && LDS_POPS && !INPLACE) ? 2 : 1][(STENCIL && LDS_POPS) ? NWORD : 1][(STENCIL && LDS_POPS) ? NT : 1];

    const int tid = threadIdx.x;
    const int tw = HAS_Y ? (GEN ? P.tile_x : kTileX) : NT, th = HAS_Y ? (GEN ? P.tile_y : kTileY) : 1;
    const int lx = tw + 2;  // a row of phi with its ring
    // lanes beyond the tile repeat its last row (nothing of theirs is stored)
    const int row = HAS_Y ? (GEN ? (tid * P.tile_inv) >> 16 : tid / kTileX) : 0;
    const int tx = tid - row * tw, ty = GEN ? min(row, th - 1) : row;
    // tile of this work-group: x fastest, then y, then the z chunk
    const int tile = xcd_tile(blockIdx.x, P.tiles_x * P.tiles_y * P.tiles_z);
    const int bx = tile % P.tiles_x;
    const int by = (tile / P.tiles_x) % P.tiles_y;
    const int bz = tile / (P.tiles_x * P.tiles_y);
    const int x = bx * tw + tx;
    const int y = by * th + ty;
    const bool active = (!GEN || row < th) && (x < P.nx) && (y < P.ny);
    const int cell = HAS_Y ? (ty + 1) * lx + tx + 1 : tx + 1;  // phi of this node in sphi
    // the source copy holds raw populations at the x and y walls and this tile or its ring
    // touches one: its pulls bounce back there (a second variant of the loads)
    const bool edge = HAS_Y && GEN && P.raw_xy &&
                      ((P.wall_x && (bx * tw <= 1 || (bx + 1) * tw >= P.nx - 1)) ||
                       (P.wall_y && (by * th <= 1 || (by + 1) * th >= P.ny - 1)));
    // does the pull of a population moving along (ex, ey, ez) at node (xx, yy, .) bounce back:
    // at a z wall (zlo / zhi, wave-uniform), or at an x or y wall of a raw copy (per lane)?
    auto bounces = [&](auto ex_, auto ey_, auto ez_, bool zlo, bool zhi, int xx, int yy)
                       __attribute__((always_inline)) -> bool {
        constexpr int ex = decltype(ex_)::value, ey = decltype(ey_)::value;
        bool b = false;
        if constexpr (ex != 0) b = P.wall_x && xx == (ex > 0 ? 0 : P.nx - 1);
        if constexpr (ey != 0) b = b || (P.wall_y && yy == (ey > 0 ? 0 : P.ny - 1));
        return (HAS_Y && GEN && P.raw_xy && b) || zbounce<decltype(ez_)::value>(zlo, zhi);
    };

    const int z0 = bz * P.zc;
    const int z1 = min(z0 + P.zc, P.nz);

    using SLT = std::common_type<SL>;  // type tags of the lattices
    using FLT = std::common_type<FL>;

    // wave-uniform slot bases of the source and destination copies.  The 2 x Q_tot
    // 64-bit bases do not fit in the SGPR file, and computing each from a copy base and
    // the slot strides costs about eight scalar instructions.  The host stores every
    // base in the parameter block; the kernel reads them through a kernel-argument
    // pointer that refresh_bases() makes opaque at the top of every plane, so each base
    // is one scalar load (merged with its neighbours) next to its use, and nothing is
    // hoisted into the SGPR file and spilled.
    using kconst = __attribute__((address_space(4))) const char;
    using kslot = __attribute__((address_space(4))) const unsigned long long;
    static_assert(offsetof(KParams, dst_slot) == offsetof(KParams, src_slot) + kMaxSlots * sizeof(void*),
                  "slot tables are adjacent");
    // the parameter block is the kernel's only argument, at offset 0 of the segment
    kconst* kargs = (kconst*)__builtin_amdgcn_kernarg_segment_ptr();
    auto refresh_bases = [&]() __attribute__((always_inline)) { asm volatile("" : "+s"(kargs)); };
    // the table entries lose the address space; the casts restore `global` so the
    // accesses stay global_* with a 32-bit voffset instead of flat_* with 64-bit addresses
    using gconst = __attribute__((address_space(1))) const char;
    using gmut = __attribute__((address_space(1))) char;
    auto src = [&](auto s_) __attribute__((always_inline)) -> const char* {
        constexpr int S = decltype(s_)::value;
        const unsigned long long b = reinterpret_cast<kslot*>(kargs + offsetof(KParams, src_slot))[S];
        return (const char*)(gconst*)b;
    };
    auto dst = [&](auto s_) __attribute__((always_inline)) -> char* {
        constexpr int S = decltype(s_)::value;
        const unsigned long long b = reinterpret_cast<kslot*>(kargs + offsetof(KParams, dst_slot))[S];
        return (char*)(gmut*)b;
    };
    auto wref_dec = [&](auto s_, auto k_, auto lat_) __attribute__((always_inline)) -> float {
        return NODE::wref_dec(P, s_, k_, lat_);
    };
    // fluid populations that arrive without an x shift are read by this work-group
    // only (no ring, no x neighbour shares their lines): streamed past the caches.
    // Measured: +1.7% for the 3D step, -1.7% for 2D (one row per work-group), so 3D only
    auto load_once = [&](auto s_, auto k_, auto lat_, unsigned idx) __attribute__((always_inline)) -> C {
        constexpr int S = decltype(s_)::value;
        using L = typename decltype(lat_)::type;
        constexpr bool ONCE = LBM_NT_FLUID && SL::DIM == 3 && L::ex(decltype(k_)::value) == 0;
        return ld_at<PREC, SLOTS::rest(S), ONCE>(src(s_), idx, wref_dec(s_, k_, lat_), P.finv[SLOTS::field(S)]);
    };
    // scalar populations arriving at node idx (pull from idx - e_k; the node's own opposite
    // population where that crosses a z wall: zlo / zhi, wave-uniform).  REPL: bounce_pops
    // replaces those that bounce back at any wall (a branch that only planes and tiles at a
    // wall take, its loads in the same batch)
    // The scalar populations of a node in their stored form (RAW: 16-bit storage keeps
    // the bits of the moving populations and of the FP32 rest population, decoded later;
    // FP32 / FP64 the values), field-major: g, hA, hB (, hC), QS each
    constexpr bool RAW16 = PREC == P16 || PREC == PB16;
    constexpr int NSC = (1 + NC) * QS;
    using RW = typename std::conditional<RAW16, unsigned, C>::type;
    auto one_pop = [&](auto s_, unsigned t) __attribute__((always_inline)) -> RW {
        constexpr int S = decltype(s_)::value;
        if constexpr (!RAW16) return ld_at<PREC, SLOTS::rest(S)>(src(s_), t, 0.0f, 1.0f);
        else if constexpr (SLOTS::rest(S)) return __builtin_bit_cast(unsigned, ld_at<PREC, true>(src(s_), t, 0.0f, 1.0f));
        else return *reinterpret_cast<const unsigned short*>(src(s_) + t * 2u);
    };
    // every field's population k from slot kk at node t
    auto pops_at = [&](auto k_, auto kk_, unsigned t, RW (&raw)[NSC]) __attribute__((always_inline)) {
        constexpr int k = decltype(k_)::value, kk = decltype(kk_)::value;
        raw[k] = one_pop(IC<G0 + kk>{}, t);
        raw[QS + k] = one_pop(IC<A0 + kk>{}, t);
        raw[2 * QS + k] = one_pop(IC<B0 + kk>{}, t);
        if constexpr (NC3) raw[3 * QS + k] = one_pop(IC<HC0 + kk>{}, t);
    };
    auto load_pops = [&](unsigned idx, const Nbr& nb, bool zlo, bool zhi, RW (&raw)[NSC]) __attribute__((always_inline)) {
        static_for<0, QS>([&](auto kc) __attribute__((always_inline)) {
            constexpr int k = decltype(kc)::value, o = SL::opp(k);
            if (!REPL && zbounce<SL::ez(k)>(zlo, zhi)) pops_at(kc, IC<o>{}, idx, raw);
            else pops_at(kc, kc, unsigned(int(idx) + pull_offset<SL::ex(k), SL::ey(k), SL::ez(k)>(nb)), raw);
        });
    };
    auto bounce_pops = [&](unsigned idx, bool zlo, bool zhi, int xx, int yy, RW (&raw)[NSC]) __attribute__((always_inline)) {
        static_for<1, QS>([&](auto kc) __attribute__((always_inline)) {
            constexpr int k = decltype(kc)::value, o = SL::opp(k);
            if (bounces(IC<SL::ex(k)>{}, IC<SL::ey(k)>{}, IC<SL::ez(k)>{}, zlo, zhi, xx, yy)) pops_at(kc, IC<o>{}, idx, raw);
        });
    };
    // decoded values of one field (base slot B, first raw entry R0)
    auto decode_field = [&](auto b_, const RW* raw, C (&x)[QS]) __attribute__((always_inline)) {
        constexpr int B = decltype(b_)::value;
        static_for<0, QS>([&](auto kc) __attribute__((always_inline)) {
            constexpr int k = decltype(kc)::value;
            if constexpr (!RAW16) x[k] = raw[k];
            else if constexpr (k == 0) x[0] = __builtin_bit_cast(float, raw[0]);
            else x[k] = dec_lo<PREC>(raw[k], wref_dec(IC<B + k>{}, kc, SLT{}), P.finv[SLOTS::field(B)]);
        });
    };
    auto decode_pops = [&](const RW (&raw)[NSC], C (&gg)[QS], C (&aa)[QS], C (&bb)[QS], C (&qq)[QC])
                           __attribute__((always_inline)) {
        decode_field(IC<G0>{}, raw, gg);
        decode_field(IC<A0>{}, raw + QS, aa);
        decode_field(IC<B0>{}, raw + 2 * QS, bb);
        if constexpr (NC3) decode_field(IC<HC0>{}, raw + 3 * QS, qq);
    };
    auto load_scalars = [&](unsigned idx, const Nbr& nb, bool zlo, bool zhi, C (&gg)[QS], C (&aa)[QS],
                            C (&bb)[QS], C (&qq)[QC], double& phis, double& cA, double& cB, double& cC)
                            __attribute__((always_inline)) {
        RW raw[NSC];
        load_pops(idx, nb, zlo, zhi, raw);
        if (REPL && (zlo || zhi || edge)) bounce_pops(idx, zlo, zhi, x, y, raw);
        decode_pops(raw, gg, aa, bb, qq);
        NODE::pop_sums(gg, aa, bb, qq, phis, cA, cB, cC);
    };
    // phi of a node from its population sums (Eqs. Moment0_Phi, PotChem)
    auto phi_from = [&](double ps, double sa, double sb, double sc) __attribute__((always_inline)) -> double {
        double muC;
        return NODE::scalars(ps, sa, sb, sc, P, muC).phi;
    };

    auto node_phi = [&](int xx, int yy, int zz, bool zlo, bool zhi) __attribute__((always_inline)) -> C {
        C tg[QS], ta[QS], tb[QS], tq[QC];
        double ps, sa, sb, sc;
        load_scalars(unsigned((zz * P.ny + yy) * P.nx + xx), neighbours(xx, yy, zz, P), zlo, zhi, tg, ta, tb, tq,
                     ps, sa, sb, sc);
        return C(phi_from(ps, sa, sb, sc));
    };

    // scalar populations and sums of this thread's node: current plane (c*) and next plane (n*)
    C cg[QS], ca[QS], cb[QS], ng[QS], na[QS], nb[QS], cq[QC], nq[QC];
    double c_ps = 0.0, c_cA = 0.0, c_cB = 0.0, n_ps = 0.0, n_cA = 0.0, n_cB = 0.0, c_cC = 0.0, n_cC = 0.0;

    // PACKED: this node's own scalar populations (stored form) into the LDS ring (per
    // field: the FP32 rest population, then the moving populations of k and opp(k) in one
    // word) and their zeroth moments (the moving populations summed as moving_sum does)
    auto finish_packed = [&](const RW (&raw)[NSC], int pbuf, double& phis, double& cA, double& cB, double& cC)
                             __attribute__((always_inline)) {
      if constexpr (PACKED) {
        auto field = [&](auto b_, auto w0_, const RW* r, double& sum) __attribute__((always_inline)) {
            constexpr int B = decltype(b_)::value;    // slot of the field's rest population
            constexpr int W0 = decltype(w0_)::value;  // the field's first LDS word
            constexpr int F = SLOTS::field(B);
            spop[pbuf][W0][tid] = r[0];
            C m = C(0);
            static_for<1, QS>([&](auto kc) __attribute__((always_inline)) {
                constexpr int k = decltype(kc)::value, o = SL::opp(k);
                if constexpr (k < o) {
                    constexpr int PI = pair_index<SL, k>();
                    const unsigned w = r[k] | (r[o] << 16);
                    spop[pbuf][W0 + 1 + PI][tid] = w;
                    const C dk = dec_lo<PREC>(w, wref_dec(IC<B + k>{}, kc, SLT{}), P.finv[F]);
                    const C dd = dec_hi<PREC>(w, wref_dec(IC<B + o>{}, IC<o>{}, SLT{}), P.finv[F]);
                    if constexpr (PI == 0) m = dk + dd;
                    else m = (m + dk) + dd;
                }
            });
            sum = double(__builtin_bit_cast(float, r[0])) + double(m);
        };
        field(IC<G0>{}, IC<0>{}, raw, phis);
        field(IC<A0>{}, IC<1 + NPAIR>{}, raw + QS, cA);
        field(IC<B0>{}, IC<2 * (1 + NPAIR)>{}, raw + 2 * QS, cB);
        if constexpr (NC3) field(IC<HC0>{}, IC<3 * (1 + NPAIR)>{}, raw + 3 * QS, cC);
        else cC = 0.0;
      }
    };
    auto fill_packed = [&](unsigned idx, const Nbr& nb, bool zlo, bool zhi, int pbuf, double& phis, double& cA,
                           double& cB, double& cC) __attribute__((always_inline)) {
        RW raw[NSC];
        load_pops(idx, nb, zlo, zhi, raw);
        if (REPL && (zlo || zhi)) bounce_pops(idx, zlo, zhi, x, y, raw);
        finish_packed(raw, pbuf, phis, cA, cB, cC);
    };

    // 3D plane fill with one memory round trip: every lane loads its own node (lanes
    // outside the domain an in-range stand-in) and one ring node (lanes beyond the ring
    // repeat its last node) in one basic block, so that all loads go out together; only
    // the waves that hold ring nodes decode them (a wave-uniform branch).  The stores
    // need no conditions: a lane's private LDS ring entries and the phi cells of lanes
    // outside the domain are never read, and a repeated node writes the same value to the
    // same cell.
    const int NH = 2 * lx + 2 * th;
    auto ring_cell = [&](int& hx, int& hy) __attribute__((always_inline)) {
        const int i = min(tid, NH - 1);
        if (i < lx) { hx = i; hy = 0; }
        else if (i < 2 * lx) { hx = i - lx; hy = th + 1; }
        else if (i < 2 * lx + th) { hx = 0; hy = i - 2 * lx + 1; }
        else { hx = lx - 1; hy = i - 2 * lx - th + 1; }
    };
    auto fill_load = [&](int zm, bool zlo, bool zhi, RW (&own)[NSC], RW (&ring)[NSC])
                         __attribute__((always_inline)) {
        static_assert(NT % 64 == 0, "whole waves");
        const int ox = map_coord(min(x, P.nx), P.nx, P.wall_x), oy = map_coord(min(y, P.ny), P.ny, P.wall_y);
        int hx, hy;
        ring_cell(hx, hy);
        const int rx = map_coord(min(bx * tw + hx - 1, P.nx), P.nx, P.wall_x);
        const int ry = map_coord(min(by * th + hy - 1, P.ny), P.ny, P.wall_y);
        const unsigned oi = unsigned((zm * P.ny + oy) * P.nx + ox), ri = unsigned((zm * P.ny + ry) * P.nx + rx);
        load_pops(oi, neighbours(ox, oy, zm, P), zlo, zhi, own);
        load_pops(ri, neighbours(rx, ry, zm, P), zlo, zhi, ring);
        if (REPL && (zlo || zhi || edge)) {
            bounce_pops(oi, zlo, zhi, ox, oy, own);
            bounce_pops(ri, zlo, zhi, rx, ry, ring);
        }
    };
    auto fill_finish = [&](const RW (&own)[NSC], const RW (&ring)[NSC], int slot, int pbuf, double& ps, double& cA,
                           double& cB, double& cC) __attribute__((always_inline)) {
        if constexpr (PACKED) {
            finish_packed(own, pbuf, ps, cA, cB, cC);
        } else if constexpr (LDS_POPS) {
            C gg[QS], aa[QS], bb[QS], qq[QC];
            decode_pops(own, gg, aa, bb, qq);
            if constexpr (INPLACE) {
                // the current plane's populations come out (of the prologue's fills nothing does)
#pragma unroll
                for (int k = 0; k < QS; ++k) {
                    cg[k] = spop[0][k][tid];
                    ca[k] = spop[0][QS + k][tid];
                    cb[k] = spop[0][2 * QS + k][tid];
                    if constexpr (NC3) cq[k] = spop[0][3 * QS + k][tid];
                }
                pbuf = 0;
            }
#pragma unroll
            for (int k = 0; k < QS; ++k) {
                spop[pbuf][k][tid] = gg[k];
                spop[pbuf][QS + k][tid] = aa[k];
                spop[pbuf][2 * QS + k][tid] = bb[k];
                if constexpr (NC3) spop[pbuf][3 * QS + k][tid] = qq[k];
            }
            NODE::pop_sums(gg, aa, bb, qq, ps, cA, cB, cC);
        } else {
            decode_pops(own, ng, na, nb, nq);
            NODE::pop_sums(ng, na, nb, nq, ps, cA, cB, cC);
        }
        sphi[slot][cell] = C(phi_from(ps, cA, cB, cC));
        // the first lane of this wave holds a ring node (wave-uniform)
        if (__builtin_amdgcn_readfirstlane(tid) < NH) {
            C tg[QS], ta[QS], tb[QS], tq[QC];
            double rps, rsa, rsb, rsc;
            int hx, hy;
            ring_cell(hx, hy);
            decode_pops(ring, tg, ta, tb, tq);
            NODE::pop_sums(tg, ta, tb, tq, rps, rsa, rsb, rsc);
            sphi[slot][hy * lx + hx] = C(phi_from(rps, rsa, rsb, rsc));
        }
    };

    // 2D: a row segment and the nodes on both sides of it
    auto fill_row = [&](int zm, bool zlo, bool zhi, int slot, int pbuf, double& ps, double& cA, double& cB,
                        double& cC) __attribute__((always_inline)) {
        if (active) {
            if constexpr (PACKED) {
                fill_packed(unsigned(zm * P.nx + x), neighbours(x, 0, zm, P), zlo, zhi, pbuf, ps, cA, cB, cC);
            } else if constexpr (LDS_POPS) {
                C gg[QS], aa[QS], bb[QS], qq[QC];
                load_scalars(unsigned(zm * P.nx + x), neighbours(x, 0, zm, P), zlo, zhi, gg, aa, bb, qq, ps, cA,
                             cB, cC);
#pragma unroll
                for (int k = 0; k < QS; ++k) {
                    spop[pbuf][k][tid] = gg[k];
                    spop[pbuf][QS + k][tid] = aa[k];
                    spop[pbuf][2 * QS + k][tid] = bb[k];
                    if constexpr (NC3) spop[pbuf][3 * QS + k][tid] = qq[k];
                }
            } else {
                load_scalars(unsigned(zm * P.nx + x), neighbours(x, 0, zm, P), zlo, zhi, ng, na, nb, nq, ps, cA,
                             cB, cC);
            }
            sphi[slot][cell] = C(phi_from(ps, cA, cB, cC));
        } else if (x <= P.nx) {
            // ghost column just beyond the domain edge
            sphi[slot][cell] = node_phi(map_coord(x, P.nx, P.wall_x), 0, zm, zlo, zhi);
        }
        for (int i = tid; i < 2; i += NT) {
            const int hx = (i == 0) ? 0 : lx - 1;
            const int gx = bx * tw + hx - 1;
            if (gx > P.nx) continue;  // beyond the ghost layer: never read
            sphi[slot][hx] = node_phi(map_coord(gx, P.nx, P.wall_x), 0, zm, zlo, zhi);
        }
    };

    // phi of plane zz (tile + ring) into LDS slot `slot`; this thread's own node populations
    // go to the private LDS ring entry `pbuf`
    auto fill_body = [&](int zm, bool zlo, bool zhi, int slot, int pbuf, double& ps, double& cA, double& cB,
                         double& cC) __attribute__((always_inline)) {
        if constexpr (HAS_Y) {
            RW own[NSC], ring[NSC];
            fill_load(zm, zlo, zhi, own, ring);
            // keep the scheduler from moving the decode and sums of the own node between the
            // loads (it would then wait for them before the ring loads go out)
            __builtin_amdgcn_sched_barrier(0);
            fill_finish(own, ring, slot, pbuf, ps, cA, cB, cC);
        } else {
            fill_row(zm, zlo, zhi, slot, pbuf, ps, cA, cB, cC);
        }
    };
    auto fill_plane = [&](int zz, int slot, int pbuf, double& ps, double& cA, double& cB, double& cC)
                          __attribute__((always_inline)) {
        const int zm = map_coord(zz, P.nz, P.wall_z);
        const bool zlo = P.wall_z && zm == 0, zhi = P.wall_z && zm == P.nz - 1;
        // not REPL: a z wall plane is a separate, uniform branch, and the interior planes keep
        // the plain loads
        if (REPL || zlo || zhi) fill_body(zm, zlo, zhi, slot, pbuf, ps, cA, cB, cC);
        else fill_body(zm, false, false, slot, pbuf, ps, cA, cB, cC);
    };

    // diagnostics: the kNumDiag reductions, then sum c^C with a third composition
    constexpr int NACC = (MODE == MODE_DIAG) ? (NC3 ? kNumDiag + 1 : kNumDiag) : 1;
    // this node's scalar populations of plane z from the private LDS ring into registers
    // (read right after the barrier: reading them only where the g and h collisions use
    // them frees about 18 VGPRs but measured 17 % slower, the LDS latency exposed)
    auto fetch_pops = [&](int zz) __attribute__((always_inline)) {
        if constexpr (PACKED && STENCIL) {
            if (active) {
                const int pb = (zz - z0) & 1;
                auto field = [&](auto b_, auto w0_, C(&x)[QS]) __attribute__((always_inline)) {
                    constexpr int B = decltype(b_)::value;
                    constexpr int W0 = decltype(w0_)::value;
                    constexpr int F = SLOTS::field(B);
                    x[0] = __builtin_bit_cast(float, spop[pb][W0][tid]);
                    static_for<1, QS>([&](auto kc) __attribute__((always_inline)) {
                        constexpr int k = decltype(kc)::value, o = SL::opp(k);
                        if constexpr (k < o) {
                            const unsigned w = spop[pb][W0 + 1 + pair_index<SL, k>()][tid];
                            x[k] = dec_lo<PREC>(w, wref_dec(IC<B + k>{}, kc, SLT{}), P.finv[F]);
                            x[o] = dec_hi<PREC>(w, wref_dec(IC<B + o>{}, IC<o>{}, SLT{}), P.finv[F]);
                        }
                    });
                };
                field(IC<G0>{}, IC<0>{}, cg);
                field(IC<A0>{}, IC<1 + NPAIR>{}, ca);
                field(IC<B0>{}, IC<2 * (1 + NPAIR)>{}, cb);
                if constexpr (NC3) field(IC<HC0>{}, IC<3 * (1 + NPAIR)>{}, cq);
            }
        } else if constexpr (LDS_POPS && STENCIL && !INPLACE) {
            if (active) {
                const int pb = (zz - z0) & 1;
#pragma unroll
                for (int k = 0; k < QS; ++k) {
                    cg[k] = spop[pb][k][tid];
                    ca[k] = spop[pb][QS + k][tid];
                    cb[k] = spop[pb][2 * QS + k][tid];
                    if constexpr (NC3) cq[k] = spop[pb][3 * QS + k][tid];
                }
            }
        }
    };
    double acc[NACC];
#pragma unroll
    for (int i = 0; i < NACC; ++i) acc[i] = 0.0;

    const double phi_ref = P.mean_subtract ? *P.phi_ref : 0.0;
    if constexpr (MODE == MODE_STEP || MODE == MODE_STEP_PHI) {
        // a step between caller checkpoints carries the buffered <phi> over
        if (P.ref_copy && blockIdx.x == 0 && tid == 0) *P.ref_copy = *P.phi_ref;
    }

    if constexpr (STENCIL) {
        if (z0 < z1) {
            fill_plane(z0 - 1, 0, 1, n_ps, n_cA, n_cB, n_cC);  // ring only; own entries overwritten next
            fill_plane(z0, 1, 0, c_ps, c_cA, c_cB, c_cC);
            if constexpr (!LDS_POPS) {
#pragma unroll
                for (int k = 0; k < QS; ++k) { cg[k] = ng[k]; ca[k] = na[k]; cb[k] = nb[k]; }
                if constexpr (NC3) {
#pragma unroll
                    for (int k = 0; k < QS; ++k) cq[k] = nq[k];
                }
            }
        }
    }

    for (int z = z0; z < z1; ++z) {
        refresh_bases();
        int sm = 0, sc = 0, sp = 0;
        const unsigned idx = unsigned((z * P.ny + y) * P.nx + x);
        const Nbr nbr = neighbours(x, y, z, P);
        C fpop[QF > 0 ? QF : 1];
        // 16-bit storage: the moving f arrive as raw bits and are decoded where the flow
        // moments need them, so that no wait for them sits before the plane fill's loads
        constexpr bool FRAW = LBM_FRAW && (PREC == P16 || PREC == PB16);
        unsigned fraw[(QF > 0 && FRAW) ? QF : 1];
        auto one_f = [&](auto kc, auto from_, unsigned t) __attribute__((always_inline)) {
            constexpr int k = decltype(kc)::value;
            if constexpr (FRAW && k != 0) {
                constexpr bool ONCE = LBM_NT_FLUID && SL::DIM == 3 && FL::ex(k) == 0;
                fraw[k] = ld_raw<unsigned short, ONCE>(reinterpret_cast<const unsigned short*>(src(from_) + t * 2u));
            } else {
                fpop[k] = load_once(from_, from_, FLT{}, t);
            }
        };
        auto load_f_body = [&](bool zlo, bool zhi) __attribute__((always_inline)) {
            static_for<0, QF>([&](auto kc) __attribute__((always_inline)) {
                constexpr int k = decltype(kc)::value;
                if (!REPL && zbounce<FL::ez(k)>(zlo, zhi)) one_f(kc, IC<FL::opp(k)>{}, idx);
                else one_f(kc, kc, unsigned(int(idx) + pull_offset<FL::ex(k), FL::ey(k), FL::ez(k)>(nbr)));
            });
        };
        auto bounce_f = [&](bool zlo, bool zhi) __attribute__((always_inline)) {
            static_for<1, QF>([&](auto kc) __attribute__((always_inline)) {
                constexpr int k = decltype(kc)::value;
                if (bounces(IC<FL::ex(k)>{}, IC<FL::ey(k)>{}, IC<FL::ez(k)>{}, zlo, zhi, x, y)) one_f(kc, IC<FL::opp(k)>{}, idx);
            });
        };
        // 16-bit storage: z-wall bounce-back by selecting the source slot and node (no
        // branch: the loads stay in one basic block with the plane fill's)
        auto load_f_sel = [&]() __attribute__((always_inline)) {
            const bool zlo = P.wall_z && z == 0, zhi = P.wall_z && z == P.nz - 1;
            // lanes outside the domain load an in-range node (their values are not used)
            const int fx = min(x, P.nx - 1), fy = min(y, P.ny - 1);
            const unsigned fidx = unsigned((z * P.ny + fy) * P.nx + fx);
            const Nbr fnb = neighbours(fx, fy, z, P);
            static_for<0, QF>([&](auto kc) __attribute__((always_inline)) {
                constexpr int k = decltype(kc)::value, o = FL::opp(k);
                if constexpr (k != 0) {
                    constexpr bool ONCE = LBM_NT_FLUID && SL::DIM == 3 && FL::ex(k) == 0;
                    const unsigned pulled = unsigned(int(fidx) + pull_offset<FL::ex(k), FL::ey(k), FL::ez(k)>(fnb));
                    const char* base = src(kc);
                    unsigned t = pulled;
                    if constexpr (FL::ez(k) != 0) {
                        const bool b = zbounce<FL::ez(k)>(zlo, zhi);
                        base = b ? src(IC<o>{}) : base;
                        t = b ? fidx : pulled;
                    }
                    fraw[k] = ld_raw<unsigned short, ONCE>(reinterpret_cast<const unsigned short*>(base + t * 2u));
                } else {
                    fpop[0] = load_once(kc, kc, FLT{}, fidx);
                }
            });
        };
        auto load_f = [&]() __attribute__((always_inline)) {
            if constexpr (FLOW) {
                const bool zlo = P.wall_z && z == 0, zhi = P.wall_z && z == P.nz - 1;
                if constexpr (FRAW && HAS_Y) {
                    load_f_sel();  // every lane loads (lanes outside the domain: in-range stand-ins)
                    if (GEN && edge && active) bounce_f(zlo, zhi);
                } else if (active) {
                    if (REPL || zlo || zhi) load_f_body(zlo, zhi);
                    else load_f_body(false, false);
                    if (REPL && (zlo || zhi || edge)) bounce_f(zlo, zhi);
                }
            }
        };
        // fluid populations of this node do not depend on the LDS plane: with
        // LBM_EARLY_F they are issued before the plane fill to overlap its latency
        if constexpr (LBM_EARLY_F) load_f();
        if constexpr (STENCIL) {
            sm = (z - z0) % 3;
            sc = (z - z0 + 1) % 3;
            sp = (z - z0 + 2) % 3;
            fill_plane(z + 1, sp, (z - z0 + 1) & 1, n_ps, n_cA, n_cB, n_cC);
            __syncthreads();
            if constexpr (LDS_POPS) fetch_pops(z);
        } else {
            if (active) {
                const bool zlo = P.wall_z && z == 0, zhi = P.wall_z && z == P.nz - 1;
                if (REPL || zlo || zhi) load_scalars(idx, nbr, zlo, zhi, cg, ca, cb, cq, c_ps, c_cA, c_cB, c_cC);
                else load_scalars(idx, nbr, false, false, cg, ca, cb, cq, c_ps, c_cA, c_cB, c_cC);
            }
        }
        if constexpr (!LBM_EARLY_F) load_f();
        const C(&g)[QS] = cg;
        const C(&a)[QS] = ca;
        const C(&b)[QS] = cb;
        const double sA = c_cA, sB = c_cB, sC = c_cC;

        if (active) {
            double muC;  // potential of a third composition
            const Scalars m = NODE::scalars(c_ps, sA, sB, sC, P, muC);
            const C phi = C(m.phi);

            C grad[3] = {C(0), C(0), C(0)};
            C lap = C(0);
            if constexpr (STENCIL) {
                NODE::stencil(
                    [&](auto ex_, auto ey_, auto ez_) __attribute__((always_inline)) -> C {
                        constexpr int ex = decltype(ex_)::value, ey = decltype(ey_)::value, ez = decltype(ez_)::value;
                        return sphi[ez == 0 ? sc : (ez > 0 ? sp : sm)][cell + ey * lx + ex];
                    },
                    sphi[sc][cell], grad, lap);
            }

            C u[3] = {C(0), C(0), C(0)};
            C p_h = C(0);  // pressure variable of f: p_h, or p* with variable density
            C F[3] = {C(0), C(0), C(0)};
            C irho = C(1);  // 1 / rho(phi) (variable density)
            if constexpr (FLOW) {
                if constexpr (FRAW) {
                    static_for<1, QF>([&](auto kc) __attribute__((always_inline)) {
                        fpop[decltype(kc)::value] = dec_lo<PREC>(fraw[decltype(kc)::value], wref_dec(kc, kc, FLT{}), P.finv[0]);
                    });
                }
                NODE::flow(P, fpop, m.phi, phi, phi_ref, grad, lap, F, u, p_h, irho);
            }

            if constexpr (MODE == MODE_STEP || MODE == MODE_STEP_PHI) {
                if (P.mean_subtract) acc[0] += m.phi;
                // phi of the source state, as the stencil saw it (for the adjoint)
                if constexpr (MODE == MODE_STEP_PHI) static_cast<C*>(P.phi_out)[idx] = phi;

                // post-collision populations go to this node's own slots of the other copy
                NODE::collide(P, fpop, g, a, b, cq, c_ps, sA, sB, sC, m, muC, phi, F, u, p_h, irho,
                              [&](auto s_, auto v) __attribute__((always_inline)) { st_raw<!GEN>(dst(s_), idx, v); });
            } else if constexpr (MODE == MODE_MOMENTS || MODE == MODE_SCALARS) {
                // hydrodynamic pressure: p_h, or rho c_s^2 p* with variable density
                const double p_out = VD && FLOW ? double(p_h) / (3.0 * double(irho)) : double(p_h);
                const double vals[kNumMom] = {m.phi, sA, sB, m.muA, m.muB, p_out,
                                              double(u[0]), double(u[1]), double(u[2]), sC, muC};
                constexpr int NMOM = NC3 ? kNumMom : kNumMom - 2;
#pragma unroll
                for (int i = 0; i < NMOM; ++i) {
                    if (P.mout[i]) {
                        if (P.mout_f32) static_cast<float*>(P.mout[i])[idx] = float(vals[i]);
                        else static_cast<double*>(P.mout[i])[idx] = vals[i];
                    }
                }
            } else {  // MODE_DIAG
                const double u2 = double(u[0]) * double(u[0]) + double(u[1]) * double(u[1]) +
                                  double(u[2]) * double(u[2]);
                const double g2 = double(grad[0]) * double(grad[0]) + double(grad[1]) * double(grad[1]) +
                                  double(grad[2]) * double(grad[2]);
                acc[0] += sA;
                acc[1] += sB;
                acc[2] += m.phi;
                acc[3] += 0.5 * (VD ? P.rho0 + P.drho * m.phi : P.rho0) * u2;
                acc[4] = fmax(acc[4], sqrt(u2));
                acc[5] += (4.0 / P.W) * m.phi * (1.0 - m.phi);
                if constexpr (NC3) {
                    acc[6] += 0.5 * P.W * P.W * g2 + dwell(m.phi) +
                              P.lam * 0.5 * (m.muA * m.muA + m.muB * m.muB + muC * muC);
                    acc[7] += (isfinite(m.phi) && isfinite(sA) && isfinite(sB) && isfinite(sC)) ? 0.0 : 1.0;
                    acc[NACC - 1] += sC;
                } else {
                    acc[6] += 0.5 * P.W * P.W * g2 + dwell(m.phi) + P.lam * bulk_free_energy<GK>(m.phi, m.muA, m.muB, P);
                    acc[7] += (isfinite(m.phi) && isfinite(sA) && isfinite(sB)) ? 0.0 : 1.0;
                }
                P.mask_out[idx] = m.phi >= 0.5 ? 1 : 0;
            }
        }
        if constexpr (STENCIL) {
            // the next plane becomes the current one
            if constexpr (!LDS_POPS) {
#pragma unroll
                for (int k = 0; k < QS; ++k) { cg[k] = ng[k]; ca[k] = na[k]; cb[k] = nb[k]; }
                if constexpr (NC3) {
#pragma unroll
                    for (int k = 0; k < QS; ++k) cq[k] = nq[k];
                }
            }
            c_ps = n_ps; c_cA = n_cA; c_cB = n_cB; c_cC = n_cC;
            __syncthreads();
        }
    }

    if constexpr (MODE == MODE_DIAG) {
        block_reduce_store<NACC, NT>(acc, 4, P.partials + NACC * tile);
    } else if constexpr (MODE == MODE_STEP || MODE == MODE_STEP_PHI) {
        if (P.mean_subtract) block_reduce_store<1, NT>(acc, -1, P.partials + tile);
    }
}

// ---------------------------------------------------------------------------
// half-way bounce-back as a fix-up between steps (Section 4.2.4: walls at rest
// with zero normal flux).  The next step pulls X_k(x) from slot k at
// wrap(x - e_k).  When x - e_k lies across a wall, bounce-back wants instead the
// post-collision population that left x towards the wall, slot opp(k) at x.
// Node x' = wrap(x - e_k) is in the mirror situation: it pulls slot opp(k) at x
// and wants its own slot k.  Exchanging the two entries serves both.  Each
// exchange is done once, by the node x and direction k with k < opp(k); each
// wall node is visited by exactly one thread: the face of its lowest-index wall
// axis.

template <class SL, class FL, int PREC, int NC = 2>
__global__ void __launch_bounds__(256) k_walls(const KParams P, int axis) {
    using SLOTS = Slots<FL::Q, SL::Q, NC>;
    // enumerate the two faces of `axis`: (b, c) span the other two axes
    const int n[3] = {P.nx, P.ny, P.nz};
    const int ab = axis == 0 ? 1 : 0, ac = axis == 2 ? 1 : 2;
    const long long face = (long long)n[ab] * n[ac];
    const long long t = (long long)blockIdx.x * blockDim.x + threadIdx.x;
    if (t >= 2 * face) return;
    int c[3];
    c[axis] = t < face ? 0 : n[axis] - 1;
    const long long r = t % face;
    c[ab] = int(r % n[ab]);
    c[ac] = int(r / n[ab]);
    // walls on x and y only: the z walls bounce back when the next step pulls
    const int wall[3] = {P.wall_x, P.wall_y, 0};
    // skip nodes owned by the face of a lower wall axis
    for (int a = 0; a < axis; ++a)
        if (wall[a] && (c[a] == 0 || c[a] == n[a] - 1)) return;
    if (n[axis] == 1 && t >= face) return;  // both faces are the same plane
    const int idx = (c[2] * P.ny + c[1]) * P.nx + c[0];

    // does x - e lie across an x or y wall (and not across a z wall, which the pull
    // handles)?
    auto crosses = [&](int ex, int ey, int ez) {
        if (P.wall_z && ez != 0 && (c[2] - ez < 0 || c[2] - ez >= n[2])) return false;
        const int e[3] = {ex, ey, ez};
        for (int a = 0; a < 3; ++a)
            if (wall[a] && e[a] != 0 && (c[a] - e[a] < 0 || c[a] - e[a] >= n[a])) return true;
        return false;
    };
    // index of wrap(x - e)
    auto source = [&](int ex, int ey, int ez) {
        const int e[3] = {ex, ey, ez};
        int q[3];
        for (int a = 0; a < 3; ++a) q[a] = (c[a] - e[a] + n[a]) % n[a];
        return (q[2] * P.ny + q[1]) * P.nx + q[0];
    };
    // raw storage word of slot S at node i
    using Word = typename std::conditional<PREC == P64, double,
                                           typename std::conditional<PREC == P32, float, unsigned short>::type>::type;
    auto word = [&](auto s_, int i) -> Word* {
        constexpr int S = decltype(s_)::value;
        return reinterpret_cast<Word*>(P.dst_base + slot_offset<SLOTS, S>(P)) + i;
    };
    // every exchange pair (slot k at wrap(x - e_k), slot opp(k) at x), k < opp(k);
    // 16-bit formats: moving populations only (equal references for k and opp(k))
    auto pairs = [&](auto&& fn) {
        auto lattice = [&](auto lat_, auto base_) {
            using L = typename decltype(lat_)::type;
            constexpr int B = decltype(base_)::value;
            static_for<1, L::Q>([&](auto kc) {
                constexpr int k = decltype(kc)::value;
                constexpr int o = L::opp(k);
                if constexpr (k < o) fn(IC<B + k>{}, IC<B + o>{}, IC<L::ex(k)>{}, IC<L::ey(k)>{}, IC<L::ez(k)>{});
            });
        };
        if constexpr (FL::Q > 0) lattice(std::common_type<FL>{}, IC<0>{});
        lattice(std::common_type<SL>{}, IC<SLOTS::G0>{});
        lattice(std::common_type<SL>{}, IC<SLOTS::A0>{});
        lattice(std::common_type<SL>{}, IC<SLOTS::B0>{});
        if constexpr (NC >= 3) lattice(std::common_type<SL>{}, IC<SLOTS::C0>{});
    };
    constexpr int NP = (FL::Q > 0 ? (FL::Q - 1) / 2 : 0) + (1 + NC) * ((SL::Q - 1) / 2);
    // all loads first, then all stores: the round trips overlap
    Word va[NP], vb[NP];
    bool cr[NP];
    int np = 0;
    pairs([&](auto s_, auto o_, auto ex_, auto ey_, auto ez_) {
        const int p = np++;
        cr[p] = crosses(ex_.value, ey_.value, ez_.value);
        if (cr[p]) {
            va[p] = *word(s_, source(ex_.value, ey_.value, ez_.value));
            vb[p] = *word(o_, idx);
        }
    });
    np = 0;
    pairs([&](auto s_, auto o_, auto ex_, auto ey_, auto ez_) {
        const int p = np++;
        if (cr[p]) {
            *word(s_, source(ex_.value, ey_.value, ez_.value)) = vb[p];
            *word(o_, idx) = va[p];
        }
    });
}

// ---------------------------------------------------------------------------
// initialisation at rest (Section 4.2.1): equilibrium populations from (phi_0, mu_0).
// A copy holds post-collision populations at the node that computed them; the
// next step pulls X_k(x) from slot k at wrap(x - e_k).  The equilibrium X_k(x) is
// therefore written to slot k at wrap(x - e_k).

template <class SL, class FL, int PREC, int NC = 2>
__global__ void __launch_bounds__(256) k_init(const KParams P, const double* __restrict__ phi0,
                                              const double* __restrict__ muA0,
                                              const double* __restrict__ muB0,
                                              const double* __restrict__ muC0) {
    using C = typename Stor<PREC>::C;
    using SLOTS = Slots<FL::Q, SL::Q, NC>;
    constexpr int G0 = SLOTS::G0, A0 = SLOTS::A0, B0 = SLOTS::B0, HC0 = SLOTS::C0;
    using STL = typename std::conditional<SL::DIM == 2, D2Q9K, D3Q19K>::type;
    const int x = blockIdx.x * blockDim.x + threadIdx.x;
    const int y = blockIdx.y, z = blockIdx.z;
    if (x >= P.nx) return;
    const int idx = (z * P.ny + y) * P.nx + x;
    const Nbr nb = neighbours(x, y, z, P);
    const double phi = phi0[idx], muA = muA0[idx], muB = muB0[idx];
    const double pp = interp_p(phi);
    // Eq. species_closure (general curvatures: c = c^eq(phi) + kappa(phi) mu), unless the
    // compositions are given (initial condition of Section 4.2.1: c stepped at phi = 1/2
    // with mu = 0)
    double kA = muA, kB = muB;  // kappa(phi) mu
    double domega = -(muA * (P.c0A - P.c1A) + muB * (P.c0B - P.c1B));
    if (P.general_k) {
        const double kAA = P.kap0[0] + pp * (P.kap1[0] - P.kap0[0]);
        const double kAB = P.kap0[1] + pp * (P.kap1[1] - P.kap0[1]);
        const double kBB = P.kap0[2] + pp * (P.kap1[2] - P.kap0[2]);
        kA = kAA * muA + kAB * muB;
        kB = kAB * muA + kBB * muB;
        const double dAA = P.kap0[0] - P.kap1[0], dAB = P.kap0[1] - P.kap1[1], dBB = P.kap0[2] - P.kap1[2];
        domega -= 0.5 * (dAA * muA * muA + 2.0 * dAB * muA * muB + dBB * muB * muB);
    }
    const double cA = P.init_c[0] ? P.init_c[0][idx] : kA + P.c0A + pp * (P.c1A - P.c0A);
    const double cB = P.init_c[1] ? P.init_c[1][idx] : kB + P.c0B + pp * (P.c1B - P.c0B);
    // a third composition: the same closure, and its share of Delta omega
    double muC = 0.0, cC = 0.0;
    if constexpr (NC >= 3) {
        muC = muC0[idx];
        cC = P.init_c[2] ? P.init_c[2][idx] : muC + P.c0C + pp * (P.c1C - P.c0C);
        domega -= muC * (P.c0C - P.c1C);
    }
    const double S0 = P.mphi_w2 * (P.lam * interp_dp(phi) * domega - dwell_d(phi));

    // returns the rounding residue (value - stored value); 16-bit storage adds the
    // residues of a field's moving populations to its rest population, written last
    auto put = [&](auto s_, auto k_, auto lat_, double v) -> double {
        using L = typename decltype(lat_)::type;
        constexpr int S = decltype(s_)::value, k = decltype(k_)::value;
        constexpr int F = SLOTS::field(S);
        unsigned t;
        char* slot = const_cast<char*>(pull_src<SLOTS, L, S, k>(P.dst_base, P, z, unsigned(idx), nb, t));
        return v - double(st_at_r<PREC, SLOTS::rest(S)>(slot, t, float(L::w(k)) * P.fref[F], P.fscale[F],
                                                         P.finv[F], C(v)));
    };
    double rg = 0.0, ra = 0.0, rb = 0.0, rc = 0.0;
    static_for<1, SL::Q>([&](auto kc) {
        constexpr int k = decltype(kc)::value;
        constexpr double wk = SL::w(k);
        rg += put(IC<G0 + k>{}, kc, std::common_type<SL>{}, wk * phi - 0.5 * wk * S0);
        ra += put(IC<A0 + k>{}, kc, std::common_type<SL>{}, wk * muA);
        rb += put(IC<B0 + k>{}, kc, std::common_type<SL>{}, wk * muB);
        if constexpr (NC >= 3) rc += put(IC<HC0 + k>{}, kc, std::common_type<SL>{}, wk * muC);
    });
    {
        constexpr double w0 = SL::w(0);
        put(IC<G0>{}, IC<0>{}, std::common_type<SL>{}, w0 * phi - 0.5 * w0 * S0 + rg);
        put(IC<A0>{}, IC<0>{}, std::common_type<SL>{}, cA - (1.0 - w0) * muA + ra);
        put(IC<B0>{}, IC<0>{}, std::common_type<SL>{}, cB - (1.0 - w0) * muB + rb);
        if constexpr (NC >= 3) put(IC<HC0>{}, IC<0>{}, std::common_type<SL>{}, cC - (1.0 - w0) * muC + rc);
    }
    if constexpr (FL::Q > 0) {
        double grad[3] = {0.0, 0.0, 0.0}, lap = 0.0;
#pragma unroll
        for (int k = 1; k < STL::Q; ++k) {
            const int xn = map_coord(x + STL::ex(k), P.nx, P.wall_x);
            const int yn = map_coord(y + STL::ey(k), P.ny, P.wall_y);
            const int zn = map_coord(z + STL::ez(k), P.nz, P.wall_z);
            const double v = phi0[(zn * P.ny + yn) * P.nx + xn];
            grad[0] += 3.0 * STL::w(k) * STL::ex(k) * v;
            grad[1] += 3.0 * STL::w(k) * STL::ey(k) * v;
            grad[2] += 3.0 * STL::w(k) * STL::ez(k) * v;
            lap += 6.0 * STL::w(k) * (v - phi);
        }
        const double phi_ref = P.mean_subtract ? *P.phi_ref : 0.0;
        const double bracket = P.cap * (dwell_d(phi) * P.inv_W2 - lap);
        const double buoy = (phi - phi_ref) * P.drho;
        const double F[3] = {buoy * P.gx + bracket * grad[0], buoy * P.gy + bracket * grad[1],
                             buoy * P.gz + bracket * grad[2]};
        double rf = 0.0;
        // variable density: dimensionless populations, forcing divided by rho(phi) c_s^2
        const double fsc = P.variable_density ? 3.0 / (P.rho0 + P.drho * phi) : 1.0;
        static_for<1, FL::Q>([&](auto kc) {
            constexpr int k = decltype(kc)::value;
            const double eF = (FL::ex(k) * F[0] + FL::ey(k) * F[1] + FL::ez(k) * F[2]) * fsc;
            // f^eq at p_h = 0, u = 0 minus F_k / 2 with Gamma_k(u = 0) = w_k
            rf += put(kc, kc, std::common_type<FL>{}, -0.5 * FL::w(k) * eF);
        });
        put(IC<0>{}, IC<0>{}, std::common_type<FL>{}, rf);  // e_0 . F = 0
    }
}

// ---------------------------------------------------------------------------
// canonical FP64 population access: X_k(x) lives in slot k at wrap(x - e_k)

template <class SL, class FL, int PREC, bool SET, int NC = 2>
__global__ void __launch_bounds__(256) k_pops(const KParams P, long long nodes, double* __restrict__ buf) {
    using C = typename Stor<PREC>::C;
    using SLOTS = Slots<FL::Q, SL::Q, NC>;
    const long long i = (long long)blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= nodes) return;
    const int x = int(i % P.nx), y = int((i / P.nx) % P.ny), z = int(i / ((long long)P.nx * P.ny));
    const Nbr nb = neighbours(x, y, z, P);
    auto one = [&](auto s_, auto k_, auto lat_) {
        using L = typename decltype(lat_)::type;
        constexpr int S = decltype(s_)::value, k = decltype(k_)::value;
        const float wref = float(L::w(k)) * P.fref[SLOTS::field(S)];
        unsigned t;
        if constexpr (SET) {
            char* slot = const_cast<char*>(pull_src<SLOTS, L, S, k>(P.dst_base, P, z, unsigned(i), nb, t));
            st_at<PREC, SLOTS::rest(S)>(slot, t, wref, P.fscale[SLOTS::field(S)], C(buf[S * nodes + i]));
        } else {
            const char* slot = pull_src<SLOTS, L, S, k>(P.src_base, P, z, unsigned(i), nb, t);
            buf[S * nodes + i] = double(ld_at<PREC, SLOTS::rest(S)>(slot, t, wref, P.finv[SLOTS::field(S)]));
        }
    };
    static_for<0, FL::Q>([&](auto kc) { one(kc, kc, std::common_type<FL>{}); });
    static_for<0, SL::Q>([&](auto kc) {
        constexpr int k = decltype(kc)::value;
        one(IC<SLOTS::G0 + k>{}, kc, std::common_type<SL>{});
        one(IC<SLOTS::A0 + k>{}, kc, std::common_type<SL>{});
        one(IC<SLOTS::B0 + k>{}, kc, std::common_type<SL>{});
        if constexpr (NC >= 3) one(IC<SLOTS::C0 + k>{}, kc, std::common_type<SL>{});
    });
}

// ---------------------------------------------------------------------------
// adjoint kernels.  The adjoint of the arriving population X_s(x) is lambda_s(x)
// (FP32 [slot][node], P.adj_in / P.adj_out) plus c_F(x) (rows of P.auxc) when s is a
// scalar population of field F.  Kernels over nodes use 256-thread work-groups; their
// theta partials accumulate in P.partials + 6 * blockIdx.x.

template <class SL, class FL>
__device__ __forceinline__ float* adj_at(const char* base, const KParams& P, int slot, unsigned long long idx) {
    return reinterpret_cast<float*>(const_cast<char*>(base) + (unsigned long long)slot * P.adj_stride + idx * 4u);
}

__device__ __forceinline__ void theta_from_K(double K_b, const KParams& P, double (&th)[6]) {
    // K = M_phi / W^2
    th[0] += K_b / (P.W * P.W);
    th[5] += K_b * (-2.0 * P.mphi_w2 / P.W);
}

// Adjoint of one step, one thread per node.  mu = dL/dQ(x) is the transposed
// streaming of the adjoint of step n + 1: mu_k(x) = Lambda_k(x + e_k), or
// Lambda_opp(k)(x) when x + e_k lies across a wall (bounce-back), where Lambda =
// lambda (+ c_F for scalar fields).  The arriving populations of state n are pulled
// as in the step; the phi stencil reads phi of state n (`phi`, written by the step
// that left state n).  lambda^n gets the local part (P.adj_out); dL/dG, dL/dN and the
// sensitivities of phi go to aux rows 0..6 for k_adj_gather; theta partials
// accumulate per work-group.
template <class SL, class FL, int PREC>
__global__ void __launch_bounds__(256)
    __attribute__((amdgpu_waves_per_eu(SL::DIM == 2 ? LBM_ADJ_WAVES_2D : LBM_ADJ_WAVES_3D)))
k_adj_node(const KParams P, long long nodes, const typename Stor<PREC>::C* __restrict__ phi) {
    using C = typename Stor<PREC>::C;
    using T = C;
    using SLOTS = Slots<FL::Q, SL::Q>;
    using STL = typename std::conditional<SL::DIM == 2, D2Q9K, D3Q19K>::type;
    constexpr int QS = SL::Q, QF = FL::Q;
    constexpr int G0 = SLOTS::G0, A0 = SLOTS::A0, B0 = SLOTS::B0;
    using SLT = std::common_type<SL>;
    using FLT = std::common_type<FL>;
    // 32-bit node index (nodes < 2^31): keeps every access in the voffset + saddr form
    const unsigned idx = blockIdx.x * 256u + threadIdx.x;
    double th[6] = {0, 0, 0, 0, 0, 0};
    if (idx < (unsigned long long)nodes) {
        const unsigned nxny = unsigned(P.nx) * unsigned(P.ny);
        const int z = int(idx / nxny), r = int(idx - unsigned(z) * nxny);
        const int y = r / P.nx, x = r - y * P.nx;
        const Nbr nbr = neighbours(x, y, z, P);
        auto load = [&](auto s_, auto k_, auto lat_) __attribute__((always_inline)) -> C {
            using L = typename decltype(lat_)::type;
            constexpr int S = decltype(s_)::value, k = decltype(k_)::value;
            unsigned t;
            const char* slot = pull_src<SLOTS, L, S, k>(P.src_base, P, z, idx, nbr, t);
            return ld_at<PREC, SLOTS::rest(S)>(slot, t, float(L::w(k)) * P.fref[SLOTS::field(S)],
                                               P.finv[SLOTS::field(S)]);
        };
        C fpop[QF > 0 ? QF : 1], g[QS], a[QS], b[QS];
        static_for<0, QF>([&](auto kc) __attribute__((always_inline)) { fpop[kc.value] = load(kc, kc, FLT{}); });
        static_for<0, QS>([&](auto kc) __attribute__((always_inline)) {
            g[kc.value] = load(IC<G0 + kc.value>{}, kc, SLT{});
            a[kc.value] = load(IC<A0 + kc.value>{}, kc, SLT{});
            b[kc.value] = load(IC<B0 + kc.value>{}, kc, SLT{});
        });
        // phi stencil inputs of Eqs. Grad and Laplacian (mirror ghosts at walls)
        double G[3] = {0.0, 0.0, 0.0}, Nsum = 0.0, pc = 0.0;
        if constexpr (QF > 0) {
            const Nbr sn = stencil_neighbours(x, y, z, P);
            const char* pb = reinterpret_cast<const char*>(phi);
            pc = double(*reinterpret_cast<const C*>(pb + voff(idx * unsigned(sizeof(C)))));
            static_for<1, STL::Q>([&](auto kc) __attribute__((always_inline)) {
                constexpr int k = decltype(kc)::value;
                constexpr int ex = STL::ex(k), ey = STL::ey(k), ez = STL::ez(k);
                const unsigned t = unsigned(int(idx) + push_offset<ex, ey, ez>(sn));
                const double v = double(*reinterpret_cast<const C*>(pb + voff(t * unsigned(sizeof(C))))) *
                                 (3.0 * STL::w(k));
                if constexpr (ex != 0) G[0] += ex > 0 ? v : -v;
                if constexpr (ey != 0) G[1] += ey > 0 ? v : -v;
                if constexpr (ez != 0) G[2] += ez > 0 ? v : -v;
                Nsum += v;
            });
        }
        const float* cin = P.auxc;
        const unsigned own = voff(idx * 4u);
        const bool lo[3] = {P.wall_x && x == 0, P.wall_y && y == 0, P.wall_z && z == 0};
        const bool hi[3] = {P.wall_x && x == P.nx - 1, P.wall_y && y == P.ny - 1, P.wall_z && z == P.nz - 1};
        // mu_s(x) = Lambda_s(wrap(x + e_s)), or Lambda_opp(s)(x) across a wall
        auto mu_of = [&](auto s_) __attribute__((always_inline)) -> T {
            constexpr int S = decltype(s_)::value;
            constexpr bool FLUID = S < G0;
            constexpr int F = FLUID ? -1 : (S - G0) / QS;  // scalar field 0 g, 1 hA, 2 hB
            constexpr int k = FLUID ? S : (S - G0) % QS;
            using L = typename std::conditional<FLUID, FL, SL>::type;
            // wave-uniform bases, 32-bit byte offsets (global_load voffset, saddr)
            const unsigned t = unsigned(int(idx) + push_offset<L::ex(k), L::ey(k), L::ez(k)>(nbr));
            const char* ls = P.adj_in + (unsigned long long)S * P.adj_stride;
            const unsigned o = voff(t * 4u);
            float v = *reinterpret_cast<const float*>(ls + o);
            if constexpr (F >= 0) {
                const char* cf = reinterpret_cast<const char*>(cin + (unsigned long long)F * P.aux_stride);
                v += *reinterpret_cast<const float*>(cf + o);
            }
            return T(v);
        };
        // bounce-back: Lambda_opp(s)(x) at the node itself when x + e_s crosses a wall
        auto mu_wall = [&](auto s_, T& v) __attribute__((always_inline)) {
            constexpr int S = decltype(s_)::value;
            constexpr bool FLUID = S < G0;
            constexpr int F = FLUID ? -1 : (S - G0) / QS;
            constexpr int k = FLUID ? S : (S - G0) % QS;
            using L = typename std::conditional<FLUID, FL, SL>::type;
            constexpr int ex = L::ex(k), ey = L::ey(k), ez = L::ez(k);
            if constexpr (ex != 0 || ey != 0 || ez != 0) {
                bool cross = false;
                if constexpr (ex > 0) cross = cross || hi[0];
                if constexpr (ex < 0) cross = cross || lo[0];
                if constexpr (ey > 0) cross = cross || hi[1];
                if constexpr (ey < 0) cross = cross || lo[1];
                if constexpr (ez > 0) cross = cross || hi[2];
                if constexpr (ez < 0) cross = cross || lo[2];
                if (cross) {
                    constexpr int O = S - k + L::opp(k);
                    const char* lo_ = P.adj_in + (unsigned long long)O * P.adj_stride;
                    float w = *reinterpret_cast<const float*>(lo_ + own);
                    if constexpr (F >= 0)
                        w += *reinterpret_cast<const float*>(
                            reinterpret_cast<const char*>(cin + (unsigned long long)F * P.aux_stride) + own);
                    v = T(w);
                }
            }
        };
        // adjoint of step n + 1 read once into registers: every neighbour load first,
        // then the wall lanes' replacements (a region that other waves skip)
        T muv[SLOTS::N];
        static_for<0, SLOTS::N>([&](auto sc) __attribute__((always_inline)) { muv[sc.value] = mu_of(sc); });
        const bool wall_lane = lo[0] || lo[1] || lo[2] || hi[0] || hi[1] || hi[2];
        if (wall_lane)
            static_for<0, SLOTS::N>([&](auto sc) __attribute__((always_inline)) { mu_wall(sc, muv[sc.value]); });
        auto mu_reg = [&](auto s_) __attribute__((always_inline)) -> T { return muv[decltype(s_)::value]; };
        auto put = [&](auto s_, T v) __attribute__((always_inline)) {
            char* o = P.adj_out + (unsigned long long)decltype(s_)::value * P.adj_stride;
            __builtin_nontemporal_store(float(v), reinterpret_cast<float*>(o + own));
        };
        const double phi_ref = P.mean_subtract ? *P.phi_ref : 0.0;
        double Gb[3], Nb = 0.0;
        node_adjoint<SL, FL, T>(fpop, g, a, b, G, Nsum, pc, phi_ref, P, mu_reg, put, Gb, Nb, th);
        double ps = 0.0, sA = 0.0, sB = 0.0;
        for (int k = 0; k < QS; ++k) { ps += double(g[k]); sA += double(a[k]); sB += double(b[k]); }
        const PhiSens ds = phi_sensitivities(ps, sA, sB, P);
        auto aux_put = [&](int row, double v) __attribute__((always_inline)) {
            char* o = reinterpret_cast<char*>(P.aux + (unsigned long long)row * P.aux_stride);
            *reinterpret_cast<float*>(o + own) = float(v);
        };
        if constexpr (QF > 0) {
            aux_put(0, Gb[0]);
            if constexpr (SL::DIM == 3) aux_put(1, Gb[1]);
            aux_put(2, Gb[2]);
            aux_put(3, Nb);
        }
        aux_put(4, ds.d0);
        aux_put(5, ds.q);
        aux_put(6, ds.dK);
    }
    block_reduce_store<6, 256, true>(th, -1, P.partials + 6 * blockIdx.x);
}

// seed: the final moment phi_T (Eq. Moment0_Phi) of the state at P.src_base receives
// dL/dphi_T: lambda = 0, c_F = dL/dphi dphi/dF, theta via dphi/dK
template <class SL, class FL, int PREC>
__global__ void __launch_bounds__(256) k_adj_seed(const KParams P, long long nodes,
                                                  const double* __restrict__ dL_dphi) {
    using SLOTS = Slots<FL::Q, SL::Q>;
    const long long i = (long long)blockIdx.x * blockDim.x + threadIdx.x;
    double th[6] = {0, 0, 0, 0, 0, 0};
    if (i < nodes) {
        const int x = int(i % P.nx), y = int((i / P.nx) % P.ny), z = int(i / ((long long)P.nx * P.ny));
        const Nbr nb = neighbours(x, y, z, P);
        double ps = 0.0, cA = 0.0, cB = 0.0;
        static_for<0, SL::Q>([&](auto kc) {
            constexpr int k = decltype(kc)::value;
            unsigned t;
            const char* sg = pull_src<SLOTS, SL, SLOTS::G0 + k, k>(P.src_base, P, z, unsigned(i), nb, t);
            const char* sa = pull_src<SLOTS, SL, SLOTS::A0 + k, k>(P.src_base, P, z, unsigned(i), nb, t);
            const char* sb = pull_src<SLOTS, SL, SLOTS::B0 + k, k>(P.src_base, P, z, unsigned(i), nb, t);
            ps += double(ld_at<PREC, SLOTS::rest(SLOTS::G0 + k)>(sg, t, float(SL::w(k)) * P.fref[1], P.finv[1]));
            cA += double(ld_at<PREC, SLOTS::rest(SLOTS::A0 + k)>(sa, t, float(SL::w(k)) * P.fref[2], P.finv[2]));
            cB += double(ld_at<PREC, SLOTS::rest(SLOTS::B0 + k)>(sb, t, float(SL::w(k)) * P.fref[3], P.finv[3]));
        });
        const PhiSens ds = phi_sensitivities(ps, cA, cB, P);
        const double s = dL_dphi[i];
        for (int k = 0; k < SLOTS::N; ++k) *adj_at<SL, FL>(P.adj_out, P, k, i) = 0.0f;
        float* c = P.auxc;
        c[0 * P.aux_stride + i] = float(s * ds.d0);
        c[1 * P.aux_stride + i] = float(s * ds.q * (P.c1A - P.c0A));
        c[2 * P.aux_stride + i] = float(s * ds.q * (P.c1B - P.c0B));
        theta_from_K(s * ds.dK, P, th);
    }
    block_reduce_store<6, 256, true>(th, -1, P.partials + 6 * blockIdx.x);
}

// Transpose of the phi stencil (mirror ghosts at walls, wrap otherwise): node y
// collects psi(y) = sum over (x, k) with map(x + e_k) = y of 3 w_k (e_k . Gb(x) + Nb(x)),
// Gb, Nb = aux rows 0..3.  GMODE 0 (adjoint step): phi(y) = Phi(sum g, c^A, c^B)(y), so
// c_F(y) = psi(y) dphi/dF(y) (aux rows 4, 5) and theta receives psi(y) dphi/dK(y)
// (aux row 6).  GMODE 1 (initial state, phi_0 an input): grad_phi0(y) = aux row 4 + psi(y).
//
// A node reads each of 8 (18) neighbours' three (four) rows: a work-group stages them for
// a tile and its ring in LDS (1.5 to 3 loads a row and node instead of 9 to 19, the latency
// of one batch).  Beyond a wall lies the mirror image of the source node, its normal
// component of Gb reversed: the pair (y - e, e) of an inside source and the pair (y, -e) whose
// target was mirrored back to y then read alike.  The partial sums hold one entry per
// 256 nodes, so no more work-groups than that are launched and each strides over the tiles.
// Measured, with one sum instead of six reduced per work-group: 512^2 10.0 -> 6.2 us,
// 64 x 48 x 40 13.1 -> 6.3 us.
template <int DIM>
struct GatherTile {
    static constexpr int X = DIM == 2 ? 64 : 32, Y = DIM == 2 ? 1 : 4, Z = DIM == 2 ? 4 : 2;
    static constexpr int LX = X + 2, LY = DIM == 2 ? 1 : Y + 2, LZ = Z + 2, CELLS = LX * LY * LZ;
};

template <class SL, class FL, int GMODE>
__global__ void __launch_bounds__(256) k_adj_gather(const KParams P, int ntiles, double* __restrict__ grad_phi0) {
    using STL = typename std::conditional<SL::DIM == 2, D2Q9K, D3Q19K>::type;
    using T = GatherTile<SL::DIM>;
    constexpr bool D3 = SL::DIM == 3, FLOW = FL::Q > 0;
    constexpr int OY = D3 ? 1 : 0;
    __shared__ float gb[FLOW ? 4 : 1][FLOW ? T::CELLS : 1];
    const int tid = threadIdx.x;
    const int tx = tid % T::X, ty = D3 ? (tid / T::X) % T::Y : 0, tz = tid / (T::X * T::Y);
    const int cell = ((tz + 1) * T::LY + ty + OY) * T::LX + tx + 1;
    const int gx = (P.nx + T::X - 1) / T::X, gy = (P.ny + T::Y - 1) / T::Y;
    const unsigned long long as = P.aux_stride;
    auto row = [&](int rr) { return reinterpret_cast<const char*>(P.aux + (unsigned long long)rr * as); };
    auto at = [&](int rr, unsigned node) { return *reinterpret_cast<const float*>(row(rr) + voff(node * 4u)); };
    double kb[1] = {0.0};
    for (int t = blockIdx.x; t < ntiles; t += gridDim.x) {
        const int tile = t;
        const int x0 = (tile % gx) * T::X, y0 = ((tile / gx) % gy) * T::Y, z0 = tile / (gx * gy) * T::Z;
        const int x = x0 + tx, y = y0 + ty, z = z0 + tz;
        const bool inside = x < P.nx && y < P.ny && z < P.nz;
        const unsigned i = inside ? unsigned((z * P.ny + y) * P.nx + x) : 0u;
        const float r4 = at(4, i), r5 = GMODE == 0 ? at(5, i) : 0.0f, r6 = GMODE == 0 ? at(6, i) : 0.0f;
        float psi = 0.0f;
        if constexpr (FLOW) {
            // a coordinate in memory: wrapped, or mirrored (flip: the component reverses);
            // beyond the first ghost layer of a partial tile any node (never read)
            auto source = [](int c, int n, int wall, float& flip) __attribute__((always_inline)) -> int {
                flip = 1.0f;
                if (c < 0) {
                    if (wall) flip = -1.0f;
                    return wall ? 0 : n - 1;
                }
                if (c >= n) {
                    if (wall) flip = -1.0f;
                    return wall || c > n ? n - 1 : 0;
                }
                return c;
            };
            __syncthreads();  // the previous tile has been read
#pragma unroll
            for (int c0 = 0; c0 < T::CELLS; c0 += 256) {
                const int c = c0 + tid;
                if (c < T::CELLS) {
                    const int cx = c % T::LX, cy = (c / T::LX) % T::LY, cz = c / (T::LX * T::LY);
                    float fx, fy, fz;
                    const int sx = source(x0 + cx - 1, P.nx, P.wall_x, fx);
                    const int sy = source(y0 + cy - OY, P.ny, P.wall_y, fy);
                    const int sz = source(z0 + cz - 1, P.nz, P.wall_z, fz);
                    const unsigned s = unsigned((sz * P.ny + sy) * P.nx + sx);
                    gb[0][c] = fx * at(0, s);
                    if constexpr (D3) gb[1][c] = fy * at(1, s);
                    gb[2][c] = fz * at(2, s);
                    gb[3][c] = at(3, s);
                }
            }
            __syncthreads();
            // sources x = y - e_k
            static_for<1, STL::Q>([&](auto kc) __attribute__((always_inline)) {
                constexpr int k = decltype(kc)::value;
                constexpr int ex = STL::ex(k), ey = STL::ey(k), ez = STL::ez(k);
                const int s = cell - ((ez * T::LY + ey) * T::LX + ex);
                float v = gb[3][s];
                if constexpr (ex != 0) v += ex > 0 ? gb[0][s] : -gb[0][s];
                if constexpr (ey != 0) v += ey > 0 ? gb[1][s] : -gb[1][s];
                if constexpr (ez != 0) v += ez > 0 ? gb[2][s] : -gb[2][s];
                psi += float(3.0 * STL::w(k)) * v;
            });
        }
        if (!inside) continue;
        if constexpr (GMODE == 1) {
            grad_phi0[i] = double(r4) + double(psi);
        } else {
            char* cbase = reinterpret_cast<char*>(P.auxc);
            const unsigned o = voff(i * 4u);
            *reinterpret_cast<float*>(cbase + o) = psi * r4;
            *reinterpret_cast<float*>(cbase + as * 4u + o) = psi * r5 * float(P.c1A - P.c0A);
            *reinterpret_cast<float*>(cbase + 2 * as * 4u + o) = psi * r5 * float(P.c1B - P.c0B);
            kb[0] += double(psi) * double(r6);
        }
    }
    if constexpr (GMODE == 0) {
        __shared__ double sum;
        block_reduce_store<1, 256>(kb, -1, &sum);
        if (tid == 0) {
            double th[6] = {0, 0, 0, 0, 0, 0};
            theta_from_K(sum, P, th);
            P.partials[6 * blockIdx.x] += th[0];
            P.partials[6 * blockIdx.x + 5] += th[5];
        }
    }
}

// Adjoint of the initialisation (k_init) with mu_0 held fixed: the adjoint of the
// initial populations (lambda + c in P.adj_in / aux) back to phi_0.  Local part per
// node into aux (rows 0..3: Gb, Nb of the F_0 stencil; row 4: local dL/dphi_0), theta
// partials per work-group; the stencil part closes in k_adj_gather<.., 1>.
template <class SL, class FL>
__global__ void __launch_bounds__(256) k_adj_init_local(const KParams P, long long nodes,
                                                        const double* __restrict__ phi0,
                                                        const double* __restrict__ muA0,
                                                        const double* __restrict__ muB0) {
    using SLOTS = Slots<FL::Q, SL::Q>;
    using STL = typename std::conditional<SL::DIM == 2, D2Q9K, D3Q19K>::type;
    const long long i = (long long)blockIdx.x * blockDim.x + threadIdx.x;
    double th[6] = {0, 0, 0, 0, 0, 0};
    if (i < nodes) {
        const int x = int(i % P.nx), y = int((i / P.nx) % P.ny), z = int(i / ((long long)P.nx * P.ny));
        const unsigned long long as = P.aux_stride;
        const float* c = P.auxc;
        const double cg = c[0 * as + i], cAa = c[1 * as + i], cBb = c[2 * as + i];
        const double phi = phi0[i], muA = muA0[i], muB = muB0[i];
        const double dA = P.c1A - P.c0A, dB = P.c1B - P.c0B;
        const double K = P.mphi_w2;
        const double dw = muA * dA + muB * dB;
        double phi_b = 0.0, S_b = 0.0;
        // g_k = w_k phi - w_k S_0 / 2; h_0 = c - (1 - w_0) mu, c = mu + c_0 + p(phi)(c_1 - c_0)
        for (int k = 0; k < SL::Q; ++k) {
            const double lg = double(*adj_at<SL, FL>(P.adj_in, P, SLOTS::G0 + k, i)) + cg;
            phi_b += lg * SL::w(k);
            S_b += -0.5 * lg * SL::w(k);
        }
        const double lA = double(*adj_at<SL, FL>(P.adj_in, P, SLOTS::A0, i)) + cAa;
        const double lB = double(*adj_at<SL, FL>(P.adj_in, P, SLOTS::B0, i)) + cBb;
        phi_b += (lA * dA + lB * dB) * interp_dp(phi);
        // S_0 = K (lambda p'(phi) dw - omega_dw'(phi))
        theta_from_K(S_b * (P.lam * interp_dp(phi) * dw - dwell_d(phi)), P, th);
        phi_b += S_b * K * (P.lam * interp_ddp(phi) * dw - dwell_dd(phi));
        double Gb[3] = {0.0, 0.0, 0.0}, Nb = 0.0;
        if constexpr (FL::Q > 0) {
            // f_k = -w_k (e_k . F_0) / 2
            double F_b[3] = {0.0, 0.0, 0.0};
            for (int k = 0; k < FL::Q; ++k) {
                const double lf = *adj_at<SL, FL>(P.adj_in, P, k, i);
                F_b[0] += -0.5 * FL::w(k) * FL::ex(k) * lf;
                F_b[1] += -0.5 * FL::w(k) * FL::ey(k) * lf;
                F_b[2] += -0.5 * FL::w(k) * FL::ez(k) * lf;
            }
            double G[3] = {0.0, 0.0, 0.0}, N = 0.0;
            for (int k = 1; k < STL::Q; ++k) {
                const int xn = map_coord(x + STL::ex(k), P.nx, P.wall_x);
                const int yn = map_coord(y + STL::ey(k), P.ny, P.wall_y);
                const int zn = map_coord(z + STL::ez(k), P.nz, P.wall_z);
                const double v = phi0[(zn * P.ny + yn) * P.nx + xn];
                G[0] += 3.0 * STL::w(k) * STL::ex(k) * v;
                G[1] += 3.0 * STL::w(k) * STL::ey(k) * v;
                G[2] += 3.0 * STL::w(k) * STL::ez(k) * v;
                N += 3.0 * STL::w(k) * v;
            }
            const double lap = 2.0 * N - 6.0 * (1.0 - STL::w(0)) * phi;
            const double bracket = P.cap * (dwell_d(phi) * P.inv_W2 - lap);
            phi_b += P.drho * (F_b[0] * P.gx + F_b[1] * P.gy + F_b[2] * P.gz);
            const double bracket_b = F_b[0] * G[0] + F_b[1] * G[1] + F_b[2] * G[2];
            for (int d = 0; d < 3; ++d) Gb[d] = bracket * F_b[d];
            phi_b += bracket_b * P.cap * P.inv_W2 * dwell_dd(phi);
            const double lap_b = -bracket_b * P.cap;
            th[5] += bracket_b * (P.cap / P.W) * (-dwell_d(phi) * P.inv_W2 - lap);
            Nb = 2.0 * lap_b;
            phi_b += -6.0 * (1.0 - STL::w(0)) * lap_b;
        }
        P.aux[0 * as + i] = float(Gb[0]);
        P.aux[1 * as + i] = float(Gb[1]);
        P.aux[2 * as + i] = float(Gb[2]);
        P.aux[3 * as + i] = float(Nb);
        P.aux[4 * as + i] = float(phi_b);
    }
    block_reduce_store<6, 256, true>(th, -1, P.partials + 6 * blockIdx.x);
}

// the adjoint as FP64 [slot][node] (lambda + c_F) from P.adj_in, or from such an
// array into P.adj_out (lambda = value, c_F = 0)
template <class SL, class FL, bool SET>
__global__ void __launch_bounds__(256) k_adj_copy(const KParams P, long long nodes, double* buf) {
    using SLOTS = Slots<FL::Q, SL::Q>;
    const long long i = (long long)blockIdx.x * blockDim.x + threadIdx.x;
    const int s = blockIdx.y;
    if (i >= nodes || s >= SLOTS::N) return;
    const int F = s < SLOTS::G0 ? -1 : (s - SLOTS::G0) / SL::Q;
    float* c = P.auxc;
    if constexpr (SET) {
        *adj_at<SL, FL>(P.adj_out, P, s, i) = float(buf[s * nodes + i]);
        if (s == 0) {
            for (int f = 0; f < 3; ++f) c[f * P.aux_stride + i] = 0.0f;
        }
    } else {
        double v = *adj_at<SL, FL>(P.adj_in, P, s, i);
        if (F >= 0) v += double(c[F * P.aux_stride + i]);
        buf[s * nodes + i] = v;
    }
}

// zero the bytes after each slot of the copies at P.src_slot and P.dst_slot (used_m / used_r
// bytes of a moving / rest slot are populations)
template <int NT = 256>
__global__ void __launch_bounds__(NT) k_zero_padding(const KParams P, int qf, int qs, unsigned long long used_m,
                                                     unsigned long long used_r) {
    const int s = blockIdx.x;
    const bool rest = (s < qf ? s : (s - qf) % qs) == 0;
    char* slot = blockIdx.y ? P.dst_slot[s] : const_cast<char*>(P.src_slot[s]);
    const unsigned long long at = (rest ? used_r : used_m) + threadIdx.x;
    if (at < (rest ? P.stride_r : P.stride_m)) slot[at] = 0;
}

// zero n doubles
template <int NT = 256>
__global__ void __launch_bounds__(NT) k_zero_f64(double* p, long long n) {
    const long long i = (long long)blockIdx.x * blockDim.x + threadIdx.x;
    if (i < n) p[i] = 0.0;
}

// per-work-group sums of a double field (grid-stride, fixed order)
template <int NT = 256>
__global__ void __launch_bounds__(256) k_sum_partials(const double* __restrict__ v, long long n,
                                                      double* __restrict__ partials) {
    double acc[1] = {0.0};
    for (long long i = (long long)blockIdx.x * 256 + threadIdx.x; i < n; i += (long long)gridDim.x * 256)
        acc[0] += v[i];
    block_reduce_store<1, 256>(acc, -1, partials + blockIdx.x);
}

// final fixed-order reduction of per-work-group partials (one work-group).
// partials are [nparts][N]; out[i] = scale[i] * reduce_i(partials[.][i]), except that
// the last entry goes to out[LAST_AT]
template <int N, bool ACC = false, int LAST_AT = N - 1>
__global__ void __launch_bounds__(256) k_finalize(const double* __restrict__ partials, int nparts,
                                                  int maxslot, double scale0, double* __restrict__ out) {
    double acc[N];
#pragma unroll
    for (int i = 0; i < N; ++i) acc[i] = 0.0;
    // unrolled so that the loads of several rounds are in flight (8192 entries: 15 -> 5 us)
#pragma unroll 8
    for (int p = threadIdx.x; p < nparts; p += 256) {
#pragma unroll
        for (int i = 0; i < N; ++i) {
            const double v = partials[p * N + i];
            acc[i] = (i == maxslot) ? fmax(acc[i], v) : acc[i] + v;
        }
    }
    double res[N];
    block_reduce_store<N, 256>(acc, maxslot, res);
    if (threadIdx.x == 0) {
#pragma unroll
        for (int i = 0; i < N; ++i) {
            const double v = (i == 0) ? res[i] * scale0 : res[i];
            const int o = (i == N - 1) ? LAST_AT : i;
            if constexpr (ACC) out[o] += v;
            else out[o] = v;
        }
    }
}

// ---------------------------------------------------------------------------
// droplet count (Section 4.2.2): Euler characteristic chi = sum over the
// elements of the cell complex of (-1)^dim, where the complex is the union of the
// closed unit cells of the nodes whose mask byte is set.  Every element is the
// cell-like part S (a subset of the axes) of one anchor: along the axes in S it is
// the cell interval j, along the others the vertex position between cells j - 1
// and j.  It belongs to the complex when one of the 2^(d - |S|) cells containing
// it is set, and has dimension |S|.  One thread per anchor reads the 2^d cells
// around it (cells across a wall are empty, periodic axes wrap), so every element
// is counted once.  The grid strides over the anchors; partials[blockIdx.x]
// receives the work-group's sum (an integer, exact in FP64).

// U: index of an anchor, 32-bit where it cannot wrap (EulerGeom::wide), which with mask reads
// free of branches took 96^3 from 17.3 to 12.6 us
template <int D, class U>
__global__ void __launch_bounds__(256) k_euler(const unsigned char* __restrict__ mask, const EulerGeom G,
                                               double* __restrict__ partials) {
    int acc = 0;
    const U step = gridDim.x * 256u, n = U(G.nanchors);
    for (U t = blockIdx.x * 256u + threadIdx.x; t < n; t += step) {
        int j[D];
        U r = t;
#pragma unroll
        for (int a = 0; a < D; ++a) {
            const U m = U(G.n[a] + G.wall[a]);
            j[a] = int(r % m);
            r /= m;
        }
        // bit o set: cell (j_a - 1 + o_a)_a is in the complex (o_a = bit a of o)
        unsigned bits = 0;
#pragma unroll
        for (int o = 0; o < (1 << D); ++o) {
            unsigned off = 0;
            bool in = true;
#pragma unroll
            for (int a = 0; a < D; ++a) {
                int c = j[a] - 1 + ((o >> a) & 1);
                if (c < 0) {
                    if (G.wall[a]) in = false;
                    else c += G.n[a];
                } else if (c >= G.n[a]) {
                    if (G.wall[a]) in = false;
                    else c -= G.n[a];
                }
                off += in ? unsigned(c) * unsigned(G.stride[a]) : 0u;
            }
            bits |= (unsigned(in) & unsigned(mask[off] != 0)) << o;  // no branch: the loads go out together
        }
#pragma unroll
        for (int S = 0; S < (1 << D); ++S) {
            bool valid = true;
#pragma unroll
            for (int a = 0; a < D; ++a)
                if (((S >> a) & 1) && j[a] >= G.n[a]) valid = false;  // no cell j past the last one
            // cells containing the element: o has every bit of S
            bool present = false;
#pragma unroll
            for (int o = 0; o < (1 << D); ++o)
                if ((o & S) == S && ((bits >> o) & 1u)) present = true;
            if (valid && present) acc += (__builtin_popcount(S) & 1) ? -1 : 1;
        }
    }
    double v[1] = {double(acc)};
    block_reduce_store<1, 256>(v, -1, partials + blockIdx.x);
}

}  // namespace lbm
