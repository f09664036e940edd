// Launch plans (no HIP types: host programs include it as well).
#pragma once

#include <algorithm>
#include <cmath>

namespace lbm {

enum Prec : int { P64 = 0, P32 = 1, P16 = 2, PB16 = 3 };
// collision operator of the fused step: the paper's BGK, or two relaxation times
// (flags): COLL_TRT two relaxation times, COLL_VD the variable-density flow model
// COLL_GK general curvature matrices of the free energies (2 x 2 closure per node)
// COLL_MRT multiple relaxation times on the lattice's moment basis
enum Coll : int { COLL_BGK = 0, COLL_TRT = 1, COLL_VD = 2, COLL_GK = 4, COLL_MRT = 8 };

// a launch takes fewer than 2^32 threads along an axis of its grid
constexpr long long kMaxThreads = 0xFFFFFFFFLL;

// threads of a 3D work-group, and the largest tile with its ring of one node
constexpr int kTileNodes = 256, kTileCells = 464;
// a tile of w x h nodes that a 3D work-group can take: one node and one ring node per thread
constexpr bool tile_fits(int w, int h) {
    return w >= 1 && h >= 1 && w <= kTileNodes && h <= kTileNodes && w * h <= kTileNodes &&
           (w + 2) * (h + 2) <= kTileCells && 2 * (w + 2) + 2 * h <= kTileNodes;
}

// planes per work-group of the 3D kernels without the phi stencil, for `cols` columns of
// tiles: one, two on large grids (96^3 FP64 step 67.2 -> 61.2 us, 256^3 FP32 580 -> 550 us
// against the chunks of the other kernels); 0, those chunks, where the launch would be too
// large (long narrow boxes: 4 x 4 x 2^25)
constexpr int flat_chunk(long long cols, long long nz, int threads) {
    const int zc = cols * nz > 8192 ? 2 : 1;
    return cols * ((nz + zc - 1) / zc) * threads > kMaxThreads ? 0 : zc;
}

// Windows of the several-steps kernel (2D): 2^lw nodes wide, halo (hx, hz), owned nodes
// ix x iz per window; full_*: the axis fits into the window whole (no halo, wraps inside).
// nsub: steps per launch.  raw_x: the source copy holds raw post-collision populations at
// the x walls (left by a launch of this kernel), else exchanged ones (k_walls).
struct BlockGeom {
    int lw, hx, hz, ix, iz, tiles_x, tiles_z, full_x, full_z, nsub, raw_x;
};

// LDS bytes of a window of nt nodes: the moving populations in their stored form, and phi
constexpr int window_lds(int qf, int qs, int prec, int nc, int nt) {
    const int moving = qf + (1 + nc) * qs - ((qf > 0 ? 1 : 0) + 1 + nc);
    const int word = prec == P64 ? 8 : prec == P32 ? 4 : 2;
    return nt * (moving * word + (qf > 0 ? (prec == P64 ? 8 : 4) : 0));
}

// threads of the small window, and of the large one.  Without flow 512: two or three of them
// share a compute unit and one loads while another collides (2048^2 D2Q5 FP32 46 us a step
// against 49 with 1024; D2Q9 FP32 75 against 85, BF16 69 against 73).  With flow each step
// costs two rings, so the share of the window that is owned matters more: 1024 where the
// populations fit in LDS and in a quarter of the registers (2048^2 D2Q9 + 3 x D2Q9 FP32
// 221 us against 304 with 512).
constexpr int kSmallWindow = 256;
constexpr int large_window(int qf, int qs, int prec, int coll, int nc) {
    const int regs = (qf + (1 + nc) * qs) * (prec == P64 ? 2 : 1);
    const int most = (coll & (COLL_MRT | COLL_GK)) != 0 ? 30 : 36;  // these need more temporaries
    return (qf > 0 && regs <= most && window_lds(qf, qs, prec, nc, 1024) <= 160 * 1024) ? 1024 : 512;
}

// what the plan of a 2D call depends on
struct PlanInput {
    int nx, nz;            // kernel frame
    int qf, nslots, prec;
    double copy_bytes;     // of one population copy
    bool whole;            // every row of a slot is whole 128-byte lines
    bool wall_x;
    int coll;              // flags of Coll
    int nt[2];             // threads of the small and the large window
    bool keep_copy;        // the state ends in the copy where single steps would leave it
};

// windows of nt nodes, 2^lw wide, for up to k steps per launch; false: the halo leaves none
inline bool block_geometry(const PlanInput& in, int nt, int lw, int k, BlockGeom& g) {
    const int bw = 1 << lw, bh = nt >> lw;
    const int halo = in.qf ? 2 * k - 1 : k - 1;
    g = BlockGeom{};
    g.lw = lw;
    g.full_x = in.nx <= bw;
    g.full_z = in.nz <= bh;
    g.hx = g.full_x ? 0 : halo;
    g.hz = g.full_z ? 0 : halo;
    g.ix = g.full_x ? in.nx : bw - 2 * halo;
    g.iz = g.full_z ? in.nz : bh - 2 * halo;
    if (g.ix < 1 || g.iz < 1) return false;
    g.tiles_x = (in.nx + g.ix - 1) / g.ix;
    g.tiles_z = (in.nz + g.iz - 1) / g.iz;
    return true;
}

// steps of launch i of `launches` that share n steps
constexpr long long steps_of_launch(long long n, long long launches, long long i) {
    return n / launches + (i < n % launches ? 1 : 0);
}

// launches of a call of n steps with at most k steps each.  keep_copy: an even number for an
// even number of steps and an odd one for an odd number, as with one step per launch
constexpr long long launches_of(long long n, int k, bool keep_copy) {
    const long long l = (n + k - 1) / k;
    return l + (keep_copy ? (l ^ n) & 1 : 0);
}

struct BlockPlan {
    int nt = 0;  // 0: one step per launch with the marching kernel
    long long launches = 0;
    BlockGeom g;
};

// How a call of n steps is cut into windows: the estimate of its time in us, smallest over
// the windows of both sizes (256 and 512 or 1024 nodes) of every power-of-two width and the
// numbers of launches that the call can take with up to 128 steps each.  The windows are those
// of the steps that are run, ceil(n / launches).  A launch takes 4 us, each step its barriers
// (0.36 us, 0.68 with flow), and a window its loads, collisions and stores: alone on a
// compute unit the latency of these, else their throughput.  The windows of all 256 units
// share the memory (`mem`, with the part of a 128-byte line that a row's ends waste, and
// less while both copies stay in the last-level cache); the collisions, `cmp`, overlap with
// it where several windows share a unit.  One window of 1024 nodes has a unit to itself, so
// these run in whole rounds; one of 512 FP64 nodes with flow leaves part of a unit idle.
// The constants are a fit to 1900 timings (ten families, 64^2 to 2047^2): the choice is
// within 0.8 % of the fastest on average (6 % with a fit to fewer: 150 x 93 D2Q9 + 3 x D2Q5
// FP32 closed 3.01 us a step, 2.71 now; 2047^2 D2Q9 BF16 68.1, 59.2 now; 512^2 D2Q9 + 3 x
// D2Q5 FP64 18.5, 15.9 now).  The marching kernel stays where its own estimate is lower.
inline BlockPlan block_plan(const PlanInput& in, long long n) {
    BlockPlan best;
    const double nodes = double(in.nx) * in.nz, flow = in.qf ? 1.0 : 0.0;
    const double bytes = in.copy_bytes / nodes;  // of a node's populations
    const double word = bytes / in.nslots;
    const double cmp = 0.0067 * in.nslots * (13.0 + 14.4 * flow);  // of 1024 nodes, one step
    const double rate = 2.0 * bytes * nodes > 124e6 ? 33.7e3 : 47e3;  // bytes/us of one unit
    // the marching kernel's time, and how much longer than the estimate the best windows take
    // (`heavy`): with flow the collisions of the less usual models and the conversions of
    // 16-bit storage count, most for boxes beyond the last-level cache (2048^2 D2Q9 + 3 x D2Q5,
    // march / windows: BF16 112 / 109 us, FP16 116 / 128, BF16 with TRT 116 / 131; 1500^2, whose
    // rows are not whole lines, BF16 74 / 52)
    const bool s16 = word < 3.5, trt = (in.coll & COLL_TRT) != 0;
    const bool wide = (in.coll & (COLL_MRT | COLL_GK)) != 0;
    double heavy = 1.0, march = in.whole ? 1.0 : (s16 ? 1.25 : 1.1);
    if (flow > 0.0 && s16) {
        heavy = (in.prec == P16 ? 1.39 : 1.2) * (wide ? 1.3 : trt ? 1.15 : 1.0) *
                ((in.coll & COLL_VD) != 0 ? 1.125 : 1.0);
        march *= wide ? 1.23 : 1.12;
    } else if (flow > 0.0 && word > 6.0 && wide) {
        heavy = 1.28;  // 2048^2 D2Q9 + 3 x D2Q5 FP64, MRT: 344 / 363 us
    }
    // the longest launch of every way to share the steps among fewer launches
    int longest[128], ways = 0;
    for (int k = int(std::min(n, 128LL)); k > 0; --k) {
        const long long launches = launches_of(n, k, in.keep_copy);
        k = int((n + launches - 1) / launches);
        longest[ways++] = k;
    }
    double cost = 1e30, loaded = 1e30;  // of the call
    for (int nt : in.nt) {
        for (int lw = 4; (1 << lw) <= nt; ++lw) {
            for (int i = ways - 1; i >= 0; --i) {
                BlockGeom g;
                if (!block_geometry(in, nt, lw, longest[i], g)) break;
                const double windows = double(g.tiles_x) * g.tiles_z, share = std::min(1.0, nodes / (windows * nt));
                if (windows * nt > double(kMaxThreads)) break;  // more with every further step
                const long long launches = launches_of(n, longest[i], in.keep_copy);
                const double k = double(n) / double(launches);
                const double mem = bytes * 1024.0 / rate *
                                   (1.0 + 16.5 / ((1 << lw) * word) + share * (1.0 + 44.0 / (g.ix * word)));
                const double alone = nt / 1024.0 * (0.44 + 0.456 * k * cmp);
                double rounds = windows * nt / (256.0 * 1024.0);
                if (nt == 1024 && rounds > 1.0) rounds = std::ceil(rounds);
                if (nt > 256 && flow > 0.0 && word > 6.0) rounds *= 1.43;
                // 1024 nodes with TRT on the D2Q9 lattices spill 33 registers (512^2 BF16: 20 us
                // a step, 15.5 with the marching kernel)
                const double spill = trt && s16 && in.nslots > 30 && nt == 1024 ? 1.9 : 1.0;
                const double busy = rounds * spill * (mem + (0.395 - 0.087 * flow) * k * cmp);
                const double base = 3.95 + (0.364 + 0.314 * flow) * k;
                const double t = double(launches) * (base + std::max(alone, busy));
                if (t < cost) {
                    cost = t;
                    loaded = double(launches) * (base + std::max(alone, busy * heavy));
                    best.nt = nt;
                    best.launches = launches;
                    best.g = g;
                }
            }
        }
    }
    // x walls: an exchange (5 us) after every step of the marching kernel, after the last launch
    // of windows
    const double walls = in.wall_x ? 5.0 : 0.0;
    if (loaded + walls >= double(n) * (3.6 + 3.5 * flow + 2.0 * bytes * nodes / 4.85e6 * march + walls)) best.nt = 0;
    return best;
}

}  // namespace lbm
