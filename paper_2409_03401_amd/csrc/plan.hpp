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

// lanes of the 64-wide tiles of a row, over its nodes
constexpr double tile_lanes(int nx) { return 64.0 * ((nx + 63) / 64) / nx; }
// Steps of a 3D box whose rows are whole lines, but not of 64-wide tiles: the general kernel
// where 64-wide tiles waste a sixth of their lanes and more, else its plain stores cost more than
// the lanes (us a step, general / 64 x 4, D3Q7 with flow FP64: 80^3 80 / 91, 160^3 582 / 592,
// 224 x 128 x 128 537 / 505; D3Q7 FP64 without flow 80^3 28 / 39, 224 x 128 x 128 251 / 246).  FP32 with flow gains
// only on boxes that the last-level cache holds in good part (96^3 59 / 71, 96 x 200 x 150 215 /
// 209, 160 x 96 x 80 95 / 90), and on D3Q19 scalars where half the lanes idle (32 x 128 x 128
// 79 / 89, 96^3 150 / 143, 160^3 675 / 619)
constexpr bool general_tiles(int nx, long long nodes, int prec, int qf, int qs) {
    const double lanes = tile_lanes(nx);
    if (qf > 0 && prec == P32) return qs == 19 ? lanes >= 1.5 : lanes > 1.2 && nodes < (3 << 19);
    return lanes >= 1.2;
}

// 3D calls of several steps with x or y walls (`axes` of them), rows of whole lines and steps in
// 64-wide tiles: does the general kernel, which bounces back there when it pulls, cost less than
// an exchange after each step?  The exchange takes 10 to 50 us, the general kernel a share of a
// step, most of it with flow on D3Q19 scalars and where its tiles are ragged.  Us a step, pulled /
// exchanged: D3Q7 with flow FP32, closed, 128^3 170 / 193, 256^3 1304 / 1152, 288 x 96 x 64 152 / 164,
// with x walls only 151 / 145; D3Q19 scalars with flow, x walls, 64^3 BF16 47 / 65, 160 x 96 x 80 FP64
// 421 / 426, 128^3 FP64 670 / 622, BF16 279 / 263
constexpr bool pull_walls(int nx, long long nodes, int qf, int qs, int axes) {
    return nodes < (qf > 0 && qs == 19 ? 5 << 18 : qf > 0 && tile_lanes(nx) > 1.0 ? (axes > 1 ? 4 << 19 : 3 << 19) : 1 << 22);
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

// rows of a marching work-group in 2D, whose columns are `threads` nodes wide: about 2048
// work-groups (8 per compute unit); a 512^2 box then takes one or two rows per group, the
// fastest on one MI355X (measured)
constexpr int row_chunk(int nx, int nz, int threads) {
    const int cols = (nx + threads - 1) / threads, groups = std::max(1, std::min(nz, 2048 / cols));
    return (nz + groups - 1) / groups;
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

// us that the chip takes for the collisions of 2^18 nodes, a factor of the model and one of the
// storage format: [model][scalar lattice of 5 or 9 directions][with flow], [with flow][precision]
constexpr double collision_time(int qf, int nslots, int coll, int prec) {
    constexpr double model[7][2][2] = {
        {{0.618, 1.11}, {0.965, 1.7}},     // BGK
        {{0.759, 1.71}, {1.22, 2.32}},     // TRT
        {{0.898, 1.88}, {1.83, 3.1}},      // MRT
        {{0.0, 1.36}, {0.0, 1.94}},        // variable density
        {{0.0, 1.98}, {0.0, 2.61}},        // variable density, TRT
        {{0.98, 1.72}, {1.33, 2.15}},      // general curvatures
        {{0.796, 1.38}, {0.0, 0.0}},       // three compositions
    };
    constexpr double store[2][4] = {{1.46, 1.1, 1.6, 1.3}, {1.37, 0.975, 1.44, 1.23}};
    const int flow = qf > 0 ? 1 : 0, ns = nslots - qf;
    const int m = ns == 20 ? 6 : (coll & COLL_GK) ? 5 : (coll & COLL_MRT) ? 2
                : (coll & COLL_VD) ? ((coll & COLL_TRT) ? 4 : 3) : (coll & COLL_TRT) ? 1 : 0;
    return model[m][ns == 27 ? 1 : 0][flow] * store[flow][prec];
}

// waves that a SIMD holds for kernels of v vector registers
constexpr int waves_of(double v) { return std::max(1, std::min(8, 512 / ((int(v) + 7) / 8 * 8))); }

// share of the `traffic` of a step, in bytes, that stays in the last-level cache
inline double cached(double traffic, double size) {
    const double r = traffic / size, r2 = r * r;
    return 1.0 / (1.0 + r2 * r2);
}

// us of one step with the marching kernel, `work` from collision_time: the latency of a
// work-group's rows (with flow two more than it updates), in rounds of the groups that are
// resident (about as many registers as the kernels have, and the LDS ring of scalar
// populations), or the time of the bytes (rows of whole lines take non-temporal stores) and of
// the collisions
inline double march_time(const PlanInput& in, int qs, int nc, double work) {
    const bool flow = in.qf > 0, wide = (in.coll & (COLL_MRT | COLL_GK)) != 0, s16 = in.prec == P16 || in.prec == PB16;
    const int ns = in.nslots;
    int resident = waves_of(!flow ? (in.prec == P64 ? 32 + 2.8 * ns : 38 + 1.5 * ns + (wide ? 20 : 0))
                            : in.prec == P64 ? 6.5 * ns - 10 + (wide ? 25 : 0)
                            : s16 ? 90 + ns + (wide ? 15 : 0) : 40 + 2.6 * ns + (wide ? 12 : 0));
    if (flow) {
        const int word = in.prec == P64 ? 8 : 4;
        const int ring = 2 * 256 * word * (1 + nc) * (s16 ? 1 + (qs - 1) / 2 : qs);
        if (ring <= 96 * 1024) resident = std::min(resident, 160 * 1024 / (ring + 3 * 258 * word));
    }
    const int zc = row_chunk(in.nx, in.nz, 256), cols = (in.nx + 255) / 256;
    const double x = double(cols) * ((in.nz + zc - 1) / zc) / 256.0 / resident;
    const double rounds = x <= 1.0 ? 1.0 : 0.89 * std::ceil(x) + 0.11 * x;
    const double fill = flow ? 2.0 / zc : 0.0;  // rows read besides those updated
    const double traffic = 2.0 * in.copy_bytes, hit = cached(traffic, 311e6);
    const double mem = traffic * (in.whole ? hit / 5.92e6 + (1.0 - hit) / 5.52e6 : hit / 7.63e6 + (1.0 - hit) / 4.49e6);
    const double lanes = 256.0 * cols / in.nx;  // of a row's work-groups, over its nodes
    const double cmp = 0.583 * work * double(in.nx) * in.nz / 262144.0 * lanes * lanes * lanes;
    const double busy = mem * (1.0 + 0.167 * fill) + cmp * (1.0 + 0.057 * fill);
    const double alone = rounds * (zc + (flow ? 2 : 0)) * (1.31 + 0.442 * work);
    return 2.09 + std::sqrt(alone * alone + busy * busy);
}

// windows of nt nodes that a compute unit holds, by LDS and about as many registers as the
// kernels have
constexpr int resident_windows(const PlanInput& in, int qs, int nc, int nt) {
    const bool flow = in.qf > 0, s16 = in.prec == P16 || in.prec == PB16;
    double v = in.prec == P64 ? 26 + 4.4 * in.nslots + (flow ? 20 : 0)
                              : 28 + 2.4 * in.nslots + (flow ? 14 : 0) + (s16 ? 4 : 0);
    if (flow && (in.coll & (COLL_MRT | COLL_GK)) != 0) v += 12;
    if (flow && s16 && qs == 9 && (in.coll & (COLL_TRT | COLL_MRT)) != 0) v += 24;
    return std::max(1, std::min(std::min(160 * 1024 / window_lds(in.qf, qs, in.prec, nc, nt), 2048 / nt),
                                waves_of(v) * 256 / nt));
}

// us of one launch of windows of nt nodes, `resident` of them on a unit, k steps each; `mem`: us
// that the chip takes for the bytes of a copy of 2^18 nodes.  A launch takes 4 us, and a round of
// resident windows the latency of its steps' collisions and barriers and the throughput of its
// loads and stores, which share the memory (a row's ends waste parts of 128-byte lines), and of
// its collisions.  Windows of one unit overlap the two; a window that has the unit to itself
// hardly, and its rounds are whole.
inline double window_time(const PlanInput& in, const BlockGeom& g, int nt, int resident, double k, double work, double mem) {
    const double nodes = double(in.nx) * in.nz, bytes = in.copy_bytes / nodes, word = bytes / in.nslots;
    const double windows = double(g.tiles_x) * g.tiles_z, share = std::min(1.0, nodes / (windows * nt));
    // 1024 nodes with TRT on the D2Q9 lattices spill 33 registers (512^2 BF16: 20 us a step,
    // 15.5 with the marching kernel)
    if (nt == 1024 && (in.coll & COLL_TRT) != 0 && word < 3.5 && in.nslots > 30) work *= 1.57;
    const double move = mem * (1.0 + share * (1.0 + 57.5 / (g.ix * word))), collide = k * work;
    const double busy = (std::max(move, collide) + (resident == 1 ? 0.65 : 0.48) * std::min(move, collide)) *
                        (resident == 1 && nt == 512 && windows > 256.0 ? 1.22 : 1.0);
    const double x = windows / 256.0, held = std::min(std::ceil(x), double(resident));
    const double r = x / resident, rounds = r <= 1.0 ? 1.0 : resident == 1 ? std::ceil(r) : 0.41 * std::ceil(r) + 0.59 * r;
    const double load = nt == 1024 ? 0.0146 * bytes : 0.0;  // nothing else runs while the one window loads
    return (in.qf ? 3.72 : 3.13) + rounds * (load + (in.qf ? 0.208 * k : 0.0) + 0.353 * collide + held * nt / 1024.0 * busy);
}

// How a call of n steps is cut into windows: the smallest estimate of its time over the
// windows of both sizes and every power-of-two width and over the numbers of launches that the
// call can take with up to 128 steps each (the windows are those of the steps that run,
// ceil(n / launches)).  The marching kernel stays unless that is below its own estimate by
// what the two may err.  The constants above are a fit to 27 000 timings (22 families in four
// precisions, 256 x 1 to 3001 x 1111 nodes, windows of 1 to 16 steps): windows within 7 % (rms),
// the marching kernel within 9 %.  Over calls of 1 to 40 steps on these grids the plan takes
// 1.7 % longer than the best choice on average, and in one call of 90 over 2 % longer than the
// marching kernel (an estimate that knew nothing of the models' collisions: 4.9 %, one of 25,
// the worst MRT on D2Q9 FP16 without flow, 512^2 in 10 steps, 139 us against 87).
inline BlockPlan block_plan(const PlanInput& in, long long n) {
    BlockPlan best;
    const double work = collision_time(in.qf, in.nslots, in.coll, in.prec);
    const int qs = (in.nslots - in.qf) % 9 == 0 ? 9 : 5, nc = (in.nslots - in.qf) / qs - 1;
    // the ways to share the steps among launches: their number and the longest of them
    long long launches[128];
    int longest[128], ways = 0;
    for (int k = int(std::min(n, 128LL)); k > 0; --k) {
        launches[ways] = launches_of(n, k, in.keep_copy);
        k = longest[ways] = int((n + launches[ways] - 1) / launches[ways]);
        ++ways;
    }
    // x walls: an exchange (5 us) after every step of the marching kernel, after the last launch
    // of windows
    const double walls = in.wall_x ? 5.0 : 0.0;
    double cost = double(n) * (march_time(in, qs, nc, work) + walls);  // of the call
    const double hit = cached(2.0 * in.copy_bytes, 296e6);
    const double mem = in.copy_bytes / (double(in.nx) * in.nz) * 1024.0 * (hit / 49.6e3 + (1.0 - hit) / 31.3e3);
    for (int nt : in.nt) {
        const int resident = resident_windows(in, qs, nc, nt);
        for (int lw = 4; (1 << lw) <= nt; ++lw) {
            for (int i = ways - 1; i >= 0; --i) {
                BlockGeom g;
                if (!block_geometry(in, nt, lw, longest[i], g)) break;
                if (double(g.tiles_x) * g.tiles_z * nt > double(kMaxThreads)) break;  // more with every further step
                const double margin = longest[i] == 1 ? 0.88 : 0.95, calls = double(launches[i]);
                const double t = (calls * window_time(in, g, nt, resident, double(n) / calls, work, mem) + walls) / margin;
                if (t < cost) {
                    cost = t;
                    best.nt = nt;
                    best.launches = launches[i];
                    best.g = g;
                }
            }
        }
    }
    return best;
}

}  // namespace lbm
