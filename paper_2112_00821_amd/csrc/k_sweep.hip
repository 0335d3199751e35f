// Host dispatch of the fused plane-sweep kernel (Alg. 1 of the paper): grid
// size, tile height and the (window, cost) variant.  The kernel itself is in
// k_sweep.hpp; k_sweep_inst.hip instantiates one variant per translation
// unit.
#include "kernels.hpp"

#include <algorithm>
#include <cmath>
#include <cstdlib>
#include <cstring>

namespace fmvs {

constexpr int kSweepTileW = 64;

template <int CW, int CH, int COST>
hipError_t sweep_launch_cfg(const SweepArgs &a, dim3 grid, int rpt, hipStream_t s);
template <int CW, int CH, int COST>
hipError_t sweep_launch_batch_cfg(const SweepArgs *list, const int *prefix, int n, int blocks, int rpt,
                                  hipStream_t s);

// Tile height / 4 (one wavefront per 4 rows): 8 halves the halo of 4, 4 gives
// more workgroups and smaller unions of label windows.
// (views in bytes: built for 4 only)
int sweep_rpt(const SweepArgs &a) {
    if (a.views[0] && !a.warped) return 4;
    return a.rows_per_thread == 4 ? 4 : (a.rows_per_thread == 8 ? 8 : (a.cost == 1 ? 4 : 8));
}

// Tile grid of one frame for tiles of 4 * rpt rows; returns the tile count.
int sweep_tiles(SweepArgs &a, int rpt) {
    a.tiles_x = (a.w + kSweepTileW - 1) / kSweepTileW;
    a.tiles_y = (a.h + 4 * rpt - 1) / (4 * rpt);
    return a.tiles_x * a.tiles_y;
}

// Split each tile's label range into chunks (workgroups of their own): a
// tile's whole label loop is long, and with few workgroups the last round
// leaves CUs idle.  `waves` wavefronts over all tiles are wanted where chunks
// keep 16 labels (shorter ones repeat the setup and write S in pieces), half
// as many down to 4 labels a chunk.  Measured: 1280x720 x 64 labels, level 0:
// 0.80 ms with 4 chunks of 16, 0.90 ms with 16 of 4; 480x270 x 128 labels:
// 0.37 ms with 8 chunks, 0.35 ms with 31; 333x187 x 16 labels, three levels:
// 0.38 ms with chunks of at least 8, 0.24 ms of at least 4.
int sweep_chunks(const SweepArgs &a, int tiles, int rpt, double waves) {
    const double per_chunk = (double)tiles * rpt;
    const int runs = std::max(1, a.D / 16), words = std::max(1, (a.D + 3) / 4);
    const int full = (int)std::min(std::ceil(waves / per_chunk), 1e6);
    const int half = (int)std::min(std::ceil(0.5 * waves / per_chunk), 1e6);
    const int n = std::max(1, std::max(std::min(full, runs), std::min(half, words)));
    // equal chunks, of whole words of four labels: 31 chunks of 32 words would
    // leave one of twice the length (480x270 x 128 labels: 0.39 ms, 0.35 ms
    // with 32).  The count is rounded up to that, so between n and twice n (17
    // chunks of 32 words become 32).  On levels with windows the kernel deals
    // out the words of a tile's window union, which are D's or more.
    const int len = std::max(1, words / n);
    return (words + len - 1) / len;
}

hipError_t launch_sweep(const SweepArgs &a0, hipStream_t s) {
    SweepArgs a = a0;
    const int rpt = sweep_rpt(a);
    const int tiles = sweep_tiles(a, rpt);
    if (tiles == 0) return hipSuccess;
    if (a.n_chunks <= 0) {
        // 32768 wavefronts are eight rounds of the 16 a CU holds.
        // FASSMVS_SWEEP_BLOCKS asks for that many workgroups instead.
        const char *e = std::getenv("FASSMVS_SWEEP_BLOCKS");
        const int target = e ? std::atoi(e) : 0;
        a.n_chunks = sweep_chunks(a, tiles, rpt, target > 0 ? (double)target * rpt : 32768.0);
    }
    dim3 grid((unsigned)(tiles * a.n_chunks));
    // (window, cost) pairs the sweep is built for
#define FMVS_SWEEP(CWv, CHv, C) \
    if (a.cost == C && a.cw == CWv && a.ch == CHv) return sweep_launch_cfg<CWv, CHv, C>(a, grid, rpt, s);
    FMVS_SWEEP(5, 5, 0)
    FMVS_SWEEP(9, 7, 0)
    FMVS_SWEEP(7, 7, 0)
    FMVS_SWEEP(3, 3, 0)
    FMVS_SWEEP(5, 5, 1)
    FMVS_SWEEP(9, 9, 1)
    FMVS_SWEEP(7, 7, 1)
    FMVS_SWEEP(3, 3, 1)
#undef FMVS_SWEEP
    return hipErrorInvalidValue;
}

// Several frames' sweeps in one launch, in two steps so the launch can be
// captured in a graph apart from the argument upload.
// prepare_sweep_batch: host[0..n-1] are the frames' args (same window and
// cost, no pre-warped input); their tile grids and chunk counts are set
// (about 4 * `target` wavefronts over all frames, each frame's share by its
// pixels x labels) and they are written with the workgroup prefix (n + 1
// ints) to out (host memory of sweep_batch_bytes(n)).  Returns the
// workgroup count, or -1 if the frames cannot share a launch.
size_t sweep_batch_bytes(int n) { return sizeof(SweepArgs) * n + sizeof(int) * (n + 1); }

int prepare_sweep_batch(SweepArgs *host, int n, int rpt, int target, void *out) {
    if (n < 1) return -1;
    double work = 0.0;
    for (int i = 0; i < n; ++i) work += (double)host[i].w * host[i].h * host[i].D;
    int *prefix = (int *)((SweepArgs *)out + n);
    prefix[0] = 0;
    for (int i = 0; i < n; ++i) {
        SweepArgs &a = host[i];
        if (a.cw != host[0].cw || a.ch != host[0].ch || a.cost != host[0].cost || a.warped) return -1;
        a.rows_per_thread = rpt;
        const int tiles = sweep_tiles(a, rpt);
        const double share = work > 0.0 ? (double)a.w * a.h * a.D / work : 1.0;
        a.n_chunks = sweep_chunks(a, tiles, rpt, 4.0 * target * share);
        prefix[i + 1] = prefix[i] + tiles * a.n_chunks;
    }
    std::memcpy(out, host, sizeof(SweepArgs) * n);
    return prefix[n];
}

// launch_sweep_batch: the args block prepared above, in device memory at
// dev, for `blocks` workgroups.
hipError_t launch_sweep_batch(const void *dev, int n, int blocks, int rpt, int cw, int ch, int cost, hipStream_t s) {
    if (blocks <= 0) return hipSuccess;
    const SweepArgs *dl = (const SweepArgs *)dev;
    const int *dp = (const int *)((const SweepArgs *)dev + n);
#define FMVS_SWEEPB(CWv, CHv, C) \
    if (cost == C && cw == CWv && ch == CHv) return sweep_launch_batch_cfg<CWv, CHv, C>(dl, dp, n, blocks, rpt, s);
    FMVS_SWEEPB(5, 5, 0)
    FMVS_SWEEPB(9, 7, 0)
    FMVS_SWEEPB(7, 7, 0)
    FMVS_SWEEPB(3, 3, 0)
    FMVS_SWEEPB(5, 5, 1)
    FMVS_SWEEPB(9, 9, 1)
    FMVS_SWEEPB(7, 7, 1)
    FMVS_SWEEPB(3, 3, 1)
#undef FMVS_SWEEPB
    return hipErrorInvalidValue;
}

}  // namespace fmvs
