// Larger FP64 grids: K red-black sweeps a launch, each wave walking down the
// rows of its own tile (the tile pipeline of blocked_pipeline.h, which says how
// a tile's half-sweeps follow one another in registers).
//
// A tile is 64 split columns wide, one a lane, of which 64 - 2 (K + 1) are its
// own, and as tall as lets all tiles run at once, two waves a SIMD.  The
// persistent kernel gives a lane two columns: fewer recomputed columns, but one
// wave a SIMD, whose dependent chain down the 2 K half-sweeps of a row nothing
// covers (8191^2: 38% of its cycles issue, 40% wait), and a tile waits for its
// neighbours' flags.  Here the tiles of a pass are independent (a pass reads one
// buffer and writes the other, halos are recomputed) and the boundary between
// launches orders the passes.  What is left is the recomputation: at 4095^2 and
// K = 6, 64 / 50 columns and (88 + 24) / 88 rows.
#include <algorithm>

#include "blocked_pipeline.h"
#include "rbgs_internal.h"

namespace rbgs {
namespace {

using namespace blocked;

template <int L, bool SOR>
__global__ __launch_bounds__(kLanes, 2) void k_pipeline(GridDesc<double> g, const int* stop, int last,
                                                        double omega) {
    if (stop && *stop) return;
    const int tile = xcd_logical_block(int(blockIdx.x), int(gridDim.x));
    process_tile<double, 1, L, SOR>(g, 0, tile, SOR || last, omega);
}

constexpr int64_t kWaves = 2048;  // two a SIMD on 256 CUs
constexpr int kTallest = 512;     // rows of a tile, where one round does not do

template <int L>
hipError_t launch(const WindowArgs<double>& a, hipStream_t s) {
    GridDesc<double> g{};
    g.red[0] = const_cast<double*>(a.in[0]);
    g.black[0] = const_cast<double*>(a.in[1]);
    g.red[1] = a.out[0];
    g.black[1] = a.out[1];
    g.f_red = a.f[0];
    g.f_black = a.f[1];
    g.n = a.n;
    g.pitch = a.pitch;
    g.h2 = a.h2;
    g.halo_q = L / 2 + 1;
    g.q_core = kLanes - 2 * g.halo_q;
    g.bands = ((a.n >> 1) + 1 + g.q_core - 1) / g.q_core;
    // as many strips as fill the chip once, or a whole number of times
    const int64_t rounds = (int64_t(g.bands) * a.n + kTallest * kWaves - 1) / (kTallest * kWaves);
    const int64_t most = std::max<int64_t>(rounds * kWaves / g.bands, 1);
    g.rows = std::max(int((a.n + most - 1) / most), 2 * L);
    g.strips = (a.n + g.rows - 1) / g.rows;
    g.ntiles = g.strips * g.bands;
    const dim3 grid{unsigned(g.ntiles)}, block{kLanes};
    if (a.omega != 1.0)
        hipLaunchKernelGGL((k_pipeline<L, true>), grid, block, 0, s, g, a.stop, a.last, a.omega);
    else
        hipLaunchKernelGGL((k_pipeline<L, false>), grid, block, 0, s, g, a.stop, a.last, a.omega);
    return hipGetLastError();
}

}  // namespace

// Measured on MI355X, FP64, us (sweeps):     windows / persistent   here
//   1500^2 (200)                                    1061            1075
//   1700^2 (200)                                    1168            1102
//   2047^2 (200)                                    1594            1107
//   3001^2 (200)                                    2823            1732
//   4095^2 (200)                                    3625            2811
//   5001^2 (200)                                    4935            3939
//   7001^2 (100)                                    4610            3892
//   8191^2 (40)                                     2688            2581
//   8191^2 (100)                                    5363            5416
//  12287^2 (20)                                     3540            3467
//  12287^2 (60)                                     7028            7474
// Calls of up to 8 sweeps stay with the windows, whose passes have no ramp.  Larger
// grids than those above: window_takes.
bool pipeline_takes(int n, size_t elem_bytes, int nsweeps) {
    return elem_bytes == 8 && nsweeps >= 9 && n >= 1600 && (n <= 8000 || nsweeps <= 30);
}

// 200 sweeps, us at K = 5, 6, 7: 3001^2 1732, 1805, 1865; 4095^2 2932, 2811,
// 2857; 5001^2 4560, 4156, 3939.
int pipeline_fuse(int n) { return n <= 3500 ? 5 : n <= 4500 ? 6 : 7; }

hipError_t launch_pipeline(const WindowArgs<double>& a, int sweeps, hipStream_t s) {
    switch (sweeps) {
        case 2: return launch<4>(a, s);
        case 3: return launch<6>(a, s);
        case 4: return launch<8>(a, s);
        case 5: return launch<10>(a, s);
        case 6: return launch<12>(a, s);
        case 7: return launch<14>(a, s);
    }
    return hipErrorInvalidValue;
}

}  // namespace rbgs
