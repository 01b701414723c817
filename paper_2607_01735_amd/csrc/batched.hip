// Batched sweeps: many independent grids of uneven sizes, by register windows
// (batched_window.hip) where the caller leaves the way open, else in one
// launch of the tile pipeline (blocked_pipeline.h); plus the batched
// pack/unpack kernels, the graph-captured plan and the autotuner, which times
// both.  Of the pipeline:
//
// Work items are (pass, grid, tile).  Tickets run pass-major, and inside a
// pass the grids are ordered largest first (longest-processing-time first),
// so the biggest grids' tiles, which bound the makespan, start earliest.
// Pass-major order is a topological order of every grid's dependency graph,
// so the deadlock-freedom argument of the single-grid kernel carries over.
// Each grid keeps its own progress flags (offset flag_base); its tiles wait
// only on their own 3 x 3 neighbourhood.
//
// Small grids (n <= lds_max_n, when both colours of u and of h^2 f fit in
// one workgroup's LDS) can leave the tile queue: k_batch_lds sweeps each in
// one workgroup, all sweeps of the call in LDS, before the persistent
// launch.  The autotuner decides whether that beats tiling them (a 63^2
// grid is one 64-lane tile with a halo as wide as the grid, but its tiles
// interleave with the large grids' instead of adding a launch).
#include <hip/hip_runtime.h>

#include <algorithm>
#include <cmath>
#include <cstdio>
#include <cstdlib>
#include <cstring>
#include <map>
#include <mutex>
#include <numeric>
#include <string>
#include <vector>

#include "blocked_pipeline.h"
#include "lds_limit.h"
#include "rbgs.h"
#include "rbgs_blocked.h"
#include "rbgs_internal.h"

namespace rbgs {
namespace {

using namespace blocked;

// Per-grid pack/unpack description (natural <-> split, both buffers).
struct PackDesc {
    const void* nat_u;
    const void* nat_f;
    void* nat_out;       // unpack destination (the caller's u)
    void* red[2];
    void* black[2];
    void* f_red;
    void* f_black;
    int64_t ld;
    int64_t pitch;
    int64_t row_start;   // first global row index of this grid
    int n;
};

__device__ __forceinline__ int find_grid(const PackDesc* d, int count, int64_t row) {
    int lo = 0, hi = count - 1;  // last grid whose row_start <= row
    while (lo < hi) {
        int mid = (lo + hi + 1) >> 1;
        if (d[mid].row_start <= row)
            lo = mid;
        else
            hi = mid - 1;
    }
    return lo;
}

// One workgroup per grid row (all grids' rows numbered consecutively).
// Packs u into both ping-pong buffers (so both hold the Dirichlet ring) and f.
template <typename W>
__global__ __launch_bounds__(256) void k_batch_pack(const PackDesc* __restrict__ descs, int count) {
    const int64_t row = blockIdx.x;
    const int gi = __builtin_amdgcn_readfirstlane(find_grid(descs, count, row));
    const PackDesc d = descs[gi];
    const int64_t i = row - d.row_start;
    const W* u = static_cast<const W*>(d.nat_u) + i * d.ld;
    const W* f = static_cast<const W*>(d.nat_f) + i * d.ld;
    const int c0 = int(i & 1);  // colour of (i, 2q); (i, 2q+1) has the other
    for (int64_t q = threadIdx.x; q < d.pitch; q += 256) {
        const int64_t j0 = 2 * q, j1 = 2 * q + 1;
        const W u0 = j0 <= d.n + 1 ? u[j0] : W(0), u1 = j1 <= d.n + 1 ? u[j1] : W(0);
        const W f0 = j0 <= d.n + 1 ? f[j0] : W(0), f1 = j1 <= d.n + 1 ? f[j1] : W(0);
        const int64_t o = i * d.pitch + q;
        W* r0 = static_cast<W*>(d.red[0]);
        W* b0 = static_cast<W*>(d.black[0]);
        W* r1 = static_cast<W*>(d.red[1]);
        W* b1 = static_cast<W*>(d.black[1]);
        (c0 ? b0 : r0)[o] = u0;
        (c0 ? r0 : b0)[o] = u1;
        (c0 ? b1 : r1)[o] = u0;
        (c0 ? r1 : b1)[o] = u1;
        (c0 ? static_cast<W*>(d.f_black) : static_cast<W*>(d.f_red))[o] = f0;
        (c0 ? static_cast<W*>(d.f_red) : static_cast<W*>(d.f_black))[o] = f1;
    }
}

// Interior points of every grid back to the caller's arrays, from buffer b.
template <typename W>
__global__ __launch_bounds__(256) void k_batch_unpack(const PackDesc* __restrict__ descs, int count,
                                                      int b) {
    const int64_t row = blockIdx.x;
    const int gi = __builtin_amdgcn_readfirstlane(find_grid(descs, count, row));
    const PackDesc d = descs[gi];
    const int64_t i = row - d.row_start;
    if (i < 1 || i > d.n) return;
    W* u = static_cast<W*>(d.nat_out) + i * d.ld;
    const W* red = static_cast<const W*>(d.red[b]);
    const W* black = static_cast<const W*>(d.black[b]);
    const W* even_src = (i & 1) ? black : red;
    const W* odd_src = (i & 1) ? red : black;
    for (int64_t q = threadIdx.x; q < d.pitch; q += 256) {
        const int64_t j0 = 2 * q, j1 = 2 * q + 1;
        if (j0 >= 1 && j0 <= d.n) u[j0] = even_src[i * d.pitch + q];
        if (j1 >= 1 && j1 <= d.n) u[j1] = odd_src[i * d.pitch + q];
    }
}

// SOR: red-black SOR with each grid's own omega (FP64 batched solves).
template <typename T, int V, int L, bool SOR>
__global__ __launch_bounds__(kLanes) void k_blocked_batched(const GridDesc<T>* __restrict__ descs,
                                                            const int* __restrict__ tile_grid,
                                                            int total_tiles, Queue qu) {
    if (stopped(qu)) return;
    const int total = qu.passes * total_tiles;
    for (;;) {
        const int tk = next_ticket(qu);
        if (tk >= total) break;
        const int pass = tk / total_tiles;
        const int idx = tk - pass * total_tiles;
        const int gi = __builtin_amdgcn_readfirstlane(tile_grid[idx]);
        const GridDesc<T> g = descs[gi];
        if (!run_item<T, V, L, false, SOR>(g, qu, pass, idx - g.flag_base, DebugModes(), 0,
                                           g.omega))
            break;
    }
}

// ---------------------------------------------------------------------------
// Host side
// ---------------------------------------------------------------------------
struct EventPair {
    hipEvent_t a = nullptr, b = nullptr;
    ~EventPair() {
        if (a) (void)hipEventDestroy(a);
        if (b) (void)hipEventDestroy(b);
    }
};

constexpr int kLdsThreads = 512;

// LDS bytes that k_batch_lds needs for an n x n grid: both colours of u and
// of h^2 f, (n + 2) rows of (n + 3) / 2 elements each.
inline size_t lds_grid_bytes(int n, size_t es) {
    return 4 * size_t(n + 2) * size_t((n + 3) / 2) * es;
}

// Largest dynamic LDS one workgroup may use on the current device.
inline size_t lds_limit_bytes() {
    int dev = 0, v = 0;
    if (hipGetDevice(&dev) != hipSuccess) return 0;
    if (hipDeviceGetAttribute(&v, hipDeviceAttributeSharedMemPerBlockOptin, dev) != hipSuccess ||
        v <= 0) {
        (void)hipGetLastError();
        if (hipDeviceGetAttribute(&v, hipDeviceAttributeMaxSharedMemoryPerBlock, dev) != hipSuccess)
            return 0;
    }
    return size_t(v);
}

// One colour's half-sweep of an LDS-resident grid.  Split layout with row
// pitch pl: colour c holds (i, j = 2q + ((i + c) & 1)) at [i][q]; the
// other colour's neighbours of that point sit at [i +- 1][q] and at
// [i][(j +- 1) / 2].  Wave w takes rows 1 + w, 1 + w + waves, ..., its lanes
// the q of a row.  Same operations, same order as every other kernel.
template <typename T, int C>
__device__ __forceinline__ void lds_half_sweep(T* __restrict__ self, const T* __restrict__ other,
                                               const T* __restrict__ hf, int n, int pl) {
    constexpr int kWaves = kLdsThreads / 64;
    const int lane = threadIdx.x & 63;
    for (int i = 1 + int(threadIdx.x >> 6); i <= n; i += kWaves) {
        const int p = (i + C) & 1;
        const T* o = other + i * pl;
        for (int q = lane; q < pl; q += 64) {
            const int j = 2 * q + p;
            if (j < 1 || j > n) continue;
            T s = o[pl + q] + o[q - pl];
            s = s + o[(j + 1) >> 1];
            s = s + o[(j - 1) >> 1];
            s = s - hf[i * pl + q];
            self[i * pl + q] = T(0.25) * s;
        }
    }
}

// One workgroup per small grid: loads buffer 0 (both colours) and h^2 f into
// LDS, runs nsweeps red-then-black sweeps there with a barrier after each
// colour (the barriers of Algorithm 1 inside one workgroup), and writes the
// iterate to buffer `out`, the one the unpack reads.
template <typename T>
__global__ __launch_bounds__(kLdsThreads) void k_batch_lds(const GridDesc<T>* __restrict__ descs,
                                                           const int* __restrict__ ids,
                                                           int nsweeps, int out) {
    extern __shared__ __align__(16) unsigned char lds_raw[];
    const int gi = __builtin_amdgcn_readfirstlane(ids[blockIdx.x]);
    const GridDesc<T>& g = descs[gi];
    const int n = g.n;
    const int64_t P = g.pitch;
    const int pl = (n + 3) / 2;
    const int cells = (n + 2) * pl;
    T* ur = reinterpret_cast<T*>(lds_raw);
    T* ub = ur + cells;
    T* hr = ub + cells;
    T* hb = hr + cells;
    const T h2 = g.h2;
    for (int k = threadIdx.x; k < cells; k += kLdsThreads) {
        const int i = k / pl;
        const int64_t at = int64_t(i) * P + (k - i * pl);
        ur[k] = g.red[0][at];
        ub[k] = g.black[0][at];
        hr[k] = h2 * g.f_red[at];
        hb[k] = h2 * g.f_black[at];
    }
    __syncthreads();
    for (int sw = 0; sw < nsweeps; ++sw) {
        lds_half_sweep<T, 0>(ur, ub, hr, n, pl);
        __syncthreads();
        lds_half_sweep<T, 1>(ub, ur, hb, n, pl);
        __syncthreads();
    }
    T* yr = g.red[out];
    T* yb = g.black[out];
    for (int k = threadIdx.x; k < cells; k += kLdsThreads) {
        const int i = k / pl;
        const int64_t at = int64_t(i) * P + (k - i * pl);
        yr[at] = ur[k];
        yb[at] = ub[k];
    }
}

size_t elem_bytes_of(rbgs_dtype dt) { return dt == RBGS_F64 ? 8 : 4; }

// Workspace layout of a batch: queue header, flags, tables, then the split
// arrays of every grid (u twice, f once; two colours each).
struct BatchLayout {
    size_t header = 0, flags = 0, gdesc = 0, pdesc = 0, tile_map = 0, small = 0, arrays = 0,
           total = 0;
    std::vector<size_t> grid_off;  // offset of each grid's six colour arrays
    std::vector<int64_t> pitch;
    int max_tiles_total = 0;
};

BatchLayout batch_layout(int count, const rbgs_grid* grids, rbgs_dtype dt) {
    BatchLayout b;
    const size_t es = elem_bytes_of(dt);
    int64_t tiles = 0;
    for (int g = 0; g < count; ++g) tiles += max_tiles(grids[g].n);
    b.max_tiles_total = int(std::min<int64_t>(tiles, INT32_MAX / 2));
    size_t off = 0;
    b.header = off;
    off += 256;
    b.flags = off;
    off += align256(size_t(tiles) * 4);
    b.gdesc = off;
    off += align256(size_t(count) * std::max(sizeof(GridDesc<double>), sizeof(GridDesc<float>)));
    b.pdesc = off;
    off += align256(size_t(count) * sizeof(PackDesc));
    b.tile_map = off;
    off += align256(size_t(tiles) * 4);
    b.small = off;
    off += align256(size_t(count) * 4);
    b.arrays = off;
    b.grid_off.resize(count);
    b.pitch.resize(count);
    for (int g = 0; g < count; ++g) {
        b.pitch[g] = split_pitch(grids[g].n, es);
        b.grid_off[g] = off;
        off += 6 * align256(size_t(grids[g].n + 2) * size_t(b.pitch[g]) * es);
    }
    b.total = off;
    return b;
}

struct BatchSetup {
    int passes = 0, rem = 0, total_tiles = 0, fuse = 0;
    int64_t total_rows = 0;
    std::vector<char> gdesc;    // GridDesc<T> table, LPT order of tiles
    std::vector<PackDesc> pdesc;
    std::vector<int> tile_map;
    std::vector<int> small_ids;  // grids swept LDS-resident by k_batch_lds
    size_t small_lds_bytes = 0;  // dynamic LDS for the largest of them
    // Swept by windows (win.passes > 0) there are no tiles and no LDS-resident grids;
    // in the workspace these tables take the place of tile_map and small_ids.
    BatchWindows win;
    std::vector<int> win_order, win_first;
};

// How a batch is swept: the persistent kernel's shape, or (windows) not by it.
struct BatchChoice {
    int fuse = 0, rows = 0, lds_max_n = 0;
    bool windows = false;
};

// Whether the caller leaves the way of sweeping a batch open.
bool batch_open(const rbgs_sweep_opts* o) {
    return !o || (o->kernel == RBGS_KERNEL_AUTO && o->fuse == 0 && o->tile_rows == 0 &&
                  o->lds_max_n == 0 && o->debug_delay == 0 && o->debug_spin_limit == 0 &&
                  o->debug_stall_tile == 0);
}

// Splits a batch into windows for nsweeps sweeps; false: too many of them.
bool split_windows(BatchSetup& s, int count, const rbgs_grid* grids, size_t es, int nsweeps) {
    std::vector<int> n(static_cast<size_t>(count));
    for (int g = 0; g < count; ++g) n[size_t(g)] = grids[g].n;
    BatchWindows b;
    if (nsweeps < 1 || !batch_windows(count, n.data(), es, nsweeps, &b, &s.win_first, &s.win_order))
        return false;
    s.win = b;
    return true;
}

// LDS-resident threshold the autotuner tries: the largest grid of the
// benchmark's size mix that fits (127 in FP32: 133 KB; 63 in FP64: 68 KB).
// Untuned batches use none: the LDS launch runs before the persistent one,
// and on the measured mixes (512 grids of 63..1023 FP32; 16 grids of
// 63..255 FP64) tiling the small grids alongside the large ones was faster.
inline int tuned_lds_candidate(size_t es) { return es == 4 ? 127 : 63; }

template <typename T>
BatchSetup build_setup(int count, const rbgs_grid* grids, void* const* u, const void* const* f,
                       const BatchLayout& lay, char* ws, const BatchChoice& how, int nsweeps) {
    BatchSetup s;
    const int fuse = how.fuse, rows_opt = how.rows, lds_max_n = how.lds_max_n;
    const size_t lds_limit = lds_max_n > 0 ? lds_limit_bytes() : 0;
    s.fuse = fuse;
    s.passes = nsweeps / fuse;
    s.rem = nsweeps - s.passes * fuse;
    const size_t es = sizeof(T);
    // largest grids first
    std::vector<int> order(count);
    std::iota(order.begin(), order.end(), 0);
    std::stable_sort(order.begin(), order.end(),
                     [&](int a, int b) { return grids[a].n > grids[b].n; });
    std::vector<GridDesc<T>> gd(count);
    s.pdesc.resize(count);
    int flag = 0;
    int64_t row = 0;
    for (int g = 0; g < count; ++g) {
        const int n = grids[g].n;
        const int64_t P = lay.pitch[g];
        const size_t colour = align256(size_t(n + 2) * size_t(P) * es);
        char* base = ws + lay.grid_off[g];
        int rows = rows_opt > 0 ? rows_opt : default_rows(n, 2 * fuse);
        if (rows < 2 * fuse) rows = 2 * fuse;
        if (rows < kMinRows) rows = kMinRows;
        const Geometry geo = geometry(n, int(es), fuse, rows);
        GridDesc<T>& d = gd[g];
        d.red[0] = reinterpret_cast<T*>(base + 0 * colour);
        d.black[0] = reinterpret_cast<T*>(base + 1 * colour);
        d.red[1] = reinterpret_cast<T*>(base + 2 * colour);
        d.black[1] = reinterpret_cast<T*>(base + 3 * colour);
        d.f_red = reinterpret_cast<const T*>(base + 4 * colour);
        d.f_black = reinterpret_cast<const T*>(base + 5 * colour);
        d.n = n;
        d.pitch = P;
        d.h2 = T(grids[g].h * grids[g].h);
        d.rows = geo.rows;
        d.halo_q = geo.halo_q;
        d.q_core = geo.q_core;
        d.strips = geo.strips;
        d.bands = geo.bands;
        d.ntiles = geo.ntiles;
        d.omega = T(1);
        PackDesc& p = s.pdesc[g];
        p.nat_u = u[g];
        p.nat_f = f[g];
        p.nat_out = u[g];
        p.red[0] = d.red[0];
        p.black[0] = d.black[0];
        p.red[1] = d.red[1];
        p.black[1] = d.black[1];
        p.f_red = base + 4 * colour;
        p.f_black = base + 5 * colour;
        p.ld = grids[g].ld;
        p.pitch = P;
        p.row_start = row;
        p.n = n;
        row += n + 2;
    }
    s.total_rows = row;
    const bool windows = how.windows && split_windows(s, count, grids, es, nsweeps);
    for (int k = 0; k < count && !windows; ++k) {
        const int g = order[k];
        const size_t lds = lds_grid_bytes(grids[g].n, es);
        if (grids[g].n <= lds_max_n && lds <= lds_limit) {
            s.small_ids.push_back(g);
            s.small_lds_bytes = std::max(s.small_lds_bytes, lds);
            gd[g].flag_base = 0;
            continue;
        }
        gd[g].flag_base = flag;
        for (int t = 0; t < gd[g].ntiles; ++t) s.tile_map.push_back(g);
        flag += gd[g].ntiles;
    }
    s.total_tiles = flag;
    s.gdesc.resize(sizeof(GridDesc<T>) * count);
    std::memcpy(s.gdesc.data(), gd.data(), s.gdesc.size());
    return s;
}

// The buffer a batch's sweeps leave their result in, from buffer 0.
int result_buffer(const BatchSetup& s) {
    if (s.win.passes > 0) return s.win.passes & 1;
    return (s.passes + (s.rem > 0 ? 1 : 0)) & 1;
}

template <typename T, int V, int L, bool SOR>
hipError_t launch_batched_k(const GridDesc<T>* d, const int* map, int total_tiles, const Queue& qu,
                            hipStream_t s) {
    int per_cu = 0, cus = 0;
    hipError_t e = persistent_occupancy(
        reinterpret_cast<const void*>(&k_blocked_batched<T, V, L, SOR>), &per_cu, &cus);
    if (e != hipSuccess) return e;
    int64_t total = int64_t(qu.passes) * total_tiles;
    int64_t grid = int64_t(cus) * per_cu;
    if (grid > total) grid = total;
    if (grid < 1) grid = 1;
    hipLaunchKernelGGL((k_blocked_batched<T, V, L, SOR>), dim3(unsigned(grid)), dim3(kLanes), 0,
                       s, d, map, total_tiles, qu);
    return hipGetLastError();
}

template <typename T, bool SOR>
hipError_t launch_batched_depth(int fuse, const GridDesc<T>* d, const int* map, int tiles,
                                const Queue& qu, hipStream_t s) {
    constexpr int V = 16 / int(sizeof(T));
    switch (fuse) {
        case 1: return launch_batched_k<T, V, 2, SOR>(d, map, tiles, qu, s);
        case 2: return launch_batched_k<T, V, 4, SOR>(d, map, tiles, qu, s);
        case 3: return launch_batched_k<T, V, 6, SOR>(d, map, tiles, qu, s);
        case 4: return launch_batched_k<T, V, 8, SOR>(d, map, tiles, qu, s);
        case 5: return launch_batched_k<T, V, 10, SOR>(d, map, tiles, qu, s);
        case 6: return launch_batched_k<T, V, 12, SOR>(d, map, tiles, qu, s);
        case 7: return launch_batched_k<T, V, 14, SOR>(d, map, tiles, qu, s);
        case 8: return launch_batched_k<T, V, 16, SOR>(d, map, tiles, qu, s);
        case 9: return launch_batched_k<T, V, 18, SOR>(d, map, tiles, qu, s);
        default: return launch_batched_k<T, V, 20, SOR>(d, map, tiles, qu, s);
    }
}

// sor: the grids' omega relax every update (FP64 only)
template <typename T>
hipError_t launch_batched_by_fuse(int fuse, const GridDesc<T>* d, const int* map, int tiles,
                                  const Queue& qu, bool sor, hipStream_t s) {
    if constexpr (std::is_same<T, double>::value) {
        if (sor) return launch_batched_depth<T, true>(fuse, d, map, tiles, qu, s);
    } else {
        if (sor) return hipErrorInvalidValue;
    }
    return launch_batched_depth<T, false>(fuse, d, map, tiles, qu, s);
}

// Enqueue the device work of one batched sweep: pack, persistent passes,
// remaining sweeps as short persistent launches of fuse 1, unpack.
template <typename T>
hipError_t enqueue_batch(const BatchSetup& su, const BatchLayout& lay, char* ws, int count,
                         const rbgs_sweep_opts* o, bool do_pack, bool do_unpack, hipStream_t s,
                         bool sor = false) {
    hipError_t e;
    const PackDesc* pd = reinterpret_cast<const PackDesc*>(ws + lay.pdesc);
    const GridDesc<T>* gd = reinterpret_cast<const GridDesc<T>*>(ws + lay.gdesc);
    const int* map = reinterpret_cast<const int*>(ws + lay.tile_map);
    if (do_pack) {
        hipLaunchKernelGGL((k_batch_pack<typename std::conditional<sizeof(T) == 8, uint64_t, uint32_t>::type>),
                           dim3(unsigned(su.total_rows)), dim3(256), 0, s, pd, count);
        if ((e = hipGetLastError()) != hipSuccess) return e;
    }
    Queue qu;
    qu.ticket = reinterpret_cast<int*>(ws + lay.header);
    qu.error = reinterpret_cast<int*>(ws + lay.header + 64);
    qu.progress = reinterpret_cast<int*>(ws + lay.flags);
    qu.spin_limit = (o && o->debug_spin_limit > 0) ? o->debug_spin_limit : (1 << 22);
    qu.delay = o ? o->debug_delay : 0;
    qu.stall_tile = o ? o->debug_stall_tile : 0;
    qu.stop = nullptr;
    // the error word is cleared once; tickets and flags before every launch
    if ((e = launch_zero(ws + lay.header, 256, s)) != hipSuccess) return e;
    if (su.win.passes > 0) {
        const int* first = reinterpret_cast<const int*>(ws + lay.small);
        for (int p = 0; p < su.win.passes; ++p)  // map: the grids' order
            if ((e = launch_batch_pass<T>(su.win, gd, first, map, p, s)) != hipSuccess) return e;
        if (do_unpack) {
            hipLaunchKernelGGL((k_batch_unpack<typename std::conditional<sizeof(T) == 8, uint64_t, uint32_t>::type>),
                               dim3(unsigned(su.total_rows)), dim3(256), 0, s, pd, count,
                               su.win.passes & 1);
            if ((e = hipGetLastError()) != hipSuccess) return e;
        }
        return hipSuccess;
    }
    int parity = 0;
    // full passes of `fuse` sweeps, then (if nsweeps is not a multiple) one
    // pass of the remaining sweeps; its smaller depth fits the same tiles,
    // whose halo was sized for `fuse`
    const int launches[2][2] = {{su.fuse, su.passes}, {su.rem, su.rem > 0 ? 1 : 0}};
    const int final_parity = (su.passes + (su.rem > 0 ? 1 : 0)) & 1;
    if (sor && !su.small_ids.empty()) return hipErrorInvalidValue;  // Gauss-Seidel only
    if (!su.small_ids.empty()) {
        // the LDS-resident grids: all their sweeps in one launch, written to
        // the buffer the unpack reads
        const int nsweeps = su.passes * su.fuse + su.rem;
        static std::atomic<uint64_t> allowed{0};  // of this T's kernel
        (void)allow_dynamic_lds(reinterpret_cast<const void*>(&k_batch_lds<T>), lds_limit_bytes(),
                                allowed);
        hipLaunchKernelGGL((k_batch_lds<T>), dim3(unsigned(su.small_ids.size())), dim3(kLdsThreads),
                           su.small_lds_bytes, s, gd, reinterpret_cast<const int*>(ws + lay.small),
                           nsweeps, final_parity);
        if ((e = hipGetLastError()) != hipSuccess) return e;
    }
    for (const auto& lp : launches) {
        if (lp[1] == 0 || su.total_tiles == 0) continue;
        if ((e = launch_zero(ws + lay.header, 64, s)) != hipSuccess) return e;
        if ((e = launch_zero(ws + lay.flags, size_t(su.total_tiles) * 4, s)) != hipSuccess) return e;
        qu.passes = lp[1];
        qu.buf_offset = parity;
        if ((e = launch_batched_by_fuse<T>(lp[0], gd, map, su.total_tiles, qu, sor, s)) !=
            hipSuccess)
            return e;
        parity = (parity + lp[1]) & 1;
    }
    parity = final_parity;
    if (do_unpack) {
        hipLaunchKernelGGL((k_batch_unpack<typename std::conditional<sizeof(T) == 8, uint64_t, uint32_t>::type>),
                           dim3(unsigned(su.total_rows)), dim3(256), 0, s, pd, count, parity);
        if ((e = hipGetLastError()) != hipSuccess) return e;
    }
    return hipSuccess;
}

thread_local std::string g_batch_error = "no error";

int bfail(int status, const std::string& msg) {
    g_batch_error = msg;
    return status;
}

int validate_batch(int32_t count, const rbgs_grid* grids, int dt, void* const* u,
                   const void* const* f, int32_t nsweeps, const rbgs_sweep_opts* o) {
    if (count < 1 || count > 65535) return bfail(RBGS_EINVAL, "count must be in [1, 65535]");
    if (!grids || !u || !f) return bfail(RBGS_EINVAL, "grids, u and f must not be NULL");
    if (dt != RBGS_F64 && dt != RBGS_F32) return bfail(RBGS_EINVAL, "unknown dtype");
    if (nsweeps < 0) return bfail(RBGS_EINVAL, "nsweeps must be >= 0");
    for (int g = 0; g < count; ++g) {
        const rbgs_grid& gr = grids[g];
        if (gr.n < 1 || gr.n > 65533 || gr.ld < int64_t(gr.n) + 2 || !(gr.h > 0.0) ||
            !std::isfinite(gr.h))
            return bfail(RBGS_EINVAL, "grid " + std::to_string(g) + " is invalid");
        if (!u[g] || !f[g]) return bfail(RBGS_EINVAL, "grid " + std::to_string(g) + ": NULL array");
    }
    if (o) {
        if (o->kernel != RBGS_KERNEL_AUTO && o->kernel != RBGS_KERNEL_BLOCKED)
            return bfail(RBGS_EINVAL, "batched sweeps use the persistent kernel");
        if (o->fuse < 0 || o->fuse > kMaxFuse) return bfail(RBGS_EINVAL, "fuse must be in [0, 10]");
        if (o->tile_rows != 0 && (o->tile_rows < kMinRows || o->tile_rows > kMaxRows))
            return bfail(RBGS_EINVAL, "tile_rows must be in [8, 65536] (0 = default)");
        if (o->tile_cols != 0) return bfail(RBGS_EINVAL, "tile_cols must be 0");
        if (o->lds_max_n < -1) return bfail(RBGS_EINVAL, "lds_max_n must be >= -1");
        if (o->debug_delay < 0 || o->debug_delay > 1000 || o->debug_spin_limit < 0 ||
            o->debug_stall_tile < 0)
            return bfail(RBGS_EINVAL, "bad debug option");
        if (o->debug_tile_order != 0 || o->debug_stamp_check != 0 || o->debug_trace != nullptr ||
            o->debug_trace_items != 0)
            return bfail(RBGS_EUNSUPPORTED,
                         "tile orders, stamp checks and traces are for single-grid sweeps");
    }
    return RBGS_OK;
}

int check_ws(void* ws, size_t bytes, size_t need) {
    if (!ws) return bfail(RBGS_EWORKSPACE, "workspace is NULL");
    if (reinterpret_cast<uintptr_t>(ws) % 256 != 0)
        return bfail(RBGS_EWORKSPACE, "workspace must be 256-byte aligned");
    if (bytes < need)
        return bfail(RBGS_EWORKSPACE, "workspace too small: need " + std::to_string(need) + " bytes");
    return RBGS_OK;
}


// --- autotuner cache --------------------------------------------------------
// The persistent kernel's best shape for a batch, and whether the windows were
// faster still (way 1) or not (0); -1: a choice that was made without timing them.
struct Tuned {
    int fuse, rows, lds_max_n, way;
};
std::mutex g_tune_mu;
std::map<std::string, Tuned> g_tune;  // batch shape -> tuned parameters

std::string tune_key(int count, const rbgs_grid* grids, int dt) {
    std::map<int, int> hist;
    for (int g = 0; g < count; ++g) hist[grids[g].n]++;
    int dev = 0, cus = 0;
    (void)hipGetDevice(&dev);
    (void)hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, dev);
    std::string k = std::string(dt == RBGS_F64 ? "/f64" : "/f32") + "/cu" + std::to_string(cus);
    for (auto& kv : hist) k += "/" + std::to_string(kv.first) + "x" + std::to_string(kv.second);
    return k;
}

void load_tune_file() {
    static bool loaded = false;
    if (loaded) return;
    loaded = true;
    const char* path = std::getenv("RBGS_TUNE_CACHE");
    if (!path) return;
    FILE* fp = std::fopen(path, "r");
    if (!fp) return;
    // one entry per line, "v3" and the key, fuse rows lds_max_n ms way; "v2" entries
    // have no way and give way to a "v3" one (other lines are skipped)
    char line[4352], key[4096];
    while (std::fgets(line, sizeof line, fp)) {
        int fuse = 0, rows = 0, lds = 0, way = -1;
        float ms = 0.f;
        const int got = std::sscanf(line, "%4095s %d %d %d %f %d", key, &fuse, &rows, &lds, &ms, &way);
        if (got < 5 || fuse < 1 || fuse > kMaxFuse || rows < kMinRows || lds < -1) continue;
        const bool v3 = std::strncmp(key, "v3/", 3) == 0;
        if (v3 ? got != 6 || way < 0 || way > 1 : std::strncmp(key, "v2/", 3) != 0) continue;
        const auto it = g_tune.find(key + 2);
        if (!v3 && it != g_tune.end() && it->second.way >= 0) continue;
        g_tune[key + 2] = Tuned{fuse, rows, lds, v3 ? way : -1};
    }
    std::fclose(fp);
}

void store_tune(const std::string& key, const Tuned& t, float ms) {
    g_tune[key] = t;
    const char* path = std::getenv("RBGS_TUNE_CACHE");
    if (!path) return;
    FILE* fp = std::fopen(path, "a");
    if (!fp) return;
    std::fprintf(fp, "v3%s %d %d %d %.6f %d\n", key.c_str(), t.fuse, t.rows, t.lds_max_n, double(ms),
                 t.way);
    std::fclose(fp);
}

// How nsweeps sweeps of a batch run: explicit options first, then the tuned
// choice, then the defaults (batch_windows_pay, default_fuse, per-grid default tile
// height, no LDS-resident grids).
BatchChoice choose(int count, const rbgs_grid* grids, int dt, const rbgs_sweep_opts* o,
                   int nsweeps) {
    BatchChoice c;
    c.fuse = (o && o->fuse > 0) ? o->fuse : 0;
    c.rows = (o && o->tile_rows > 0) ? o->tile_rows : 0;
    c.lds_max_n = o ? o->lds_max_n : 0;
    int way = -1;
    if (c.fuse == 0 || c.rows == 0 || c.lds_max_n == 0) {
        std::lock_guard<std::mutex> lk(g_tune_mu);
        load_tune_file();
        auto it = g_tune.find(tune_key(count, grids, dt));
        if (it != g_tune.end()) {
            if (c.fuse == 0) c.fuse = it->second.fuse;
            if (c.rows == 0) c.rows = it->second.rows;
            if (c.lds_max_n == 0) c.lds_max_n = it->second.lds_max_n;
            way = it->second.way;
        }
    }
    int nmax = 1;
    for (int g = 0; g < count; ++g) nmax = grids[g].n > nmax ? grids[g].n : nmax;
    const int es = dt == RBGS_F64 ? 8 : 4;
    if (c.fuse == 0) c.fuse = default_fuse(es, nmax);
    if (c.lds_max_n == 0) c.lds_max_n = -1;
    if (batch_open(o) && nsweeps > 0) {
        if (way >= 0) {
            c.windows = way == 1;
        } else {
            std::vector<int> n(static_cast<size_t>(count));
            for (int g = 0; g < count; ++g) n[size_t(g)] = grids[g].n;
            c.windows = batch_windows_pay(count, n.data(), size_t(es), nsweeps);
        }
    }
    return c;
}

template <typename T>
int upload_setup(const BatchSetup& su, const BatchLayout& lay, char* ws, int count,
                 hipStream_t s) {
    hipError_t e = hipMemcpyAsync(ws + lay.gdesc, su.gdesc.data(), su.gdesc.size(),
                                  hipMemcpyHostToDevice, s);
    if (e == hipSuccess)
        e = hipMemcpyAsync(ws + lay.pdesc, su.pdesc.data(), sizeof(PackDesc) * count,
                           hipMemcpyHostToDevice, s);
    const bool windows = su.win.passes > 0;
    const std::vector<int>& map = windows ? su.win_order : su.tile_map;
    const std::vector<int>& small = windows ? su.win_first : su.small_ids;
    if (e == hipSuccess && !map.empty())
        e = hipMemcpyAsync(ws + lay.tile_map, map.data(), sizeof(int) * map.size(),
                           hipMemcpyHostToDevice, s);
    if (e == hipSuccess && !small.empty())
        e = hipMemcpyAsync(ws + lay.small, small.data(), sizeof(int) * small.size(),
                           hipMemcpyHostToDevice, s);
    // the host tables are freed when the caller returns: wait for the copies
    if (e == hipSuccess) e = hipStreamSynchronize(s);
    if (e != hipSuccess) return bfail(RBGS_EHIP, std::string("table upload: ") + hipGetErrorString(e));
    return RBGS_OK;
}

int read_error_word(const BatchLayout& lay, char* ws, hipStream_t s) {
    int err = 0;
    hipError_t e = hipMemcpyAsync(&err, ws + lay.header + 64, sizeof err, hipMemcpyDeviceToHost, s);
    if (e == hipSuccess) e = hipStreamSynchronize(s);
    if (e != hipSuccess) return bfail(RBGS_EHIP, std::string("error word: ") + hipGetErrorString(e));
    if (err) return bfail(RBGS_ETIMEOUT, "a tile dependency wait in the batched kernel timed out");
    return RBGS_OK;
}

template <typename T>
int sweep_batched_t(int32_t count, const rbgs_grid* grids, void* const* u, const void* const* f,
                    int32_t nsweeps, const rbgs_sweep_opts* o, char* ws, hipStream_t s) {
    const rbgs_dtype dt = sizeof(T) == 8 ? RBGS_F64 : RBGS_F32;
    const BatchLayout lay = batch_layout(count, grids, dt);
    const BatchSetup su = build_setup<T>(count, grids, u, f, lay, ws,
                                         choose(count, grids, dt, o, nsweeps), nsweeps);
    int rc = upload_setup<T>(su, lay, ws, count, s);
    if (rc) return rc;
    EventPair ev;
    if (o && o->timing) {
        if (hipEventCreate(&ev.a) != hipSuccess || hipEventCreate(&ev.b) != hipSuccess)
            return bfail(RBGS_EHIP, "event create");
        (void)hipEventRecord(ev.a, s);
    }
    hipError_t e = enqueue_batch<T>(su, lay, ws, count, o, true, true, s);
    if (e != hipSuccess) return bfail(RBGS_EHIP, std::string("batched sweep: ") + hipGetErrorString(e));
    if (o && o->timing) {
        (void)hipEventRecord(ev.b, s);
        (void)hipEventSynchronize(ev.b);
        float ms = 0.f;
        (void)hipEventElapsedTime(&ms, ev.a, ev.b);
        const int tiled = su.total_tiles > 0 ? (su.passes > 0) + (su.rem > 0) : 0;
        const int launches = tiled + (su.small_ids.empty() ? 0 : 1);
        *o->timing = rbgs_timing{0.f, ms, 0.f, su.win.passes > 0 ? su.win.passes : launches};
    }
    return read_error_word(lay, ws, s);
}

// ---------------------------------------------------------------------------
// Batched solve: FP64 iterative refinement (the single-grid rbgs_solve's
// steps, grid by grid) whose FP32 inner sweeps run as one batched
// sweep over every grid that has not yet converged.
// ---------------------------------------------------------------------------

// Workspace of a batched solve: the FP32 batch (per grid: the correction e
// in two ping-pong buffers and the right-hand side r, split layout), then
// per grid the FP64 split u and f and the residual partial sums, then two
// norms per grid.
struct SolveLayout {
    BatchLayout inner;
    std::vector<size_t> u_off;    // u_red, u_black, f_red, f_black (FP64 split)
    std::vector<int64_t> pitch64;
    std::vector<size_t> part_off;
    size_t sums = 0;
    size_t total = 0;
};

SolveLayout solve_layout(int count, const rbgs_grid* grids) {
    SolveLayout L;
    L.inner = batch_layout(count, grids, RBGS_F32);
    size_t off = align256(L.inner.total);
    L.u_off.resize(count);
    L.pitch64.resize(count);
    L.part_off.resize(count);
    for (int g = 0; g < count; ++g) {
        const int n = grids[g].n;
        const int64_t P = split_pitch(n, 8);
        L.pitch64[g] = P;
        L.u_off[g] = off;
        off += 4 * align256(size_t(n + 2) * size_t(P) * 8);
        L.part_off[g] = off;
        off += align256(size_t(residual_partial_slots(n, P, 8)) * 2 * sizeof(double));
    }
    L.sums = off;
    off += align256(size_t(count) * 2 * sizeof(double));
    L.total = off;
    return L;
}

struct GridArrays {
    double *u_red, *u_black, *f_red, *f_black;
    float *e[2][2];  // [buffer][red, black]
    float *r_red, *r_black;
    int64_t p64, p32;
};

GridArrays grid_arrays(const SolveLayout& L, char* ws, const rbgs_grid* grids, int g) {
    GridArrays a;
    const int n = grids[g].n;
    const size_t c64 = align256(size_t(n + 2) * size_t(L.pitch64[g]) * 8);
    char* b64 = ws + L.u_off[g];
    a.u_red = reinterpret_cast<double*>(b64);
    a.u_black = reinterpret_cast<double*>(b64 + c64);
    a.f_red = reinterpret_cast<double*>(b64 + 2 * c64);
    a.f_black = reinterpret_cast<double*>(b64 + 3 * c64);
    const size_t c32 = align256(size_t(n + 2) * size_t(L.inner.pitch[g]) * 4);
    char* b32 = ws + L.inner.grid_off[g];  // the order build_setup assigns
    a.e[0][0] = reinterpret_cast<float*>(b32);
    a.e[0][1] = reinterpret_cast<float*>(b32 + c32);
    a.e[1][0] = reinterpret_cast<float*>(b32 + 2 * c32);
    a.e[1][1] = reinterpret_cast<float*>(b32 + 3 * c32);
    a.r_red = reinterpret_cast<float*>(b32 + 4 * c32);
    a.r_black = reinterpret_cast<float*>(b32 + 5 * c32);
    a.p64 = L.pitch64[g];
    a.p32 = L.inner.pitch[g];
    return a;
}

int solve_batched_ir(int32_t count, const rbgs_grid* grids, double* const* u,
                     const double* const* f, const rbgs_solve_opts* o, rbgs_solve_info* infos,
                     char* ws, hipStream_t s) {
    const SolveLayout L = solve_layout(count, grids);
    const int bf16 = o->precision == RBGS_PREC_BF16RHS_IR;
    const int inner = o->inner_sweeps > 0 ? o->inner_sweeps : o->check_every;
    double* sums = reinterpret_cast<double*>(ws + L.sums);
    std::vector<GridArrays> ga(count);
    hipError_t e = hipSuccess;
    for (int g = 0; g < count && e == hipSuccess; ++g) {
        ga[g] = grid_arrays(L, ws, grids, g);
        e = launch_pack(u[g], grids[g].ld, ga[g].u_red, ga[g].u_black, grids[g].n, ga[g].p64, 8, s);
        if (e == hipSuccess)
            e = launch_pack(f[g], grids[g].ld, ga[g].f_red, ga[g].f_black, grids[g].n, ga[g].p64, 8, s);
    }
    if (e != hipSuccess) return bfail(RBGS_EHIP, std::string("pack: ") + hipGetErrorString(e));
    std::vector<double> rel(count, 0.0), ab(count, 0.0), host(2 * size_t(count));
    std::vector<int> done(count, 0), outer(count, 0);
    // FP64 residual of the listed grids, with r stored in FP32 (or bfloat16)
    // as the next inner right-hand side
    auto residuals = [&](const std::vector<int>& which) -> int {
        hipError_t r = hipSuccess;
        for (int g : which) {
            r = launch_residual_split<double>(ga[g].u_red, ga[g].u_black, ga[g].f_red, ga[g].f_black,
                                              grids[g].n, ga[g].p64,
                                              1.0 / (grids[g].h * grids[g].h),
                                              reinterpret_cast<double*>(ws + L.part_off[g]),
                                              sums + 2 * g, ga[g].r_red, ga[g].r_black, ga[g].p32,
                                              bf16, s);
            if (r != hipSuccess) break;
        }
        if (r == hipSuccess)
            r = hipMemcpyAsync(host.data(), sums, host.size() * sizeof(double),
                               hipMemcpyDeviceToHost, s);
        if (r == hipSuccess) r = hipStreamSynchronize(s);
        if (r != hipSuccess) return bfail(RBGS_EHIP, std::string("residual: ") + hipGetErrorString(r));
        for (int g : which) {
            const double rn = std::sqrt(host[2 * g]), bn = std::sqrt(host[2 * g + 1]);
            ab[g] = rn;
            rel[g] = bn > 0.0 ? rn / bn : rn;
        }
        return RBGS_OK;
    };
    std::vector<int> all(count);
    std::iota(all.begin(), all.end(), 0);
    int rc = residuals(all);
    if (rc) return rc;
    for (;;) {
        // the grids still refining, grouped by this step's sweep count (a
        // grid near max_sweeps takes fewer, as in the single-grid solve)
        std::map<int, std::vector<int>> by_k;
        for (int g = 0; g < count; ++g)
            if (!(rel[g] <= o->rel_tol) && done[g] < o->max_sweeps && std::isfinite(rel[g]))
                by_k[std::min(inner, o->max_sweeps - done[g])].push_back(g);
        if (by_k.empty()) break;
        std::vector<int> stepped;
        for (const auto& kv : by_k) {
            const int k = kv.first;
            const std::vector<int>& act = kv.second;
            for (int g : act)
                for (int b = 0; b < 2 && e == hipSuccess; ++b)
                    for (int c = 0; c < 2 && e == hipSuccess; ++c)
                        e = launch_zero(ga[g].e[b][c],
                                        size_t(grids[g].n + 2) * size_t(ga[g].p32) * 4, s);
            if (e != hipSuccess) return bfail(RBGS_EHIP, std::string("zero: ") + hipGetErrorString(e));
            // one batched launch over these grids: a view of the layout with
            // their arrays only
            const int na = int(act.size());
            BatchLayout sub = L.inner;
            sub.grid_off.assign(na, 0);
            sub.pitch.assign(na, 0);
            std::vector<rbgs_grid> sg(na);
            std::vector<void*> nu(na, nullptr);
            std::vector<const void*> nf(na, nullptr);
            for (int a = 0; a < na; ++a) {
                sub.grid_off[a] = L.inner.grid_off[act[a]];
                sub.pitch[a] = L.inner.pitch[act[a]];
                sg[a] = grids[act[a]];
            }
            const BatchSetup su =
                build_setup<float>(na, sg.data(), nu.data(), nf.data(), sub, ws,
                                   choose(na, sg.data(), RBGS_F32, &o->sweep, k), k);
            if ((rc = upload_setup<float>(su, sub, ws, na, s))) return rc;
            e = enqueue_batch<float>(su, sub, ws, na, &o->sweep, false, false, s);
            if (e != hipSuccess)
                return bfail(RBGS_EHIP, std::string("inner sweeps: ") + hipGetErrorString(e));
            if ((rc = read_error_word(sub, ws, s))) return rc;
            const int out = result_buffer(su);
            for (int g : act) {
                e = launch_add_correction(ga[g].u_red, ga[g].u_black, ga[g].p64, ga[g].e[out][0],
                                          ga[g].e[out][1], ga[g].p32, grids[g].n, s);
                if (e != hipSuccess)
                    return bfail(RBGS_EHIP, std::string("correction: ") + hipGetErrorString(e));
                done[g] += k;
                ++outer[g];
                stepped.push_back(g);
            }
        }
        if ((rc = residuals(stepped))) return rc;
    }
    for (int g = 0; g < count && e == hipSuccess; ++g)
        e = launch_unpack(u[g], grids[g].ld, ga[g].u_red, ga[g].u_black, grids[g].n, ga[g].p64, 8, s);
    if (e == hipSuccess) e = hipStreamSynchronize(s);
    if (e != hipSuccess) return bfail(RBGS_EHIP, std::string("unpack: ") + hipGetErrorString(e));
    int status = RBGS_OK;
    for (int g = 0; g < count; ++g) {
        rbgs_solve_info info{done[g], outer[g], rel[g], ab[g], RBGS_OK, o->precision};
        if (!std::isfinite(rel[g]))
            info.status = RBGS_ENONFINITE;
        else if (!(rel[g] <= o->rel_tol))
            info.status = RBGS_ENOCONV;
        if (infos) infos[g] = info;
        if (info.status != RBGS_OK && status == RBGS_OK) status = info.status;
    }
    if (status == RBGS_ENOCONV) g_batch_error = "tolerance not reached by every grid";
    if (status == RBGS_ENONFINITE) g_batch_error = "a residual is not finite";
    return status;
}

// ---------------------------------------------------------------------------
// Batched FP64 solve: the single-grid FP64 solve loop (residual, then
// check_every sweeps, until rel <= rel_tol or max_sweeps), with the sweeps
// of every grid still iterating in one batched sweep; with
// omega != 1 the sweeps are red-black SOR, each grid with its own omega.
// ---------------------------------------------------------------------------

// Workspace: the FP64 batch (per grid two ping-pong buffers of u and f,
// split layout), then per grid the residual partial sums, then two norms
// per grid.
struct SolveLayoutF64 {
    BatchLayout batch;
    std::vector<size_t> part_off;
    size_t sums = 0;
    size_t total = 0;
};

SolveLayoutF64 solve_layout_f64(int count, const rbgs_grid* grids) {
    SolveLayoutF64 L;
    L.batch = batch_layout(count, grids, RBGS_F64);
    size_t off = align256(L.batch.total);
    L.part_off.resize(count);
    for (int g = 0; g < count; ++g) {
        L.part_off[g] = off;
        off += align256(size_t(residual_partial_slots(grids[g].n, L.batch.pitch[g], 8)) * 2 *
                        sizeof(double));
    }
    L.sums = off;
    off += align256(size_t(count) * 2 * sizeof(double));
    L.total = off;
    return L;
}

int solve_batched_f64(int32_t count, const rbgs_grid* grids, double* const* u,
                      const double* const* f, const rbgs_solve_opts* o, rbgs_solve_info* infos,
                      char* ws, hipStream_t s) {
    const SolveLayoutF64 L = solve_layout_f64(count, grids);
    const int check = o->check_every > 0 ? o->check_every : o->inner_sweeps;
    // omega 0: each grid's optimum for the model problem, 2 / (1 + sin(pi h))
    const bool sor = o->omega != 1.0;
    auto omega_of = [&](int g) {
        return o->omega == 0.0 ? 2.0 / (1.0 + std::sin(M_PI * grids[g].h)) : o->omega;
    };
    double* sums = reinterpret_cast<double*>(ws + L.sums);
    // colour array k of grid g in the order build_setup lays them out:
    // red, black of buffer 0, red, black of buffer 1, f red, f black
    auto arr = [&](int g, int k) {
        const size_t colour = align256(size_t(grids[g].n + 2) * size_t(L.batch.pitch[g]) * 8);
        return reinterpret_cast<double*>(ws + L.batch.grid_off[g] + size_t(k) * colour);
    };
    // u and f of every grid into the split layout (u into both buffers, so
    // both hold the Dirichlet ring)
    {
        const BatchSetup su = build_setup<double>(count, grids, reinterpret_cast<void* const*>(u),
                                                  reinterpret_cast<const void* const*>(f), L.batch,
                                                  ws, BatchChoice{1, 0, -1}, 0);
        int rc = upload_setup<double>(su, L.batch, ws, count, s);
        if (rc) return rc;
        hipError_t e = enqueue_batch<double>(su, L.batch, ws, count, nullptr, true, false, s);
        if (e != hipSuccess) return bfail(RBGS_EHIP, std::string("pack: ") + hipGetErrorString(e));
    }
    // buffer holding each grid's current iterate
    std::vector<int> cur(count, 0), done(count, 0);
    std::vector<double> rel(count, 0.0), ab(count, 0.0), host(2 * size_t(count));
    auto residuals = [&](const std::vector<int>& which) -> int {
        hipError_t r = hipSuccess;
        for (int g : which) {
            const int b = cur[g];
            r = launch_residual_split<double>(arr(g, 2 * b), arr(g, 2 * b + 1), arr(g, 4), arr(g, 5),
                                              grids[g].n, L.batch.pitch[g],
                                              1.0 / (grids[g].h * grids[g].h),
                                              reinterpret_cast<double*>(ws + L.part_off[g]),
                                              sums + 2 * g, nullptr, nullptr, 0, 0, s);
            if (r != hipSuccess) break;
        }
        if (r == hipSuccess)
            r = hipMemcpyAsync(host.data(), sums, host.size() * sizeof(double),
                               hipMemcpyDeviceToHost, s);
        if (r == hipSuccess) r = hipStreamSynchronize(s);
        if (r != hipSuccess) return bfail(RBGS_EHIP, std::string("residual: ") + hipGetErrorString(r));
        for (int g : which) {
            const double rn = std::sqrt(host[2 * g]), bn = std::sqrt(host[2 * g + 1]);
            ab[g] = rn;
            rel[g] = bn > 0.0 ? rn / bn : rn;
        }
        return RBGS_OK;
    };
    std::vector<int> all(count);
    std::iota(all.begin(), all.end(), 0);
    int rc = residuals(all);
    if (rc) return rc;
    hipError_t e = hipSuccess;
    for (;;) {
        // grids still iterating, grouped by this round's sweep count (the
        // last round of a grid near max_sweeps takes the remainder)
        std::map<int, std::vector<int>> by_k;
        for (int g = 0; g < count; ++g)
            if (!(rel[g] <= o->rel_tol) && done[g] < o->max_sweeps && std::isfinite(rel[g]))
                by_k[std::min(check, o->max_sweeps - done[g])].push_back(g);
        if (by_k.empty()) break;
        std::vector<int> stepped;
        for (const auto& kv : by_k) {
            const int k = kv.first;
            const std::vector<int>& act = kv.second;
            const int na = int(act.size());
            BatchLayout sub = L.batch;
            sub.grid_off.assign(na, 0);
            sub.pitch.assign(na, 0);
            std::vector<rbgs_grid> sg(na);
            std::vector<void*> nu(na, nullptr);
            std::vector<const void*> nf(na, nullptr);
            for (int a = 0; a < na; ++a) {
                sub.grid_off[a] = L.batch.grid_off[act[a]];
                sub.pitch[a] = L.batch.pitch[act[a]];
                sg[a] = grids[act[a]];
            }
            BatchChoice how = choose(na, sg.data(), RBGS_F64, &o->sweep, k);
            if (sor) {  // the LDS-resident sweep and the windows are Gauss-Seidel only
                how.lds_max_n = -1;
                how.windows = false;
            }
            BatchSetup su = build_setup<double>(na, sg.data(), nu.data(), nf.data(), sub, ws, how, k);
            // a grid whose iterate sits in buffer 1 runs with its buffers
            // swapped, so that every launch starts from "buffer 0"
            GridDesc<double>* gd = reinterpret_cast<GridDesc<double>*>(su.gdesc.data());
            for (int a = 0; a < na; ++a) {
                if (cur[act[a]]) {
                    std::swap(gd[a].red[0], gd[a].red[1]);
                    std::swap(gd[a].black[0], gd[a].black[1]);
                }
                gd[a].omega = omega_of(act[a]);
            }
            if ((rc = upload_setup<double>(su, sub, ws, na, s))) return rc;
            e = enqueue_batch<double>(su, sub, ws, na, &o->sweep, false, false, s, sor);
            if (e != hipSuccess) return bfail(RBGS_EHIP, std::string("sweeps: ") + hipGetErrorString(e));
            if ((rc = read_error_word(sub, ws, s))) return rc;
            const int out = result_buffer(su);
            for (int g : act) {
                cur[g] ^= out;
                done[g] += k;
                stepped.push_back(g);
            }
        }
        if ((rc = residuals(stepped))) return rc;
    }
    for (int g = 0; g < count && e == hipSuccess; ++g)
        e = launch_unpack(u[g], grids[g].ld, arr(g, 2 * cur[g]), arr(g, 2 * cur[g] + 1), grids[g].n,
                          L.batch.pitch[g], 8, s);
    if (e == hipSuccess) e = hipStreamSynchronize(s);
    if (e != hipSuccess) return bfail(RBGS_EHIP, std::string("unpack: ") + hipGetErrorString(e));
    int status = RBGS_OK;
    for (int g = 0; g < count; ++g) {
        rbgs_solve_info info{done[g], 0, rel[g], ab[g], RBGS_OK, RBGS_PREC_F64};
        if (!std::isfinite(rel[g]))
            info.status = RBGS_ENONFINITE;
        else if (!(rel[g] <= o->rel_tol))
            info.status = RBGS_ENOCONV;
        if (infos) infos[g] = info;
        if (info.status != RBGS_OK && status == RBGS_OK) status = info.status;
    }
    if (status == RBGS_ENOCONV) g_batch_error = "tolerance not reached by every grid";
    if (status == RBGS_ENONFINITE) g_batch_error = "a residual is not finite";
    return status;
}

}  // namespace
}  // namespace rbgs

using namespace rbgs;

struct rbgs_batch_plan {
    hipGraph_t graph = nullptr;
    hipGraphExec_t exec = nullptr;
    BatchLayout lay;
    char* ws = nullptr;
    int passes = 0, fuse = 0;
};

extern "C" {

size_t rbgs_batch_workspace_size(int32_t count, const rbgs_grid* grids, rbgs_dtype dt) {
    if (count < 1 || count > 65535 || !grids || (dt != RBGS_F64 && dt != RBGS_F32)) return 0;
    for (int g = 0; g < count; ++g)
        if (grids[g].n < 1 || grids[g].n > 65533 || grids[g].ld < int64_t(grids[g].n) + 2) return 0;
    return batch_layout(count, grids, dt).total;
}

const char* rbgs_batch_last_error(void) { return g_batch_error.c_str(); }

int rbgs_sweep_batched(int32_t count, const rbgs_grid* grids, rbgs_dtype dt, void* const* u,
                       const void* const* f, int32_t nsweeps, const rbgs_sweep_opts* opts,
                       void* workspace, size_t workspace_bytes, void* stream) {
    int rc = validate_batch(count, grids, dt, u, f, nsweeps, opts);
    if (rc) return rc;
    if ((rc = check_ws(workspace, workspace_bytes, batch_layout(count, grids, dt).total))) return rc;
    if (nsweeps == 0) return RBGS_OK;
    hipStream_t s = static_cast<hipStream_t>(stream);
    char* ws = static_cast<char*>(workspace);
    return dt == RBGS_F64 ? sweep_batched_t<double>(count, grids, u, f, nsweeps, opts, ws, s)
                          : sweep_batched_t<float>(count, grids, u, f, nsweeps, opts, ws, s);
}

int rbgs_batch_plan_create(rbgs_batch_plan** plan, int32_t count, const rbgs_grid* grids,
                           rbgs_dtype dt, void* const* u, const void* const* f, int32_t nsweeps,
                           const rbgs_sweep_opts* opts, void* workspace, size_t workspace_bytes) {
    if (!plan) return bfail(RBGS_EINVAL, "plan is NULL");
    *plan = nullptr;
    int rc = validate_batch(count, grids, dt, u, f, nsweeps, opts);
    if (rc) return rc;
    if (nsweeps < 1) return bfail(RBGS_EINVAL, "a plan needs nsweeps >= 1");
    BatchLayout lay = batch_layout(count, grids, dt);
    if ((rc = check_ws(workspace, workspace_bytes, lay.total))) return rc;
    char* ws = static_cast<char*>(workspace);
    hipStream_t cs = nullptr;
    if (hipStreamCreateWithFlags(&cs, hipStreamNonBlocking) != hipSuccess)
        return bfail(RBGS_EHIP, "stream create");
    const BatchChoice how = choose(count, grids, dt, opts, nsweeps);
    BatchSetup su;
    if (dt == RBGS_F64) {
        su = build_setup<double>(count, grids, u, f, lay, ws, how, nsweeps);
        rc = upload_setup<double>(su, lay, ws, count, cs);
    } else {
        su = build_setup<float>(count, grids, u, f, lay, ws, how, nsweeps);
        rc = upload_setup<float>(su, lay, ws, count, cs);
    }
    if (rc) {
        (void)hipStreamDestroy(cs);
        return rc;
    }
    rbgs_batch_plan* p = new rbgs_batch_plan;
    p->lay = lay;
    p->ws = ws;
    p->passes = su.passes;
    p->fuse = how.fuse;
    hipError_t e = hipStreamBeginCapture(cs, hipStreamCaptureModeThreadLocal);
    if (e == hipSuccess) {
        hipError_t e2 = dt == RBGS_F64 ? enqueue_batch<double>(su, lay, ws, count, opts, true, true, cs)
                                       : enqueue_batch<float>(su, lay, ws, count, opts, true, true, cs);
        e = hipStreamEndCapture(cs, &p->graph);
        if (e2 != hipSuccess) e = e2;
    }
    if (e == hipSuccess) e = hipGraphInstantiate(&p->exec, p->graph, nullptr, nullptr, 0);
    (void)hipStreamDestroy(cs);
    if (e != hipSuccess) {
        if (p->graph) (void)hipGraphDestroy(p->graph);
        delete p;
        return bfail(RBGS_EHIP, std::string("graph capture: ") + hipGetErrorString(e));
    }
    *plan = p;
    return RBGS_OK;
}

int rbgs_batch_plan_launch(rbgs_batch_plan* plan, void* stream) {
    if (!plan || !plan->exec) return bfail(RBGS_EINVAL, "plan is NULL");
    hipError_t e = hipGraphLaunch(plan->exec, static_cast<hipStream_t>(stream));
    if (e != hipSuccess) return bfail(RBGS_EHIP, std::string("graph launch: ") + hipGetErrorString(e));
    return RBGS_OK;
}

int rbgs_batch_plan_check(rbgs_batch_plan* plan, void* stream) {
    if (!plan) return bfail(RBGS_EINVAL, "plan is NULL");
    return read_error_word(plan->lay, plan->ws, static_cast<hipStream_t>(stream));
}

int rbgs_batch_plan_destroy(rbgs_batch_plan* plan) {
    if (!plan) return RBGS_OK;
    if (plan->exec) (void)hipGraphExecDestroy(plan->exec);
    if (plan->graph) (void)hipGraphDestroy(plan->graph);
    delete plan;
    return RBGS_OK;
}

int rbgs_autotune_batched(int32_t count, const rbgs_grid* grids, rbgs_dtype dt, void* const* u,
                          const void* const* f, void* workspace, size_t workspace_bytes,
                          void* stream, rbgs_sweep_opts* best, float* best_ms_per_sweep) {
    int rc = validate_batch(count, grids, dt, u, f, 0, nullptr);
    if (rc) return rc;
    BatchLayout lay = batch_layout(count, grids, dt);
    if ((rc = check_ws(workspace, workspace_bytes, lay.total))) return rc;
    hipStream_t s = static_cast<hipStream_t>(stream);
    char* ws = static_cast<char*>(workspace);
    hipEvent_t a = nullptr, b = nullptr;
    if (hipEventCreate(&a) != hipSuccess || hipEventCreate(&b) != hipSuccess)
        return bfail(RBGS_EHIP, "event create");
    const int fuses[] = {4, 5, 6, 7};
    const int rowsv[] = {64, 128, 256};
    const int lds_candidate = tuned_lds_candidate(dt == RBGS_F64 ? 8 : 4);
    bool packed = false;
    const size_t es = dt == RBGS_F64 ? 8 : 4;
    auto enqueue = [&](const BatchSetup& su) {
        const hipError_t e =
            dt == RBGS_F64 ? enqueue_batch<double>(su, lay, ws, count, nullptr, !packed, false, s)
                           : enqueue_batch<float>(su, lay, ws, count, nullptr, !packed, false, s);
        packed = true;
        return e;
    };
    // time per sweep of one candidate over nsweeps sweeps, after an untimed run of
    // warm sweeps
    auto time_one = [&](const BatchChoice& how, int warm, int nsweeps, float* per_sweep) -> int {
        auto setup = [&](int k) {
            return dt == RBGS_F64 ? build_setup<double>(count, grids, u, f, lay, ws, how, k)
                                  : build_setup<float>(count, grids, u, f, lay, ws, how, k);
        };
        hipError_t e = hipSuccess;
        for (int k : {warm, nsweeps}) {
            const BatchSetup su = setup(k);
            int r = dt == RBGS_F64 ? upload_setup<double>(su, lay, ws, count, s)
                                   : upload_setup<float>(su, lay, ws, count, s);
            if (r) return r;
            if (e == hipSuccess) e = hipEventRecord(a, s);
            if (e == hipSuccess) e = enqueue(su);
            if (e == hipSuccess) e = hipEventRecord(b, s);
            if (e == hipSuccess) e = hipEventSynchronize(b);
            if (e != hipSuccess)
                return bfail(RBGS_EHIP, std::string("autotune: ") + hipGetErrorString(e));
        }
        float ms = 0.f;
        if ((e = hipEventElapsedTime(&ms, a, b)) != hipSuccess)
            return bfail(RBGS_EHIP, std::string("autotune: ") + hipGetErrorString(e));
        int r = read_error_word(lay, ws, s);
        if (r) return r;
        *per_sweep = ms / float(nsweeps);
        return RBGS_OK;
    };
    float best_ms = 1e30f;
    BatchChoice bt{kMaxFuse, 0, -1};
    for (int fu : fuses) {
        for (int ro : rowsv) {
            float per_sweep = 0.f;
            if ((rc = time_one({fu, ro, -1}, fu, 2 * fu, &per_sweep))) break;
            if (per_sweep < best_ms) {
                best_ms = per_sweep;
                bt = BatchChoice{fu, ro, -1};
            }
        }
        if (rc) break;
    }
    if (!rc) {  // then the small grids LDS-resident instead
        float per_sweep = 0.f;
        rc = time_one({bt.fuse, bt.rows, lds_candidate}, bt.fuse, 2 * bt.fuse, &per_sweep);
        if (!rc && per_sweep < best_ms) {
            best_ms = per_sweep;
            bt.lds_max_n = lds_candidate;
        }
    }
    if (!rc) {  // the windows against the best of these, over as many sweeps
        BatchChoice wi = bt;
        wi.windows = true;
        float persistent = 0.f, windows = 0.f;
        rc = time_one(bt, bt.fuse, 8 * bt.fuse, &persistent);
        if (!rc) best_ms = persistent;
        BatchSetup probe;
        if (!rc && split_windows(probe, count, grids, es, 8 * bt.fuse)) {
            rc = time_one(wi, bt.fuse, 8 * bt.fuse, &windows);
            if (!rc && windows < persistent) {
                best_ms = windows;
                bt.windows = true;
            }
        }
    }
    (void)hipEventDestroy(a);
    (void)hipEventDestroy(b);
    if (rc) return rc;
    {
        std::lock_guard<std::mutex> lk(g_tune_mu);
        load_tune_file();
        store_tune(tune_key(count, grids, dt),
                   Tuned{bt.fuse, bt.rows, bt.lds_max_n, bt.windows ? 1 : 0}, best_ms);
    }
    if (best) {
        std::memset(best, 0, sizeof *best);
        best->kernel = bt.windows ? RBGS_KERNEL_AUTO : RBGS_KERNEL_BLOCKED;
        best->fuse = bt.fuse;
        best->tile_rows = bt.rows;
        best->lds_max_n = bt.lds_max_n;
    }
    if (best_ms_per_sweep) *best_ms_per_sweep = best_ms;
    return RBGS_OK;
}

size_t rbgs_batch_solve_workspace_size(int32_t count, const rbgs_grid* grids) {
    if (rbgs_batch_workspace_size(count, grids, RBGS_F32) == 0) return 0;
    return std::max(solve_layout(count, grids).total, solve_layout_f64(count, grids).total);
}

int rbgs_solve_batched(int32_t count, const rbgs_grid* grids, double* const* u,
                       const double* const* f, const rbgs_solve_opts* opts,
                       rbgs_solve_info* infos, void* workspace, size_t workspace_bytes,
                       void* stream) {
    if (!opts) return bfail(RBGS_EINVAL, "opts is NULL");
    if (opts->fallback != 0)
        return bfail(RBGS_EUNSUPPORTED, "the precision fallback is for single-grid solves");
    if (opts->precision != RBGS_PREC_F64 && opts->precision != RBGS_PREC_F32_IR &&
        opts->precision != RBGS_PREC_BF16RHS_IR)
        return bfail(RBGS_EINVAL, "unknown precision");
    if (!(opts->rel_tol > 0.0) || opts->max_sweeps < 0)
        return bfail(RBGS_EINVAL, "need rel_tol > 0 and max_sweeps >= 0");
    if (opts->inner_sweeps < 0 || opts->check_every < 0 ||
        (opts->inner_sweeps == 0 && opts->check_every == 0))
        return bfail(RBGS_EINVAL, "need inner_sweeps >= 1 (or check_every >= 1)");
    if (opts->omega != 1.0) {
        if (!(opts->omega == 0.0 || (opts->omega > 0.0 && opts->omega < 2.0)))
            return bfail(RBGS_EINVAL, "omega must be in (0, 2), or 0 for each grid's optimum");
        if (opts->precision != RBGS_PREC_F64)
            return bfail(RBGS_EUNSUPPORTED, "batched SOR (omega != 1) runs in FP64 without "
                                            "refinement");
    }
    int rc = validate_batch(count, grids, RBGS_F64, reinterpret_cast<void* const*>(u),
                            reinterpret_cast<const void* const*>(f), 0, &opts->sweep);
    if (rc) return rc;
    if ((rc = check_ws(workspace, workspace_bytes, rbgs_batch_solve_workspace_size(count, grids))))
        return rc;
    char* ws = static_cast<char*>(workspace);
    hipStream_t s = static_cast<hipStream_t>(stream);
    return opts->precision == RBGS_PREC_F64
               ? solve_batched_f64(count, grids, u, f, opts, infos, ws, s)
               : solve_batched_ir(count, grids, u, f, opts, infos, ws, s);
}

}  // extern "C"
