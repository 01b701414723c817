// Small and middle-sized grids: K red-black sweeps a launch, each wave with its
// own window of the grid in registers.
//
// These grids are bound by latency: a launch per half-sweep costs two launches
// a sweep, and waves that trade boundary rows (sweep_resident.hip) pay a
// handoff across dies every few sweeps.  Here a wave loads a window of
// W = R + 4 K rows by 64 split columns (one red and one black point per lane
// and row) at once, runs 2 K half-sweeps in registers, and writes the R x
// (64 - 2 K) core whose values the window determines; the next launch starts
// from those.  Windows overlap, so a launch needs no flags, and the boundary
// between launches orders the passes.  Half-sweep l only updates the rows that
// the core still depends on, l + 1 .. W - 2 - l: 2 K (R + 2 K - 1) row updates,
// every one of a half-sweep independent of the others, so one wave per SIMD
// keeps it busy.
//
// A pass reads black and f (red is recomputed from black before anything
// reads it) and writes black, and red in the last pass; windows at the ring
// also read red, whose ring values they keep.  A pass reads one buffer and
// writes the other.  Each point's operations and their order are those of the
// plain half-sweep (h^2 f is formed once per pass), so the bits are the same.
#include "sweep_window.h"

namespace rbgs {
namespace {

using namespace window_pass;

template <typename T, int K, int R, bool SOR>
__global__ __launch_bounds__(kLanes) void k_window(WindowArgs<T> a) {
    if (a.stop && *a.stop) return;
    run_window<T, K, R, core_width(K), SOR>(a, int(blockIdx.x));
}

template <typename T, int K, int R>
hipError_t launch(WindowArgs<T> a, hipStream_t s) {
    a.bands = window_bands(a.n, core_width(K));
    const dim3 grid(unsigned(a.bands * window_strips(a.n, R)));
    if constexpr (sizeof(T) == 8) {
        if (a.omega != T(1)) {
            hipLaunchKernelGGL((k_window<T, K, R, true>), grid, dim3(kLanes), 0, s, a);
            return hipGetLastError();
        }
    }
    hipLaunchKernelGGL((k_window<T, K, R, false>), grid, dim3(kLanes), 0, s, a);
    return hipGetLastError();
}

// The shape for a grid: most sweeps a launch (k) and rows a window writes (r).
// Small grids are latency-bound and want short windows on many SIMDs; larger
// ones want a smaller share of recomputed rows ((r + 4 k) / r).  Measured on
// MI355X, 240 sweeps, us by (k, r):
//   FP64  255^2  (5,4) 330  (5,8) 399  (4,16) 580   resident 1059
//         640^2  (5,4) 429  (5,8) 448  (4,16) 619   blocked 1402
//         900^2  (5,4) 700  (5,8) 564  (4,16) 642   blocked 1465
//        1023^2  (5,4) 878  (5,8) 875  (4,16) 736   blocked 1536
//        2047^2             (5,8) 2193 (4,16) 1928  blocked 2305
//        2400^2             (5,8) 2549 (4,16) 2441  blocked 2392
//   FP32  511^2  (6,4) 294  (6,8) 337  (6,16) 445   resident 1179
//         767^2  (6,4) 363  (6,8) 343  (6,16) 454   resident 1859
//        1000^2  (6,8) 544  (6,16) 492 (6,24) 608   plain 1661
//        2600^2  (6,8) 1948 (6,16) 1509 (6,24) 1367 blocked 2534
//        8191^2 (60 sweeps)  (6,16) 2461 (6,24) 2279 blocked 2710
//       16383^2 (60 sweeps)  (6,16) 12161 (6,24) 10383 blocked 7193
struct Shape {
    int k, r;
};
Shape shape(int n, size_t elem_bytes) {
    if (elem_bytes == 8) {
        if (n <= 650) return {5, 4};
        return n <= 950 ? Shape{5, 8} : Shape{4, 16};
    }
    if (n <= 512) return {6, 4};
    if (n <= 800) return {6, 8};
    return n <= 1100 ? Shape{6, 16} : Shape{6, 24};
}

}  // namespace

// Where the windows are the choice (against the plain, resident and blocked
// kernels, MI355X): always up to 2300 (FP64; from 1600 and nine sweeps the row
// pipeline is the faster one) / 10000 (FP32), the figures above; beyond, calls of
// few sweeps, where the persistent kernel's ramp or two launches a sweep cost
// more (FP64 4095^2: 7 sweeps 341 us against 683; 8191^2: 8 sweeps 1341 against
// 1436; FP32 12287^2: 24 sweeps 2463 against 2788); not for one sweep of a
// large grid, which the half-sweeps do in fewer bytes (FP64 4095^2 243 against
// 223; FP32 12287^2 1248 against 1127).
bool window_takes(int n, size_t elem_bytes, int nsweeps) {
    if (pipeline_takes(n, elem_bytes, nsweeps)) return true;
    const bool f64 = elem_bytes == 8;
    if (nsweeps == 1) return n <= (f64 ? 3000 : 4500);
    if (n <= (f64 ? 2300 : 10000)) return true;
    return nsweeps <= (f64 ? 8 : 24);
}

int window_fuse(int n, size_t elem_bytes, int nsweeps) {
    return pipeline_takes(n, elem_bytes, nsweeps) ? pipeline_fuse(n) : shape(n, elem_bytes).k;
}

// A call's passes run at depth k or k - 1 where it has enough sweeps; depths
// below that (calls of a few sweeps) all take eight rows.
template <>
hipError_t launch_window<double>(const WindowArgs<double>& a, int sweeps, hipStream_t s) {
    if (a.deep) return launch_pipeline(a, sweeps, s);
    const int r = shape(a.n, 8).r;
    switch (sweeps) {
        case 1: return launch<double, 1, 8>(a, s);
        case 2: return launch<double, 2, 8>(a, s);
        case 3: return r == 16 ? launch<double, 3, 16>(a, s) : launch<double, 3, 8>(a, s);
        case 4:
            if (r == 4) return launch<double, 4, 4>(a, s);
            return r == 8 ? launch<double, 4, 8>(a, s) : launch<double, 4, 16>(a, s);
        case 5: return r == 4 ? launch<double, 5, 4>(a, s) : launch<double, 5, 8>(a, s);
    }
    return hipErrorInvalidValue;
}

template <int K>
hipError_t launch_rows(const WindowArgs<float>& a, int r, hipStream_t s) {
    if (r == 4) return launch<float, K, 4>(a, s);
    if (r == 8) return launch<float, K, 8>(a, s);
    return r == 16 ? launch<float, K, 16>(a, s) : launch<float, K, 24>(a, s);
}

template <>
hipError_t launch_window<float>(const WindowArgs<float>& a, int sweeps, hipStream_t s) {
    const int r = shape(a.n, 4).r;
    switch (sweeps) {
        case 1: return launch<float, 1, 8>(a, s);
        case 2: return launch<float, 2, 8>(a, s);
        case 3: return launch<float, 3, 8>(a, s);
        case 4: return launch<float, 4, 8>(a, s);
        case 5: return launch_rows<5>(a, r, s);
        case 6: return launch_rows<6>(a, r, s);
    }
    return hipErrorInvalidValue;
}

}  // namespace rbgs
