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

// Whether the windows (or, pipeline_takes, the row pipeline) are the choice
// against the plain, resident and blocked kernels.  in_place: the sweeps have to
// end in the buffer they start from, which makes an odd number of passes one more,
// and shallower.  MI355X, us, here against the others:
//   one sweep of a large grid, which the half-sweeps do in fewer bytes, or in
//     place: FP64 4095^2 243 / 223; FP32 12287^2 1248 / 1127
//   two in place, as two passes: FP64 7001^2 0.93 of it, 8191^2 581 / 573, 12287^2
//     1266 / 1231; FP32 5001^2 0.95, 7001^2 1.06, 12287^2 703 / 636; SOR, whose
//     passes move red too, 1800^2 0.98, 4095^2 1.12
//   up to seven: all sizes (FP64 24575^2 x 7 11019 / 22153, FP32 32767^2 0.76)
//   FP64 up to 8000: always; beyond, up to 30 sweeps, until the ramp of the
//     persistent kernel no longer counts: x 9 8191^2 1250 / 1443, 12287^2 2764 /
//     2897, 15001^2 1.00, 16383^2 5144 / 4934, 24575^2 11446 / 10585; with a pass
//     more: x 16 12287^2 2716 / 3270, x 20 14001^2 1.03, x 30 8191^2 1759 / 2045,
//     12287^2 4006 / 3936, 14001^2 1.11
//   FP32: always up to 9200 (x 100 8191^2 3622 / 4076); above, passes of four
//     sweeps, which have short windows, cost too much (x 8 10001^2 1454 / 1360,
//     12287^2 2176 / 1890), and above 10000 so do more passes than the persistent
//     kernel takes (x 18 12287^2 2066 / 2405, x 20 2690 / 2504); 16383^2 x 12 3347
//     / 3098, x 24 5114 / 4265.  With a pass more: x 14, down to four and three
//     sweeps a pass, 4095^2 281 / 316, 5001^2 1.14, 12287^2 2363 / 1255; x 16
//     6001^2 1.03, 7001^2 0.79, 8191^2 1201 / 966; x 26 5001^2 0.99, 6001^2 1.07;
//     x 38 7001^2 0.79, 9001^2 1.16
bool window_takes(int n, size_t elem_bytes, int nsweeps, bool in_place, bool sor) {
    const bool f64 = elem_bytes == 8;
    if (nsweeps == 1) return !in_place && n <= (f64 ? 3000 : 4500);
    if (nsweeps == 2 && in_place) return n <= (sor ? 1900 : f64 ? 7500 : 5500);
    if (nsweeps < 8) return true;
    const int passes = window_passes(n, elem_bytes, nsweeps, in_place);
    const bool more = passes > window_passes(n, elem_bytes, nsweeps, false);
    if (f64) {
        const int most = !more ? 15500 : nsweeps <= 20 ? 13000 : 12000;
        return n <= 8000 || (nsweeps <= 30 && n <= most);
    }
    const int depth = nsweeps / passes;  // of the shallower passes
    if (more) {
        if (depth < 4) return n <= 4300;
        if (2 * int64_t(nsweeps) < 9 * int64_t(passes)) return n <= (passes <= 4 ? 7100 : 5500);
        return n <= 8200;
    }
    if (n <= 9200) return true;
    if (n <= 10000) return depth >= 5;
    return n <= 12500 && nsweeps <= 24 && depth >= 5 && passes <= (nsweeps + 6) / 7;
}

int window_passes(int n, size_t elem_bytes, int nsweeps, bool in_place) {
    const int k = window_fuse(n, elem_bytes, nsweeps);
    const int passes = nsweeps / k + (nsweeps % k ? 1 : 0);
    return in_place && (passes & 1) && nsweeps > passes ? passes + 1 : passes;
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
