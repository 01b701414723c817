// The register windows of sweep_window.hip over a batch of grids of uneven
// sizes: a pass is one launch over the windows of every grid, numbered grid by
// grid, largest first.  A workgroup (one wave) finds its grid by bisection in
// the table of first windows, scalar loads from cache.  64 grids of 63 ..
// 1023 in FP32 (19.7 million points) run at 1.2e12 point sweeps a second;
// tiles handed out by a queue, each waiting for its neighbours' pass, ran at
// 0.47e12.  Windows of one pass do
// not depend on one another, so there is no queue and nothing to wait for.
#include <algorithm>
#include <climits>

#include "blocked_pipeline.h"
#include "rbgs_blocked.h"
#include "rbgs_internal.h"
#include "sweep_window.h"

namespace rbgs {
namespace {

using namespace window_pass;

// first[k]: the first window of the k-th grid in order; grids[order[k]] is it.
// K <= TOP, the deepest pass of the call, whose core width numbers the windows.
template <typename T, int K, int TOP, int R>
__global__ __launch_bounds__(kLanes) void k_window_batch(const blocked::GridDesc<T>* __restrict__ grids,
                                                         const int* __restrict__ first,
                                                         const int* __restrict__ order, int count,
                                                         int buffer, int last) {
    const int w = int(blockIdx.x);
    int lo = 0, hi = count - 1;  // the last k with first[k] <= w
    while (lo < hi) {
        const int mid = (lo + hi + 1) >> 1;
        if (first[mid] <= w)
            lo = mid;
        else
            hi = mid - 1;
    }
    const blocked::GridDesc<T>& g = grids[order[lo]];
    WindowArgs<T> a;
    a.in[0] = g.red[buffer];
    a.in[1] = g.black[buffer];
    a.out[0] = g.red[1 - buffer];
    a.out[1] = g.black[1 - buffer];
    a.f[0] = g.f_red;
    a.f[1] = g.f_black;
    a.stop = nullptr;
    a.pitch = g.pitch;
    a.h2 = g.h2;
    a.omega = T(1);
    a.n = g.n;
    a.last = last;
    a.bands = ((g.n >> 1) + core_width(TOP)) / core_width(TOP);
    run_window<T, K, R, core_width(TOP), false>(a, w - first[lo]);
}

template <typename T, int TOP, int R>
hipError_t launch(const BatchWindows& b, const blocked::GridDesc<T>* g, const int* first,
                  const int* order, int k, int buffer, bool last, hipStream_t s) {
    const dim3 grid{unsigned(b.windows)};
    if (k == TOP)
        hipLaunchKernelGGL((k_window_batch<T, TOP, TOP, R>), grid, dim3(kLanes), 0, s, g, first, order,
                           b.count, buffer, int(last));
    else if constexpr (TOP > 1)
        hipLaunchKernelGGL((k_window_batch<T, TOP - 1, TOP, R>), grid, dim3(kLanes), 0, s, g, first,
                           order, b.count, buffer, int(last));
    return hipGetLastError();
}

template <typename T, int R>
hipError_t launch_top(const BatchWindows& b, const blocked::GridDesc<T>* g, const int* first,
                      const int* order, int k, int buffer, bool last, hipStream_t s) {
    switch (b.top) {
        case 1: return launch<T, 1, 8>(b, g, first, order, k, buffer, last, s);
        case 2: return launch<T, 2, 8>(b, g, first, order, k, buffer, last, s);
        case 3: return launch<T, 3, 8>(b, g, first, order, k, buffer, last, s);
        case 4: return launch<T, 4, R>(b, g, first, order, k, buffer, last, s);
        case 5: return launch<T, 5, R>(b, g, first, order, k, buffer, last, s);
        case 6:
            if constexpr (sizeof(T) == 4) return launch<T, 6, R>(b, g, first, order, k, buffer, last, s);
    }
    return hipErrorInvalidValue;
}

}  // namespace

// The split of a batch into passes and windows.  The shapes follow those of one
// grid of as many points.
bool batch_windows(int count, const int* n, size_t elem_bytes, int nsweeps, BatchWindows* b,
                   std::vector<int>* first, std::vector<int>* order) {
    double points = 0.0;
    for (int g = 0; g < count; ++g) points += double(n[g]) * n[g];
    const int deepest = batch_deepest(count, n, elem_bytes);
    b->count = count;
    b->nsweeps = nsweeps;
    b->passes = (nsweeps - 1) / deepest + 1;
    b->top = (nsweeps - 1) / b->passes + 1;
    const int tall = elem_bytes == 8 ? 16 : 24;
    b->rows = b->top <= 3 ? 8 : points > (elem_bytes == 8 ? 8e5 : 2e6) ? tall : 8;
    order->resize(size_t(count));
    for (int g = 0; g < count; ++g) (*order)[size_t(g)] = g;
    std::stable_sort(order->begin(), order->end(), [&](int x, int y) { return n[x] > n[y]; });
    int64_t at = 0;
    first->resize(size_t(count));
    for (int k = 0; k < count; ++k) {
        (*first)[size_t(k)] = int(at);
        const int m = n[(*order)[size_t(k)]];
        at += int64_t(window_bands(m, core_width(b->top))) * window_strips(m, b->rows);
        if (at > INT32_MAX / kLanes) return false;  // threads of a launch
    }
    b->windows = int(at);
    return true;
}

int batch_deepest(int count, const int* n, size_t elem_bytes) {
    if (elem_bytes != 8) return 6;
    double points = 0.0;
    for (int g = 0; g < count; ++g) points += double(n[g]) * n[g];
    return points > 8e5 ? 4 : 5;
}

// Windows against the persistent kernel at its default shape, MI355X, us: 64 grids
// of 63 .. 1023, 100 sweeps FP32 1706 against 4178, FP64 3352 against 4650, 4
// sweeps 405 against 562 and 566 against 692, one sweep 389 against 517; 4095^2
// with two small ones FP64 60 sweeps 1750 against 3577; 2 of 10000^2 FP32 100 sweeps
// 10038 against 10635.  Above 4095 (FP64) / 10000 (FP32) the persistent kernel's
// deeper passes gain on one grid too.
// FP64 batches of several large grids: the persistent kernel moves less once its
// tiles fill the chip, which the windows, a pass every four sweeps, do not make up
// in long calls.  Measured, 8 of 4095^2: 20 sweeps 4953 windows, 4694 persistent,
// 100 sweeps 17898 and 14487; 16 of 3500^2, 10 sweeps 1.07, 100 1.42; 16 of 2300^2 20
// sweeps 3235 and 3300, 100 11537 and 9809; 4 of 4095^2 20 2515 and 2763, 100 9113
// and 7990; 8 of 2300^2 100 5933 and 6900; 48 of 1800^2 (a last strip of 8 rows) 50
// 0.98, 100 1.02.  The rule compares
//   windows      5 us per million points and pass
//   persistent   400 us of ramp more, and 0.355 us per tile of 256 rows and pass (the
//                28 halo rows are rows too; a pass below depth 7, 0.65 + 0.05 depth
//                of it), for at least 1250 tiles, which is when the chip is full
// and so takes the faster one, or one within 3% of it, in 159 of the 165 calls timed
// (30 batches with grids of 1600^2 .. 4095^2, 1 to 100 sweeps), and is 6% off at worst.
// FP32: 3 of 8191^2 x 14, which the persistent kernel does in two passes of seven,
// 3156 and 2888, 3 of 10000^2 4744 and 4097; x 20 to 100 0.81 to 1.02 but for 8 of
// 6000^2, 100 sweeps 18178 and 16194 (the autotuner times both).
bool batch_windows_pay(int count, const int* n, size_t elem_bytes, int nsweeps) {
    const bool f64 = elem_bytes == 8;
    int most = 0;
    double points = 0.0;
    for (int g = 0; g < count; ++g) {
        most = std::max(most, n[g]);
        points += double(n[g]) * n[g];
    }
    if (most > (f64 ? 4095 : 10000)) return false;
    constexpr int fuse = 7;  // of the persistent kernel, where the largest grid has 1536
    if (default_fuse(int(elem_bytes), most) != fuse) return true;
    double tiles = 0.0;
    for (int g = 0; g < count; ++g) {
        const int rows = default_rows(n[g], 2 * fuse);
        tiles += double(geometry(n[g], int(elem_bytes), fuse, rows).ntiles) * (rows + 4 * fuse) /
                 (256 + 4 * fuse);
    }
    if (!f64) return !(nsweeps == 2 * fuse && most > 7000 && tiles >= 1700.0);
    const int rest = nsweeps % fuse;
    const double passes = nsweeps / fuse + (rest ? 0.65 + 0.05 * rest : 0.0);
    const double windows = 5e-6 * points * ((nsweeps - 1) / batch_deepest(count, n, elem_bytes) + 1);
    return windows <= 400.0 + 0.355 * std::max(tiles, 1250.0) * passes;
}

template <typename T>
hipError_t launch_batch_pass(const BatchWindows& b, const void* grids, const int* first,
                             const int* order, int pass, hipStream_t s) {
    const blocked::GridDesc<T>* g = static_cast<const blocked::GridDesc<T>*>(grids);
    const int k = b.nsweeps / b.passes + (pass < b.nsweeps % b.passes ? 1 : 0);
    const bool last = pass == b.passes - 1;
    constexpr int kTall = sizeof(T) == 8 ? 16 : 24;
    return b.rows == 8 ? launch_top<T, 8>(b, g, first, order, k, pass & 1, last, s)
                       : launch_top<T, kTall>(b, g, first, order, k, pass & 1, last, s);
}

template hipError_t launch_batch_pass<float>(const BatchWindows&, const void*, const int*, const int*,
                                             int, hipStream_t);
template hipError_t launch_batch_pass<double>(const BatchWindows&, const void*, const int*, const int*,
                                              int, hipStream_t);

}  // namespace rbgs
