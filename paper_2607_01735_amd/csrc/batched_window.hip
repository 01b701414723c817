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

// Windows against the persistent kernel, MI355X, us: 64 grids of 63 .. 1023,
// 100 sweeps FP32 1706 against 4178, FP64 3352 against 4650, 4 sweeps 405
// against 562 and 566 against 692, one sweep 389 against 517; 300 such grids
// FP32 30 sweeps 3303 against 5198; 8 grids of 2300^2 FP64 100 sweeps 5936
// against 6889, 4095^2 with two small ones 60 sweeps 1750 against 3577; 2 of
// 10000^2 FP32 60 sweeps 6550 against 7218.  Larger grids, where the
// persistent kernel's deeper passes gain on one grid too, keep it.  The
// shapes follow those of one grid of as many points.
bool batch_windows(int count, const int* n, size_t elem_bytes, int nsweeps, BatchWindows* b,
                   std::vector<int>* first, std::vector<int>* order) {
    double points = 0.0;
    for (int g = 0; g < count; ++g) {
        if (n[g] > (elem_bytes == 8 ? 4095 : 10000)) return false;
        points += double(n[g]) * n[g];
    }
    const int deepest = elem_bytes == 8 ? (points > 8e5 ? 4 : 5) : 6;
    b->count = count;
    b->passes = (nsweeps + deepest - 1) / deepest;
    b->top = (nsweeps + b->passes - 1) / b->passes;
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
        if (at > INT32_MAX / 2) return false;
    }
    b->windows = int(at);
    return true;
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
