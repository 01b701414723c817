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
#include <type_traits>

#include "rbgs_internal.h"

namespace rbgs {
namespace {

constexpr int kLanes = 64;

template <int N>
using IC = std::integral_constant<int, N>;

template <int B, int E, typename F>
__device__ __forceinline__ void static_for(F&& f) {
    if constexpr (B < E) {
        f(IC<B>{});
        static_for<B + 1, E>(f);
    }
}

template <int CTRL>
__device__ __forceinline__ double lane_shift(double v) {
    const int lo = __builtin_amdgcn_mov_dpp(__double2loint(v), CTRL, 0xf, 0xf, true);
    const int hi = __builtin_amdgcn_mov_dpp(__double2hiint(v), CTRL, 0xf, 0xf, true);
    return __hiloint2double(hi, lo);
}
template <int CTRL>
__device__ __forceinline__ float lane_shift(float v) {
    return __int_as_float(__builtin_amdgcn_mov_dpp(__float_as_int(v), CTRL, 0xf, 0xf, true));
}
// lane i receives lane i + 1's / i - 1's value (the end lane 0: it is halo)
template <typename T>
__device__ __forceinline__ T next(T v) { return lane_shift<0x130>(v); }
template <typename T>
__device__ __forceinline__ T prev(T v) { return lane_shift<0x138>(v); }

typedef __attribute__((address_space(1))) char gchar;

// The element at byte offset `bytes` (wave-uniform) + `lane` of p, as a global
// access with a scalar base and a 32-bit vector offset (the empty asm keeps the
// compiler from forming 64-bit vector addresses).
template <typename T>
__device__ __forceinline__ auto element(const T* p, int64_t bytes, uint32_t lane) {
    typedef __attribute__((address_space(1))) T gelem;
    gchar* g = (gchar*)(reinterpret_cast<uintptr_t>(p) + uintptr_t(bytes));
    asm("" : "+s"(g), "+v"(lane));
    return (gelem*)(g + lane);
}

// m ? a : b bitwise, m 0 or ~0 (a conditional becomes a branch around a)
__device__ __forceinline__ float blend(uint32_t m, float a, float b) {
    return __uint_as_float((m & __float_as_uint(a)) | (~m & __float_as_uint(b)));
}
__device__ __forceinline__ double blend(uint32_t m, double a, double b) {
    const uint32_t lo = (m & uint32_t(__double2loint(a))) | (~m & uint32_t(__double2loint(b)));
    const uint32_t hi = (m & uint32_t(__double2hiint(a))) | (~m & uint32_t(__double2hiint(b)));
    return __hiloint2double(int(hi), int(lo));
}

// EDGE: the window holds points of the ring.
// SOR: u <- u + omega (g - u), each operation rounded once; red is then read
// and written by every pass.
template <typename T, int K, int R, bool EDGE, bool SOR>
__device__ __forceinline__ void window(const WindowArgs<T>& a, int base, int q, bool core) {
    constexpr int W = R + 4 * K;
    const int n = a.n;
    const uint32_t qb = uint32_t(q < 0 ? 0 : (q < int(a.pitch) ? q : int(a.pitch) - 1)) *
                        uint32_t(sizeof(T));
    T u[2][W], hf[2][W];  // red, black by window row (row i = base + r, base even)
    // rows outside the grid are clamped into it: they reach only rows that are
    // not written
    auto row = [&](int r, int lo, int hi) {
        const int i = base + r;
        return int64_t(i < lo ? lo : (i > hi ? hi : i)) * (a.pitch * int64_t(sizeof(T)));
    };
#pragma unroll
    for (int r = 0; r < W; ++r) {
        u[1][r] = *element(a.in[1], row(r, 0, n + 1), qb);
        u[0][r] = EDGE || SOR ? *element(a.in[0], row(r, 0, n + 1), qb) : T(0);
        hf[0][r] = *element(a.f[0], row(r, 1, n), qb);
        hf[1][r] = *element(a.f[1], row(r, 1, n), qb);
    }
    __builtin_amdgcn_sched_barrier(0);  // all loads first
#pragma unroll
    for (int r = 0; r < W; ++r) {
        hf[0][r] = a.h2 * hf[0][r];
        hf[1][r] = a.h2 * hf[1][r];
    }
    // columns 0 and n + 1 by the parity p of a point's column
    const uint64_t ring_rows = (base <= 0 && base > -W ? uint64_t(1) << -base : 0) |
                               (n + 1 >= base && n + 1 < base + W ? uint64_t(1) << (n + 1 - base) : 0);
    const bool ring[2] = {q == 0 || 2 * q == n + 1, 2 * q + 1 == n + 1};
    const uint32_t ring_mask[2] = {ring[0] ? ~0u : 0u, ring[1] ? ~0u : 0u};
    static_for<0, 2 * K>([&](auto lc) {
        constexpr int l = decltype(lc)::value;
        constexpr int c = l & 1;
        T (&self)[W] = u[c];
        const T (&o)[W] = u[1 - c];
        static_for<l + 1, W - 1 - l>([&](auto rc) {
            constexpr int r = decltype(rc)::value;
            constexpr int p = (r + c) & 1;
            const T right = p ? next(o[r]) : o[r];
            const T left = p ? o[r] : prev(o[r]);
            T s = o[r + 1] + o[r - 1];
            s = s + right;
            s = s + left;
            s = s - hf[c][r];
            T v = T(0.25) * s;
            if constexpr (SOR) {
                const T d = v - self[r];
                const T w = a.omega * d;
                v = self[r] + w;
            }
            if constexpr (EDGE) {
                const uint32_t row_mask = ((ring_rows >> r) & 1) != 0 ? ~0u : 0u;
                self[r] = blend(ring_mask[p] | row_mask, self[r], v);
            } else {
                self[r] = v;
            }
        });
    });
    if (!core) return;
    static_for<0, R>([&](auto rc) {
        constexpr int r = 2 * K + decltype(rc)::value;
        const int i = base + r;
        if (i < 1 || i > n) return;
        const int64_t at = int64_t(i) * (a.pitch * int64_t(sizeof(T)));
        constexpr int p = (r + 1) & 1;  // black's
        if (!EDGE || (!ring[p] && 2 * q + p <= n)) *element(a.out[1], at, qb) = u[1][r];
        if ((SOR || a.last) && (!EDGE || (!ring[1 - p] && 2 * q + 1 - p <= n)))
            *element(a.out[0], at, qb) = u[0][r];
    });
}

template <typename T, int K, int R, bool SOR>
__global__ __launch_bounds__(kLanes) void k_window(WindowArgs<T> a) {
    if (a.stop && *a.stop) return;
    constexpr int kCore = kLanes - 2 * K;
    const int strip = int(blockIdx.x) / a.bands, band = int(blockIdx.x) - strip * a.bands;
    const int base = strip * R - 2 * K;
    const int lane = int(threadIdx.x);
    const int first = band * kCore - K;
    const int q = first + lane;
    const bool core = lane >= K && lane < kLanes - K && 2 * q <= a.n;
    const bool interior = base >= 1 && base + R + 4 * K - 1 <= a.n && first >= 1 &&
                          2 * (first + kLanes - 1) + 1 <= a.n;
    if (interior)
        window<T, K, R, false, SOR>(a, base, q, core);
    else
        window<T, K, R, true, SOR>(a, base, q, core);
}

template <typename T, int K, int R>
hipError_t launch(WindowArgs<T> a, hipStream_t s) {
    constexpr int kCore = kLanes - 2 * K;
    a.bands = ((a.n >> 1) + 1 + kCore - 1) / kCore;
    const dim3 grid(unsigned(a.bands * ((a.n + 1 + R - 1) / R)));
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
// kernels, MI355X): always up to 2300 (FP64) / 10000 (FP32), the figures above;
// beyond, calls of few sweeps, where the persistent kernel's ramp or two
// launches a sweep cost more (FP64 4095^2: 7 sweeps 341 us against 683, 24
// sweeps 704 against 757; 8191^2: 8 sweeps 1341 against 1436, 10 sweeps 1549
// against 1475; FP32 12287^2: 24 sweeps 2463 against 2788); not for one sweep
// of a large grid, which the half-sweeps do in fewer bytes (FP64 4095^2 243
// against 223; FP32 12287^2 1248 against 1127).
bool window_takes(int n, size_t elem_bytes, int nsweeps) {
    const bool f64 = elem_bytes == 8;
    if (nsweeps == 1) return n <= (f64 ? 3000 : 4500);
    if (n <= (f64 ? 2300 : 10000)) return true;
    return nsweeps <= (f64 && n > 4500 ? 8 : 24);
}

int window_fuse(int n, size_t elem_bytes) { return shape(n, elem_bytes).k; }

// A call's passes run at depth k or k - 1 where it has enough sweeps; depths
// below that (calls of a few sweeps) all take eight rows.
template <>
hipError_t launch_window<double>(const WindowArgs<double>& a, int sweeps, hipStream_t s) {
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
