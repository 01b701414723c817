// Device side of the register windows (sweep_window.hip says how they work and
// what bounds them), shared by the kernels of one grid and of a batch.
#pragma once

#include <type_traits>

#include "rbgs_internal.h"

namespace rbgs {
namespace window_pass {

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

// Window w of a grid, numbered band by band in strips of R rows, the core
// columns of a window kCore wide (at most 64 - 2 K).
template <typename T, int K, int R, int kCore, bool SOR>
__device__ __forceinline__ void run_window(const WindowArgs<T>& a, int w) {
    const int strip = w / a.bands, band = w - strip * a.bands;
    const int base = strip * R - 2 * K;
    const int lane = int(threadIdx.x);
    const int first = band * kCore - K;
    const int q = first + lane;
    const bool core = lane >= K && lane < K + kCore && 2 * q <= a.n;
    const bool interior = base >= 1 && base + R + 4 * K - 1 <= a.n && first >= 1 &&
                          2 * (first + kLanes - 1) + 1 <= a.n;
    if (interior)
        window<T, K, R, false, SOR>(a, base, q, core);
    else
        window<T, K, R, true, SOR>(a, base, q, core);
}

constexpr int core_width(int k) { return kLanes - 2 * k; }

inline int window_bands(int n, int core) { return ((n >> 1) + 1 + core - 1) / core; }
inline int window_strips(int n, int r) { return (n + 1 + r - 1) / r; }

}  // namespace window_pass
}  // namespace rbgs
