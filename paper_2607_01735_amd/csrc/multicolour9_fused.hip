// Several four-colour sweeps of the 9-point system in one pass over the grid.
//
// A launch per colour (multicolour9.hip) moves 40 B per grid point and sweep:
// every quarter-sweep streams three colours, its own f and its own colour.
// Here a wave marches down a strip of colour rows with K sweeps pipelined in
// registers, so a pass reads colours 1, 2, 3 and f once and writes colours
// 1, 2, 3 once (20 B per point; colour 0 is recomputed from the others before
// anything reads it and is written by the last pass only): 6.7 B per point
// and sweep at K = 3.
//
// Pair t of rows is rows 2t (colours 0, 2) and 2t + 1 (colours 1, 3).  At
// step t sweep s works around pair P = t - 2 s:
//   colour 0 of pair P      from colours 1, 3 of P - 1, P and 2 of P (before),
//   colour 1 of pair P - 1  from colour 0 of P - 1, P (new), 2 of P - 1, P and
//                           3 of P - 1 (before),
//   colour 2 of pair P - 1  from colour 0 of P - 1, 1 of P - 2, P - 1 (new) and
//                           3 of P - 2, P - 1 (before),
//   colour 3 of pair P - 2  from colours 0, 2 of P - 2, P - 1 and 1 of P - 2;
// pair P - 2 is then complete and enters sweep s + 1.  The rows that a level
// needs later stay in registers, and so do the products c6 f (each formed
// once).  A lane holds one column of each colour (64 columns of the colour
// arrays, 8-byte loads); the neighbours at J - 1 and J + 1 come through DPP
// lane shifts.  Tiles overlap by K columns a side (colours 0, 1 need J - 1 and
// colours 2, 3 need J + 1, so a sweep spoils one column a side) and 2 K pairs
// above and below, which are recomputed and not written; a pass reads one
// buffer and writes the other, so tiles are independent.
//
// 50 sweeps at 4001^2: 5.13 ms with a launch per colour, 1.54 here; a pass of
// three sweeps takes 87 us and moves 426 MB by the counters (4.9 TB/s; 320 MB
// without the columns and pairs that tiles share), two waves a SIMD, which issue in
// 41% of their cycles.  What bounds it is the serial chain of twelve levels a step
// and the bytes in flight, not the 148 FP64 instructions a step (a third of the
// time).
//
// Each point's operations and their order are k_mc9_quarter's; the division
// by 20 is div20 below, which gives the same bits.
#include <type_traits>

#include "rbgs_internal.h"

namespace rbgs {
namespace {

constexpr int kLanes = 64;
constexpr int kPrefetch = 2;            // pairs loaded ahead of their use
constexpr int kSimds = 256 * 4;         // of the chip: CUs x 4

constexpr int pmod(int a, int m) { return ((a % m) + m) % m; }

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
// lane i receives lane i + 1's / i - 1's value (the end lane 0: it is halo)
__device__ __forceinline__ double next(double v) { return lane_shift<0x130>(v); }
__device__ __forceinline__ double prev(double v) { return lane_shift<0x138>(v); }

// s / 20, correctly rounded, by multiplication.  q = s * RN(1/20) is within
// one unit in the last place (RN(1/20) is off by 2^-54 relative),
// r = 20 q - s is exact in one FMA, and RN(q - r RN(1/20)) is then the rounded
// quotient (Markstein, "Computation of elementary functions on the IBM RISC
// System/6000 processor", 1990, Theorem 8) unless it is subnormal (a tie may
// go the wrong way) or s is infinite or NaN (the result is NaN).  Those raise
// `odd`, and the tile is computed again with the division itself.  Signed
// zeros come out right.  EXACT: the division.
template <bool EXACT>
__device__ __forceinline__ double div20(double s) {
    if constexpr (EXACT) return s / 20.0;
    const double rcp = 1.0 / 20.0;
    const double q = s * rcp;
    const double r = __builtin_fma(20.0, q, -s);
    return __builtin_fma(-r, rcp, q);
}

// NaN or subnormal (class bits: signalling and quiet NaN, the subnormals)
__device__ __forceinline__ bool odd_class(double v) {
    return __builtin_amdgcn_class(v, 0x001 | 0x002 | 0x010 | 0x080);
}

template <bool EDGE>
struct In {
    double c0, c1, c2, c3, f0, f1, f2, f3;
};

// Ring length of the row registers: steps unrolled, so that every index is a
// constant.  A product c6 f lives for 2 K - 1 steps.
template <int K>
constexpr int unroll() { return K < 2 ? 4 : 2 * K; }

template <int K, bool EDGE>
struct State {
    static constexpr int U = unroll<K>();
    double v[K + 1][4][U];  // v[s][c]: colour c before sweep s, by pair (slot pair mod U)
    double f[4][U];         // c6 f
    In<EDGE> in[U];
    int64_t row[U];         // row offsets, by pair
};

struct Tile {
    uint32_t jb;    // byte offset in a row of the column loaded (clamped into it)
    int J, p0, p1;  // column, first and last pair written
    bool core;      // this lane's column is written
    // the ring's last row or column n + 1 as a pair or J of the even colours
    // (n odd) or of the odd ones (n even), else -1; and whether this lane's
    // even and odd column is off the ring
    int ring_even, ring_odd;
    bool even_in, odd_in;
};

__device__ __forceinline__ int64_t clampi(int64_t x, int64_t lo, int64_t hi) {
    return x < lo ? lo : (x > hi ? hi : x);
}

// Byte offset of a pair's row.  Rows outside the arrays are clamped into
// them: they reach only pairs that are not written.
__device__ __forceinline__ int64_t row_offset(const Mc9PassArgs& a, int pair) {
    return int64_t(pair < 0 ? 0 : (pair < a.rows ? pair : a.rows - 1)) * (a.pitch * 8);
}

// The inputs of step t from the row offsets of pairs t, t - 1, t - 2 (scalar
// bases, 32-bit lane offset).
template <bool EDGE>
__device__ __forceinline__ In<EDGE> load_in(const Mc9PassArgs& a, const Tile& g, int64_t r0,
                                            int64_t r1, int64_t r2) {
    auto at = [&](const double* p, int64_t row) {
        return *reinterpret_cast<const double*>(reinterpret_cast<const char*>(p) + row + g.jb);
    };
    In<EDGE> in;
    in.c1 = at(a.in[1], r0);
    in.c2 = at(a.in[2], r0);
    in.c3 = at(a.in[3], r0);
    in.c0 = EDGE ? at(a.in[0], r0) : 0.0;  // ring values only
    in.f0 = at(a.f[0], r0);
    in.f1 = at(a.f[1], r1);
    in.f2 = at(a.f[2], r1);
    in.f3 = at(a.f[3], r2);
    return in;
}

template <bool EXACT>
__device__ __forceinline__ double update(double ns_dn, double ns_up, double ew_e, double ew_w,
                                         double dn_e, double dn_w, double up_e, double up_w,
                                         double t) {
    double e = ns_dn + ns_up;
    e = e + ew_e;
    e = e + ew_w;
    double c = dn_e + dn_w;
    c = c + up_e;
    c = c + up_w;
    double s = 4.0 * e + c;
    s = s - t;
    return div20<EXACT>(s);
}

template <int K, bool EDGE, bool EXACT, int S>
__device__ __forceinline__ void step(State<K, EDGE>& st, const Mc9PassArgs& a, const Tile& g,
                                     int t, bool& odd) {
    constexpr int U = unroll<K>();
    const In<EDGE> cur = st.in[S];
    constexpr int A = (S + kPrefetch) % U;
    st.row[A] = row_offset(a, t + kPrefetch);
    st.in[A] = load_in<EDGE>(a, g, st.row[A], st.row[pmod(A - 1, U)], st.row[pmod(A - 2, U)]);
    st.v[0][0][S] = cur.c0;
    st.v[0][1][S] = cur.c1;
    st.v[0][2][S] = cur.c2;
    st.v[0][3][S] = cur.c3;
    st.f[0][S] = a.c6 * cur.f0;
    st.f[1][pmod(S - 1, U)] = a.c6 * cur.f1;
    st.f[2][pmod(S - 1, U)] = a.c6 * cur.f2;
    st.f[3][pmod(S - 2, U)] = a.c6 * cur.f3;
    static_for<0, K>([&](auto sc) {
        constexpr int s = decltype(sc)::value;
        constexpr int P0 = pmod(S - 2 * s, U), P1 = pmod(S - 2 * s - 1, U), P2 = pmod(S - 2 * s - 2, U);
        const int P = t - 2 * s;
        auto& o = st.v[s];      // before this sweep
        auto& w = st.v[s + 1];  // after it
        // ring points keep their value (points beyond the ring reach no point
        // that is written); row_in is wave-uniform
        auto keep = [&](double v, double old, bool row_in, bool col_in) {
            const bool in = !EDGE || (row_in && col_in);
            if constexpr (!EXACT) odd = odd || (in && odd_class(v));
            return EDGE ? (in ? v : old) : v;
        };
        const bool r0 = P != 0 && P != g.ring_even, r1 = P - 1 != g.ring_odd;
        const bool r2 = P - 1 != 0 && P - 1 != g.ring_even, r3 = P - 2 != g.ring_odd;
        w[0][P0] = keep(update<EXACT>(o[1][P0], o[1][P1], o[2][P0], prev(o[2][P0]), o[3][P0],
                               prev(o[3][P0]), o[3][P1], prev(o[3][P1]), st.f[0][P0]),
                        o[0][P0], r0, g.even_in);
        w[1][P1] = keep(update<EXACT>(w[0][P0], w[0][P1], o[3][P1], prev(o[3][P1]), o[2][P0],
                               prev(o[2][P0]), o[2][P1], prev(o[2][P1]), st.f[1][P1]),
                        o[1][P1], r1, g.even_in);
        w[2][P1] = keep(update<EXACT>(o[3][P1], o[3][P2], next(w[0][P1]), w[0][P1], next(w[1][P1]),
                               w[1][P1], next(w[1][P2]), w[1][P2], st.f[2][P1]),
                        o[2][P1], r2, g.odd_in);
        w[3][P2] = keep(update<EXACT>(w[2][P1], w[2][P2], next(w[1][P2]), w[1][P2], next(w[0][P1]),
                               w[0][P1], next(w[0][P2]), w[0][P2], st.f[3][P2]),
                        o[3][P2], r3, g.odd_in);
    });
    const int pair = t - 2 * K;
    if (pair >= g.p0 && pair <= g.p1 && g.core) {
        constexpr int D = pmod(S - 2 * K, U);
        const int64_t row = int64_t(pair) * a.pitch;
        const bool even_row = !EDGE || (pair != 0 && pair != g.ring_even);
        const bool odd_row = !EDGE || pair != g.ring_odd;
        const bool even_col = !EDGE || g.even_in, odd_col = !EDGE || g.odd_in;
        // n odd: the pair (column) of the ring's last row (column) has no odd row
        const bool beyond_row = EDGE && pair == g.ring_even, beyond_col = EDGE && g.J == g.ring_even;
        auto store = [&](double* rowp, double v) {
            *reinterpret_cast<double*>(reinterpret_cast<char*>(rowp) + g.jb) = v;
        };
        if (a.last && even_row && even_col) store(a.out[0] + row, st.v[K][0][D]);
        if (odd_row && even_col && !beyond_row) store(a.out[1] + row, st.v[K][1][D]);
        if (even_row && odd_col && !beyond_col) store(a.out[2] + row, st.v[K][2][D]);
        if (odd_row && odd_col && !beyond_row && !beyond_col) store(a.out[3] + row, st.v[K][3][D]);
    }
}

// Steps S .. U - 1 from step t; false after the last one.  (Leaving between
// steps keeps no register of a step not taken alive, as a branch around each
// step would.)
template <int K, bool EDGE, bool EXACT, int S>
__device__ __forceinline__ bool steps(State<K, EDGE>& st, const Mc9PassArgs& a, const Tile& g,
                                      int t, int t_last, bool& odd) {
    step<K, EDGE, EXACT, S>(st, a, g, t + S, odd);
    if (t + S >= t_last) return false;
    if constexpr (S + 1 < unroll<K>())
        return steps<K, EDGE, EXACT, S + 1>(st, a, g, t, t_last, odd);
    else
        return true;
}

// Returns whether a point of this lane wants the division itself.
template <int K, bool EDGE, bool EXACT>
__device__ __forceinline__ bool march(const Mc9PassArgs& a, const Tile& g, int t0, int t_last) {
    constexpr int U = unroll<K>();
    State<K, EDGE> st;
#pragma unroll
    for (int k = 0; k < U; ++k) {
#pragma unroll
        for (int s = 0; s <= K; ++s)
            st.v[s][0][k] = st.v[s][1][k] = st.v[s][2][k] = st.v[s][3][k] = 0.0;
        st.f[0][k] = st.f[1][k] = st.f[2][k] = st.f[3][k] = 0.0;
    }
#pragma unroll
    for (int d = -2; d < kPrefetch; ++d) st.row[pmod(d, U)] = row_offset(a, t0 + d);
#pragma unroll
    for (int d = 0; d < kPrefetch; ++d)
        st.in[d] = load_in<EDGE>(a, g, st.row[d], st.row[pmod(d - 1, U)], st.row[pmod(d - 2, U)]);
    bool odd = false;
    for (int t = t0; steps<K, EDGE, EXACT, 0>(st, a, g, t, t_last, odd); t += U) {
    }
    return odd;
}

template <int K>
__global__ __launch_bounds__(kLanes, 2) void k_mc9_pass(Mc9PassArgs a) {
    if (a.stop && *a.stop) return;
    constexpr int core = kLanes - 2 * K;
    const int tile = xcd_logical_block(int(blockIdx.x), int(gridDim.x));
    const int strip = tile / a.bands, band = tile - strip * a.bands;
    const int lane = int(threadIdx.x);
    Tile g;
    g.p0 = strip * a.pairs;
    g.p1 = g.p0 + a.pairs - 1 < a.rows - 1 ? g.p0 + a.pairs - 1 : a.rows - 1;
    const int first = band * core - K;  // first column loaded
    g.J = first + lane;
    g.jb = uint32_t(clampi(g.J, 0, a.pitch - 1)) * 8u;
    g.core = lane >= K && lane < kLanes - K && 2 * g.J <= a.n;
    g.ring_even = (a.n & 1) ? (a.n + 1) >> 1 : -1;
    g.ring_odd = (a.n & 1) ? -1 : a.n >> 1;
    g.even_in = g.J != 0 && g.J != g.ring_even;
    g.odd_in = g.J != g.ring_odd;
    const int t0 = g.p0 - 2 * K > 0 ? g.p0 - 2 * K : 0;
    const int t_last = g.p1 + 2 * K;
    const bool interior = g.p0 - 2 * K >= 1 && 2 * t_last + 1 <= a.n && first >= 1 &&
                          2 * (first + kLanes - 1) + 1 <= a.n;
    // tiles at the ring divide (they would not fit the register file beside
    // both the ring's selects and the check)
    if (!interior || __builtin_expect(__any(march<K, false, false>(a, g, t0, t_last)), 0))
        march<K, true, true>(a, g, t0, t_last);
}

// Pairs a strip: as few as leave all tiles resident at once, with one or two
// waves per SIMD.  A strip takes pairs + 4 K steps, and two waves on a SIMD
// take about 1.5 times as long as one (60 sweeps of 1023^2 at two a pass: 387
// us with 6 pairs, 774 tiles; 466 with 4, 1152 tiles; 2047^2: 788 with 12,
// 1548 tiles; 834 with 16, 1152 tiles).  Where one round would need strips
// above 48 pairs, several rounds of 32 (8191^2, 12 sweeps: 2.13 ms against
// 2.24 with 160 pairs in one round, 2.38 with 142, a few tiles over).  A
// single sweep holds half the registers, four waves per SIMD, and wants the
// bytes in flight (4001^2: 68 us a pass with 16 pairs, 74 with 40).
int pass_pairs(int rows, int bands, int sweeps) {
    auto fit = [&](int waves) {
        const int strips = waves / bands > 1 ? waves / bands : 1;
        const int p = (rows + strips - 1) / strips;
        return p > 2 ? p : 2;
    };
    if (sweeps == 1) {
        const int p = fit(4 * kSimds);
        return p <= 16 ? p : 16;
    }
    const int one = fit(kSimds), two = fit(2 * kSimds);
    const int p = 2 * (one + 4 * sweeps) <= 3 * (two + 4 * sweeps) ? one : two;
    return p <= 48 ? p : 32;
}

}  // namespace

// Three sweeps a pass are the fewest bytes per sweep that fit the registers
// (four spill); small grids are bound by the steps of a strip, of which a
// sweep adds four, and by launches.  Measured on MI355X, 60 sweeps: 255^2
// 271 us at two a pass, 316 at three, 326 at one; 2047^2 788, 818 and 1125;
// 4001^2 (50 sweeps) 2.03 ms at two and 1.62 at three, 1.54 since the ring is
// packed with u.
int mc9_fuse(int n) { return n < 3000 ? 2 : 3; }

hipError_t launch_mc9_pass(double* const in[4], double* const out[4], double* const f[4], int n,
                           double c6, int sweeps, bool last, const int* stop, hipStream_t s) {
    if (sweeps < 1 || sweeps > kMc9MaxFuse) return hipErrorInvalidValue;
    Mc9PassArgs a;
    for (int c = 0; c < 4; ++c) {
        a.in[c] = in[c];
        a.out[c] = out[c];
        a.f[c] = f[c];
    }
    a.n = n;
    a.pitch = mc9_pitch(n);
    a.rows = mc9_rows(n);
    a.c6 = c6;
    a.last = last;
    a.stop = stop;
    const int core = kLanes - 2 * sweeps;
    a.bands = ((n >> 1) + 1 + core - 1) / core;
    a.pairs = pass_pairs(a.rows, a.bands, sweeps);
    const dim3 grid(unsigned(a.bands) * unsigned((a.rows + a.pairs - 1) / a.pairs));
    switch (sweeps) {
        case 1: hipLaunchKernelGGL(k_mc9_pass<1>, grid, dim3(kLanes), 0, s, a); break;
        case 2: hipLaunchKernelGGL(k_mc9_pass<2>, grid, dim3(kLanes), 0, s, a); break;
        default: hipLaunchKernelGGL(k_mc9_pass<3>, grid, dim3(kLanes), 0, s, a); break;
    }
    return hipGetLastError();
}

}  // namespace rbgs
