// Fused legs of the multigrid cycle on split (red/black) FP64 arrays.
//
// A level's half of the V-cycle is one pass over the level instead of one
// launch per half-sweep and transfer:
//   down: NU red-black sweeps (Eq. (1)), the residual, its full weighting
//         onto the coarse right-hand side;
//   up:   the interpolant added to black, NU sweeps, and on the finest level
//         optionally the sum of squares of the residual that follows.
// The launch-per-step cycle moves 133 B per fine point of a V(2,2) cycle
// with its residual check (48 + 20 down, 13 + 36 + 16 up); these passes move
// 18 down (black and f read, black and the coarse right-hand side written;
// 14 on a coarse level, whose iterate starts at zero and is not read) and 22
// up.  Each point's operations and their order are those of the single
// kernels (sweep_plain.hip, multigrid.hip, residual.hip), so the iterate is
// the same bit for bit.
//
// A wave takes a tile: 128 split columns (two per lane, 16-byte loads) by a
// strip of rows.  Levels l = 0 .. L-1 (L = 2 NU half-sweeps) are pipelined
// down the strip in registers: at input row x level l updates row x - 1 - l
// from the three rows that level l - 1 produced last, and the residual of
// row x - 1 - L follows from the last two levels' rows.  Every input is read
// once per pass; horizontal neighbours come through DPP lane shifts; f rows
// stay in registers for the later levels.  Tiles overlap: rows and columns
// next to the core are recomputed (4 split columns and L + 1 rows a side)
// and not written, so tiles are independent and need no flags.  Input and
// output buffers differ (down: first to second, up: second to first), so no
// tile reads what another writes.
//
// Only black crosses between the legs: the first red half-sweep of either
// leg overwrites every red value without reading it.
#include "rbgs_internal.h"

namespace rbgs {
namespace {

constexpr int kLanes = 64;
constexpr int kHalo = 4;                    // split columns a side (even)
constexpr int kCore = 2 * kLanes - 2 * kHalo;
constexpr int kPrefetch = 2;                // rows loaded ahead of their use (1 and 3 ran alike)
constexpr int kLegWaves = 256 * 4 * 2;      // resident waves: CUs x SIMDs x 2

struct alignas(16) V2 {
    double v[2];
};

struct In {
    V2 b, r, f0, f1;
    double e[2];
};

template <int L>
struct State {
    V2 win[L][3];   // level l: rows of the other colour (ring of 3)
    V2 blk[3];      // final black rows
    V2 red_in[2];   // red ring values, which pass through level 0
    V2 fr[6], fb[6];
    In in[6];
    double ec[2][2];  // coarse rows (x - 1) >> 1 and the next (up)
    double wt[2], wm[2];  // weighted residual rows 2I - 1 and 2I (down)
};

constexpr int pmod(int a, int m) { return ((a % m) + m) % m; }

template <int CTRL>
__device__ __forceinline__ double lane_shift(double v) {
    const int lo = __builtin_amdgcn_mov_dpp(__double2loint(v), CTRL, 0xf, 0xf, true);
    const int hi = __builtin_amdgcn_mov_dpp(__double2hiint(v), CTRL, 0xf, 0xf, true);
    return __hiloint2double(hi, lo);
}
constexpr int kFromNext = 0x130;  // wave_shl:1, the last lane gets 0 (it is halo)
constexpr int kFromPrev = 0x138;  // wave_shr:1

// c ? a : b as a bitwise blend (no branch around the computation of a)
__device__ __forceinline__ double blend(bool c, double a, double b) {
    const uint64_t m = uint64_t(0) - uint64_t(c);
    return __longlong_as_double(
        (long long)((uint64_t(__double_as_longlong(a)) & m) | (uint64_t(__double_as_longlong(b)) & ~m)));
}

struct Geo {
    int x, r0, r1, x_last;
    int64_t q0, qv, qc0, qc1, cq;
    bool in_core;
};

__device__ __forceinline__ int clampi(int x, int lo, int hi) {
    return x < lo ? lo : (x > hi ? hi : x);
}

// Rows outside the grid are clamped into it: their values only reach rows
// that are not written.
template <bool UP, bool EDGE, bool ZERO>
__device__ __forceinline__ In load_in(const MgLegArgs& a, int x, const Geo& g, bool odd) {
    In in;
    const int64_t row = int64_t(clampi(x, 0, a.n + 1)) * a.pitch + g.qv;
    const V2 zero{{0.0, 0.0}};
    in.b = ZERO ? zero : *reinterpret_cast<const V2*>(a.b_in + row);
    in.r = (EDGE && !ZERO) ? *reinterpret_cast<const V2*>(a.r_in + row) : zero;
    in.f0 = *reinterpret_cast<const V2*>(a.f_red + int64_t(clampi(x - 1, 1, a.n)) * a.pitch + g.qv);
    in.f1 = *reinterpret_cast<const V2*>(a.f_black + int64_t(clampi(x - 2, 1, a.n)) * a.pitch + g.qv);
    in.e[0] = in.e[1] = 0.0;
    if (UP && odd) {  // coarse row (x + 1) / 2 comes into use
        const int I = clampi((x + 1) >> 1, 0, a.nc + 1);
        const double* even = (I & 1) ? a.e_black : a.e_red;  // column 2Q has colour I & 1
        const double* oddc = (I & 1) ? a.e_red : a.e_black;
        in.e[0] = even[int64_t(I) * a.cpitch + g.cq];
        in.e[1] = oddc[int64_t(I) * a.cpitch + g.cq];
    }
    return in;
}

// Columns q .. q + 1 of one row, the points of the core that lie inside.
__device__ __forceinline__ void store_row(double* row, const V2& v, const Geo& g, int p, int n) {
    const int64_t lo = g.qc0 > 1 - p ? g.qc0 : 1 - p;
    const int64_t in = (int64_t(n) - p) >> 1;
    const int64_t hi = g.qc1 - 1 < in ? g.qc1 - 1 : in;
    if (g.q0 >= lo && g.q0 + 1 <= hi) {
        *reinterpret_cast<V2*>(row + g.q0) = v;
    } else {
        if (g.q0 >= lo && g.q0 <= hi) row[g.q0] = v.v[0];
        if (g.q0 + 1 >= lo && g.q0 + 1 <= hi) row[g.q0 + 1] = v.v[1];
    }
}

__device__ __forceinline__ double weight_row(double a, double b, double c) {
    return (a + 2.0 * b) + c;
}

// One input row; S = (x - first row) mod 6 with an even first row fixes the
// register slots (periods 3 and 6) and the row parities at compile time.
template <int L, bool UP, bool EDGE, bool ZERO, bool NORM, int S>
__device__ __forceinline__ void step(State<L>& st, const MgLegArgs& a, const Geo& g, int x,
                                     double& acc) {
    const int n = a.n;
    const In cur = st.in[S];
    st.in[(S + kPrefetch) % 6] =
        load_in<UP, EDGE, ZERO>(a, x + kPrefetch, g, ((S + kPrefetch) & 1) != 0);
    st.fr[S] = cur.f0;
    st.fb[S] = cur.f1;
    V2 carry = cur.b;
    if constexpr (UP) {
        // black plus the interpolant (multigrid.hip's prolongation); ring
        // points take none
        double v[2];
        if constexpr ((S & 1) == 0) {  // x even: columns 4Q + 1, 4Q + 3, coarse row x / 2
            const double nx = lane_shift<kFromNext>(st.ec[1][0]);
            v[0] = (st.ec[1][0] + st.ec[1][1]) * 0.5;
            v[1] = (st.ec[1][1] + nx) * 0.5;
        } else {  // x odd: columns 4Q, 4Q + 2, coarse rows (x - 1) / 2 and (x + 1) / 2
#pragma unroll
            for (int k = 0; k < 2; ++k) {
                st.ec[0][k] = st.ec[1][k];
                st.ec[1][k] = cur.e[k];
                v[k] = (st.ec[0][k] + st.ec[1][k]) * 0.5;
            }
        }
        constexpr int p = (S + 1) & 1;
#pragma unroll
        for (int k = 0; k < 2; ++k) {
            const double c = cur.b.v[k] + v[k];
            if constexpr (EDGE) {
                const int64_t q = g.q0 + k;
                carry.v[k] = blend(x >= 1 && x <= n && q >= 1 - p && q <= ((int64_t(n) - p) >> 1),
                                   c, cur.b.v[k]);
            } else {
                carry.v[k] = c;
            }
        }
    }
    V2 red_old;  // final red row x - L - 2, about to leave its ring
    auto level = [&](auto lc) {
        constexpr int l = decltype(lc)::value;
        constexpr int s_new = pmod(S - l, 3);      // row x - l
        constexpr int s_mid = pmod(S - l - 1, 3);  // row y = x - 1 - l
        constexpr int s_up = pmod(S - l - 2, 3);   // row y - 1
        constexpr int p = pmod(S - 1 - l + (l & 1), 2);
        if constexpr (l == L - 1) red_old = st.win[l][s_new];
        st.win[l][s_new] = carry;
        const V2& up = st.win[l][s_up];
        const V2& mid = st.win[l][s_mid];
        const V2& dn = st.win[l][s_new];
        double extra;
        if constexpr (p == 1)
            extra = lane_shift<kFromNext>(mid.v[0]);
        else
            extra = lane_shift<kFromPrev>(mid.v[1]);
        const V2& f = (l & 1) ? st.fb[pmod(S + 1 - l, 6)] : st.fr[pmod(S - l, 6)];
        const int y = x - 1 - l;
        V2 out;
#pragma unroll
        for (int e = 0; e < 2; ++e) {
            const double right = p ? (e == 0 ? mid.v[1] : extra) : mid.v[e];
            const double left = p ? mid.v[e] : (e == 1 ? mid.v[0] : extra);
            double s = dn.v[e] + up.v[e];
            s = s + right;
            s = s + left;
            const double t = a.h2 * f.v[e];
            s = s - t;
            const double nv = 0.25 * s;
            if constexpr (EDGE) {
                double prev;
                if constexpr (l == 0)
                    prev = st.red_in[pmod(S - 1, 2)].v[e];
                else
                    prev = st.win[l - 1][pmod(S - l - 1, 3)].v[e];
                const int64_t q = g.q0 + e;
                out.v[e] = blend(y >= 1 && y <= n && q >= 1 - p && q <= ((int64_t(n) - p) >> 1),
                                 nv, prev);
            } else {
                out.v[e] = nv;
            }
        }
        carry = out;
    };
    level(std::integral_constant<int, 0>{});
    level(std::integral_constant<int, 1>{});
    if constexpr (L > 2) {
        level(std::integral_constant<int, 2>{});
        level(std::integral_constant<int, 3>{});
    }
    if constexpr (EDGE) st.red_in[S & 1] = cur.r;
    constexpr int b_new = pmod(S, 3), b_mid = pmod(S - 1, 3), b_up = pmod(S - 2, 3);
    st.blk[b_new] = carry;  // final black row x - L
    {
        const int y = x - L;
        constexpr int pb = pmod(S + 1, 2);  // L even: parity of (y + 1)
        if (y >= g.r0 && y <= g.r1) {
            double* brow = a.b_out + int64_t(y) * a.pitch;
            const V2& red = st.win[L - 1][pmod(S - L, 3)];
            if constexpr (EDGE) {
                store_row(brow, carry, g, pb, n);
                if constexpr (UP) store_row(a.r_out + int64_t(y) * a.pitch, red, g, 1 - pb, n);
            } else if (g.in_core) {
                *reinterpret_cast<V2*>(brow + g.q0) = carry;
                if constexpr (UP)
                    *reinterpret_cast<V2*>(a.r_out + int64_t(y) * a.pitch + g.q0) = red;
            }
        }
    }
    if constexpr (!UP || NORM) {
        // residual of row y = x - L - 1: rev at columns 4Q, 4Q + 2, rod at
        // 4Q + 1, 4Q + 3
        const int y = x - L - 1;
        constexpr int py = pmod(S + 1, 2);  // parity of y
        const V2 red[3] = {red_old, st.win[L - 1][pmod(S - L - 1, 3)], st.win[L - 1][pmod(S - L, 3)]};
        const V2 black[3] = {st.blk[b_up], st.blk[b_mid], st.blk[b_new]};
        const V2(&ev)[3] = py ? black : red;  // even columns have colour y & 1
        const V2(&od)[3] = py ? red : black;
        const V2& f_red = st.fr[pmod(S - L, 6)];
        const V2& f_black = st.fb[pmod(S - L + 1, 6)];
        const V2& fe = py ? f_black : f_red;
        const V2& fo = py ? f_red : f_black;
        const double ev_next = lane_shift<kFromNext>(ev[1].v[0]);
        const double od_prev = lane_shift<kFromPrev>(od[1].v[1]);
        double rev[2], rod[2];
#pragma unroll
        for (int e = 0; e < 2; ++e) {
            double s = od[2].v[e] + od[0].v[e];  // even columns: neighbours are odd ones
            // (i +- 1, j) of an even column lies in the other colour's array at the same q
            s = s + od[1].v[e];
            s = s + (e == 1 ? od[1].v[0] : od_prev);
            rev[e] = fe.v[e] - (s - 4.0 * ev[1].v[e]) * a.inv_h2;
            double t = ev[2].v[e] + ev[0].v[e];
            t = t + (e == 0 ? ev[1].v[1] : ev_next);
            t = t + ev[1].v[e];
            rod[e] = fo.v[e] - (t - 4.0 * od[1].v[e]) * a.inv_h2;
        }
        if constexpr (NORM) {
            if (y >= g.r0 && y <= g.r1) {
                double sq = 0.0;
#pragma unroll
                for (int e = 0; e < 2; ++e) {
                    const int64_t q = g.q0 + e;
                    const bool core = q >= g.qc0 && q < g.qc1;
                    const bool oke = EDGE ? core && q >= 1 && q <= (int64_t(n) >> 1) : core;
                    const bool oko = EDGE ? core && q <= ((int64_t(n) - 1) >> 1) : core;
                    sq = sq + blend(oke, rev[e] * rev[e], 0.0);
                    sq = sq + blend(oko, rod[e] * rod[e], 0.0);
                }
                acc = acc + sq;
            }
        } else {
            const double rod_prev = lane_shift<kFromPrev>(rod[1]);
            const double w0 = weight_row(rod_prev, rev[0], rod[0]);  // J = 2Q
            const double w1 = weight_row(rod[0], rev[1], rod[1]);    // J = 2Q + 1
            if constexpr (py == 1) {  // y = 2I + 1 closes coarse row I
                const int I = (y - 1) >> 1;
                if (y - 1 >= g.r0 && I >= 1 && I <= a.nc && y - 1 <= g.r1) {
                    const double c0 = ((st.wt[0] + 2.0 * st.wm[0]) + w0) * 0.0625;
                    const double c1 = ((st.wt[1] + 2.0 * st.wm[1]) + w1) * 0.0625;
                    const int64_t Q = g.q0 >> 1;
                    double* even = ((I & 1) ? a.fc_black : a.fc_red) + int64_t(I) * a.cpitch;
                    double* oddc = ((I & 1) ? a.fc_red : a.fc_black) + int64_t(I) * a.cpitch;
                    const bool core = g.q0 >= g.qc0 && g.q0 < g.qc1;
                    if (core && Q >= 1 && 2 * Q <= a.nc) even[Q] = c0;
                    if (core && 2 * Q + 1 <= a.nc) oddc[Q] = c1;
                }
                st.wt[0] = w0;
                st.wt[1] = w1;
            } else {
                st.wm[0] = w0;
                st.wm[1] = w1;
            }
        }
    }
}

template <int L, bool UP, bool EDGE, bool ZERO, bool NORM>
__device__ __forceinline__ double march(const MgLegArgs& a, const Geo& g, int xs) {
    State<L> st;
    const V2 zero{{0.0, 0.0}};
#pragma unroll
    for (int l = 0; l < L; ++l) st.win[l][0] = st.win[l][1] = st.win[l][2] = zero;
    st.blk[0] = st.blk[1] = st.blk[2] = zero;
    st.red_in[0] = st.red_in[1] = zero;
#pragma unroll
    for (int k = 0; k < 6; ++k) st.fr[k] = st.fb[k] = zero;
    st.wt[0] = st.wt[1] = st.wm[0] = st.wm[1] = 0.0;
    double acc = 0.0;
#pragma unroll
    for (int d = 0; d < kPrefetch; ++d)
        st.in[d] = load_in<UP, EDGE, ZERO>(a, xs + d, g, (d & 1) != 0);
    if constexpr (UP) {  // coarse row xs / 2 (xs even)
        const In first = load_in<UP, EDGE, ZERO>(a, xs - 1, g, true);
        st.ec[0][0] = st.ec[0][1] = 0.0;
        st.ec[1][0] = first.e[0];
        st.ec[1][1] = first.e[1];
    }
    for (int x = xs; x <= g.x_last; x += 6) {
        step<L, UP, EDGE, ZERO, NORM, 0>(st, a, g, x, acc);
        step<L, UP, EDGE, ZERO, NORM, 1>(st, a, g, x + 1, acc);
        if (x + 2 > g.x_last) break;
        step<L, UP, EDGE, ZERO, NORM, 2>(st, a, g, x + 2, acc);
        step<L, UP, EDGE, ZERO, NORM, 3>(st, a, g, x + 3, acc);
        if (x + 4 > g.x_last) break;
        step<L, UP, EDGE, ZERO, NORM, 4>(st, a, g, x + 4, acc);
        step<L, UP, EDGE, ZERO, NORM, 5>(st, a, g, x + 5, acc);
    }
    return acc;
}

// Two waves per SIMD: the pipeline of two sweeps holds about 200 registers.
template <int L, bool UP, bool ZERO, bool NORM>
__global__ __launch_bounds__(kLanes, 2) void k_mg_leg(MgLegArgs a) {
    if (a.stop && *a.stop) return;
    const int nb = int(gridDim.x);
    const int tile = xcd_logical_block(int(blockIdx.x), nb);
    const int strip = tile / a.bands, band = tile - strip * a.bands;
    const int n = a.n;
    Geo g;
    g.r0 = 1 + strip * a.rows;  // odd
    g.r1 = g.r0 + a.rows - 1 < n ? g.r0 + a.rows - 1 : n;
    g.x_last = UP ? (NORM ? g.r1 + 1 + L : g.r1 + L) : g.r1 + 2 + L;
    const int xs = g.r0 - 1 - L > 0 ? g.r0 - 1 - L : 0;  // even
    g.qc0 = int64_t(band) * kCore;
    const int64_t qmax = int64_t(n >> 1);
    g.qc1 = g.qc0 + kCore < qmax + 1 ? g.qc0 + kCore : qmax + 1;
    g.q0 = g.qc0 - kHalo + 2 * int64_t(threadIdx.x);
    g.qv = g.q0 < 0 ? 0 : (g.q0 > a.pitch - 2 ? a.pitch - 2 : g.q0);
    const int64_t cq = g.q0 >> 1;
    g.cq = cq < 0 ? 0 : (cq > a.cpitch - 1 ? a.cpitch - 1 : cq);
    g.in_core = g.q0 >= g.qc0 && g.q0 + 2 <= g.qc1;
    const int64_t qa = g.qc0 - kHalo;
    const bool interior = g.r0 - 1 - L >= 1 && g.r1 + 2 + L <= n && qa >= 1 &&
                          qa + 2 * kLanes - 1 <= (int64_t(n) - 1) >> 1 &&
                          g.qc1 - g.qc0 == kCore;
    double acc;
    if (interior)
        acc = march<L, UP, false, ZERO, NORM>(a, g, xs);
    else
        acc = march<L, UP, true, ZERO, NORM>(a, g, xs);
    if constexpr (NORM) {  // the wave's sum in a fixed order
        __shared__ double part[kLanes];
        part[threadIdx.x] = acc;
        __syncthreads();
#pragma unroll
        for (int w = kLanes / 2; w > 0; w >>= 1) {
            if (int(threadIdx.x) < w) part[threadIdx.x] += part[threadIdx.x + w];
            __syncthreads();
        }
        if (threadIdx.x == 0) a.partials[tile] = part[0];
    }
}

constexpr int kReduceThreads = 256;

// sums[0] <- the tiles' partial sums in a fixed order.
__global__ __launch_bounds__(kReduceThreads) void k_mg_norm(const double* __restrict__ partials,
                                                            int count, double* __restrict__ sums,
                                                            const int* stop) {
    if (stop && *stop) return;
    __shared__ double part[kReduceThreads];
    double r = 0.0;
    for (int k = threadIdx.x; k < count; k += kReduceThreads) r += partials[k];
    part[threadIdx.x] = r;
    __syncthreads();
    for (int w = kReduceThreads / 2; w > 0; w >>= 1) {
        if (int(threadIdx.x) < w) part[threadIdx.x] += part[threadIdx.x + w];
        __syncthreads();
    }
    if (threadIdx.x == 0) sums[0] = part[0];
}

template <int L, bool UP, bool ZERO, bool NORM>
void launch_one(const MgLegArgs& a, hipStream_t s) {
    hipLaunchKernelGGL((k_mg_leg<L, UP, ZERO, NORM>), dim3(unsigned(a.bands * a.strips)),
                       dim3(kLanes), 0, s, a);
}

}  // namespace

// Strips as tall as leaves all tiles resident at once (every tile recomputes
// 2 L + 3 rows, and a second round of waves would be nearly empty), but at
// least 8 rows, where a small level wants more waves.  A V(2,2) solve at
// 8191^2 takes 7.30 ms with 160 rows (1820 tiles), 7.60 with 64 (4480) and
// 7.71 with 128 (2240: a tenth of them in a round of their own); V(1,1) at
// 1023^2 1.07 ms with 8 rows, 1.16 with 16.
MgLegGeometry mg_leg_geometry(int n) {
    MgLegGeometry g;
    g.bands = int(((n >> 1) + 1 + kCore - 1) / kCore);
    const int most = kLegWaves / g.bands > 1 ? kLegWaves / g.bands : 1;
    const int rows = (n + most - 1) / most;
    g.rows = rows <= 8 ? 8 : (rows + 1) / 2 * 2;
    g.strips = (n + g.rows - 1) / g.rows;
    return g;
}

hipError_t launch_mg_leg(MgLegArgs a, int sweeps, bool up, bool zero, bool norm, hipStream_t s) {
    if (sweeps < 1 || sweeps > 2 || a.n < 3 || (a.n & 1) == 0) return hipErrorInvalidValue;
    const MgLegGeometry g = mg_leg_geometry(a.n);
    a.bands = g.bands;
    a.rows = g.rows;
    a.strips = g.strips;
    if (!up) {
        if (sweeps == 1)
            zero ? launch_one<2, false, true, false>(a, s) : launch_one<2, false, false, false>(a, s);
        else
            zero ? launch_one<4, false, true, false>(a, s) : launch_one<4, false, false, false>(a, s);
    } else if (sweeps == 1) {
        norm ? launch_one<2, true, false, true>(a, s) : launch_one<2, true, false, false>(a, s);
    } else {
        norm ? launch_one<4, true, false, true>(a, s) : launch_one<4, true, false, false>(a, s);
    }
    hipError_t e = hipGetLastError();
    if (e != hipSuccess || !norm) return e;
    hipLaunchKernelGGL(k_mg_norm, dim3(1), dim3(kReduceThreads), 0, s, a.partials,
                       g.bands * g.strips, a.sums, a.stop);
    return hipGetLastError();
}

}  // namespace rbgs
