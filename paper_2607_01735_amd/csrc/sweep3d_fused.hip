// Several 3D red-black sweeps in one pass over the grid.
//
// A launch per half-sweep (sweep3d.hip) moves 24 B per grid point and sweep.
// Here a workgroup marches along i over a tile of rows (j) and split columns
// (q) with L = 2 K half-sweeps pipelined in registers, so a pass reads black
// and f once and writes black once (16 B per point; red is recomputed from
// black before anything reads it and is written by the last pass only):
// 8 B per point and sweep at K = 2.
//
// At input plane x level l updates plane y = x - 1 - l of colour l & 1 from
// the other colour's planes y - 1, y, y + 1 that level l - 1 produced last.  A
// wave holds kR rows of 64 columns, a lane one column of each row: the i
// neighbours are its own registers, the k neighbour outside its column comes
// from the next lane (DPP), j neighbours are its own registers or, at the
// first and last of its rows, the neighbouring wave's, which that wave left in
// LDS.  Only plane y needs j neighbours, and level l - 1 produced it a step
// earlier, so one barrier per step orders the exchange for all levels.
//
// Tiles overlap by L rows, L / 2 columns and L planes a side, which are
// recomputed and not written; a pass reads one black array and writes another,
// so workgroups are independent.  Ring points keep their value by a select
// (black's are in both arrays; red's are loaded where they are needed).
//
// 40 sweeps at 383^3: 12.6 ms with a launch per half-sweep, 5.8 here; a pass of
// two sweeps takes 270 us, of which 220 remain when every load hits a cache:
// it is bound by instruction issue (283 vector instructions per wave and step,
// 168 of them the update's FP64; two waves a SIMD, which the registers allow)
// and by the halo's share of them, then by memory (1.44 GB a pass by the
// counters, 5.3 TB/s).
//
// Each point's operations and their order are k_rb3_half's; the division by 6
// is div6 below, which gives the same bits.
#include <type_traits>

#include "rbgs_internal.h"

namespace rbgs {
namespace {

constexpr int kLanes = 64;
constexpr int kWaves = 8;      // waves of a workgroup, along j
constexpr int kR = 4;          // rows of a wave (even: fixes the row parities)
constexpr int kRows = kWaves * kR;
constexpr int kPrefetch = 1;   // planes loaded ahead of their use
constexpr int kCus = 256;      // one workgroup of 8 waves (two per SIMD) fills a CU

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

// s / 6, correctly rounded, by multiplication: q = s * RN(1/6) is within one
// unit in the last place (RN(1/6) is off by 2^-54 relative), r = 6 q - s is
// exact in one FMA, and RN(q - r RN(1/6)) is then the rounded quotient
// (Markstein, "Computation of elementary functions on the IBM RISC System/6000
// processor", 1990, Theorem 8) unless it is subnormal (a tie may go the wrong
// way) or s is infinite or NaN (the result is NaN).  A tile that meets such a
// result is computed again with the division itself (EXACT).  Signed zeros
// come out right.
template <bool EXACT>
__device__ __forceinline__ double div6(double s) {
    if constexpr (EXACT) return s / 6.0;
    const double rcp = 1.0 / 6.0;
    const double q = s * rcp;
    const double r = __builtin_fma(6.0, q, -s);
    return __builtin_fma(-r, rcp, q);
}

// NaN or subnormal (class bits: signalling and quiet NaN, the subnormals)
__device__ __forceinline__ bool odd_class(double v) {
    return __builtin_amdgcn_class(v, 0x001 | 0x002 | 0x010 | 0x080);
}

struct In {
    double b[kR], r[kR], f0[kR], f1[kR];
};

template <int L>
struct State {
    double win[L][3][kR];  // level l: planes of the other colour (ring of 3)
    In in[6];
};

struct Tile {
    int wave, j0;         // this wave and its first row (even)
    int i0, i1;           // planes written
    uint32_t rows_in;     // bit r: row j0 + r is interior
    uint32_t rows_core;   // bit r: row j0 + r is written
    bool ring0, ring1;    // this lane's column 2 q / 2 q + 1 is on the ring
    bool has_ring;        // some point of this wave's rows is (wave-uniform)
    bool core;            // this lane's column is written
    uint32_t at[kR];      // byte offset in a plane of row j0 + r at this lane's column, clamped
};

template <int L>
struct Lds {
    // rows 0 and kR - 1 of every wave and level, by step parity
    double edge[2][L][kWaves][2][kLanes];
    // h^2 f that levels 0 and 1 used, for levels 2 and 3 two steps later (each
    // thread's own; in registers they would spill)
    double f[L > 2 ? 2 : 1][2][L > 2 ? kRows : 1][kLanes];
};

__device__ __forceinline__ int clampi(int x, int lo, int hi) {
    return x < lo ? lo : (x > hi ? hi : x);
}

// The element at byte offset `bytes` (wave-uniform) + `lane` of p.  The empty
// asm keeps the two apart, a scalar base and a 32-bit vector offset: left alone
// the compiler forms (array + lane offset) ahead of the loop, a 64-bit vector
// address per array and row, and spills.
typedef __attribute__((address_space(1))) char gchar;  // stays a global access
typedef __attribute__((address_space(1))) double gdouble;

__device__ __forceinline__ gdouble* element(const double* p, int64_t bytes, uint32_t lane) {
    gchar* g = (gchar*)(reinterpret_cast<uintptr_t>(p) + uintptr_t(bytes));
    asm("" : "+s"(g), "+v"(lane));
    return (gdouble*)(g + lane);
}

// The inputs of step x.  Planes outside the grid are clamped into it: they
// reach only planes that are not written.
template <int PX>
__device__ __forceinline__ In load_in(const Rb3PassArgs& a, const Tile& g, int x) {
    const int n1 = a.n + 1;
    const int64_t pl = int64_t(a.n + 2) * a.pitch * 8;
    auto at = [&](const double* p, int plane, int r) {  // scalar base, 32-bit lane offset
        return *element(p, clampi(plane, 0, n1) * pl, g.at[r]);
    };
    In in;
    const bool ring_plane = x - 1 == 0 || x - 1 == n1;
#pragma unroll
    for (int r = 0; r < kR; ++r) {
        in.b[r] = at(a.b_in, x, r);
        in.f0[r] = at(a.f_red, x - 1, r);
        in.f1[r] = at(a.f_black, x - 2, r);
        in.r[r] = 0.0;
    }
    if (ring_plane || g.has_ring) {
#pragma unroll
        for (int r = 0; r < kR; ++r) {
            // red ring values of plane x - 1 (column parity of red in row j0 + r)
            const bool col = ((PX - 1 + r) & 1) ? g.ring1 : g.ring0;
            if (ring_plane || !((g.rows_in >> r) & 1) || col) in.r[r] = at(a.red, x - 1, r);
        }
    }
    return in;
}

template <int L, bool NEVEN, bool EXACT, int S>
__device__ __forceinline__ void step(State<L>& st, Lds<L>& lds, const Rb3PassArgs& a,
                                     const Tile& g, int x, bool& odd) {
    const int lane = int(threadIdx.x) & (kLanes - 1);
    const int n = a.n;
    const In cur = st.in[S];
    st.in[(S + kPrefetch) % 6] = load_in<(S + kPrefetch) & 1>(a, g, x + kPrefetch);
    double carry[kR];
#pragma unroll
    for (int r = 0; r < kR; ++r) carry[r] = cur.b[r];
    static_for<0, L>([&](auto lc) {
        constexpr int l = decltype(lc)::value;
        constexpr int s_new = pmod(S - l, 3);      // plane x - l
        constexpr int s_mid = pmod(S - l - 1, 3);  // plane y = x - 1 - l
        constexpr int s_up = pmod(S - l - 2, 3);   // plane y - 1
        const int y = x - 1 - l;
        // this colour's previous value of row r: what ring points keep
        auto keep = [&](auto rc) -> double {
            if constexpr (l == 0)
                return cur.r[decltype(rc)::value];
            else
                return st.win[l - 1][pmod(S - l - 1, 3)][decltype(rc)::value];
        };
#pragma unroll
        for (int r = 0; r < kR; ++r) st.win[l][s_new][r] = carry[r];
        // j neighbours across waves, left in LDS by the previous step
        const double above = lds.edge[(S + 1) & 1][l][g.wave > 0 ? g.wave - 1 : 0][1][lane];
        const double below = lds.edge[(S + 1) & 1][l][g.wave + 1 < kWaves ? g.wave + 1 : g.wave][0][lane];
        lds.edge[S & 1][l][g.wave][0][lane] = carry[0];
        lds.edge[S & 1][l][g.wave][1][lane] = carry[kR - 1];
        // h^2 f of plane y: levels 0 and 1 form it (red plane x - 1, black
        // plane x - 2), levels 2 and 3 take what those formed two steps ago
        double hf[kR];
#pragma unroll
        for (int r = 0; r < kR; ++r) {
            const double own = a.h2 * (l & 1 ? cur.f1[r] : cur.f0[r]);
            if constexpr (l < 2) {
                hf[r] = own;
            } else {
                double& slot = lds.f[l & 1][S & 1][g.wave * kR + r][lane];
                hf[r] = slot;
                slot = own;
            }
        }
        double out[kR];
        static_for<0, kR>([&](auto rc) {
            constexpr int r = decltype(rc)::value;
            constexpr int p = pmod(S - 1 + r, 2);  // (y + j + colour) & 1: level l's colour is l & 1
            const double(&mid)[kR] = st.win[l][s_mid];
            const double jp = r + 1 < kR ? mid[r + 1 < kR ? r + 1 : r] : below;
            const double jm = r > 0 ? mid[r > 0 ? r - 1 : r] : above;
            const double right = p ? next(mid[r]) : mid[r];
            const double left = p ? mid[r] : prev(mid[r]);
            double s = st.win[l][s_new][r] + st.win[l][s_up][r];
            s = s + jp;
            s = s + jm;
            s = s + right;
            s = s + left;
            s = s - hf[r];
            const double v = div6<EXACT>(s);
            if constexpr (!EXACT) odd = odd || odd_class(v);
            // columns 0 and n + 1: k = n + 1 has p = 1 when n is even, else
            // both have p = 0 (points beyond the ring reach none inside it)
            if constexpr (p == 0)
                out[r] = g.ring0 ? keep(IC<r>{}) : v;
            else if constexpr (NEVEN)
                out[r] = g.ring1 ? keep(IC<r>{}) : v;
            else
                out[r] = v;
        });
        if (y == 0 || y == n + 1) {
            static_for<0, kR>([&](auto rc) { out[decltype(rc)::value] = keep(rc); });
        } else if (g.rows_in != (1u << kR) - 1u) {
            static_for<0, kR>([&](auto rc) {
                constexpr int r = decltype(rc)::value;
                if (!((g.rows_in >> r) & 1)) out[r] = keep(rc);
            });
        }
#pragma unroll
        for (int r = 0; r < kR; ++r) carry[r] = out[r];
    });
    const int y = x - L;
    if (y >= g.i0 && y <= g.i1 && g.core) {
        const int64_t pl = int64_t(y) * (int64_t(n + 2) * a.pitch * 8);
        static_for<0, kR>([&](auto rc) {
            constexpr int r = decltype(rc)::value;
            constexpr int pb = pmod(S - L + r + 1, 2);  // black's column parity in row j0 + r
            if ((g.rows_core >> r) & 1) {
                auto store = [&](double* p, double v) {
                    __builtin_nontemporal_store(v, element(p, pl, g.at[r]));
                };
                if (pb ? !g.ring1 : !g.ring0) store(a.b_out, carry[r]);
                if (a.last && (pb ? !g.ring0 : !g.ring1)) store(a.red, st.win[L - 1][pmod(S - L, 3)][r]);
            }
        });
    }
    __syncthreads();
}

// Steps S .. 5 from step x; false after the last one.
template <int L, bool NEVEN, bool EXACT, int S>
__device__ __forceinline__ bool steps(State<L>& st, Lds<L>& lds, const Rb3PassArgs& a,
                                      const Tile& g, int x, int x_last, bool& odd) {
    step<L, NEVEN, EXACT, S>(st, lds, a, g, x + S, odd);
    if (x + S >= x_last) return false;
    if constexpr (S < 5)
        return steps<L, NEVEN, EXACT, S + 1>(st, lds, a, g, x, x_last, odd);
    else
        return true;
}

// Returns whether a point of this lane wants the division itself.
template <int L, bool NEVEN, bool EXACT>
__device__ __forceinline__ bool march(Lds<L>& lds, const Rb3PassArgs& a, const Tile& g, int xs,
                                      int x_last) {
    State<L> st;
#pragma unroll
    for (int r = 0; r < kR; ++r) {
#pragma unroll
        for (int l = 0; l < L; ++l) st.win[l][0][r] = st.win[l][1][r] = st.win[l][2][r] = 0.0;
    }
    // the first step's j neighbours only reach planes that are not written,
    // or the ring plane, which keeps its value
    const int lane = int(threadIdx.x) & (kLanes - 1);
#pragma unroll
    for (int l = 0; l < L; ++l)
        lds.edge[1][l][g.wave][0][lane] = lds.edge[1][l][g.wave][1][lane] = 0.0;
    if constexpr (L > 2) {
#pragma unroll
        for (int k = 0; k < 4; ++k)
#pragma unroll
            for (int r = 0; r < kR; ++r) lds.f[k & 1][k >> 1][g.wave * kR + r][lane] = 0.0;
    }
    static_for<0, kPrefetch>([&](auto dc) {
        constexpr int d = decltype(dc)::value;
        st.in[d] = load_in<d & 1>(a, g, xs + d);
    });
    __syncthreads();
    bool odd = false;
    for (int x = xs; steps<L, NEVEN, EXACT, 0>(st, lds, a, g, x, x_last, odd); x += 6) {
    }
    return odd;
}

template <int L, bool NEVEN>
__global__ __launch_bounds__(kWaves* kLanes, 2) void k_rb3_pass(Rb3PassArgs a) {
    if (a.stop && *a.stop) return;
    __shared__ Lds<L> lds;
    const int tile = xcd_logical_block(int(blockIdx.x), int(gridDim.x));
    const int band = tile % a.bands, jt = (tile / a.bands) % a.jtiles;
    const int chunk = tile / (a.bands * a.jtiles);
    const int lane = int(threadIdx.x) & (kLanes - 1);
    const int n = a.n;
    Tile g;
    g.wave = __builtin_amdgcn_readfirstlane(int(threadIdx.x) / kLanes);
    const int jc0 = jt * (kRows - 2 * L);  // rows written: jc0 .. jc0 + kRows - 2 L - 1
    g.j0 = jc0 - L + g.wave * kR;
    g.i0 = chunk * a.planes;
    g.i1 = g.i0 + a.planes - 1 < n ? g.i0 + a.planes - 1 : n;
    // lanes past the band's halo repeat its last column
    const int q = band * a.qcore - L / 2 + (lane < a.qcore + L ? lane : a.qcore + L - 1);
    const uint32_t qb = uint32_t(clampi(q, 0, int(a.pitch) - 1)) * 8u;
    g.rows_in = g.rows_core = 0;
#pragma unroll
    for (int r = 0; r < kR; ++r) {
        const int j = g.j0 + r;
        if (j >= 1 && j <= n) {
            g.rows_in |= 1u << r;
            if (j >= jc0 && j < jc0 + kRows - 2 * L) g.rows_core |= 1u << r;
        }
        g.at[r] = uint32_t(clampi(j, 0, n + 1)) * uint32_t(a.pitch * 8) + qb;
    }
    g.ring0 = q == 0 || 2 * q == n + 1;
    g.ring1 = 2 * q + 1 == n + 1;
    g.has_ring = g.rows_in != (1u << kR) - 1u || __any(g.ring0 || g.ring1);
    g.core = lane >= L / 2 && lane < L / 2 + a.qcore && 2 * q <= n + 1 && !(g.ring0 && 2 * q > n);
    const int xs = g.i0 - L > 0 ? g.i0 - L : 0;  // even
    const int x_last = g.i1 + L;
    const bool odd = march<L, NEVEN, false>(lds, a, g, xs, x_last);
    if (__builtin_expect(__syncthreads_or(odd), 0)) march<L, NEVEN, true>(lds, a, g, xs, x_last);
}

}  // namespace

hipError_t launch_rb3_pass(const double* b_in, double* b_out, double* red, const double* f_red,
                           const double* f_black, int n, int64_t pitch, double h2, int sweeps,
                           bool last, const int* stop, hipStream_t s) {
    if (sweeps < 1 || sweeps > kRb3MaxFuse) return hipErrorInvalidValue;
    Rb3PassArgs a;
    a.b_in = b_in;
    a.b_out = b_out;
    a.red = red;
    a.f_red = f_red;
    a.f_black = f_black;
    a.stop = stop;
    a.pitch = pitch;
    a.h2 = h2;
    a.n = n;
    a.last = last;
    const int L = 2 * sweeps;
    const int qs = (n >> 1) + 1;
    a.bands = (qs + kLanes - L - 1) / (kLanes - L);
    a.qcore = (qs + a.bands - 1) / a.bands;
    a.jtiles = (n + 1 + kRows - 2 * L - 1) / (kRows - 2 * L);
    // chunks of planes: the fewest steps over all rounds of workgroups
    const int64_t area = int64_t(a.bands) * a.jtiles;
    int64_t best = INT64_MAX;
    int chunks = 1;
    for (int c = 1; c <= n + 1; ++c) {
        const int planes = ((n + 1 + c - 1) / c + 1) / 2 * 2;
        if (planes < 4 && c > 1) break;
        const int64_t cost = (area * c + kCus - 1) / kCus * (planes + 2 * L);
        if (cost < best) {
            best = cost;
            chunks = c;
        }
    }
    a.planes = ((n + 1 + chunks - 1) / chunks + 1) / 2 * 2;  // even: fixes the plane parities
    chunks = (n + 1 + a.planes - 1) / a.planes;
    const dim3 grid{unsigned(area * chunks)}, block{kWaves * kLanes};
    const bool even = (n & 1) == 0;
    if (sweeps == 1 && even)
        hipLaunchKernelGGL((k_rb3_pass<2, true>), grid, block, 0, s, a);
    else if (sweeps == 1)
        hipLaunchKernelGGL((k_rb3_pass<2, false>), grid, block, 0, s, a);
    else if (even)
        hipLaunchKernelGGL((k_rb3_pass<4, true>), grid, block, 0, s, a);
    else
        hipLaunchKernelGGL((k_rb3_pass<4, false>), grid, block, 0, s, a);
    return hipGetLastError();
}

}  // namespace rbgs
