// Grid transfers of the multigrid cycle on split (red/black) arrays.
//
// The cycle uses red-black Gauss-Seidel as its smoother: an extension beyond
// the paper, whose conclusion (Section 5) names multilevel odd-even
// techniques as future work.  The hierarchy is vertex-centred: a fine grid of
// n_f = 2 n_c + 1 interior points per side holds coarse point (I, J) at fine
// point (2I, 2J), the ring being index 0 and n+1 on every level.
//
// k_mg_restrict: the fine residual r = f - A_h u (the residual of Eq. (1)'s
//   system, same operations in the same order as the residual kernel), its
//   full weighting onto the coarse right-hand side, and a zero coarse
//   iterate, in one pass.  The fine residual is never stored.
// k_mg_prolong_add: u += bilinear interpolation of the coarse iterate.
//
// Rounding order (every + and * rounded once, no contraction):
//   full weighting: row_a = (r[a][2J-1] + 2 r[a][2J]) + r[a][2J+1] for the
//   fine rows a = 2I-1, 2I, 2I+1, then ((row_0 + 2 row_1) + row_2) * 0.0625;
//   prolongation at fine (i, j) with I = i >> 1, J = j >> 1: e[I][J] (both
//   even), (e[I][J] + e[I+1][J]) * 0.5 (i odd), (e[I][J] + e[I][J+1]) * 0.5
//   (j odd), ((e[I][J] + e[I][J+1]) + (e[I+1][J] + e[I+1][J+1])) * 0.25
//   (both odd); then u + v.
#include "lds_limit.h"
#include "rbgs_internal.h"

namespace rbgs {
namespace {

constexpr int kMgThreads = 256;

// One colour of a level with its ring in LDS, (n + 2) rows of (n + 3) / 2.
__host__ __device__ constexpr int mg_coarse_cells(int n) { return (n + 2) * ((n + 3) / 2); }

// LDS of the largest coarse end: four colour arrays of every level from
// kMgCoarseN down to a single point and the top level's residual.
constexpr size_t mg_coarse_lds() {
    size_t cells = size_t(kMgCoarseN + 2) * size_t(kMgCoarseN + 2);
    for (int n = kMgCoarseN; n >= 1; n = (n - 1) / 2) cells += 4 * size_t(mg_coarse_cells(n));
    return cells * sizeof(double);
}
constexpr size_t kMgCoarseLds = mg_coarse_lds();

constexpr int kRestrictRows = 4;  // coarse rows one thread marches down

// Element k of a split row, 0 outside [0, pitch): only ever used for points
// whose values are discarded.
__device__ __forceinline__ double at_or_zero(const double* row, int64_t k, int64_t pitch) {
    return (k >= 0 && k < pitch) ? row[k] : 0.0;
}

// The seven u values of fine row i at columns 4q-2 .. 4q+4.  Even columns
// of row i have colour i & 1, odd columns the other; column j sits at j >> 1.
__device__ __forceinline__ void load_u7(const double* __restrict__ u_red,
                                        const double* __restrict__ u_black, int64_t i, int64_t q,
                                        int64_t pitch, double out[7]) {
    const double* ev = ((i & 1) ? u_black : u_red) + i * pitch;
    const double* od = ((i & 1) ? u_red : u_black) + i * pitch;
    out[0] = at_or_zero(ev, 2 * q - 1, pitch);  // 4q - 2
    out[1] = at_or_zero(od, 2 * q - 1, pitch);  // 4q - 1
    out[2] = at_or_zero(ev, 2 * q, pitch);      // 4q
    out[3] = at_or_zero(od, 2 * q, pitch);      // 4q + 1
    out[4] = at_or_zero(ev, 2 * q + 1, pitch);  // 4q + 2
    out[5] = at_or_zero(od, 2 * q + 1, pitch);  // 4q + 3
    out[6] = at_or_zero(ev, 2 * q + 2, pitch);  // 4q + 4
}

// Residual of fine row i at columns 4q-1 .. 4q+3 from u rows i-1, i, i+1.
__device__ __forceinline__ void residual5(const double up[7], const double mid[7],
                                          const double dn[7], const double* __restrict__ f_red,
                                          const double* __restrict__ f_black, int64_t i,
                                          int64_t q, int64_t pitch, double inv_h2,
                                          double r[5]) {
    const double* ev = ((i & 1) ? f_black : f_red) + i * pitch;
    const double* od = ((i & 1) ? f_red : f_black) + i * pitch;
    double f[5];
    f[0] = at_or_zero(od, 2 * q - 1, pitch);  // 4q - 1
    f[1] = at_or_zero(ev, 2 * q, pitch);      // 4q
    f[2] = at_or_zero(od, 2 * q, pitch);      // 4q + 1
    f[3] = at_or_zero(ev, 2 * q + 1, pitch);  // 4q + 2
    f[4] = at_or_zero(od, 2 * q + 1, pitch);  // 4q + 3
#pragma unroll
    for (int k = 0; k < 5; ++k) {
        double s = dn[k + 1] + up[k + 1];
        s = s + mid[k + 2];
        s = s + mid[k];
        const double lap = (s - 4.0 * mid[k + 1]) * inv_h2;
        r[k] = f[k] - lap;
    }
}

__device__ __forceinline__ double weight_row(double a, double b, double c) {
    return (a + 2.0 * b) + c;
}

// One thread per coarse q (coarse columns J = 2q and 2q + 1) and a strip of
// kRestrictRows coarse rows; it keeps three fine u rows and the previous
// fine residual row in registers while marching down.
__global__ __launch_bounds__(kMgThreads) void k_mg_restrict(
    const double* __restrict__ u_red, const double* __restrict__ u_black,
    const double* __restrict__ f_red, const double* __restrict__ f_black, int64_t pitch,
    double inv_h2, double* __restrict__ fc_red, double* __restrict__ fc_black,
    double* __restrict__ uc_red, double* __restrict__ uc_black, int nc, int64_t cpitch,
    const int* stop) {
    if (stop && *stop) return;
    const int64_t q = int64_t(blockIdx.x) * kMgThreads + threadIdx.x;
    if (q >= cpitch) return;
    const int64_t I0 = int64_t(blockIdx.y) * kRestrictRows + 1;
    const int64_t I1 = I0 + kRestrictRows - 1 < nc ? I0 + kRestrictRows - 1 : nc;
    for (int64_t I = I0; I <= I1; ++I) {  // a zero coarse iterate (ring columns stay zero)
        uc_red[I * cpitch + q] = 0.0;
        uc_black[I * cpitch + q] = 0.0;
    }
    const bool j0_ok = q >= 1 && 2 * q <= nc;
    const bool j1_ok = 2 * q + 1 <= nc;
    if (!j0_ok && !j1_ok) return;
    double a[7], b[7], c[7];
    double r_top[5], r_mid[5], r_bot[5];
    load_u7(u_red, u_black, 2 * I0 - 2, q, pitch, a);
    load_u7(u_red, u_black, 2 * I0 - 1, q, pitch, b);
    load_u7(u_red, u_black, 2 * I0, q, pitch, c);
    residual5(a, b, c, f_red, f_black, 2 * I0 - 1, q, pitch, inv_h2, r_top);
    // window now: a = row 2I-2, b = 2I-1, c = 2I
    for (int64_t I = I0; I <= I1; ++I) {
        const int64_t i = 2 * I;
#pragma unroll
        for (int m = 0; m < 7; ++m) a[m] = b[m];
#pragma unroll
        for (int m = 0; m < 7; ++m) b[m] = c[m];
        load_u7(u_red, u_black, i + 1, q, pitch, c);  // a, b, c = rows 2I-1, 2I, 2I+1
        residual5(a, b, c, f_red, f_black, i, q, pitch, inv_h2, r_mid);
#pragma unroll
        for (int m = 0; m < 7; ++m) a[m] = b[m];
#pragma unroll
        for (int m = 0; m < 7; ++m) b[m] = c[m];
        load_u7(u_red, u_black, i + 2, q, pitch, c);  // rows 2I, 2I+1, 2I+2
        residual5(a, b, c, f_red, f_black, i + 1, q, pitch, inv_h2, r_bot);
        // coarse (I, 2q) has colour I & 1; (I, 2q + 1) the other
        double* even_dst = (I & 1) ? fc_black : fc_red;
        double* odd_dst = (I & 1) ? fc_red : fc_black;
        if (j0_ok) {
            const double t = weight_row(r_top[0], r_top[1], r_top[2]);
            const double m = weight_row(r_mid[0], r_mid[1], r_mid[2]);
            const double bt = weight_row(r_bot[0], r_bot[1], r_bot[2]);
            even_dst[I * cpitch + q] = ((t + 2.0 * m) + bt) * 0.0625;
        }
        if (j1_ok) {
            const double t = weight_row(r_top[2], r_top[3], r_top[4]);
            const double m = weight_row(r_mid[2], r_mid[3], r_mid[4]);
            const double bt = weight_row(r_bot[2], r_bot[3], r_bot[4]);
            odd_dst[I * cpitch + q] = ((t + 2.0 * m) + bt) * 0.0625;
        }
#pragma unroll
        for (int k = 0; k < 5; ++k) r_top[k] = r_bot[k];
    }
}

// Coarse value e[I][J] of a split coarse grid.
__device__ __forceinline__ double coarse_at(const double* __restrict__ e_red,
                                            const double* __restrict__ e_black, int64_t I,
                                            int64_t J, int64_t cpitch) {
    const double* a = ((I + J) & 1) ? e_black : e_red;
    return a[I * cpitch + (J >> 1)];
}

// One thread per fine (i, q): the two fine points (i, 2q) and (i, 2q + 1),
// one of each colour, both at split column q.
__global__ __launch_bounds__(kMgThreads) void k_mg_prolong_add(
    double* __restrict__ u_red, double* __restrict__ u_black, int64_t pitch, int nf,
    const double* __restrict__ e_red, const double* __restrict__ e_black, int64_t cpitch,
    const int* stop) {
    if (stop && *stop) return;
    const int64_t q = int64_t(blockIdx.x) * kMgThreads + threadIdx.x;
    const int64_t i = int64_t(blockIdx.y) + 1;
    if (2 * q > nf) return;
    const int64_t I = i >> 1;
    double* ev = ((i & 1) ? u_black : u_red) + i * pitch + q;  // (i, 2q)
    double* od = ((i & 1) ? u_red : u_black) + i * pitch + q;  // (i, 2q + 1)
    const double e00 = coarse_at(e_red, e_black, I, q, cpitch);
    const double e01 = coarse_at(e_red, e_black, I, q + 1, cpitch);
    double v_even, v_odd;
    if ((i & 1) == 0) {
        v_even = e00;
        v_odd = (e00 + e01) * 0.5;
    } else {
        const double e10 = coarse_at(e_red, e_black, I + 1, q, cpitch);
        const double e11 = coarse_at(e_red, e_black, I + 1, q + 1, cpitch);
        v_even = (e00 + e10) * 0.5;
        v_odd = ((e00 + e01) + (e10 + e11)) * 0.25;
    }
    if (q >= 1) *ev = *ev + v_even;
    if (2 * q + 1 <= nf) *od = *od + v_odd;
}

// ----- prolongation fused into the first post-smoothing red half-sweep ------
// The red half-sweep after the coarse correction overwrites every red value
// without reading it, and the black half-sweep after it overwrites every
// black value without reading it; so "u += P e, red half-sweep" needs the
// corrected values of the black neighbours only, formed on the fly (black +
// interpolant, ring values unchanged) and never stored.  The red values and,
// after the black half-sweep, the black values are bitwise those of the
// unfused sequence.  13 B per fine point (black and red f read, red written,
// the coarse grid through the cache) instead of 18 + 12.

// One thread per red point (i, j), i + j even.  The interpolants of its four
// black neighbours need five coarse values when i and j are even (the cross
// around (I, J) = (i/2, j/2)) and four when both are odd (the block (I, J) ..
// (I+1, J+1), I = i >> 1, J = j >> 1); each is loaded once and every
// interpolant is formed exactly as k_mg_prolong_add forms it for that
// point's parity.  Neighbours on the ring take no correction.
__global__ __launch_bounds__(kMgThreads) void k_mg_prolong_red(
    double* __restrict__ u_red, const double* __restrict__ u_black,
    const double* __restrict__ f_red, int64_t pitch, int nf, double h2,
    const double* __restrict__ e_red, const double* __restrict__ e_black, int64_t cpitch,
    const int* stop) {
    if (stop && *stop) return;
    const int64_t q = int64_t(blockIdx.x) * kMgThreads + threadIdx.x;
    const int64_t i = int64_t(blockIdx.y) + 1;
    const int64_t p = i & 1;
    if (q < 1 - p || q > ((int64_t(nf) - p) >> 1)) return;
    const int64_t j = 2 * q + p;
    const int64_t I = i >> 1, J = j >> 1;
    // black neighbours: (i+1, j), (i-1, j), (i, j+1), (i, j-1); black (i', j')
    // sits at u_black[i' pitch + (j' >> 1)]
    const double b_dn = u_black[(i + 1) * pitch + (j >> 1)];
    const double b_up = u_black[(i - 1) * pitch + (j >> 1)];
    const double b_rt = u_black[i * pitch + ((j + 1) >> 1)];
    const double b_lt = u_black[i * pitch + ((j - 1) >> 1)];
    double v_dn, v_up, v_rt, v_lt;
    if (p == 0) {  // i, j even
        const double c = coarse_at(e_red, e_black, I, J, cpitch);
        const double cn = coarse_at(e_red, e_black, I + 1, J, cpitch);
        const double cs = coarse_at(e_red, e_black, I - 1, J, cpitch);
        const double ce = coarse_at(e_red, e_black, I, J + 1, cpitch);
        const double cw = coarse_at(e_red, e_black, I, J - 1, cpitch);
        v_dn = (c + cn) * 0.5;   // (i+1, j): i+1 odd, j even, I' = I
        v_up = (cs + c) * 0.5;   // (i-1, j): I' = I - 1
        v_rt = (c + ce) * 0.5;   // (i, j+1): i even, j+1 odd, J' = J
        v_lt = (cw + c) * 0.5;   // (i, j-1): J' = J - 1
    } else {  // i, j odd
        const double e00 = coarse_at(e_red, e_black, I, J, cpitch);
        const double e01 = coarse_at(e_red, e_black, I, J + 1, cpitch);
        const double e10 = coarse_at(e_red, e_black, I + 1, J, cpitch);
        const double e11 = coarse_at(e_red, e_black, I + 1, J + 1, cpitch);
        v_dn = (e10 + e11) * 0.5;  // (i+1, j): i+1 even, j odd, I' = I + 1, J' = J
        v_up = (e00 + e01) * 0.5;  // (i-1, j): I' = I
        v_rt = (e01 + e11) * 0.5;  // (i, j+1): i odd, j+1 even, J' = J + 1
        v_lt = (e00 + e10) * 0.5;  // (i, j-1): J' = J
    }
    const double dn = i + 1 <= nf ? b_dn + v_dn : b_dn;
    const double up = i - 1 >= 1 ? b_up + v_up : b_up;
    const double right = j + 1 <= nf ? b_rt + v_rt : b_rt;
    const double left = j - 1 >= 1 ? b_lt + v_lt : b_lt;
    double s = dn + up;
    s = s + right;
    s = s + left;
    const double t = h2 * __builtin_nontemporal_load(f_red + i * pitch + q);  // read once
    s = s - t;
    u_red[i * pitch + q] = 0.25 * s;
}

// ----- the coarse end of the cycle in one workgroup ------------------------
// Levels of at most kMgCoarseN = 63 points per side cost little work but a
// launch per step; below that size the rest of the V-cycle (its smoothing,
// transfers and coarsest sweeps, in the order of the level-by-level cycle)
// runs in one workgroup of kCoarseThreads threads with a barrier between
// phases, all levels' u and f in LDS (94 KB from 63^2 down, and 33 KB for the
// residual of the level being restricted; a 127^2 level would need 270 KB).
// Only the top level's f (and u, unless it starts at zero) is read and only
// its u is written.  Every point's arithmetic is the kernels' above, so the
// iterate is the same bit for bit.  It is bound by the LDS round trip and the
// barrier of each phase: 127^2 down in global memory (L2) took 94 us a cycle.

constexpr int kCoarseThreads = 1024;
constexpr int kCoarseQ = 32;  // split columns of a phase: (kMgCoarseN + 1) / 2
constexpr int kCoarseRows = kCoarseThreads / kCoarseQ;

// One level in LDS: split rows 0 .. n + 1 of `w` columns; u and f are element
// offsets of their red arrays, black follows `cells` elements later.
struct CwLevel {
    int u, f, n, w, cells;
    double h2, inv_h2;
};

extern __shared__ __align__(16) double cw_lds[];

// Element of the array pair at `a` that holds point (i, j).
__device__ __forceinline__ double cw_at(const CwLevel& L, int a, int i, int j) {
    return cw_lds[a + ((i + j) & 1) * L.cells + i * L.w + (j >> 1)];
}

__device__ __forceinline__ void cw_half_sweep(const CwLevel& L, int colour) {
    const int self = L.u + colour * L.cells, other = L.u + (1 - colour) * L.cells;
    const int f = L.f + colour * L.cells;
    const int q = threadIdx.x % kCoarseQ;
    for (int i = int(threadIdx.x / kCoarseQ) + 1; i <= L.n; i += kCoarseRows) {
        const int p = (i + colour) & 1;
        if (q < 1 - p || q > ((L.n - p) >> 1)) continue;
        const int at = i * L.w + q;
        double s = cw_lds[other + at + L.w] + cw_lds[other + at - L.w];
        s = s + cw_lds[other + at + p];
        s = s + cw_lds[other + at - 1 + p];
        const double t = L.h2 * cw_lds[f + at];
        s = s - t;
        cw_lds[self + at] = 0.25 * s;
    }
}

__device__ __forceinline__ void cw_sweeps(const CwLevel& L, int count) {
    for (int s = 0; s < count; ++s) {
        cw_half_sweep(L, 0);
        __syncthreads();
        cw_half_sweep(L, 1);
        __syncthreads();
    }
}

// The residual of every interior point into the natural array at r (pitch
// n + 2).
__device__ __forceinline__ void cw_residual(const CwLevel& L, int r) {
    const int q = threadIdx.x % kCoarseQ;
    for (int i = int(threadIdx.x / kCoarseQ) + 1; i <= L.n; i += kCoarseRows) {
#pragma unroll
        for (int e = 0; e < 2; ++e) {
            const int j = 2 * q + e;
            if (j < 1 || j > L.n) continue;
            double s = cw_at(L, L.u, i + 1, j) + cw_at(L, L.u, i - 1, j);
            s = s + cw_at(L, L.u, i, j + 1);
            s = s + cw_at(L, L.u, i, j - 1);
            const double lap = (s - 4.0 * cw_at(L, L.u, i, j)) * L.inv_h2;
            cw_lds[r + i * (L.n + 2) + j] = cw_at(L, L.f, i, j) - lap;
        }
    }
}

__device__ __forceinline__ void cw_restrict(int r, int nf, const CwLevel& C) {
    const int J = threadIdx.x % kCoarseQ + 1;
    for (int I = int(threadIdx.x / kCoarseQ) + 1; I <= C.n && J <= C.n; I += kCoarseRows) {
        double row[3];
#pragma unroll
        for (int a = 0; a < 3; ++a) {
            const int at = r + (2 * I - 1 + a) * (nf + 2) + 2 * J;
            row[a] = weight_row(cw_lds[at - 1], cw_lds[at], cw_lds[at + 1]);
        }
        cw_lds[C.f + ((I + J) & 1) * C.cells + I * C.w + (J >> 1)] =
            ((row[0] + 2.0 * row[1]) + row[2]) * 0.0625;
    }
}

__device__ __forceinline__ void cw_prolong_add(const CwLevel& C, const CwLevel& F) {
    const int q = threadIdx.x % kCoarseQ;
    for (int i = int(threadIdx.x / kCoarseQ) + 1; i <= F.n && 2 * q <= F.n; i += kCoarseRows) {
        const int I = i >> 1;
        const double e00 = cw_at(C, C.u, I, q), e01 = cw_at(C, C.u, I, q + 1);
        double v_even, v_odd;
        if ((i & 1) == 0) {
            v_even = e00;
            v_odd = (e00 + e01) * 0.5;
        } else {
            const double e10 = cw_at(C, C.u, I + 1, q), e11 = cw_at(C, C.u, I + 1, q + 1);
            v_even = (e00 + e10) * 0.5;
            v_odd = ((e00 + e01) + (e10 + e11)) * 0.25;
        }
        const int at = F.u + i * F.w + q;
        const int even = at + (i & 1) * F.cells, odd = at + (1 - (i & 1)) * F.cells;
        if (q >= 1) cw_lds[even] = cw_lds[even] + v_even;
        if (2 * q + 1 <= F.n) cw_lds[odd] = cw_lds[odd] + v_odd;
    }
}

__device__ __forceinline__ CwLevel cw_level(const MgCoarseLevels& lv, int l) {
    CwLevel L;
    L.u = 0;
    for (int k = 0; k < l; ++k) L.u += 4 * mg_coarse_cells(lv.level[k].n);
    L.n = lv.level[l].n;
    L.w = (L.n + 3) / 2;
    L.cells = mg_coarse_cells(L.n);
    L.f = L.u + 2 * L.cells;
    L.h2 = lv.level[l].h2;
    L.inv_h2 = lv.level[l].inv_h2;
    return L;
}

__global__ __launch_bounds__(kCoarseThreads) void k_mg_coarse_vcycle(MgCoarseLevels lv, int nu1,
                                                                    int nu2, int coarse_sweeps,
                                                                    const int* stop) {
    if (stop && *stop) return;
    const int m = lv.count;
    const CwLevel last = cw_level(lv, m - 1);
    const int total = last.u + 4 * last.cells;  // the residual's array follows
    const MgCoarseLevel& g = lv.level[0];
    const CwLevel top = cw_level(lv, 0);
    for (int k = threadIdx.x; k < total; k += kCoarseThreads) cw_lds[k] = 0.0;
    __syncthreads();
    // rows of kCoarseQ columns, then the ring column's (w = 33 for n = 62, 63)
    auto in = [&](int i, int q) {
        const int64_t src = int64_t(i) * g.pitch + q;
        const int at = i * top.w + q;
        cw_lds[top.f + at] = g.f_red[src];
        cw_lds[top.f + top.cells + at] = g.f_black[src];
        if (!lv.zero_top) {
            cw_lds[top.u + at] = g.u_red[src];
            cw_lds[top.u + top.cells + at] = g.u_black[src];
        }
    };
    const int tq = threadIdx.x % kCoarseQ, ti = threadIdx.x / kCoarseQ;
    for (int i = ti; i <= top.n + 1 && tq < top.w; i += kCoarseRows) in(i, tq);
    if (top.w > kCoarseQ && int(threadIdx.x) <= top.n + 1) in(int(threadIdx.x), kCoarseQ);
    __syncthreads();
    for (int l = 0; l + 1 < m; ++l) {
        const CwLevel L = cw_level(lv, l);
        cw_sweeps(L, nu1);
        cw_residual(L, total);
        __syncthreads();
        cw_restrict(total, L.n, cw_level(lv, l + 1));
        __syncthreads();
    }
    cw_sweeps(last, coarse_sweeps);
    for (int l = m - 2; l >= 0; --l) {
        const CwLevel L = cw_level(lv, l);
        cw_prolong_add(cw_level(lv, l + 1), L);
        __syncthreads();
        cw_sweeps(L, nu2);
    }
    for (int i = ti + 1; i <= top.n; i += kCoarseRows) {
        const int p = i & 1;  // red's column parity; black has the other
        const int at = i * top.w + tq;
        const int64_t dst = int64_t(i) * g.pitch + tq;
        if (2 * tq + p >= 1 && 2 * tq + p <= top.n) g.u_red[dst] = cw_lds[top.u + at];
        if (2 * tq + 1 - p >= 1 && 2 * tq + 1 - p <= top.n)
            g.u_black[dst] = cw_lds[top.u + top.cells + at];
    }
}

// One workgroup row (blockIdx.y) per level, its threads over the rows.
__global__ __launch_bounds__(kMgThreads) void k_mg_init(MgInit init) {
    const MgInitLevel& lv = init.level[blockIdx.y];
    if (blockIdx.x == 0 && threadIdx.x < 2 && lv.error[threadIdx.x]) *lv.error[threadIdx.x] = 0;
    if (lv.n == 0) return;
    const int n1 = lv.n + 1;
    for (int i = int(blockIdx.x); i <= n1; i += int(gridDim.x)) {
        const bool whole = i == 0 || i == n1;
        // the ring columns 0 and n + 1 of either colour sit at q = 0 and
        // (n + 1) >> 1; a row of the ring is cleared whole
        for (int64_t q = threadIdx.x; q < lv.pitch; q += kMgThreads) {
            for (int k = 0; k < 4; ++k) {
                const int64_t j = 2 * q + ((i + k) & 1);  // k & 1 is the colour
                if (whole || j == 0 || j >= n1) lv.u[k][int64_t(i) * lv.pitch + q] = 0.0;
            }
        }
    }
}

}  // namespace

hipError_t launch_mg_init(const MgInit& init, hipStream_t s) {
    if (init.count < 1 || init.count > kMgInitLevels) return hipErrorInvalidValue;
    hipLaunchKernelGGL(k_mg_init, dim3(512, unsigned(init.count)), dim3(kMgThreads), 0, s, init);
    return hipGetLastError();
}

hipError_t launch_mg_coarse_vcycle(const MgCoarseLevels& levels, int nu1, int nu2,
                                   int coarse_sweeps, const int* stop, hipStream_t s) {
    if (levels.count < 1 || levels.count > kMgMaxCoarseLevels || levels.level[0].n > kMgCoarseN)
        return hipErrorInvalidValue;
    static std::atomic<uint64_t> allowed{0};
    hipError_t e = allow_dynamic_lds(reinterpret_cast<const void*>(&k_mg_coarse_vcycle),
                                     kMgCoarseLds, allowed);
    if (e != hipSuccess) return e;
    size_t cells = size_t(levels.level[0].n + 2) * size_t(levels.level[0].n + 2);  // the residual
    for (int l = 0; l < levels.count; ++l) cells += 4 * size_t(mg_coarse_cells(levels.level[l].n));
    const size_t lds = cells * sizeof(double);
    hipLaunchKernelGGL(k_mg_coarse_vcycle, dim3(1), dim3(kCoarseThreads), lds, s, levels, nu1, nu2,
                       coarse_sweeps, stop);
    return hipGetLastError();
}

hipError_t launch_mg_prolong_red(double* u_red, const double* u_black, const double* f_red,
                                 int64_t pitch, int nf, double h2, const double* e_red,
                                 const double* e_black, int64_t cpitch, const int* stop,
                                 hipStream_t s) {
    if (nf < 3) return hipSuccess;
    const int64_t qs = int64_t(nf) / 2 + 1;
    const dim3 grid(unsigned((qs + kMgThreads - 1) / kMgThreads), unsigned(nf));
    hipLaunchKernelGGL(k_mg_prolong_red, grid, dim3(kMgThreads), 0, s, u_red, u_black, f_red,
                       pitch, nf, h2, e_red, e_black, cpitch, stop);
    return hipGetLastError();
}

hipError_t launch_mg_restrict(const double* u_red, const double* u_black, const double* f_red,
                              const double* f_black, int64_t pitch, double inv_h2,
                              double* fc_red, double* fc_black, double* uc_red, double* uc_black,
                              int nc, int64_t cpitch, const int* stop, hipStream_t s) {
    if (nc < 1) return hipSuccess;
    const dim3 grid(unsigned((cpitch + kMgThreads - 1) / kMgThreads),
                    unsigned((nc + kRestrictRows - 1) / kRestrictRows));
    hipLaunchKernelGGL(k_mg_restrict, grid, dim3(kMgThreads), 0, s, u_red, u_black, f_red,
                       f_black, pitch, inv_h2, fc_red, fc_black, uc_red, uc_black, nc, cpitch,
                       stop);
    return hipGetLastError();
}

hipError_t launch_mg_prolong_add(double* u_red, double* u_black, int64_t pitch, int nf,
                                 const double* e_red, const double* e_black, int64_t cpitch,
                                 const int* stop, hipStream_t s) {
    if (nf < 3) return hipSuccess;
    const int64_t qs = int64_t(nf) / 2 + 1;  // q = 0 .. n_c
    const dim3 grid(unsigned((qs + kMgThreads - 1) / kMgThreads), unsigned(nf));
    hipLaunchKernelGGL(k_mg_prolong_add, grid, dim3(kMgThreads), 0, s, u_red, u_black, pitch, nf,
                       e_red, e_black, cpitch, stop);
    return hipGetLastError();
}

}  // namespace rbgs
