// Runs the fused passes (register windows, row pipeline, multigrid legs, 9-point
// passes: paper_2607_01735_amd/csrc, their kernels and launchers unchanged) on the
// CPU.  A workgroup is a wave of 64 lanes as fibers (hip/hip_runtime.h); the
// workgroups of a launch do not depend on one another and run one by one.  Every
// array is its own heap block of exactly the size the library gives it, so an
// AddressSanitizer build reports any access outside it; blocks start as NaN, so a
// read of anything that was not written shows in the result.  Test infrastructure
// only: tests/test_passes_emu.py builds it and compares with the oracle bit for bit.
//
// Build: -DEMU_PIPELINE, -DEMU_LEGS, -DEMU_MC9 or nothing (windows)
// Run:   emu type n sweeps fuse omega h in.bin out.bin
//   type    float64, or float32 (windows)
//   in.bin  u then f, natural (n+2) x (n+2) arrays of that type, row major
//   out.bin u after the sweeps, at most `fuse` a pass (legs: after a V(sweeps, sweeps)
//           cycle of two levels with three sweeps on the coarse one), then a double:
//           the legs' sum of squares of the residual
#include <hip/hip_runtime.h>

#include <stdio.h>
#include <stdlib.h>

#include <functional>
#include <vector>

namespace emu {
thread_local int nthreads = kLanes;
thread_local int current = 0;
thread_local jmp_buf lane_jmp[kMaxThreads];
thread_local bool lane_done[kMaxThreads];
thread_local uint64_t lane_slot[kMaxThreads];
thread_local int bar_arrived = 0, bar_generation = 0;
int yield_every = 0;
thread_local unsigned switches = 0;
thread_local int workgroup = 0;
Dim grid = {1, 1, 1};
}  // namespace emu

struct dim3 {
    unsigned x, y, z;
    dim3(unsigned a = 1, unsigned b = 1, unsigned c = 1) : x(a), y(b), z(c) {}
};
constexpr hipError_t hipSuccess = 0, hipErrorInvalidValue = 1;
inline hipError_t hipGetLastError() { return hipSuccess; }

static thread_local ucontext_t g_host_ctx, g_start_ctx[emu::kMaxThreads];
static thread_local jmp_buf g_host_jmp;
static std::function<void()> g_body;

static void lane_start(int lane) {
    if (_setjmp(emu::lane_jmp[lane]) == 0) swapcontext(&g_start_ctx[lane], &g_host_ctx);
    g_body();
    emu::lane_done[lane] = true;
    for (int k = 1; k < emu::nthreads; ++k) {
        const int nx = (lane + k) % emu::nthreads;
        if (!emu::lane_done[nx]) emu::jump_to_lane(nx);
    }
    _longjmp(g_host_jmp, 1);
}

static void emu_launch(std::function<void()> body, dim3 grid, dim3 block) {
    static std::vector<char> stacks(size_t(emu::kMaxThreads) << 20);
    if (grid.y != 1 || grid.z != 1 || block.x > unsigned(emu::kMaxThreads)) abort();
    g_body = body;
    emu::grid = {grid.x, 1, 1};
    emu::nthreads = int(block.x);
    for (unsigned b = 0; b < grid.x; ++b) {
        emu::workgroup = int(b);
        emu::current = 0;
        emu::bar_arrived = emu::bar_generation = 0;
        for (int l = 0; l < emu::nthreads; ++l) {
            if (getcontext(&g_start_ctx[l]) != 0) abort();
            g_start_ctx[l].uc_stack.ss_sp = &stacks[size_t(l) << 20];
            g_start_ctx[l].uc_stack.ss_size = size_t(1) << 20;
            g_start_ctx[l].uc_link = nullptr;
            makecontext(&g_start_ctx[l], reinterpret_cast<void (*)()>(lane_start), 1, l);
            emu::lane_done[l] = false;
            if (swapcontext(&g_host_ctx, &g_start_ctx[l]) != 0) abort();  // parks lane l
        }
        if (_setjmp(g_host_jmp) == 0) emu::jump_to_lane(0);
    }
}

inline bool emu_class(double v, int mask) {
    uint64_t b;
    memcpy(&b, &v, 8);
    const bool neg = b >> 63, nan = (b << 1) > 0xffe0000000000000ull;
    const bool sub = (b << 1) != 0 && (b << 1) < 0x0020000000000000ull;
    return (nan && (mask & 3)) || (sub && (mask & (neg ? 0x010 : 0x080)));
}

#define gridDim (emu::grid)
#define hipLaunchKernelGGL(kernel, grid, block, lds, stream, ...) \
    emu_launch([=] { kernel(__VA_ARGS__); }, grid, block)
#define __builtin_amdgcn_class(v, mask) emu_class(v, mask)
#define asm(...)  // the empty ones that keep a scalar base and a vector offset apart

#undef __any
#define __any(...) emu::vote((__VA_ARGS__), false)

#if defined(EMU_MC9)
#include "multicolour9_fused.hip"
namespace rbgs {  // multicolour9.hip's sizes
int mc9_rows(int n) { return ((n + 1) >> 1) + 1; }
int64_t mc9_pitch(int n) { return ((((int64_t(n) + 1) >> 1) + 1) + 31) / 32 * 32; }
}  // namespace rbgs
#elif defined(EMU_LEGS)
#include "multigrid_fused.hip"
#elif defined(EMU_PIPELINE)
#include "sweep_pipeline.hip"
namespace rbgs {
template <typename T>
hipError_t launch_window(const WindowArgs<T>& a, int sweeps, hipStream_t s) {
    if constexpr (sizeof(T) == 8) return launch_pipeline(a, sweeps, s);
    return hipErrorInvalidValue;
}
}  // namespace rbgs
#else
#include "sweep_window.hip"
namespace rbgs {
bool pipeline_takes(int, size_t, int) { return false; }
int pipeline_fuse(int) { return 0; }
hipError_t launch_pipeline(const WindowArgs<double>&, int, hipStream_t) { return hipErrorInvalidValue; }
}  // namespace rbgs
#endif

using namespace rbgs;

template <typename T>
T* block_of(size_t count) {
    T* p = static_cast<T*>(malloc(count * sizeof(T)));
    if (!p) abort();
    for (size_t k = 0; k < count; ++k) p[k] = T(__builtin_nan(""));
    return p;
}

template <typename T>
struct Split {  // one colour pair
    int n;
    int64_t pitch;
    T* c[2];
    explicit Split(int n_) : n(n_), pitch(split_pitch(n_, sizeof(T))) {
        for (auto& p : c) p = block_of<T>(size_t(n + 2) * size_t(pitch));
    }
    T& at(int i, int j) { return c[(i + j) & 1][int64_t(i) * pitch + (j >> 1)]; }
    bool ring(int i, int j) const { return i == 0 || j == 0 || i == n + 1 || j == n + 1; }
    void pack(const std::vector<T>& nat, bool only_ring = false) {
        for (int i = 0; i <= n + 1; ++i)
            for (int j = 0; j <= n + 1; ++j)
                if (!only_ring || ring(i, j)) at(i, j) = nat[size_t(i) * size_t(n + 2) + size_t(j)];
    }
    void unpack(std::vector<T>& nat) {
        for (int i = 1; i <= n; ++i)
            for (int j = 1; j <= n; ++j) nat[size_t(i) * size_t(n + 2) + size_t(j)] = at(i, j);
    }
};

#if defined(EMU_LEGS)
// plain half-sweeps, for the coarse level
void run_sweeps(Split<double>& u, Split<double>& f, int sweeps, double h) {
    for (int l = 0; l < 2 * sweeps; ++l)
        for (int i = 1; i <= u.n; ++i)
            for (int j = 1; j <= u.n; ++j) {
                if (((i + j) & 1) != (l & 1)) continue;
                double s = u.at(i + 1, j) + u.at(i - 1, j);
                s = s + u.at(i, j + 1);
                s = s + u.at(i, j - 1);
                const double t = (h * h) * f.at(i, j);
                u.at(i, j) = 0.25 * (s - t);
            }
}
#elif !defined(EMU_MC9)
// sweeps from buffer u[0], at most `fuse` a pass; the buffer of the result
template <typename T>
int run_sweeps(Split<T>* u, Split<T>& f, int sweeps, int fuse, bool deep, double h, double omega) {
    const int passes = (sweeps + fuse - 1) / fuse;
    for (int p = 0; p < passes; ++p) {
        WindowArgs<T> a{};
        for (int c = 0; c < 2; ++c) {
            a.in[c] = u[p & 1].c[c];
            a.out[c] = u[1 - (p & 1)].c[c];
            a.f[c] = f.c[c];
        }
        a.pitch = f.pitch;
        a.h2 = T(h * h);
        a.omega = T(omega);
        a.n = f.n;
        a.deep = deep;
        a.last = p == passes - 1;
        if (launch_window<T>(a, sweeps / passes + (p < sweeps % passes ? 1 : 0), nullptr) != hipSuccess)
            abort();
    }
    return passes & 1;
}
#endif

template <typename T>
int run(int n, int sweeps, int fuse, double omega, double h, const char* in, const char* out) {
    (void)fuse;
    (void)omega;
    std::vector<T> u(size_t(n + 2) * size_t(n + 2)), f(u.size());
    FILE* fh = fopen(in, "rb");
    if (!fh || fread(u.data(), sizeof(T), u.size(), fh) != u.size() ||
        fread(f.data(), sizeof(T), f.size(), fh) != f.size())
        return 2;
    fclose(fh);
    double extra = 0.0;
#if defined(EMU_MC9)
    const int rows = mc9_rows(n);
    const int64_t pitch = mc9_pitch(n);
    double *b[2][4], *fc[4];
    for (int c = 0; c < 4; ++c) {
        for (auto& x : b) x[c] = block_of<double>(size_t(rows) * size_t(pitch));
        fc[c] = block_of<double>(size_t(rows) * size_t(pitch));
    }
    for (int i = 0; i <= n + 1; ++i)
        for (int j = 0; j <= n + 1; ++j) {
            const int c = (i & 1) + 2 * (j & 1);
            const int64_t at = int64_t(i >> 1) * pitch + (j >> 1);
            const size_t nat = size_t(i) * size_t(n + 2) + size_t(j);
            b[0][c][at] = u[nat];
            fc[c][at] = f[nat];
            if (i == 0 || j == 0 || i == n + 1 || j == n + 1) b[1][c][at] = u[nat];
        }
    const int passes = (sweeps + fuse - 1) / fuse;
    for (int p = 0; p < passes; ++p)
        if (launch_mc9_pass(b[p & 1], b[1 - (p & 1)], fc, n, 6.0 * (h * h),
                            sweeps / passes + (p < sweeps % passes ? 1 : 0), p == passes - 1, nullptr,
                            nullptr) != hipSuccess)
            abort();
    for (int i = 1; i <= n; ++i)
        for (int j = 1; j <= n; ++j)
            u[size_t(i) * size_t(n + 2) + size_t(j)] =
                b[passes & 1][(i & 1) + 2 * (j & 1)][int64_t(i >> 1) * pitch + (j >> 1)];
#else
    Split<T> us[2] = {Split<T>(n), Split<T>(n)}, fs(n);
    us[0].pack(u);
    us[1].pack(u, true);
    fs.pack(f);
#if defined(EMU_LEGS)
    if constexpr (sizeof(T) == 8) {
        const int nc = (n - 1) / 2;
        const double hc = 2.0 * h;
        std::vector<T> zero(size_t(nc + 2) * size_t(nc + 2), 0.0);
        Split<T> uc(nc), fcs(nc);
        uc.pack(zero);
        const MgLegGeometry geo = mg_leg_geometry(n);
        double* partials = block_of<double>(size_t(geo.bands) * size_t(geo.strips));
        MgLegArgs a{};
        a.b_in = us[0].c[1];
        a.r_in = us[0].c[0];
        a.b_out = us[1].c[1];
        a.f_red = fs.c[0];
        a.f_black = fs.c[1];
        a.pitch = fs.pitch;
        a.n = n;
        a.nc = nc;
        a.h2 = h * h;
        a.inv_h2 = 1.0 / (h * h);
        a.fc_red = fcs.c[0];
        a.fc_black = fcs.c[1];
        a.cpitch = fcs.pitch;
        if (launch_mg_leg(a, sweeps, false, false, false, nullptr) != hipSuccess) abort();
        run_sweeps(uc, fcs, 3, hc);
        a.b_in = us[1].c[1];
        a.r_in = us[1].c[0];
        a.b_out = us[0].c[1];
        a.r_out = us[0].c[0];
        a.e_red = uc.c[0];
        a.e_black = uc.c[1];
        // the norm's reduction runs 256 threads a workgroup: add the tiles' sums here
        a.partials = partials;
        a.sums = nullptr;
        a.bands = geo.bands;
        a.rows = geo.rows;
        a.strips = geo.strips;
        if (sweeps == 1)
            launch_one<2, true, false, true>(a, nullptr);
        else
            launch_one<4, true, false, true>(a, nullptr);
        for (int k = 0; k < geo.bands * geo.strips; ++k) extra += partials[k];
        us[0].unpack(u);
    }
#else
#if defined(EMU_PIPELINE)
    const bool deep = true;
#else
    const bool deep = false;
#endif
    us[run_sweeps<T>(us, fs, sweeps, fuse, deep, h, omega)].unpack(u);
#endif
#endif
    fh = fopen(out, "wb");
    if (!fh || fwrite(u.data(), sizeof(T), u.size(), fh) != u.size() || fwrite(&extra, 8, 1, fh) != 1)
        return 2;
    fclose(fh);
    return 0;
}

int main(int argc, char** argv) {
    if (argc != 9) return 2;
    const int n = atoi(argv[2]), sweeps = atoi(argv[3]), fuse = atoi(argv[4]);
    const double omega = atof(argv[5]), h = atof(argv[6]);
#if !defined(EMU_PIPELINE) && !defined(EMU_LEGS) && !defined(EMU_MC9)
    if (strcmp(argv[1], "float32") == 0) return run<float>(n, sweeps, fuse, omega, h, argv[7], argv[8]);
#endif
    return run<double>(n, sweeps, fuse, omega, h, argv[7], argv[8]);
}
