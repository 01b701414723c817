// Learned initial guess: a small U-Net, trained and run by hand-written
// kernels (BF16 activations and weights, FP32 accumulation on MFMA, FP32
// master weights and Adam).
//
// Network: input x0 = f / rms(f) on the N x N interior; four levels on
// grids N_l = (N_{l-1} + 1)/F - 1 (coarsening factor F = 2 or 4) with
// 16/32/64/128 channels; each encoder level is conv3x3+ReLU twice, levels
// are linked by the averaging restriction R; each decoder level
// takes the bilinear prolongation P = F^2 R^T of the level below beside
// the encoder's output of its own level (the concatenation) and applies conv3x3+ReLU twice; a
// 1x1 head gives y, and u0 = y * rms(f).  With F = 4 the coarsest level's
// 3x3 convolutions span the whole grid (N = 511: levels 511, 127, 31, 7).
// The restriction/prolongation pair is the multigrid transfer pair, fixed
// (no weights).  Loss: mean squared error against u*/rms(f).
//
// Tensors are NHWC (batch, row, column, channel) in bfloat16; a tensor view
// has a pixel stride (channels per pixel of its buffer).  The two halves of
// a decoder's concatenated input stay two tensors that the kernels read as
// one.  Convolutions are implicit GEMMs on the BF16 MFMA: pixels x output
// channels, K = 9 taps x input channels.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <cmath>
#include <cstring>
#include <string>
#include <vector>

#include "rbgs.h"
#include "rbgs_internal.h"

namespace rbgs {
namespace nn {

typedef uint16_t bf16;
typedef short bf16x4 __attribute__((ext_vector_type(4)));
typedef float f32x4 __attribute__((ext_vector_type(4)));

__device__ __forceinline__ float bf2f(bf16 v) { return __uint_as_float(uint32_t(v) << 16); }

// round to nearest, ties to even (NaN kept quiet), two to a v_cvt_pk_bf16_f32
__device__ __forceinline__ bf16 f2bf(float x) { return __builtin_bit_cast(bf16, static_cast<__bf16>(x)); }

// ---------------------------------------------------------------------------
// 3x3 convolution, stride 1, zero padding 1, as an implicit GEMM:
// D[co][pixel] = sum_k W[co][k] X[k][pixel], K = 9 taps x input channels, on
// 16 x 16 x 16 BF16 MFMAs.  Lane layout (checked on the device):
//   A[m][k]: lane l holds m = l%16, k = 4(l/16)+j;  B[k][n]: n = l%16,
//   k = 4(l/16)+j;  D[m][n]: lane l holds m = 4(l/16)+i, n = l%16.
// So a lane loads four consecutive input channels of one pixel (B) and of
// one output channel's weights (A), 8 bytes each, and stores four
// consecutive output channels of one pixel.  Every kernel below adds to an
// output in the same order (16-channel chunks, in each the kernel rows, in
// each the columns, one MFMA each), so an activation has the same bits
// whichever computes it; K is therefore neither split over waves nor taken
// 32 at a time.
// X may be masked: an input element counts as 0 where mask <= 0 (this is
// how the backward pass applies the ReLU derivative of the layer output; the
// mask is a ReLU's output, so it holds no NaN).  Input and output channels
// may lie in two tensors (a decoder level's input is the prolongation of the
// level below beside the encoder's output; two tensors, so that each is read
// and written in whole lines).
// ---------------------------------------------------------------------------
constexpr int kConvGroups = 2;  // 16-pixel groups of a k_conv_march wave

struct ConvArgs {
    const bf16* x;     // input channels [0, xsplit), pixel stride xs
    int64_t xs;
    const bf16* x2;    // input channels [xsplit, cin), pixel stride xs2
    int64_t xs2;
    const bf16* mask;  // optional, same geometry as x, stride ms
    int64_t ms;
    const bf16* w;     // [cout / 16][cin / 16][9][64 lanes][4], as the A operands lie
    const float* bias; // optional
    bf16* y;           // output channels [0, ysplit), pixel stride ys
    int64_t ys;
    bf16* y2;          // output channels [ysplit, cout), pixel stride ys2
    int64_t ys2;
    int batch, h, wd, cin, cout, relu, xsplit, ysplit;
    int rows;          // k_conv_march: rows of a wave
    // k_conv_march<1, 1, false, false, true>: instead of y, the head's output
    // times rms goes to u (natural layout)
    const float *head, *rms;  // head: 16 weights, bias
    double* u;
    int64_t ld, gstride;
};

typedef uint32_t u32x2 __attribute__((ext_vector_type(2)));
typedef short s16x2 __attribute__((ext_vector_type(2)));

__device__ __forceinline__ f32x4 mfma16(u32x2 a, u32x2 b, f32x4 c) {
    return __builtin_amdgcn_mfma_f32_16x16x16bf16_1k(__builtin_bit_cast(bf16x4, a),
                                                     __builtin_bit_cast(bf16x4, b), c, 0, 0, 0);
}

__device__ __forceinline__ uint32_t pack2(float lo, float hi) {
    return uint32_t(f2bf(lo)) | (uint32_t(f2bf(hi)) << 16);
}

// all ones in the halves of m that are > 0 (as a BF16 that is no NaN)
__device__ __forceinline__ uint32_t positive(uint32_t m) {
    const s16x2 v = __builtin_bit_cast(s16x2, m);
    const s16x2 one = {1, 1}, zero = {0, 0};
    return __builtin_bit_cast(
        uint32_t, s16x2(zero - __builtin_elementwise_min(__builtin_elementwise_max(v, zero), one)));
}

template <int CTRL>
__device__ __forceinline__ u32x2 dpp(u32x2 old, u32x2 v) {
    return u32x2{uint32_t(__builtin_amdgcn_update_dpp(int(old[0]), int(v[0]), CTRL, 0xf, 0xf, false)),
                 uint32_t(__builtin_amdgcn_update_dpp(int(old[1]), int(v[1]), CTRL, 0xf, 0xf, false))};
}

// The head of one pixel, its 16 channels in the four lane groups (v, four a
// lane): bias + w[0] d[0] + w[1] d[1] ..., in that order, each lane group
// handing its sum to the next.  (Inference: the last activations are neither
// written nor read again, 30 us of 401 at 511^2 x 8.)
__device__ __forceinline__ float head_pixel(f32x4 v, f32x4 bias, const float (&w)[4], float head_bias,
                                            int lane) {
    float d[4];
#pragma unroll
    for (int i = 0; i < 4; ++i) {
        const float r = v[i] + bias[i];
        d[i] = bf2f(f2bf(r > 0.f ? r : 0.f));
    }
    float s = head_bias;
#pragma unroll
    for (int k = 0; k < 4; ++k) {
        float t = s;
#pragma unroll
        for (int i = 0; i < 4; ++i) t += w[i] * d[i];
        s = __shfl(t, k * 16 + (lane & 15), 64);
    }
    return s;
}

__device__ __forceinline__ void store_pixel(const ConvArgs& a, int64_t pix, int co, f32x4 v,
                                            f32x4 bias) {
    float r[4];
#pragma unroll
    for (int i = 0; i < 4; ++i) {
        r[i] = v[i] + bias[i];
        if (a.relu) r[i] = r[i] > 0.f ? r[i] : 0.f;
    }
    const u32x2 out = {pack2(r[0], r[1]), pack2(r[2], r[3])};
    bf16* p = co < a.ysplit ? a.y + pix * a.ys + co : a.y2 + pix * a.ys2 + (co - a.ysplit);
    *reinterpret_cast<u32x2*>(p) = out;
}

// Four channels of PG x 16 pixels of a row and of the two pixels beside
// them, as loaded: of group g's pixels, then (lanes n < 8) the pixel before
// the strip or (the others) the one after it.
template <int PG>
struct RowPixels {
    u32x2 v[PG + 1];
};

// A wave's pixels in a row; outside the grid they read a pixel inside and
// are zeroed.
template <int PG>
struct RowLanes {
    int px[PG + 1];
    uint32_t ok[PG + 1];
    __device__ RowLanes(int x0, int n, int wd) {
#pragma unroll
        for (int g = 0; g <= PG; ++g) {
            const int x = g < PG ? x0 + g * 16 + n : (n < 8 ? x0 - 1 : x0 + 16 * PG);
            ok[g] = x >= 0 && x < wd ? ~0u : 0u;
            px[g] = x < 0 ? 0 : x < wd ? x : wd - 1;
        }
    }
    __device__ void load(RowPixels<PG>& r, const bf16* p, uint32_t stride, uint32_t ch) const {
#pragma unroll
        for (int g = 0; g <= PG; ++g)
            r.v[g] = *reinterpret_cast<const u32x2*>(p + (uint32_t(px[g]) * stride + ch));
    }
    // one channel of 16 (the network's input), the others 0
    __device__ void load_one(RowPixels<PG>& r, const bf16* p, int kq) const {
#pragma unroll
        for (int g = 0; g <= PG; ++g) r.v[g] = u32x2{kq == 0 ? uint32_t(p[uint32_t(px[g])]) : 0u, 0u};
    }
    // The B operands of the three taps of a kernel row: the pixels shifted
    // by a lane either way (DPP), op[column * step + group].
    template <bool MASK>
    __device__ void taps(const RowPixels<PG>& r, const RowPixels<PG>& m, uint32_t row_ok, u32x2* op,
                         int step) const {
        u32x2 v[PG + 1];
#pragma unroll
        for (int g = 0; g <= PG; ++g) {
            v[g] = r.v[g] & (ok[g] & row_ok);
            if (MASK) {
                v[g][0] &= positive(m.v[g][0]);
                v[g][1] &= positive(m.v[g][1]);
            }
        }
#pragma unroll
        for (int g = 0; g < PG; ++g) {
            const u32x2 zero = {0u, 0u};
            // row_ror:1 / row_ror:15 bring the neighbouring group's edge pixel
            const u32x2 lo = g == 0 ? v[PG] : dpp<0x121>(zero, v[g ? g - 1 : 0]);
            const u32x2 hi = g == PG - 1 ? v[PG] : dpp<0x12f>(zero, v[g + 1]);
            op[g] = dpp<0x111>(lo, v[g]);             // row_shr:1
            op[step + g] = v[g];
            op[2 * step + g] = dpp<0x101>(hi, v[g]);  // row_shl:1
        }
    }
};

// Few channels, many pixels (cin = 16, 32 or 48: the finest level, and the next
// but for its 96).  Bound by memory: 16 -> 16 channels moves 64
// bytes a pixel for 9 MFMAs per 16 pixels.  So every input element is loaded
// once: a wave takes kConvGroups x 16 pixels of `rows` rows and walks down
// them with the layer's weights and the operands of three rows in registers.
// A row is loaded three rows ahead of its use, 8 bytes a lane, a whole
// 512-byte line per 16 pixels and chunk.  511^2 x 8: 16 -> 16 channels 30 us
// (134 MB, 4.5 TB/s), 48 -> 16 67 us, masked 16 -> 16 39 us, 16 -> 48 85 us;
// a wave per 32 outputs of a row, which loaded three rows three times over
// behind its loads of weights, took 86, 255, 109 and 194 us.  32 -> 32 at
// 127^2 x 8 10 us, masked 12 (k_conv_deep 15 and 24).
template <int CK, int NT, bool MASK, bool ONE = false, bool HEAD = false>
__global__ __launch_bounds__(256) void k_conv_march(ConvArgs a) {
    constexpr int PG = kConvGroups;
    const int lane = threadIdx.x & 63;
    int wave = int(blockIdx.x) * 4 + int(threadIdx.x >> 6);
    const int strips = (a.wd + 16 * PG - 1) / (16 * PG);
    const int bands = (a.h + a.rows - 1) / a.rows;
    const int cts = a.cout / (16 * NT);
    if (wave >= a.batch * bands * strips * cts) return;
    wave = __builtin_amdgcn_readfirstlane(wave);
    const int t0 = (wave % cts) * NT;  // first output tile
    wave /= cts;
    const int x0 = (wave % strips) * 16 * PG;
    const int band = (wave / strips) % bands;
    const int b = wave / (strips * bands);
    const int y0 = band * a.rows, y1 = y0 + a.rows < a.h ? y0 + a.rows : a.h;
    const int n = lane & 15, kq = (lane >> 4) * 4;

    u32x2 w[CK][9][NT];
#pragma unroll
    for (int c = 0; c < CK; ++c)
#pragma unroll
        for (int k = 0; k < 9; ++k)
#pragma unroll
            for (int t = 0; t < NT; ++t)
                w[c][k][t] = *reinterpret_cast<const u32x2*>(
                    a.w + ((((t0 + t) * CK + c) * 9 + k) * 64 + lane) * 4);
    f32x4 bias[NT];
#pragma unroll
    for (int t = 0; t < NT; ++t)
#pragma unroll
        for (int i = 0; i < 4; ++i) bias[t][i] = a.bias ? a.bias[(t0 + t) * 16 + kq + i] : 0.f;

    const RowLanes<PG> lanes(x0, n, a.wd);
    RowPixels<PG> raw[3][CK], msk[3][CK];
    auto fetch = [&](int slot, int row) {
        const int64_t pix = int64_t(b * a.h + (row < 0 ? 0 : row < a.h ? row : a.h - 1)) * a.wd;
#pragma unroll
        for (int c = 0; c < CK; ++c) {
            if (ONE)
                lanes.load_one(raw[slot][c], a.x + pix, kq);
            else if (c * 16 < a.xsplit)
                lanes.load(raw[slot][c], a.x + pix * a.xs + c * 16, uint32_t(a.xs), uint32_t(kq));
            else
                lanes.load(raw[slot][c], a.x2 + pix * a.xs2 + (c * 16 - a.xsplit), uint32_t(a.xs2),
                           uint32_t(kq));
            if (MASK)
                lanes.load(msk[slot][c], a.mask + pix * a.ms + c * 16, uint32_t(a.ms), uint32_t(kq));
        }
    };
    float hw[4], hb = 0.f, rms = 0.f;
    if (HEAD) {
#pragma unroll
        for (int i = 0; i < 4; ++i) hw[i] = a.head[kq + i];
        hb = a.head[16];
        rms = a.rms[b];
    }
    u32x2 op[3][CK][3 * PG];  // three input rows' operands
#pragma unroll
    for (int k = 0; k < 3; ++k) fetch(k, y0 - 1 + k);
    for (int base = y0 - 1; base <= y1; base += 3) {
#pragma unroll
        for (int u = 0; u < 3; ++u) {
            const int yi = base + u;  // input row, slot u; completes output row yi - 1
            const uint32_t row_ok = yi >= 0 && yi < a.h ? ~0u : 0u;
#pragma unroll
            for (int c = 0; c < CK; ++c)
                lanes.template taps<MASK>(raw[u][c], msk[u][c], row_ok, op[u][c], PG);
            fetch(u, yi + 3);
            if (yi - 1 < y0 || yi > y1) continue;
            f32x4 acc[PG][NT];
#pragma unroll
            for (int g = 0; g < PG; ++g)
#pragma unroll
                for (int t = 0; t < NT; ++t) acc[g][t] = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
            for (int c = 0; c < CK; ++c)
#pragma unroll
                for (int k = 0; k < 9; ++k)
#pragma unroll
                    for (int g = 0; g < PG; ++g)
#pragma unroll
                        for (int t = 0; t < NT; ++t)
                            acc[g][t] = mfma16(w[c][k][t], op[(u + 1 + k / 3) % 3][c][(k % 3) * PG + g],
                                               acc[g][t]);
            const int64_t pix = int64_t(b * a.h + yi - 1) * a.wd;
            if constexpr (HEAD) {
                double* u = a.u + int64_t(b) * a.gstride + int64_t(yi) * a.ld + 1;  // row yi - 1
#pragma unroll
                for (int g = 0; g < PG; ++g) {
                    const float y = head_pixel(acc[g][0], bias[0], hw, hb, lane);
                    if (lanes.ok[g] && kq == 0) u[lanes.px[g]] = double(y) * double(rms);
                }
                continue;
            }
#pragma unroll
            for (int g = 0; g < PG; ++g)
                if (lanes.ok[g])
#pragma unroll
                    for (int t = 0; t < NT; ++t)
                        store_pixel(a, pix + lanes.px[g], (t0 + t) * 16 + kq, acc[g][t],
                                    bias[t]);
        }
    }
}

// Many channels, fewer pixels (cin a multiple of 32: the coarser levels, with 32
// channels those of them that have too few rows for k_conv_march).
// D divides the number of chunks.  Bound by latency: an output's 9 cin / 16 MFMAs are a chain of at most 108,
// under a microsecond, but each group of them waits for its loads.  So a
// wave takes few outputs (PG x 16 pixels, NT x 16 channels) and keeps the
// operands of D chunks in flight, which it reads in the order of the chain.
// 8 samples: 128 -> 128 at 7^2 9 us, 64 -> 64 at 31^2 9 us, 192 -> 64 there
// 21 us, 96 -> 32 at 127^2 37 us (one chunk and kernel row at a time: 82, 36,
// 93 and 69 us).
template <int PG, int NT, int D, bool MASK>
__global__ __launch_bounds__(256) void k_conv_deep(ConvArgs a) {
    const int lane = threadIdx.x & 63;
    const int segs = (a.wd + 16 * PG - 1) / (16 * PG);
    const int cts = a.cout / (16 * NT);
    int r = int(blockIdx.x) * 4 + int(threadIdx.x >> 6);
    if (r >= a.batch * a.h * segs * cts) return;
    r = __builtin_amdgcn_readfirstlane(r);
    const int ct = r % cts;
    r /= cts;
    const int x0 = (r % segs) * 16 * PG;
    r /= segs;
    const int row = r % a.h, b = r / a.h;
    const int n = lane & 15, kq = (lane >> 4) * 4;
    const int chunks = a.cin / 16;
    const RowLanes<PG> lanes(x0, n, a.wd);
    RowPixels<PG> raw[D][3], msk[D][3];
    u32x2 w[D][9][NT];
    int64_t pix[3];
    uint32_t row_ok[3];
#pragma unroll
    for (int d = 0; d < 3; ++d) {
        const int yy = row + d - 1;
        row_ok[d] = yy >= 0 && yy < a.h ? ~0u : 0u;
        pix[d] = int64_t(b * a.h + (row_ok[d] ? yy : row)) * a.wd;
    }
    const bf16* wbase = a.w + int64_t(ct * NT) * chunks * 9 * 256;
    auto fetch = [&](int slot, int c) {
        const int c0 = c * 16;
        const bool first = c0 < a.xsplit;
        const bf16* xb = first ? a.x + c0 : a.x2 + (c0 - a.xsplit);
        const int64_t st = first ? a.xs : a.xs2;
#pragma unroll
        for (int d = 0; d < 3; ++d) {
            lanes.load(raw[slot][d], xb + pix[d] * st, uint32_t(st), uint32_t(kq));
            if (MASK) lanes.load(msk[slot][d], a.mask + pix[d] * a.ms + c0, uint32_t(a.ms), uint32_t(kq));
        }
#pragma unroll
        for (int k = 0; k < 9; ++k)
#pragma unroll
            for (int t = 0; t < NT; ++t)
                w[slot][k][t] = *reinterpret_cast<const u32x2*>(
                    wbase + uint32_t((((t * chunks + c) * 9 + k) * 64 + lane) * 4));
    };
    f32x4 acc[PG][NT];
#pragma unroll
    for (int g = 0; g < PG; ++g)
#pragma unroll
        for (int t = 0; t < NT; ++t) acc[g][t] = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int k = 0; k < D; ++k) fetch(k, k);
    for (int base = 0; base < chunks; base += D) {
#pragma unroll
        for (int u = 0; u < D; ++u) {
            const int c = base + u + D;  // the chunk loaded next
#pragma unroll
            for (int d = 0; d < 3; ++d) {
                u32x2 op[3 * PG];
                lanes.template taps<MASK>(raw[u][d], msk[u][d], row_ok[d], op, PG);
#pragma unroll
                for (int dx = 0; dx < 3; ++dx)
#pragma unroll
                    for (int g = 0; g < PG; ++g)
#pragma unroll
                        for (int t = 0; t < NT; ++t)
                            acc[g][t] = mfma16(w[u][d * 3 + dx][t], op[dx * PG + g], acc[g][t]);
            }
            fetch(u, c < chunks ? c : chunks - 1);
        }
    }
#pragma unroll
    for (int t = 0; t < NT; ++t) {
        const int co = (ct * NT + t) * 16 + kq;
        f32x4 bias = {0.f, 0.f, 0.f, 0.f};
        if (a.bias)
#pragma unroll
            for (int i = 0; i < 4; ++i) bias[i] = a.bias[co + i];
#pragma unroll
        for (int g = 0; g < PG; ++g)
            if (lanes.ok[g])
                store_pixel(a, int64_t(b * a.h + row) * a.wd + lanes.px[g], co, acc[g][t], bias);
    }
}

// Weight gradient dW[co][ci][tap] = sum_p dZ[p][co] * X[p + off(tap)][ci] and
// bias gradient db[co] = sum_p dZ[p][co], dZ = dY masked by (Y > 0): a
// contraction over pixels, on the 16x16x32 MFMA with M = 16 output channels,
// N = 16 input channels, K = 32 pixels of a row (the bias against ones).
// The operands need four pixels of one channel a lane, where memory has the
// channels of a pixel together: rows are loaded as they lie, 8 bytes a lane,
// put into the wave's LDS, and read back through the transposing LDS load
// (ds_read_b64_tr_b16: lane l of the 64 gets channel l%16 of pixels
// 4(l/16)+j; the three columns of taps are three addresses of one row).
// Bound by memory on the finest level (200 MB for 16 -> 16 channels at
// 511^2 x 8), so a wave takes TI x TO tiles of channels and walks down
// `rows` rows of a 32-pixel strip, loading three rows ahead: X once, dY and
// Y once.  Three rows of dZ operands stay in registers: row y of X meets
// rows y + 1, y and y - 1 of dZ.  511^2 x 8: 16 -> 16 channels 44 us, 48 ->
// 16 81 us (one wave a row with 26 two-byte loads for 16 pixels: 112-162 and
// 361 us, and 24-63 us more for the bias); 96 -> 32 at 127^2 32 us (93).
// The workgroup's four waves (consecutive bands of rows) meet in LDS and are
// added as (w0 + w1) + (w2 + w3) into the workgroup's slot
// (part[slot][cout x cin x 9, then cout]); k_reduce_slots adds the slots in a
// fixed order, so the gradient has the same bits on every run.
struct WGradArgs {
    const bf16* x;     // input channels [0, xsplit), pixel stride xs
    int64_t xs;
    const bf16* x2;    // input channels [xsplit, cin), pixel stride xs2
    int64_t xs2;
    int xsplit;
    const bf16* dy;
    int64_t dys;
    const bf16* y;  // layer output (mask), stride ys
    int64_t ys;
    float* part;
    int batch, h, wd, cin, cout, rows;
    int cin_w;      // input channels of the weight tensor (cin is padded to 16)
};

constexpr int kWgradWaves = 4;
typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));
typedef __bf16 bfx8 __attribute__((ext_vector_type(8)));

__device__ __forceinline__ f32x4 mfma32(u32x4 a, u32x4 b, f32x4 c) {
    return __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bfx8, a),
                                                   __builtin_bit_cast(bfx8, b), c, 0, 0, 0);
}

typedef __attribute__((address_space(3))) bf16x4* lds4;

// Two transposed groups of 16 pixels (16 channels, 32 bytes a pixel in LDS).
__device__ __forceinline__ u32x4 read_pixels(bf16* lane_base, int pixel) {
    const bf16x4 a = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds4)(lane_base + pixel * 16));
    const bf16x4 b = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds4)(lane_base + (pixel + 16) * 16));
    const u32x2 lo = __builtin_bit_cast(u32x2, a), hi = __builtin_bit_cast(u32x2, b);
    return u32x4{lo[0], lo[1], hi[0], hi[1]};
}

template <int TI, int TO, bool ONE = false>
__global__ __launch_bounds__(64 * kWgradWaves) void k_conv3x3_wgrad(WGradArgs a) {
    constexpr int kXElems = 34 * 16, kZElems = 32 * 16;      // one tile's row in LDS
    constexpr int kStage = TI * kXElems + TO * kZElems;      // a wave's
    constexpr int kStageBytes = kWgradWaves * kStage * 2;
    constexpr int kSumBytes = kWgradWaves * 9 * 256 * 4;
    __shared__ __attribute__((aligned(16))) char smem[kStageBytes > kSumBytes ? kStageBytes : kSumBytes];
    const int lane = threadIdx.x & 63;
    const int wv = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int cig = a.cin / (16 * TI), cog = a.cout / (16 * TO);
    const int strips = (a.wd + 31) / 32;
    const int groups = (a.h + a.rows * kWgradWaves - 1) / (a.rows * kWgradWaves);
    int r = blockIdx.x;  // the grid is exactly batch x groups x strips x cig x cog
    const int co_t = (r % cog) * TO;
    r /= cog;
    const int ci_t = (r % cig) * TI;
    r /= cig;
    const int strip = r % strips;
    r /= strips;
    const int group = r % groups, b = r / groups;
    const int x0 = strip * 32;
    const int y0 = (group * kWgradWaves + wv) * a.rows;
    const int y1 = y0 + a.rows < a.h ? y0 + a.rows : a.h;
    const int n = lane & 15, kq = (lane >> 4) * 4;

    f32x4 acc[TI][TO][9], accb[TO];
#pragma unroll
    for (int to = 0; to < TO; ++to) {
        accb[to] = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
        for (int ti = 0; ti < TI; ++ti)
#pragma unroll
            for (int t = 0; t < 9; ++t) acc[ti][to][t] = f32x4{0.f, 0.f, 0.f, 0.f};
    }
    if (y0 < a.h) {
        bf16* stage = reinterpret_cast<bf16*>(smem) + wv * kStage;
        bf16* zstage = stage + TI * kXElems;
        const RowLanes<2> lanes(x0, n, a.wd);
        // pixel x = wd of the strip is no pixel: X one column left of it is kept out
        u32x4 inside;
#pragma unroll
        for (int k = 0; k < 4; ++k) {
            const int x = x0 + (k >> 1) * 16 + kq + (k & 1) * 2;
            inside[k] = (x < a.wd ? 0xffffu : 0u) | (x + 1 < a.wd ? 0xffff0000u : 0u);
        }
        RowPixels<2> rx[3][TI];
        u32x2 rdy[3][TO][2], ry[3][TO][2];
        // row `row` of X and the row below it of dY and Y
        auto fetch = [&](int slot, int row) {
            const int64_t px = int64_t(b * a.h + (row < 0 ? 0 : row < a.h ? row : a.h - 1)) * a.wd;
            const int64_t pz = int64_t(b * a.h + (row + 1 < a.h ? row + 1 : a.h - 1)) * a.wd;
#pragma unroll
            for (int ti = 0; ti < TI; ++ti) {
                const int c0 = (ci_t + ti) * 16;
                if (ONE)
                    lanes.load_one(rx[slot][ti], a.x + px, kq);
                else if (c0 < a.xsplit)
                    lanes.load(rx[slot][ti], a.x + px * a.xs + c0, uint32_t(a.xs), uint32_t(kq));
                else
                    lanes.load(rx[slot][ti], a.x2 + px * a.xs2 + (c0 - a.xsplit), uint32_t(a.xs2),
                               uint32_t(kq));
            }
#pragma unroll
            for (int to = 0; to < TO; ++to)
#pragma unroll
                for (int g = 0; g < 2; ++g) {
                    const uint32_t c0 = uint32_t((co_t + to) * 16 + kq), p = uint32_t(lanes.px[g]);
                    rdy[slot][to][g] = *reinterpret_cast<const u32x2*>(
                        a.dy + pz * a.dys + (p * uint32_t(a.dys) + c0));
                    ry[slot][to][g] = *reinterpret_cast<const u32x2*>(
                        a.y + pz * a.ys + (p * uint32_t(a.ys) + c0));
                }
        };
        u32x4 dz[3][TO];
#pragma unroll
        for (int k = 0; k < 3; ++k)
#pragma unroll
            for (int to = 0; to < TO; ++to) dz[k][to] = u32x4{0u, 0u, 0u, 0u};
        const u32x4 ones = {0x3f803f80u, 0x3f803f80u, 0x3f803f80u, 0x3f803f80u};
#pragma unroll
        for (int k = 0; k < 3; ++k) fetch(k, y0 - 1 + k);
        for (int base = y0 - 1; base <= y1; base += 3) {
#pragma unroll
            for (int u = 0; u < 3; ++u) {
                const int yi = base + u;
                const uint32_t row_ok = yi >= 0 && yi < a.h ? ~0u : 0u;
#pragma unroll
                for (int ti = 0; ti < TI; ++ti) {
                    bf16* p = stage + ti * kXElems + kq;
#pragma unroll
                    for (int g = 0; g < 2; ++g)
                        *reinterpret_cast<u32x2*>(p + (g * 16 + n + 1) * 16) =
                            rx[u][ti].v[g] & (lanes.ok[g] & row_ok);
                    if (n == 0 || n == 15)
                        *reinterpret_cast<u32x2*>(p + (n == 0 ? 0 : 33) * 16) =
                            rx[u][ti].v[2] & (lanes.ok[2] & row_ok);
                }
#pragma unroll
                for (int to = 0; to < TO; ++to)
#pragma unroll
                    for (int g = 0; g < 2; ++g) {
                        u32x2 v = rdy[u][to][g] & lanes.ok[g];
                        v[0] &= positive(ry[u][to][g][0]);
                        v[1] &= positive(ry[u][to][g][1]);
                        *reinterpret_cast<u32x2*>(zstage + to * kZElems + (g * 16 + n) * 16 + kq) = v;
                    }
                fetch(u, yi + 3);
                // the wave's own LDS, in order: no barrier, but no reordering either
                __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
                __builtin_amdgcn_wave_barrier();
                u32x4 xo[TI][3];
#pragma unroll
                for (int ti = 0; ti < TI; ++ti) {
#pragma unroll
                    for (int dx = 0; dx < 3; ++dx)
                        xo[ti][dx] = read_pixels(stage + ti * kXElems + lane * 4, dx);
                    xo[ti][0] &= inside;
                }
#pragma unroll
                for (int to = 0; to < TO; ++to)
                    dz[u][to] = read_pixels(zstage + to * kZElems + lane * 4, 0);
                __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
                __builtin_amdgcn_wave_barrier();
                if (row_ok)
#pragma unroll
                    for (int d = 0; d < 3; ++d) {
                        const int row = yi + 1 - d;  // of dZ
                        if (row < y0 || row >= y1) continue;
#pragma unroll
                        for (int ti = 0; ti < TI; ++ti)
#pragma unroll
                            for (int to = 0; to < TO; ++to)
#pragma unroll
                                for (int dx = 0; dx < 3; ++dx)
                                    acc[ti][to][d * 3 + dx] = mfma32(dz[(u + 3 - d) % 3][to], xo[ti][dx],
                                                                     acc[ti][to][d * 3 + dx]);
                    }
                if (ci_t == 0 && yi >= y0 && yi < y1)
#pragma unroll
                    for (int to = 0; to < TO; ++to) accb[to] = mfma32(dz[(u + 2) % 3][to], ones, accb[to]);
            }
        }
    }
    // per pair of tiles: [wave][tap][co][ci] in LDS, then the sum over the waves
    float* sh = reinterpret_cast<float*>(smem);
    const int64_t wcount = int64_t(a.cout) * a.cin_w * 9;
    float* slot = a.part + ((int64_t(b) * groups + group) * strips + strip) * (wcount + a.cout);
#pragma unroll
    for (int ti = 0; ti < TI; ++ti)
#pragma unroll
        for (int to = 0; to < TO; ++to) {
            __syncthreads();
#pragma unroll
            for (int t = 0; t < 9; ++t)
#pragma unroll
                for (int i = 0; i < 4; ++i) sh[((wv * 9 + t) * 16 + kq + i) * 16 + n] = acc[ti][to][t][i];
            __syncthreads();
            for (int e = threadIdx.x; e < 16 * 16 * 9; e += 64 * kWgradWaves) {
                const int tap = e % 9, ci = (e / 9) % 16, co = e / 144;
                const float* p = sh + (tap * 16 + co) * 16 + ci;
                const float v = (p[0] + p[9 * 256]) + (p[2 * 9 * 256] + p[3 * 9 * 256]);
                const int ci_g = (ci_t + ti) * 16 + ci, co_g = (co_t + to) * 16 + co;
                if (ci_g < a.cin_w) slot[(int64_t(co_g) * a.cin_w + ci_g) * 9 + tap] = v;
            }
        }
    if (ci_t != 0) return;
    __syncthreads();
    if (n == 0)
#pragma unroll
        for (int to = 0; to < TO; ++to)
#pragma unroll
            for (int i = 0; i < 4; ++i) sh[(wv * TO + to) * 16 + kq + i] = accb[to][i];
    __syncthreads();
    if (threadIdx.x < TO * 16) {
        const float* p = sh + threadIdx.x;
        slot[wcount + co_t * 16 + threadIdx.x] =
            (p[0] + p[TO * 16]) + (p[2 * TO * 16] + p[3 * TO * 16]);
    }
}

// out[e] = sum over slots k = 0 .. nparts-1 of part[k * count + e], in a
// fixed order: one block per element, thread t adds slots t, t + 256, ...
// in turn, then a fixed tree over the block (no atomics: the same bits on
// every run).
__global__ __launch_bounds__(256) void k_reduce_parts(const float* __restrict__ part,
                                                      int64_t nparts, int64_t count,
                                                      float* __restrict__ out) {
    const int64_t e = blockIdx.x;
    float s = 0.f;
    // eight loads at a time, added in slot order
    for (int64_t k0 = threadIdx.x; k0 < nparts; k0 += 8 * 256) {
        float v[8];
#pragma unroll
        for (int i = 0; i < 8; ++i) v[i] = k0 + i * 256 < nparts ? part[(k0 + i * 256) * count + e] : 0.f;
#pragma unroll
        for (int i = 0; i < 8; ++i)
            if (k0 + i * 256 < nparts) s += v[i];
    }
    __shared__ float sh[256];
    sh[threadIdx.x] = s;
    __syncthreads();
    for (int st = 128; st > 0; st >>= 1) {
        if (int(threadIdx.x) < st) sh[threadIdx.x] += sh[threadIdx.x + st];
        __syncthreads();
    }
    if (threadIdx.x == 0) out[e] = sh[0];
}

// The same sums for many elements and several layers at once (all of them, where
// their partial sums fit the workspace's share), coalesced: `ways`
// waves share 64 consecutive elements of a layer, taking the slots w, w +
// ways, ... (64 consecutive floats of a slot at a time, four partial sums),
// whose sums are added in the waves' order.  A block of 16 waves takes 64
// elements of a layer with many slots (16 ways), 256 of one with up to 64,
// which would leave most waves a single load.  A fixed order again.  (A launch a layer
// took 4.5 to 7 us, 14 times, 76 in all at 511^2 x 8; 16 ways throughout 46; now
// 29.)
constexpr int kReduceWaves = 16;
constexpr int kMaxLayers = 16;

struct ReduceArgs {
    int layers = 0;
    struct {
        const float* part;
        float* out;
        int64_t slots, count;
        int first;  // block
        int ways;   // 16 or 4
    } l[kMaxLayers];
};

__global__ __launch_bounds__(64 * kReduceWaves) void k_reduce_slots(ReduceArgs a) {
    int layer = a.layers - 1;
    while (layer > 0 && int(blockIdx.x) < a.l[layer].first) --layer;
    const auto& L = a.l[layer];
    const float* __restrict__ part = L.part;
    const int64_t nparts = L.slots, count = L.count;
    const int ways = L.ways;
    const int l = threadIdx.x & 63, w = threadIdx.x >> 6, g = w & (ways - 1);
    const int64_t e = int64_t(int(blockIdx.x) - L.first) * (64 * (kReduceWaves / ways)) +
                      (w / ways) * 64 + l;
    float acc[4] = {0.f, 0.f, 0.f, 0.f};
    if (e < count)
        for (int64_t k = g; k < nparts; k += 4 * ways) {
            float v[4];
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                const int64_t ki = k + int64_t(i) * ways;
                v[i] = ki < nparts ? part[ki * count + e] : 0.f;
            }
#pragma unroll
            for (int i = 0; i < 4; ++i) acc[i] += v[i];
        }
    __shared__ float sh[kReduceWaves][64];
    sh[w][l] = (acc[0] + acc[1]) + (acc[2] + acc[3]);
    __syncthreads();
    if (g == 0 && e < count) {
        float s = sh[w][l];
        for (int k = 1; k < ways; ++k) s += sh[w + k][l];
        L.out[e] = s;
    }
}

// Grid transfers between levels coarsened by a factor F (2 or 4): fine
// n_f = F n_c + F - 1, and coarse interior point (I, J) (0-based) sits on
// fine interior point (F I + F - 1, F J + F - 1).  Restriction averages the
// fine points within F - 1 of that point with the separable weights
// (F - |d|) / F^2 per axis (full weighting for F = 2: (1, 2, 1) / 4);
// prolongation is bilinear interpolation, P = F^2 R^T (1-D weights
// (F - |d|) / F).  Per channel, scaled by `scale`; accumulate != 0 adds into
// the output instead of overwriting.
// One thread per (pixel, group of 8 channels): 16-byte loads and stores,
// the index split and the weights formed once per 8 channels.  The host
// keeps batch x pixels x c / 8 (and the grid) below 2^32 (32-bit indexing)
// and c, the pixel strides and the base addresses in whole groups of 8.
struct bf16x8 {
    uint4 v;
    __device__ float get(int k) const {
        const uint32_t w = (&v.x)[k >> 1];
        return __uint_as_float((k & 1) ? (w & 0xffff0000u) : (w << 16));
    }
};

__device__ __forceinline__ bf16x8 load8(const bf16* p) {
    return bf16x8{*reinterpret_cast<const uint4*>(p)};
}

// F (the coarsening factor, 2 or 4) is a template parameter so that the
// window loops unroll and their loads are in flight together.
template <int F>
__global__ __launch_bounds__(256) void k_restrict(const bf16* in, int64_t is, bf16* out, int64_t os,
                                                  int batch, int nc, int c, float scale,
                                                  int accumulate) {
    const int c8 = c / 8;
    const uint32_t idx = blockIdx.x * 256u + threadIdx.x;
    const uint32_t total = uint32_t(batch) * uint32_t(nc) * uint32_t(nc) * uint32_t(c8);
    if (idx >= total) return;
    const int ch = int(idx % uint32_t(c8)) * 8;
    uint32_t r = idx / uint32_t(c8);
    const int J = int(r % uint32_t(nc));
    r /= uint32_t(nc);
    const int I = int(r % uint32_t(nc));
    const int b = int(r / uint32_t(nc));
    const int nf = F * nc + F - 1;
    const int ci = F * I + F - 1, cj = F * J + F - 1;
    float s[8];
#pragma unroll
    for (int k = 0; k < 8; ++k) s[k] = 0.f;
#pragma unroll
    for (int di = 1 - F; di < F; ++di) {
        const float wi = float(F - (di < 0 ? -di : di));
        const bf16* row = in + ((int64_t(b) * nf + ci + di) * nf + cj) * is + ch;
        float t[8];
#pragma unroll
        for (int k = 0; k < 8; ++k) t[k] = 0.f;
#pragma unroll
        for (int dj = 1 - F; dj < F; ++dj) {
            const float wj = float(F - (dj < 0 ? -dj : dj));
            const bf16x8 x = load8(row + dj * is);
#pragma unroll
            for (int k = 0; k < 8; ++k) t[k] += wj * x.get(k);
        }
#pragma unroll
        for (int k = 0; k < 8; ++k) s[k] += wi * t[k];
    }
    bf16* o = out + ((int64_t(b) * nc + I) * nc + J) * os + ch;
    bf16x8 prev = accumulate ? load8(o) : bf16x8{make_uint4(0, 0, 0, 0)};
#pragma unroll
    for (int k = 0; k < 8; ++k) {
        s[k] *= scale / float(F * F * F * F);
        if (accumulate) s[k] += prev.get(k);
    }
    *reinterpret_cast<uint4*>(o) = make_uint4(pack2(s[0], s[1]), pack2(s[2], s[3]), pack2(s[4], s[5]),
                                              pack2(s[6], s[7]));
}

// One thread per coarse interval of a fine row: the F fine points from the
// coarse point J on (J = -1: the F - 1 points before the first) and 8
// channels, from the same two coarse columns; the row's coarse rows and
// weights are the block's.  The weights are multiples of 1 / F^2, so a
// product is exact and the FMA rounds as the sum does; a neighbour outside
// the grid counts as 0, which changes no sum.  One fine point a thread took
// its index apart by three divisions and was bound by the vector unit: 65 us
// for 32 channels to 511^2 x 8 (134 MB), now 33 us.
template <int F>
__global__ __launch_bounds__(256) void k_prolong(const bf16* in, int64_t is, bf16* out, int64_t os,
                                                 int nc, int c8_shift, float scale, int accumulate) {
    const int nf = F * nc + F - 1;
    const int idx = int(blockIdx.x) * 256 + int(threadIdx.x);
    const int ch = (idx & ((1 << c8_shift) - 1)) * 8;
    const int J = (idx >> c8_shift) - 1;
    if (J >= nc) return;
    const int i = blockIdx.y, b = blockIdx.z;
    const int I = (i + 1) / F - 1, ki = (i + 1) % F;
    const float invF = 1.f / float(F);
    float x[2][2][8];  // coarse rows I and I + 1, columns J and J + 1
#pragma unroll
    for (int r = 0; r < 2; ++r) {
        const bool row_ok = I + r >= 0 && I + r < nc && (r == 0 || ki != 0);
#pragma unroll
        for (int q = 0; q < 2; ++q) {
            bf16x8 v{make_uint4(0, 0, 0, 0)};
            if (row_ok && J + q >= 0 && J + q < nc)
                v = load8(in + ((int64_t(b) * nc + I + r) * nc + J + q) * is + ch);
#pragma unroll
            for (int k = 0; k < 8; ++k) x[r][q][k] = v.get(k);
        }
    }
    const float wi[2] = {float(F - ki) * invF, float(ki) * invF};
    bf16* o = out + ((int64_t(b) * nf + i) * nf + F * (J + 1) - 1) * os + ch;
#pragma unroll
    for (int kj = 0; kj < F; ++kj) {
        if (kj == 0 && J < 0) continue;
        const float wj[2] = {float(F - kj) * invF, float(kj) * invF};
        float s[8];
#pragma unroll
        for (int k = 0; k < 8; ++k) s[k] = 0.f;
#pragma unroll
        for (int r = 0; r < 2; ++r)
#pragma unroll
            for (int q = 0; q < (kj == 0 ? 1 : 2); ++q)
#pragma unroll
                for (int k = 0; k < 8; ++k) s[k] = fmaf(wi[r] * wj[q], x[r][q][k], s[k]);
        const bf16x8 prev = accumulate ? load8(o + kj * os) : bf16x8{make_uint4(0, 0, 0, 0)};
#pragma unroll
        for (int k = 0; k < 8; ++k) {
            s[k] *= scale;
            if (accumulate) s[k] += prev.get(k);
        }
        *reinterpret_cast<uint4*>(o + kj * os) = make_uint4(
            pack2(s[0], s[1]), pack2(s[2], s[3]), pack2(s[4], s[5]), pack2(s[6], s[7]));
    }
}

// Sum of one double per thread over a block of 256, by a fixed tree; every
// thread gets the total.
__device__ __forceinline__ double block_sum_f64(double v) {
    __shared__ double sh[256];
    sh[threadIdx.x] = v;
    __syncthreads();
    for (int st = 128; st > 0; st >>= 1) {
        if (int(threadIdx.x) < st) sh[threadIdx.x] += sh[threadIdx.x + st];
        __syncthreads();
    }
    const double total = sh[0];
    __syncthreads();
    return total;
}

// Per-sample rms of f over the interior, FP64 sums in a fixed order: one
// block per (sample, interior row) adds the row's squares (thread t takes
// columns t, t + 256, ..., then a tree), then one block per sample adds its
// rows' sums the same way.
__global__ __launch_bounds__(256) void k_rms_rows(const double* f, int n, int64_t ld,
                                                  int64_t gstride, double* part) {
    const int b = int(blockIdx.x) / n, row = int(blockIdx.x) % n;
    const double* fr = f + int64_t(b) * gstride + int64_t(row + 1) * ld + 1;
    double s = 0.0;
    for (int j = threadIdx.x; j < n; j += 256) {
        const double v = fr[j];
        s += v * v;
    }
    s = block_sum_f64(s);
    if (threadIdx.x == 0) part[blockIdx.x] = s;
}

__global__ __launch_bounds__(256) void k_rms_final(const double* part, int n, float* rms) {
    const int b = blockIdx.x;
    double s = 0.0;
    for (int r = threadIdx.x; r < n; r += 256) s += part[int64_t(b) * n + r];
    s = block_sum_f64(s);
    if (threadIdx.x == 0) {
        const double r = sqrt(s / (double(n) * n));
        rms[b] = r > 0.0 ? float(r) : 1.f;
    }
}

// Network input f / rms, one channel (the first convolution's 15 others are
// zeros that it does not load).
__global__ __launch_bounds__(256) void k_input(const double* f, int n, int64_t ld, int64_t gstride,
                                               const float* rms, bf16* x) {
    const int j = int(blockIdx.x) * 256 + int(threadIdx.x), i = blockIdx.y, b = blockIdx.z;
    if (j >= n) return;
    const float v = float(f[int64_t(b) * gstride + int64_t(i + 1) * ld + j + 1] / double(rms[b]));
    x[(int64_t(b) * n + i) * n + j] = f2bf(v);
}

// Head: y[p] = sum_c w[c] d[p][c] + b (FP32 out).  c = 16 channels at
// pixel stride ds (a multiple of 8, 16-byte aligned rows): two 16-byte
// loads per pixel.
__global__ __launch_bounds__(256) void k_head(const bf16* d, int64_t ds, const float* w,
                                              const float* bias, float* y, int64_t npix) {
    const int64_t p = int64_t(blockIdx.x) * 256 + threadIdx.x;
    if (p >= npix) return;
    const bf16x8 lo = load8(d + p * ds), hi = load8(d + p * ds + 8);
    float s = bias[0];
#pragma unroll
    for (int ch = 0; ch < 16; ++ch) s += w[ch] * (ch < 8 ? lo.get(ch) : hi.get(ch - 8));
    y[p] = s;
}

// MSE against u*/rms: dy = 2 (y - t) / count, loss accumulated in FP32.
__global__ __launch_bounds__(256) void k_mse(const float* y, const double* u, const float* rms,
                                             int n, int64_t ld, int64_t gstride, int batch,
                                             float* dy, float* loss_part) {
    const int64_t idx = int64_t(blockIdx.x) * 256 + threadIdx.x;
    const int64_t count = int64_t(batch) * n * n;
    float d = 0.f;
    if (idx < count) {  // (count < 2^31)
        const uint32_t px = uint32_t(n) * uint32_t(n);
        const int b = int(uint32_t(idx) / px);
        const uint32_t k = uint32_t(idx) % px;
        const int64_t i = k / uint32_t(n) + 1, j = k % uint32_t(n) + 1;
        const float t = float(u[int64_t(b) * gstride + i * ld + j] / double(rms[b]));
        d = y[idx] - t;
        dy[idx] = 2.f * d / float(count);
    }
    __shared__ float sh[256];
    sh[threadIdx.x] = d * d;
    __syncthreads();
    for (int st = 128; st > 0; st >>= 1) {
        if (threadIdx.x < st) sh[threadIdx.x] += sh[threadIdx.x + st];
        __syncthreads();
    }
    if (threadIdx.x == 0) loss_part[blockIdx.x] = sh[0] / float(count);
}

// Head backward: dd[p][c] = w[c] dy[p] (BF16); per block, the partial sums
// of dy d[c] (c < 16) and of dy go to part[block][0..16] (k_reduce_parts
// adds the blocks in order into dw[0..15], db = dw[16]).  A thread adds its
// kHeadPixels pixels, then a fixed butterfly over each wave's 64 lanes, then
// the four waves in order: a butterfly of 17 sums for every pixel was what
// bound this kernel (43 us at 511^2 x 8, now 31).  d and dd: 16 channels
// at pixel strides that are multiples of 8, moved as two 16-byte accesses
// per pixel.
constexpr int kHeadPixels = 8;

__global__ __launch_bounds__(256) void k_head_grad(const bf16* d, int64_t ds, const float* w,
                                                   const float* dy, bf16* dd, int64_t dds,
                                                   float* part, int64_t npix) {
    const int64_t p0 = int64_t(blockIdx.x) * (256 * kHeadPixels) + threadIdx.x;
    float v[17];
#pragma unroll
    for (int ch = 0; ch < 17; ++ch) v[ch] = 0.f;
#pragma unroll 4
    for (int k = 0; k < kHeadPixels; ++k) {
        const int64_t p = p0 + k * 256;
        if (p >= npix) continue;
        const float g = dy[p];
        const bf16x8 x[2] = {load8(d + p * ds), load8(d + p * ds + 8)};
#pragma unroll
        for (int h = 0; h < 2; ++h) {
            float o[8];
#pragma unroll
            for (int ch = 0; ch < 8; ++ch) {
                o[ch] = w[8 * h + ch] * g;
                v[8 * h + ch] += g * x[h].get(ch);
            }
            *reinterpret_cast<uint4*>(dd + p * dds + 8 * h) = make_uint4(
                pack2(o[0], o[1]), pack2(o[2], o[3]), pack2(o[4], o[5]), pack2(o[6], o[7]));
        }
        v[16] += g;
    }
#pragma unroll
    for (int off = 32; off > 0; off >>= 1)
#pragma unroll
        for (int k = 0; k < 17; ++k) v[k] += __shfl_xor(v[k], off, 64);
    __shared__ float sw[4][17];
    const int lane = threadIdx.x & 63, wv = threadIdx.x >> 6;
    if (lane == 0)
#pragma unroll
        for (int k = 0; k < 17; ++k) sw[wv][k] = v[k];
    __syncthreads();
    if (threadIdx.x < 17)
        part[int64_t(blockIdx.x) * 17 + threadIdx.x] =
            ((sw[0][threadIdx.x] + sw[1][threadIdx.x]) + sw[2][threadIdx.x]) + sw[3][threadIdx.x];
}

// Master FP32 weights [co][ci][9] -> BF16 operands of the convolutions:
// forward (input channels zero-padded to cin_p), and backward-data (rows ci,
// columns co, taps flipped; not for the first layer, whose input has no
// gradient).  An operand is one 512-byte line, [tile of 16 rows][chunk of 16
// columns][tap][lane][4]: a lane's four columns of one row (ConvArgs); as
// [row][tap][column] each 8-byte load touched 16 lines.  One launch for all
// layers: a layer's elements start at block `first`.
struct PrepArgs {
    const float* param;
    int layers;
    struct {
        size_t w_off;
        bf16 *wf, *wb;
        int cout, cin, cin_p, first;
    } l[kMaxLayers];
};

__device__ __forceinline__ int64_t operand_index(int row, int tap, int col, int cols) {
    const int lane = ((col & 15) >> 2) * 16 + (row & 15);
    return (((int64_t(row >> 4) * (cols >> 4) + (col >> 4)) * 9 + tap) * 64 + lane) * 4 + (col & 3);
}

__global__ __launch_bounds__(256) void k_prep_weights(PrepArgs a) {
    int k = a.layers - 1;
    while (k > 0 && int(blockIdx.x) < a.l[k].first) --k;
    const auto& L = a.l[k];
    const int idx = (int(blockIdx.x) - L.first) * 256 + int(threadIdx.x);
    if (idx >= L.cout * L.cin_p * 9) return;
    const int ci = idx % L.cin_p;
    const int tap = (idx / L.cin_p) % 9;
    const int co = idx / (L.cin_p * 9);
    const bf16 v = ci < L.cin ? f2bf(a.param[L.w_off + (int64_t(co) * L.cin + ci) * 9 + tap]) : bf16(0);
    L.wf[operand_index(co, tap, ci, L.cin_p)] = v;
    if (L.wb && ci < L.cin) L.wb[operand_index(ci, 8 - tap, co, L.cout)] = v;
}

// Adam: b1, b2 and their complements 1 - b1, 1 - b2 and the bias corrections
// c1 = 1 - b1^t, c2 = 1 - b2^t are formed in FP64 on the host and rounded
// once (1 - b2^t in binary32 loses four digits to cancellation at small t).
__global__ __launch_bounds__(256) void k_adam(float* p, const float* g, float* m, float* v,
                                              int64_t count, float lr, float b1, float omb1,
                                              float b2, float omb2, float eps, float c1, float c2) {
    const int64_t k = int64_t(blockIdx.x) * 256 + threadIdx.x;
    if (k >= count) return;
    const float gk = g[k];
    const float mk = b1 * m[k] + omb1 * gk;
    const float vk = b2 * v[k] + omb2 * gk * gk;
    m[k] = mk;
    v[k] = vk;
    p[k] -= lr * (mk / c1) / (sqrtf(vk / c2) + eps);
}

__global__ __launch_bounds__(256) void k_fill(uint32_t* p, int64_t words) {
    const int64_t k = int64_t(blockIdx.x) * 256 + threadIdx.x;
    if (k < words) p[k] = 0u;
}

}  // namespace nn
}  // namespace rbgs

// ===========================================================================
// Host side: the network object and the C ABI.
// ===========================================================================
namespace rbgs {
namespace nn {
namespace {

constexpr int kLevels = 4;
constexpr int kC[kLevels] = {16, 32, 64, 128};

struct Layer {
    const char* name;
    int cin, cin_p, cout, level;
    size_t w_off, b_off;  // float offsets in the master parameter vector
    bf16* wf = nullptr;   // forward operands
    bf16* wb = nullptr;   // operands of the input gradient (flipped taps)
};

// Parameter order and shapes: each conv's weight (cout, cin, 3, 3) then its
// bias (cout), in the order enc0.0 ... enc3.1, dec2.0 ... dec0.1, head.
std::vector<Layer> make_layers(size_t* count) {
    std::vector<Layer> L;
    auto add = [&](const char* name, int cin, int cout, int level) {
        Layer l;
        l.name = name;
        l.cin = cin;
        l.cin_p = cin < 16 ? 16 : cin;
        l.cout = cout;
        l.level = level;
        L.push_back(l);
    };
    add("enc0.0", 1, 16, 0);
    add("enc0.1", 16, 16, 0);
    add("enc1.0", 16, 32, 1);
    add("enc1.1", 32, 32, 1);
    add("enc2.0", 32, 64, 2);
    add("enc2.1", 64, 64, 2);
    add("enc3.0", 64, 128, 3);
    add("enc3.1", 128, 128, 3);
    add("dec2.0", 192, 64, 2);
    add("dec2.1", 64, 64, 2);
    add("dec1.0", 96, 32, 1);
    add("dec1.1", 32, 32, 1);
    add("dec0.0", 48, 16, 0);
    add("dec0.1", 16, 16, 0);
    size_t off = 0;
    for (auto& l : L) {
        l.w_off = off;
        off += size_t(l.cout) * l.cin * 9;
        l.b_off = off;
        off += l.cout;
    }
    *count = off + 16 + 1;  // head weight (1, 16, 1, 1) and bias
    return L;
}

}  // namespace

struct Net {
    int n[kLevels];
    int factor = 2;  // coarsening factor between levels (2 or 4)
    int batch;
    std::vector<Layer> layers;
    size_t nparam;
    float *param, *grad, *m, *v, *rms, *loss, *y, *dy;
    float* parts = nullptr;  // partial sums of the fixed-order gradient reductions
    size_t parts_floats = 0;
    double* guess;  // natural-layout scratch grid for the learned solve
    int adam_t = 0;
    // activations (level-indexed) and their gradients
    // (enc: the encoder's outputs; up: the prolongations beside them)
    bf16 *in[kLevels], *aenc[kLevels], *enc[kLevels], *up[kLevels - 1], *adec[kLevels - 1],
        *d[kLevels - 1];
    bf16 *gd[kLevels - 1], *genc[kLevels], *gup[kLevels - 1], *gadec[kLevels - 1], *gaenc[kLevels],
        *gin[kLevels];
    size_t total = 0;
};

namespace {

int in_channels(int l) { return l == 0 ? 1 : kC[l - 1]; }

// How the weight gradient of a layer is split: TI x TO channel tiles and
// `rows` rows of a 32-pixel strip a wave.  Few rows read the two beside them
// too often and leave many slots to add, so as many as fill 256 CUs once
// with the workgroups that fit (three of one tile, one of three or four, by
// their registers), and at least four.
struct WgradSplit {
    int ti, to, rows;
    int64_t strips, groups;  // per sample; a slot each
};

WgradSplit wgrad_split(int batch, int n, int cin_p, int cout) {
    WgradSplit p;
    const int cit = cin_p / 16, cot = cout / 16;
    p.strips = (n + 31) / 32;
    const int64_t strip_rows = int64_t(batch) * p.strips * n;
    p.ti = cit == 3 ? 3 : 1;
    p.to = 1;
    // operands loaded half as often, where that leaves enough waves (8 samples
    // of 127^2, 32 -> 32: 20 us against 38; of 31^2 there are too few)
    if (cit % 2 == 0 && cot % 2 == 0 && strip_rows * (cit / 2) * (cot / 2) >= 2048) p.ti = p.to = 2;
    const int64_t column = batch * p.strips * (cit / p.ti) * (cot / p.to);  // workgroups
    const int64_t fit = p.ti * p.to == 1 ? 768 : 256;
    const int64_t bands = std::max<int64_t>(fit / column, 1) * kWgradWaves;
    p.rows = int(std::max<int64_t>((n + bands - 1) / bands, 4));
    p.groups = (n + int64_t(p.rows) * kWgradWaves - 1) / (int64_t(p.rows) * kWgradWaves);
    return p;
}

// Floats of partial sums a layer's gradients need: a slot of cout x cin x 9 and
// cout per workgroup, for the batch that has most.
size_t wgrad_floats(const Net& net, const Layer& l) {
    size_t most = 0;
    for (int b = 1; b <= net.batch; ++b) {
        const WgradSplit p = wgrad_split(b, net.n[l.level], l.cin_p, l.cout);
        most = std::max(most, size_t(b) * size_t(p.strips * p.groups));
    }
    return most * (size_t(l.cout) * size_t(l.cin) * 9 + size_t(l.cout));
}

// Floats of partial sums the fixed-order reductions need: the layers' gradients, the
// head (blocks of 17), the loss and the rms row sums.  The layers' stay until one
// launch adds them all, where that takes at most an eighth of what the rest of the
// workspace does (`others` bytes); else two and a half times the largest layer's,
// with a launch whenever they are full (grad_reduce).  511^2 x 8 with factor 4, 75 MB:
// one launch; 127^2 x 1024, whose layers need 2.1 GB together, 1.5 GB and two.
size_t parts_floats(const Net& net, size_t others) {
    size_t largest = 0, all = 0;
    const size_t B = size_t(net.batch);
    for (const auto& l : net.layers) {
        const size_t f = wgrad_floats(net, l);
        largest = std::max(largest, f);
        all += f;
    }
    size_t most = std::min(all, std::max(largest * 5 / 2, others / 8 / sizeof(float)));
    const size_t px0 = B * size_t(net.n[0]) * size_t(net.n[0]);
    most = std::max(most, (px0 + 255) / 256 * 17);
    most = std::max(most, 2 * B * size_t(net.n[0]));  // the rms row sums (doubles)
    return most;
}

// Carves every buffer; with base == nullptr only computes the size.
size_t carve(Net& net, char* base) {
    size_t off = 0;
    auto take = [&](size_t bytes) {
        char* p = base ? base + off : nullptr;
        off += align256(bytes);
        return p;
    };
    const int64_t B = net.batch;
    net.param = reinterpret_cast<float*>(take(net.nparam * 4));
    net.grad = reinterpret_cast<float*>(take(net.nparam * 4));
    net.m = reinterpret_cast<float*>(take(net.nparam * 4));
    net.v = reinterpret_cast<float*>(take(net.nparam * 4));
    for (auto& l : net.layers) {
        l.wf = reinterpret_cast<bf16*>(take(size_t(l.cout) * 9 * l.cin_p * 2));
        l.wb = reinterpret_cast<bf16*>(take(size_t(l.cin) * 9 * l.cout * 2));
    }
    net.rms = reinterpret_cast<float*>(take(B * 4));
    net.loss = reinterpret_cast<float*>(take(4));
    const int64_t px0 = int64_t(net.n[0]) * net.n[0];
    net.y = reinterpret_cast<float*>(take(B * px0 * 4));
    net.dy = reinterpret_cast<float*>(take(B * px0 * 4));
    net.guess = reinterpret_cast<double*>(take(size_t(net.n[0] + 2) * (net.n[0] + 2) * 8));
    for (int l = 0; l < kLevels; ++l) {
        const int64_t px = B * net.n[l] * net.n[l];
        auto act = [&](int ch) { return reinterpret_cast<bf16*>(take(size_t(px) * ch * 2)); };
        net.in[l] = act(in_channels(l));
        net.aenc[l] = act(kC[l]);
        net.gaenc[l] = act(kC[l]);
        net.gin[l] = act(in_channels(l));
        net.enc[l] = act(kC[l]);
        net.genc[l] = act(kC[l]);
        if (l < kLevels - 1) {
            net.up[l] = act(kC[l + 1]);
            net.gup[l] = act(kC[l + 1]);
            net.adec[l] = act(kC[l]);
            net.gadec[l] = act(kC[l]);
            net.d[l] = act(kC[l]);
            net.gd[l] = act(kC[l]);
        }
    }
    net.parts_floats = parts_floats(net, off);
    net.parts = reinterpret_cast<float*>(take(net.parts_floats * 4));
    return off;
}

unsigned blocks_for(int64_t items, int per_block = 256) {
    return unsigned((items + per_block - 1) / per_block);
}

// A convolution's channels in memory: one tensor, or two side by side.
template <typename P>
struct Channels {
    P a;
    int ca;  // channels (and pixel stride) of a
    P b = nullptr;
    int cb = 0;
    int count() const { return ca + cb; }
};
typedef Channels<const bf16*> In;
typedef Channels<bf16*> Out;

template <bool MASK>
hipError_t launch_march(const ConvArgs& a, dim3 grid, hipStream_t s) {
    const int ck = a.cin / 16, nt = a.cout / 16;
    const dim3 block(256);
    if (a.xs == 1) {
        if (MASK || ck != 1 || nt != 1 || a.u) return hipErrorInvalidValue;
        hipLaunchKernelGGL((k_conv_march<1, 1, false, true>), grid, block, 0, s, a);
        return hipGetLastError();
    }
    if (ck == 1 && nt == 1) {
        if (a.u && MASK) return hipErrorInvalidValue;
        if (a.u)
            hipLaunchKernelGGL((k_conv_march<1, 1, false, false, true>), grid, block, 0, s, a);
        else
            hipLaunchKernelGGL((k_conv_march<1, 1, MASK>), grid, block, 0, s, a);
        return hipGetLastError();
    }
    if (ck == 2 && nt % 2 == 0) {
        hipLaunchKernelGGL((k_conv_march<2, 2, MASK>), grid, block, 0, s, a);
        return hipGetLastError();
    }
    // the other shapes occur in one direction each
    if constexpr (MASK) {
        if (ck == 1 && nt == 3)
            hipLaunchKernelGGL((k_conv_march<1, 3, true>), grid, block, 0, s, a);
        else if (ck == 2 && nt == 1)
            hipLaunchKernelGGL((k_conv_march<2, 1, true>), grid, block, 0, s, a);
        else
            return hipErrorInvalidValue;
    } else if (ck == 1 && nt == 2) {
        hipLaunchKernelGGL((k_conv_march<1, 2, false>), grid, block, 0, s, a);
    } else if (ck == 3 && nt == 1) {
        hipLaunchKernelGGL((k_conv_march<3, 1, false>), grid, block, 0, s, a);
    } else {
        return hipErrorInvalidValue;
    }
    return hipGetLastError();
}

template <bool MASK>
hipError_t launch_deep(const ConvArgs& a, int pg, int nt, dim3 grid, hipStream_t s) {
    const dim3 block(256);
    const int chunks = a.cin / 16;
    if (pg == 1 && nt == 1 && chunks % 4 == 0)
        hipLaunchKernelGGL((k_conv_deep<1, 1, 4, MASK>), grid, block, 0, s, a);
    else if (pg == 1 && nt == 1 && chunks % 2 == 0)
        hipLaunchKernelGGL((k_conv_deep<1, 1, 2, MASK>), grid, block, 0, s, a);
    else if (pg == 2 && nt == 1 && chunks % 4 == 0)
        hipLaunchKernelGGL((k_conv_deep<2, 1, 4, MASK>), grid, block, 0, s, a);
    else if (pg == 2 && nt == 1 && chunks % 2 == 0)
        hipLaunchKernelGGL((k_conv_deep<2, 1, 2, MASK>), grid, block, 0, s, a);
    else if (pg == 2 && nt == 2 && chunks % 2 == 0)
        hipLaunchKernelGGL((k_conv_deep<2, 2, 2, MASK>), grid, block, 0, s, a);
    else
        return hipErrorInvalidValue;
    return hipGetLastError();
}

// The last convolution of a forward pass alone ends in the output.
struct HeadOut {
    double* u;
    int64_t ld, gstride;
};

hipError_t conv(const Net& net, const Layer& L, In x, const bf16* mask, bool forward, Out y,
                int batch, hipStream_t s, const HeadOut* head = nullptr) {
    ConvArgs a;
    a.u = nullptr;
    if (head) {
        if (!forward || L.cout != 16 || L.cin != 16) return hipErrorInvalidValue;
        a.head = net.param + (net.nparam - 17);
        a.rms = net.rms;
        a.u = head->u;
        a.ld = head->ld;
        a.gstride = head->gstride;
    }
    a.x = x.a;
    a.xs = a.xsplit = x.ca;
    a.x2 = x.b;
    a.xs2 = x.cb;
    a.mask = mask;
    a.ms = x.ca;
    a.batch = batch;
    a.h = a.wd = net.n[L.level];
    if (forward) {
        a.w = L.wf;
        a.bias = net.param + L.b_off;
        a.cin = L.cin_p;
        a.cout = L.cout;
        a.relu = 1;
    } else {  // input gradient: K runs over the layer's outputs
        a.w = L.wb;
        a.bias = nullptr;
        a.cin = L.cout;
        a.cout = L.cin;
        a.relu = 0;
    }
    a.y = y.a;
    a.ys = a.ysplit = y.ca;
    a.y2 = y.b;
    a.ys2 = y.cb;
    const bool one = forward && L.cin == 1;  // one channel in memory
    if (x.count() != (one ? 1 : a.cin) || y.count() != a.cout || (mask && x.b) ||
        int64_t(batch) * a.h * a.wd >= (int64_t(1) << 31))
        return hipErrorInvalidValue;
    // whole chunks of 16 channels, in 8-byte loads and stores
    if (((one ? 0 : x.ca) | x.cb | y.ca | y.cb) % 16 != 0 ||
        (reinterpret_cast<uintptr_t>(a.x) | reinterpret_cast<uintptr_t>(a.x2) |
         reinterpret_cast<uintptr_t>(a.y) | reinterpret_cast<uintptr_t>(a.y2) |
         reinterpret_cast<uintptr_t>(a.w) | reinterpret_cast<uintptr_t>(a.mask)) % 8 != 0)
        return hipErrorInvalidValue;
    // 32 channels: down the rows where there are waves enough for that (32 -> 64
    // at 31^2 x 8: 8.5 us against 5.6)
    const int64_t strip_rows = int64_t(batch) * a.h * ((a.wd + 31) / 32) * (a.cout / 16);
    if (a.cin % 32 != 0 || (a.cin == 32 && strip_rows >= 4096)) {
        // Rows of a wave: two rows more are read than written, so as many as
        // still fill 256 CUs once, four waves a SIMD of the 16 -> 16 form and two
        // of the others (their registers); three rows a step of the kernel, so
        // rows + 2 a multiple of 3.
        const int64_t strips = int64_t(batch) * ((a.wd + 16 * kConvGroups - 1) / (16 * kConvGroups)) *
                               (a.cin == 32 && a.cout % 32 == 0 ? a.cout / 32 : 1);
        const int64_t fit = a.cin == 16 && a.cout == 16 ? 4096 : 2048;
        const int64_t bands = std::max<int64_t>(fit / strips, 1);
        a.rows = int(std::max<int64_t>((a.h + bands - 1) / bands, 4));
        a.rows += (4 - a.rows % 3) % 3;
        const int64_t waves = strips * ((a.h + a.rows - 1) / a.rows);
        if (waves > (int64_t(1) << 31) - 4) return hipErrorInvalidValue;
        const dim3 grid(blocks_for(waves, 4));
        return mask ? launch_march<true>(a, grid, s) : launch_march<false>(a, grid, s);
    }
    a.rows = 0;
    // As many outputs a wave (up to 2 x 2 tiles, whose operands are loaded
    // half as often) as leave a wave for every SIMD.
    const auto count = [&](int pg, int nt) {
        return int64_t(batch) * a.h * ((a.wd + 16 * pg - 1) / (16 * pg)) * (a.cout / (16 * nt));
    };
    int pg = 2, nt = 2;
    if (count(pg, nt) < 1024) nt = 1;
    if (count(pg, nt) < 1024) pg = 1;
    const int64_t waves = count(pg, nt);
    if (waves > (int64_t(1) << 31) - 4) return hipErrorInvalidValue;
    const dim3 grid(blocks_for(waves, 4));
    return mask ? launch_deep<true>(a, pg, nt, grid, s) : launch_deep<false>(a, pg, nt, grid, s);
}

// The backward pass's partial sums: where the next layer's go, and what
// k_reduce_slots then adds.
struct Partials {
    ReduceArgs args;
    size_t used = 0;  // floats
    int blocks = 0;
};

// Adds the layers' partial sums so far; their room is free for the next ones.
hipError_t grad_reduce(Partials& parts, hipStream_t s) {
    if (parts.args.layers == 0) return hipSuccess;
    hipLaunchKernelGGL(k_reduce_slots, dim3(unsigned(parts.blocks)), dim3(64 * kReduceWaves), 0, s,
                       parts.args);
    parts = Partials();
    return hipGetLastError();
}

hipError_t wgrad(const Net& net, Partials& parts, const Layer& L, In x, const bf16* dy, const bf16* y,
                 int batch, hipStream_t s) {
    const int64_t dys = L.cout, ys = L.cout;
    WGradArgs a;
    a.x = x.a;
    a.xs = a.xsplit = x.ca;
    a.x2 = x.b;
    a.xs2 = x.cb;
    a.dy = dy;
    a.dys = dys;
    a.y = y;
    a.ys = ys;
    a.batch = batch;
    a.h = a.wd = net.n[L.level];
    a.cin = L.cin_p;
    a.cout = L.cout;
    a.cin_w = L.cin;  // the first layer's padded input channels feed no weight
    const bool one = L.cin == 1;  // one channel in memory
    const WgradSplit p = wgrad_split(batch, a.h, a.cin, a.cout);
    a.rows = p.rows;
    const int64_t slots = int64_t(batch) * p.strips * p.groups;
    const int64_t blocks = slots * (a.cin / (16 * p.ti)) * (a.cout / (16 * p.to));
    const int64_t count = int64_t(L.cout) * L.cin * 9 + L.cout;  // the bias follows the weights
    if (parts.used + size_t(slots * count) > net.parts_floats) {
        const hipError_t e = grad_reduce(parts, s);
        if (e != hipSuccess) return e;
    }
    a.part = net.parts + parts.used;
    if (parts.used + size_t(slots * count) > net.parts_floats || parts.args.layers == kMaxLayers ||
        blocks > (int64_t(1) << 31) - 1 ||
        L.b_off != L.w_off + size_t(count - L.cout) || ((one ? 0 : x.ca) | x.cb | a.cout) % 16 != 0 ||
        x.count() != (one ? 1 : a.cin) || (one && (p.ti != 1 || p.to != 1)) ||
        (reinterpret_cast<uintptr_t>(a.x) | reinterpret_cast<uintptr_t>(a.x2) |
         reinterpret_cast<uintptr_t>(a.dy) | reinterpret_cast<uintptr_t>(a.y)) % 8 != 0)
        return hipErrorInvalidValue;
    const dim3 grid{unsigned(blocks)}, block{64 * kWgradWaves};
    if (one) hipLaunchKernelGGL((k_conv3x3_wgrad<1, 1, true>), grid, block, 0, s, a);
    else if (p.ti == 1 && p.to == 1) hipLaunchKernelGGL((k_conv3x3_wgrad<1, 1>), grid, block, 0, s, a);
    else if (p.ti == 3 && p.to == 1) hipLaunchKernelGGL((k_conv3x3_wgrad<3, 1>), grid, block, 0, s, a);
    else if (p.ti == 2 && p.to == 2) hipLaunchKernelGGL((k_conv3x3_wgrad<2, 2>), grid, block, 0, s, a);
    else return hipErrorInvalidValue;
    const int ways = slots > 64 ? kReduceWaves : 4;
    parts.args.l[parts.args.layers++] = {a.part, net.grad + L.w_off, slots, count, parts.blocks, ways};
    parts.used += size_t(slots * count);
    const int64_t per_block = 64 * (kReduceWaves / ways);
    parts.blocks += int((count + per_block - 1) / per_block);
    return hipGetLastError();
}

}  // namespace
}  // namespace nn
}  // namespace rbgs

namespace rbgs {
namespace nn {
namespace {

#define NN_TRY(expr)                         \
    do {                                     \
        hipError_t _e = (expr);              \
        if (_e != hipSuccess) return _e;     \
    } while (0)

// The transfers move whole groups of 8 channels with 16-byte accesses.
bool transfer_ok(const bf16* in, int64_t is, const bf16* out, int64_t os, int c) {
    return c > 0 && c % 8 == 0 && is % 8 == 0 && os % 8 == 0 &&
           (reinterpret_cast<uintptr_t>(in) | reinterpret_cast<uintptr_t>(out)) % 16 == 0;
}

hipError_t restrict_op(const Net& net, const bf16* in, int64_t is, bf16* out, int64_t os, int batch,
                       int nc, int c, float scale, int acc, hipStream_t s) {
    if (!transfer_ok(in, is, out, os, c) || int64_t(batch) * nc * nc * (c / 8) > (int64_t(1) << 32) - 256)
        return hipErrorInvalidValue;
    const dim3 grid(blocks_for(int64_t(batch) * nc * nc * (c / 8)));
    if (net.factor == 2)
        hipLaunchKernelGGL(k_restrict<2>, grid, dim3(256), 0, s, in, is, out, os, batch, nc, c,
                           scale, acc);
    else if (net.factor == 4)
        hipLaunchKernelGGL(k_restrict<4>, grid, dim3(256), 0, s, in, is, out, os, batch, nc, c,
                           scale, acc);
    else
        return hipErrorInvalidValue;
    return hipGetLastError();
}

hipError_t prolong_op(const Net& net, const bf16* in, int64_t is, bf16* out, int64_t os, int batch,
                      int nc, int c, float scale, int acc, hipStream_t s) {
    const int nf = net.factor * nc + net.factor - 1;
    const int c8_shift = c >= 8 ? __builtin_ctz(unsigned(c / 8)) : 0;
    if (!transfer_ok(in, is, out, os, c) || int64_t(batch) * nf * nf * (c / 8) > (int64_t(1) << 32) - 256 ||
        (c & (c - 1)) != 0 || batch > 65535 || nf > 65535)
        return hipErrorInvalidValue;
    const dim3 grid(blocks_for(int64_t(nc + 1) << c8_shift), unsigned(nf), unsigned(batch));
    if (net.factor == 2)
        hipLaunchKernelGGL(k_prolong<2>, grid, dim3(256), 0, s, in, is, out, os, nc, c8_shift, scale,
                           acc);
    else if (net.factor == 4)
        hipLaunchKernelGGL(k_prolong<4>, grid, dim3(256), 0, s, in, is, out, os, nc, c8_shift, scale,
                           acc);
    else
        return hipErrorInvalidValue;
    return hipGetLastError();
}

hipError_t prep_weights(Net& net, hipStream_t s) {
    PrepArgs a;
    if (net.layers.size() > kMaxLayers) return hipErrorInvalidValue;
    a.param = net.param;
    a.layers = int(net.layers.size());
    unsigned blocks = 0;
    for (int k = 0; k < a.layers; ++k) {
        const Layer& l = net.layers[size_t(k)];
        a.l[k] = {l.w_off, l.wf, l.cin % 16 ? nullptr : l.wb, l.cout, l.cin, l.cin_p, int(blocks)};
        blocks += blocks_for(int64_t(l.cout) * l.cin_p * 9);
    }
    hipLaunchKernelGGL(k_prep_weights, dim3(blocks), dim3(256), 0, s, a);
    return hipGetLastError();
}

const Layer& layer(const Net& net, const char* name) {
    for (const auto& l : net.layers)
        if (std::strcmp(l.name, name) == 0) return l;
    return net.layers[0];
}

// Forward pass of `batch` samples; f: batch grids back to back (natural
// layout, gstride elements apart).  Leaves rms and, where the result is not
// wanted in u (as f lies), y (FP32, normalised) and the last activations.
hipError_t forward(Net& net, int batch, const double* f, int64_t ld, int64_t gstride, double* u,
                   hipStream_t s) {
    const HeadOut out = {u, ld, gstride};
    const int n0 = net.n[0];
    // the row sums sit in the gradient partials, which are free during a forward pass
    double* rows = reinterpret_cast<double*>(net.parts);
    hipLaunchKernelGGL(k_rms_rows, dim3(unsigned(batch * n0)), dim3(256), 0, s, f, n0, ld, gstride,
                       rows);
    NN_TRY(hipGetLastError());
    hipLaunchKernelGGL(k_rms_final, dim3(batch), dim3(256), 0, s, rows, n0, net.rms);
    NN_TRY(hipGetLastError());
    hipLaunchKernelGGL(k_input, dim3(blocks_for(n0), unsigned(n0), unsigned(batch)), dim3(256), 0, s,
                       f, n0, ld, gstride, net.rms, net.in[0]);
    NN_TRY(hipGetLastError());
    // encoder
    for (int l = 0; l < kLevels; ++l) {
        char n0name[8] = "enc0.0", n1name[8] = "enc0.1";
        n0name[3] = n1name[3] = char('0' + l);
        const Layer& c0 = layer(net, n0name);
        const Layer& c1 = layer(net, n1name);
        NN_TRY(conv(net, c0, In{net.in[l], in_channels(l)}, nullptr, true, Out{net.aenc[l], kC[l]},
                    batch, s));
        NN_TRY(conv(net, c1, In{net.aenc[l], kC[l]}, nullptr, true, Out{net.enc[l], kC[l]}, batch, s));
        if (l + 1 < kLevels)
            NN_TRY(restrict_op(net, net.enc[l], kC[l], net.in[l + 1], in_channels(l + 1), batch,
                               net.n[l + 1], kC[l], 1.f, 0, s));
    }
    // decoder
    for (int l = kLevels - 2; l >= 0; --l) {
        const bf16* below = l == kLevels - 2 ? net.enc[l + 1] : net.d[l + 1];
        NN_TRY(prolong_op(net, below, kC[l + 1], net.up[l], kC[l + 1], batch, net.n[l + 1],
                          kC[l + 1], 1.f, 0, s));
        char n0name[8] = "dec0.0", n1name[8] = "dec0.1";
        n0name[3] = n1name[3] = char('0' + l);
        NN_TRY(conv(net, layer(net, n0name), In{net.up[l], kC[l + 1], net.enc[l], kC[l]}, nullptr,
                    true, Out{net.adec[l], kC[l]}, batch, s));
        NN_TRY(conv(net, layer(net, n1name), In{net.adec[l], kC[l]}, nullptr, true,
                    Out{net.d[l], kC[l]}, batch, s, l == 0 && u ? &out : nullptr));
    }
    if (u) return hipSuccess;
    const size_t hw = net.nparam - 17;
    hipLaunchKernelGGL(k_head, dim3(blocks_for(int64_t(batch) * n0 * n0)), dim3(256), 0, s, net.d[0],
                       kC[0], net.param + hw, net.param + hw + 16, net.y, int64_t(batch) * n0 * n0);
    return hipGetLastError();
}

// Backward pass from dy (FP32, normalised output gradient) into net.grad.
hipError_t backward(Net& net, int batch, hipStream_t s) {
    const int n0 = net.n[0];
    const size_t hw = net.nparam - 17;
    const unsigned hblocks = blocks_for(int64_t(batch) * n0 * n0, 256 * kHeadPixels);
    hipLaunchKernelGGL(k_head_grad, dim3(hblocks), dim3(256), 0, s, net.d[0], kC[0],
                       net.param + hw, net.dy, net.gd[0], kC[0], net.parts,
                       int64_t(batch) * n0 * n0);
    NN_TRY(hipGetLastError());
    hipLaunchKernelGGL(k_reduce_parts, dim3(17), dim3(256), 0, s, net.parts, int64_t(hblocks),
                       int64_t(17), net.grad + hw);
    NN_TRY(hipGetLastError());
    Partials parts;
    // decoder, from level 0 (computed last) up
    for (int l = 0; l < kLevels - 1; ++l) {
        char n0name[8] = "dec0.0", n1name[8] = "dec0.1";
        n0name[3] = n1name[3] = char('0' + l);
        const Layer& c0 = layer(net, n0name);
        const Layer& c1 = layer(net, n1name);
        const int C = kC[l], U = kC[l + 1];
        NN_TRY(wgrad(net, parts, c1, In{net.adec[l], C}, net.gd[l], net.d[l], batch, s));
        NN_TRY(conv(net, c1, In{net.gd[l], C}, net.d[l], false, Out{net.gadec[l], C}, batch, s));
        NN_TRY(wgrad(net, parts, c0, In{net.up[l], U, net.enc[l], C}, net.gadec[l], net.adec[l], batch, s));
        NN_TRY(conv(net, c0, In{net.gadec[l], C}, net.adec[l], false,
                    Out{net.gup[l], U, net.genc[l], C}, batch, s));
        // up = P(d_{l+1}) with P = F^2 R^T: the gradient reaching d_{l+1} is F^2 R(dup)
        bf16* gbelow = l == kLevels - 2 ? net.genc[l + 1] : net.gd[l + 1];
        NN_TRY(restrict_op(net, net.gup[l], U, gbelow, U, batch, net.n[l + 1], U,
                           float(net.factor * net.factor), 0, s));
    }
    // encoder, from the bottom level up
    for (int l = kLevels - 1; l >= 0; --l) {
        char n0name[8] = "enc0.0", n1name[8] = "enc0.1";
        n0name[3] = n1name[3] = char('0' + l);
        const Layer& c0 = layer(net, n0name);
        const Layer& c1 = layer(net, n1name);
        const int C = kC[l];
        NN_TRY(wgrad(net, parts, c1, In{net.aenc[l], C}, net.genc[l], net.enc[l], batch, s));
        NN_TRY(conv(net, c1, In{net.genc[l], C}, net.enc[l], false, Out{net.gaenc[l], C}, batch, s));
        NN_TRY(wgrad(net, parts, c0, In{net.in[l], in_channels(l)}, net.gaenc[l], net.aenc[l], batch, s));
        if (l > 0) {
            NN_TRY(conv(net, c0, In{net.gaenc[l], C}, net.aenc[l], false,
                        Out{net.gin[l], in_channels(l)}, batch, s));
            // in_l = R(e_{l-1}): add R^T(g_in) = P(g_in)/F^2 to e_{l-1}'s gradient
            // (which already holds its skip-connection part)
            NN_TRY(prolong_op(net, net.gin[l], in_channels(l), net.genc[l - 1], kC[l - 1], batch,
                              net.n[l], in_channels(l), 1.f / float(net.factor * net.factor), 1, s));
        }
    }
    return grad_reduce(parts, s);
}

hipError_t adam(Net& net, float lr, hipStream_t s) {
    net.adam_t += 1;
    const double b1 = 0.9, b2 = 0.999, t = double(net.adam_t);
    const double c1 = -std::expm1(t * std::log(b1)), c2 = -std::expm1(t * std::log(b2));
    hipLaunchKernelGGL(k_adam, dim3(blocks_for(int64_t(net.nparam))), dim3(256), 0, s, net.param,
                       net.grad, net.m, net.v, int64_t(net.nparam), lr, float(b1), float(1.0 - b1),
                       float(b2), float(1.0 - b2), 1e-8f, float(c1), float(c2));
    NN_TRY(hipGetLastError());
    return prep_weights(net, s);
}

thread_local std::string g_nn_error = "no error";

int nnfail(int status, const std::string& msg) {
    g_nn_error = msg;
    return status;
}

int nn_hip(hipError_t e, const char* what) {
    if (e == hipSuccess) return RBGS_OK;
    return nnfail(RBGS_EHIP, std::string(what) + ": " + hipGetErrorString(e));
}

// Four levels n_l = (n_{l-1} + 1) / F - 1 with at least one point on the
// coarsest: F = 2 takes n = 2^k - 1 in [63, 8191] (coarsest >= 7 points),
// F = 4 takes n + 1 divisible by 64 in [127, 8191].
bool valid_size(int n, int factor) {
    if (n > 8191) return false;
    if (factor == 2) return n >= 63 && ((n + 1) & n) == 0;
    if (factor == 4) return n >= 127 && (n + 1) % 64 == 0;
    return false;
}

void set_levels(Net& net, int n, int factor) {
    net.factor = factor;
    net.n[0] = n;
    for (int l = 1; l < kLevels; ++l) net.n[l] = (net.n[l - 1] + 1) / factor - 1;
}

}  // namespace
}  // namespace nn
}  // namespace rbgs

using namespace rbgs;

struct rbgs_unet {
    nn::Net net;
};

extern "C" {

size_t rbgs_unet_param_count(void) {
    size_t c = 0;
    (void)nn::make_layers(&c);
    return c;
}

size_t rbgs_unet_workspace_size(int32_t n, int32_t batch, int32_t factor) {
    if (!nn::valid_size(n, factor) || batch < 1 || batch > 4096) return 0;
    nn::Net net;
    net.layers = nn::make_layers(&net.nparam);
    net.batch = batch;
    nn::set_levels(net, n, factor);
    return nn::carve(net, nullptr);
}

const char* rbgs_unet_last_error(void) { return nn::g_nn_error.c_str(); }

int rbgs_unet_create(rbgs_unet** out, int32_t n, int32_t batch, int32_t factor, void* workspace,
                     size_t workspace_bytes) {
    if (!out) return nn::nnfail(RBGS_EINVAL, "net is NULL");
    *out = nullptr;
    if (factor != 2 && factor != 4) return nn::nnfail(RBGS_EINVAL, "factor must be 2 or 4");
    if (!nn::valid_size(n, factor))
        return nn::nnfail(RBGS_EINVAL, factor == 2 ? "n must be 2^k - 1 in [63, 8191] for factor 2"
                                                   : "n + 1 must be a multiple of 64 in "
                                                     "[128, 8192] for factor 4");
    if (batch < 1 || batch > 4096) return nn::nnfail(RBGS_EINVAL, "batch must be in [1, 4096]");
    const size_t need = rbgs_unet_workspace_size(n, batch, factor);
    if (!workspace || reinterpret_cast<uintptr_t>(workspace) % 256 || workspace_bytes < need)
        return nn::nnfail(RBGS_EWORKSPACE, "workspace missing, misaligned or smaller than " +
                                               std::to_string(need) + " bytes");
    rbgs_unet* u = new rbgs_unet;
    u->net.layers = nn::make_layers(&u->net.nparam);
    u->net.batch = batch;
    nn::set_levels(u->net, n, factor);
    u->net.total = nn::carve(u->net, static_cast<char*>(workspace));
    *out = u;
    return RBGS_OK;
}

int rbgs_unet_destroy(rbgs_unet* u) {
    delete u;
    return RBGS_OK;
}

int rbgs_unet_set_params(rbgs_unet* u, const float* host, size_t count, void* stream) {
    if (!u || !host || count != u->net.nparam) return nn::nnfail(RBGS_EINVAL, "bad parameter vector");
    hipStream_t s = static_cast<hipStream_t>(stream);
    nn::Net& net = u->net;
    int rc = nn::nn_hip(hipMemcpyAsync(net.param, host, count * 4, hipMemcpyHostToDevice, s), "upload");
    if (rc) return rc;
    // a fresh parameter vector restarts Adam
    for (float* p : {net.m, net.v}) {
        hipLaunchKernelGGL(nn::k_fill, dim3(nn::blocks_for(int64_t(count))), dim3(256), 0, s,
                           reinterpret_cast<uint32_t*>(p), int64_t(count));
        if ((rc = nn::nn_hip(hipGetLastError(), "fill"))) return rc;
    }
    net.adam_t = 0;
    if ((rc = nn::nn_hip(nn::prep_weights(net, s), "weights"))) return rc;
    return nn::nn_hip(hipStreamSynchronize(s), "synchronise");
}

static int copy_out(float* host, const float* dev, size_t count, hipStream_t s) {
    int rc = nn::nn_hip(hipMemcpyAsync(host, dev, count * 4, hipMemcpyDeviceToHost, s), "download");
    if (rc) return rc;
    return nn::nn_hip(hipStreamSynchronize(s), "synchronise");
}

int rbgs_unet_get_params(rbgs_unet* u, float* host, size_t count, void* stream) {
    if (!u || !host || count != u->net.nparam) return nn::nnfail(RBGS_EINVAL, "bad parameter vector");
    return copy_out(host, u->net.param, count, static_cast<hipStream_t>(stream));
}

int rbgs_unet_get_grads(rbgs_unet* u, float* host, size_t count, void* stream) {
    if (!u || !host || count != u->net.nparam) return nn::nnfail(RBGS_EINVAL, "bad gradient vector");
    return copy_out(host, u->net.grad, count, static_cast<hipStream_t>(stream));
}

int rbgs_unet_get_adam(rbgs_unet* u, float* m, float* v, size_t count, int32_t* step,
                       void* stream) {
    if (!u || !m || !v || !step || count != u->net.nparam)
        return nn::nnfail(RBGS_EINVAL, "bad Adam state arrays");
    hipStream_t s = static_cast<hipStream_t>(stream);
    int rc = copy_out(m, u->net.m, count, s);
    if (rc) return rc;
    if ((rc = copy_out(v, u->net.v, count, s))) return rc;
    *step = int32_t(u->net.adam_t);
    return RBGS_OK;
}

int rbgs_unet_set_adam(rbgs_unet* u, const float* m, const float* v, size_t count, int32_t step,
                       void* stream) {
    if (!u || !m || !v || count != u->net.nparam || step < 0)
        return nn::nnfail(RBGS_EINVAL, "bad Adam state arrays or step");
    hipStream_t s = static_cast<hipStream_t>(stream);
    nn::Net& net = u->net;
    int rc = nn::nn_hip(hipMemcpyAsync(net.m, m, count * 4, hipMemcpyHostToDevice, s), "upload");
    if (rc) return rc;
    if ((rc = nn::nn_hip(hipMemcpyAsync(net.v, v, count * 4, hipMemcpyHostToDevice, s), "upload")))
        return rc;
    net.adam_t = step;
    return nn::nn_hip(hipStreamSynchronize(s), "synchronise");
}

int rbgs_unet_forward(rbgs_unet* u, int32_t batch, const double* f, int64_t ld, double* u0,
                      void* stream) {
    if (!u || !f || !u0) return nn::nnfail(RBGS_EINVAL, "NULL argument");
    nn::Net& net = u->net;
    if (batch < 1 || batch > net.batch) return nn::nnfail(RBGS_EINVAL, "batch out of range");
    if (ld < int64_t(net.n[0]) + 2) return nn::nnfail(RBGS_EINVAL, "ld must be >= n + 2");
    hipStream_t s = static_cast<hipStream_t>(stream);
    const int64_t gs = int64_t(net.n[0] + 2) * ld;
    return nn::nn_hip(nn::forward(net, batch, f, ld, gs, u0, s), "forward");
}

int rbgs_unet_train_step(rbgs_unet* u, int32_t batch, const double* f, const double* target,
                         int64_t ld, float lr, int32_t update, float* loss, void* stream) {
    if (!u || !f || !target) return nn::nnfail(RBGS_EINVAL, "NULL argument");
    nn::Net& net = u->net;
    if (batch < 1 || batch > net.batch) return nn::nnfail(RBGS_EINVAL, "batch out of range");
    if (ld < int64_t(net.n[0]) + 2) return nn::nnfail(RBGS_EINVAL, "ld must be >= n + 2");
    if (!(lr >= 0.f)) return nn::nnfail(RBGS_EINVAL, "lr must be >= 0");
    hipStream_t s = static_cast<hipStream_t>(stream);
    const int64_t gs = int64_t(net.n[0] + 2) * ld;
    const int n0 = net.n[0];
    int rc = nn::nn_hip(nn::forward(net, batch, f, ld, gs, nullptr, s), "forward");
    if (rc) return rc;
    const unsigned mblocks = nn::blocks_for(int64_t(batch) * n0 * n0);
    hipLaunchKernelGGL(nn::k_mse, dim3(mblocks), dim3(256), 0, s, net.y, target, net.rms, n0, ld,
                       gs, batch, net.dy, net.parts);
    if ((rc = nn::nn_hip(hipGetLastError(), "loss"))) return rc;
    hipLaunchKernelGGL(nn::k_reduce_parts, dim3(1), dim3(256), 0, s, net.parts, int64_t(mblocks),
                       int64_t(1), net.loss);
    if ((rc = nn::nn_hip(hipGetLastError(), "loss"))) return rc;
    if ((rc = nn::nn_hip(nn::backward(net, batch, s), "backward"))) return rc;
    if (update && (rc = nn::nn_hip(nn::adam(net, lr, s), "adam"))) return rc;
    if (loss) {
        if ((rc = copy_out(loss, net.loss, 1, s))) return rc;
    }
    return RBGS_OK;
}

int rbgs_solve_learned(rbgs_unet* u, const rbgs_grid* g, double* uu, const double* f,
                       const rbgs_solve_opts* o, int32_t compare_after, rbgs_solve_info* info,
                       int32_t* used_guess, double* rel_start, void* workspace,
                       size_t workspace_bytes, void* stream) {
    if (!u || !g || !uu || !f || !o) return nn::nnfail(RBGS_EINVAL, "NULL argument");
    nn::Net& net = u->net;
    if (g->n != net.n[0]) return nn::nnfail(RBGS_EINVAL, "grid size differs from the network's");
    if (g->ld != int64_t(g->n) + 2)
        return nn::nnfail(RBGS_EINVAL, "the learned solve needs a dense grid (ld = n + 2)");
    if (compare_after < 0 || compare_after > o->max_sweeps)
        return nn::nnfail(RBGS_EINVAL, "compare_after must be in [0, max_sweeps]");
    hipStream_t s = static_cast<hipStream_t>(stream);
    const int n = g->n;
    const size_t bytes = size_t(n + 2) * size_t(n + 2) * 8;
    // The caller's start (normally zero inside the Dirichlet ring) and the
    // network's guess on the same ring; after compare_after sweeps of both
    // (0: as they are), keep whichever has the lower relative residual.  The
    // plain start is both fallback and judge.
    int rc = nn::nn_hip(hipMemcpyAsync(net.guess, uu, bytes, hipMemcpyDeviceToDevice, s), "copy");
    if (rc) return rc;
    if ((rc = rbgs_unet_forward(u, 1, f, g->ld, net.guess, stream))) return rc;
    if (compare_after > 0) {
        rbgs_sweep_opts so = o->sweep;
        so.timing = nullptr;
        if ((rc = rbgs_sweep(g, RBGS_F64, uu, f, compare_after, &so, workspace, workspace_bytes, stream)) ||
            (rc = rbgs_sweep(g, RBGS_F64, net.guess, f, compare_after, &so, workspace,
                             workspace_bytes, stream)))
            return nn::nnfail(rc, rbgs_last_error());
    }
    double rel0 = 0.0, reln = 0.0;
    rc = rbgs_residual(g, RBGS_F64, uu, f, nullptr, &rel0, workspace, workspace_bytes, stream);
    if (rc) return nn::nnfail(rc, rbgs_last_error());
    rc = rbgs_residual(g, RBGS_F64, net.guess, f, nullptr, &reln, workspace, workspace_bytes, stream);
    if (rc) return nn::nnfail(rc, rbgs_last_error());
    const bool use = reln < rel0;
    if (use) {
        rc = nn::nn_hip(hipMemcpyAsync(uu, net.guess, bytes, hipMemcpyDeviceToDevice, s), "copy");
        if (rc) return rc;
    }
    if (used_guess) *used_guess = use ? 1 : 0;
    if (rel_start) *rel_start = use ? reln : rel0;
    rbgs_solve_opts rest = *o;
    rest.max_sweeps = o->max_sweeps - compare_after;
    rbgs_solve_info inner{0, 0, 0.0, 0.0, RBGS_OK};
    rc = rbgs_solve(g, RBGS_F64, uu, f, &rest, &inner, workspace, workspace_bytes, stream);
    // the work done: the comparison sweeps of both starts, then the solve
    inner.sweeps += 2 * compare_after;
    if (info) *info = inner;
    return rc;
}

}  // extern "C"
