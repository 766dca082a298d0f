// Learned surrogate: a six-layer 3x3 convolutional network that proposes
// the magnetisation ten fixed steps ahead, trained and evaluated with BF16
// MFMA (v_mfma_f32_16x16x32_bf16, FP32 accumulation).
//
//   input  x: m as a BF16 pair (hi, 256 (m - hi): 6 channels) and the
//          applied field B / 50 mT (3 channels)
//   net    conv3x3(9->32) SiLU, 4 x [conv3x3(32->32) SiLU], conv3x3(32->3)
//   output o; proposal m' = normalize(base + s o) for a base state (m or a
//          coarse step of it) and an output scale s; loss mean
//          (o - (m_t - base) / s)^2
//
// Every convolution is an implicit GEMM over (pixels) x (output channels)
// with K = 9 taps x 32 input channels.  Activations are BF16, channels
// last ([n][y][x][32], channel counts padded to 32 with zeros), weights
// BF16 [tap][cout][cin]; the data gradient is the same kernel with the
// weights flipped in space and transposed in channels, with the SiLU
// derivative of the layer below applied in its epilogue; the weight
// gradient is an MFMA reduction over pixel chunks into per-block partial
// sums that two more kernels add in a fixed order (deterministic).  Master
// weights and the Adam moments stay FP32.
#include <hip/hip_runtime.h>

#include <math.h>
#include <stdarg.h>
#include <stdio.h>
#include <string.h>

#include <algorithm>
#include <string>
#include <vector>

#include "host_common.hpp"
#include "internal.hpp"

namespace {

typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef float f32x4 __attribute__((ext_vector_type(4)));
typedef unsigned short u16;

constexpr int CH = 32;          // padded channel count of every activation
constexpr int KC = 4;           // channels of the compact network output (3 used)
constexpr int NL = 6;           // layers
constexpr int CIN[NL] = {9, 32, 32, 32, 32, 32};
constexpr int COUT[NL] = {32, 32, 32, 32, 32, 3};
constexpr float B_SCALE = 0.05f;
constexpr float LO_SCALE = 256.0f;   // the low part of m is scaled by 2^8 before its own BF16 rounding
constexpr int kVerifyPart = 4;       // start states per verification batch

// round-to-nearest-even FP32 -> BF16 bits (NaN kept quiet)
__host__ __device__ inline u16 f2bf(float f) {
    uint32_t u;
    memcpy(&u, &f, 4);
    if ((u & 0x7fffffffu) > 0x7f800000u) return (u16)((u >> 16) | 0x40);
    u += 0x7fffu + ((u >> 16) & 1u);
    return (u16)(u >> 16);
}
// the same rounding by the hardware conversion (v_cvt_pk_bf16_f32)
__device__ inline u16 f2bf_hw(float f) { return __builtin_bit_cast(u16, (__bf16)f); }
__host__ __device__ inline float bf2f(u16 h) {
    uint32_t u = (uint32_t)h << 16;
    float f;
    memcpy(&f, &u, 4);
    return f;
}

__device__ inline bf16x8 load8(const u16* p) {
    const uint4 v = *reinterpret_cast<const uint4*>(p);
    bf16x8 r;
    memcpy(&r, &v, 16);
    return r;
}
__device__ inline bf16x8 zero8() {
    bf16x8 r;
    const uint4 z = make_uint4(0, 0, 0, 0);
    memcpy(&r, &z, 16);
    return r;
}

// SiLU and its derivative on the hardware exp2 and reciprocal (about 1 ulp
// each; every result is rounded to BF16 afterwards, 2^-9)
__device__ inline float sigmoid_hw(float z) { return __builtin_amdgcn_rcpf(1.0f + __expf(-z)); }
__device__ inline float silu(float z) { return z * sigmoid_hw(z); }
__device__ inline float silu_grad(float z) {
    const float s = sigmoid_hw(z);
    return s * (1.0f + z * (1.0f - s));
}

// ---------------------------------------------------------------------------
// MFMA lane layout of v_mfma_f32_16x16x32_bf16 (C = A B, A 16x32, B 32x16):
//   A: lane l holds row (l % 16), k = 8 (l / 16) + 0..7
//   B: lane l holds column (l % 16), k = 8 (l / 16) + 0..7
//   C: lane l holds column (l % 16), rows 4 (l / 16) + 0..3
// The self-test below multiplies known matrices to confirm it.
// ---------------------------------------------------------------------------
__global__ void mfma_selftest_kernel(const u16* A, const u16* B, float* C) {
    const int l = threadIdx.x;
    bf16x8 a = load8(A + (l % 16) * 32 + 8 * (l / 16));
    u16 bt[8];
    for (int i = 0; i < 8; ++i) bt[i] = B[(8 * (l / 16) + i) * 16 + (l % 16)];
    bf16x8 b;
    memcpy(&b, bt, 16);
    f32x4 c = {0.f, 0.f, 0.f, 0.f};
    c = __builtin_amdgcn_mfma_f32_16x16x32_bf16(a, b, c, 0, 0, 0);
    for (int r = 0; r < 4; ++r) C[(4 * (l / 16) + r) * 16 + (l % 16)] = c[r];
}

// ---------------------------------------------------------------------------
// forward convolution (also the data gradient with transposed weights)
//   in   [N][H][W][32] bf16, wt [9][32 cout][32 cin] bf16, bias [32] (may be null)
//   z    [N][H][W][32] float (pre-activation, may be null)
//   zc   [N][H][W][4] float (its first four channels: the network output, may be null)
//   zb   [N][H][W][32] bf16 (pre-activation kept for the backward pass, may be null)
//   a    [N][H][W][32] bf16 (SiLU(z) if act, else z; may be null)
//   zg   [N][H][W][32] bf16 (may be null): data-gradient mode, a is then
//        z times SiLU'(zg), the gradient at the previous layer's pre-activation
// block: 4 waves, 64 pixels of `rows` consecutive rows; a wave: 16 pixels x
// 32 channels per row.  The weights are the A operand and the pixels the B
// operand, so a lane's accumulators are channels of one pixel; the output
// channels are dealt to the two accumulators (rows 4 g + i of the first:
// channel 8 g + i, of the second: 8 g + 4 + i) so that lane group g holds
// channels 8 g ... 8 g + 7, 16 contiguous bytes of every bf16 tensor.
// Bound by the bytes in flight (each pixel of a layer is read and written
// once, 192 bytes): the weight fragments sit in LDS in lane order, so that
// five waves per SIMD fit; a row is read once, the neighbour pixels coming
// from the neighbour lanes, and two rows ahead.
// ---------------------------------------------------------------------------
// lane i of each 16 lanes takes the value of lane i - 1 (LEFT) or i + 1 of c,
// the first (last) lane its own value of h
template <bool LEFT>
__device__ inline bf16x8 from_neighbour(const bf16x8& c, const bf16x8& h) {
    int cw[4], hw[4];
    memcpy(cw, &c, 16);
    memcpy(hw, &h, 16);
#pragma unroll
    for (int i = 0; i < 4; ++i)
        hw[i] = LEFT ? __builtin_amdgcn_update_dpp(hw[i], cw[i], 0x111, 0xf, 0xf, false)
                     : __builtin_amdgcn_update_dpp(hw[i], cw[i], 0x101, 0xf, 0xf, false);
    bf16x8 r;
    memcpy(&r, hw, 16);
    return r;
}

__device__ inline uint32_t pack2(float lo, float hi) { return (uint32_t)f2bf_hw(lo) | (uint32_t)f2bf_hw(hi) << 16; }

__global__ __launch_bounds__(256, 5) void conv_fwd_kernel(const u16* __restrict__ in, const u16* __restrict__ wt,
                                                       const float* __restrict__ bias, float* __restrict__ z,
                                                       float* __restrict__ zc, u16* __restrict__ zb, u16* __restrict__ a,
                                                       const u16* __restrict__ zg, int H, int W, int act, int rows) {
    __shared__ uint4 wsh[18 * 64];   // [tap][accumulator][lane]
    const int tid = threadIdx.x;
    const int lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int n = blockIdx.z;
    const int x0 = blockIdx.x * 64 + wave * 16;
    const int col = lane % 16, kg = lane / 16;
    const size_t img = (size_t)n * H * W;
    const int ya = blockIdx.y * rows, yb = min(ya + rows, H);
    const int x = x0 + col;
    const bool xin = x < W;
    const int xs = min(x, W - 1);
    // the raw fragments of a row: the lane's pixel, and for the first and
    // last lane of 16 the pixel beyond.  Every lane reads (outside the image:
    // the nearest pixel inside), so that no load is conditional and the waits
    // stay exact; what lies outside is zeroed once it has arrived.
    struct Raw {
        bf16x8 c, h;
    };
    const int hx = col == 0 ? x0 - 1 : col == 15 ? x0 + 16 : x;
    const bool hin = hx >= 0 && hx < W;
    const int co = xs * CH + 8 * kg, ho = min(max(hx, 0), W - 1) * CH + 8 * kg;
    const bool inside = x0 >= 1 && x0 + 16 < W;   // no pixel of this wave's rows outside the image
    auto load_row = [&](int yy, Raw& r) {
        const u16* src = in + (img + (size_t)min(max(yy, 0), H - 1) * W) * CH;
        r.c = load8(src + co);
        r.h = load8(src + ho);
    };
    // the fragments of taps v = 0, 1, 2
    auto expand = [&](int yy, Raw r, bf16x8 (&f)[3]) {
        const bool row = yy >= 0 && yy < H;
        if (!(row && inside)) {
            if (!(row && xin)) r.c = zero8();
            if (!(row && hin)) r.h = zero8();
        }
        f[0] = from_neighbour<true>(r.c, r.h);
        f[1] = r.c;
        f[2] = from_neighbour<false>(r.c, r.h);
    };
    Raw Ra, Rb, T0, T1;
    load_row(ya - 1, Ra);
    load_row(ya, Rb);
    load_row(ya + 1, T0);
    load_row(ya + 2, T1);
    for (int i = tid; i < 18 * 64; i += 256) {
        const int f = i >> 6, l = i & 63;      // lane l's weights of tap f / 2, accumulator f % 2
        const int c = l % 16, k = l / 16;
        const int ch = 8 * (c >> 2) + (c & 3) + 4 * (f & 1);
        wsh[i] = *reinterpret_cast<const uint4*>(wt + ((f >> 1) * CH + ch) * CH + 8 * k);
    }
    float bs[8];
#pragma unroll
    for (int i = 0; i < 8; ++i) bs[i] = bias ? bias[8 * kg + i] : 0.f;
    __syncthreads();
    bf16x8 F0[3], F1[3], F2[3];
    expand(ya - 1, Ra, F0);
    expand(ya, Rb, F1);
    const u16* wl = reinterpret_cast<const u16*>(wsh + lane);
    // one output row from input rows y-1, y, y+1: P and Q expanded, y + 1 raw
    // in T, expanded into R; row y + 3 goes into T
    auto step = [&](int y, bf16x8 (&P)[3], bf16x8 (&Q)[3], bf16x8 (&R)[3], Raw& T) {
        expand(y + 1, T, R);
        if (y + 3 <= yb) load_row(y + 3, T);
        f32x4 acc0 = {0.f, 0.f, 0.f, 0.f}, acc1 = acc0;
#pragma unroll
        for (int t = 0; t < 9; ++t) {
            const bf16x8 w0 = load8(wl + (2 * t) * 512), w1 = load8(wl + (2 * t + 1) * 512);
            const bf16x8 b = t < 3 ? P[t] : t < 6 ? Q[t - 3] : R[t - 6];
            acc0 = __builtin_amdgcn_mfma_f32_16x16x32_bf16(w0, b, acc0, 0, 0, 0);
            acc1 = __builtin_amdgcn_mfma_f32_16x16x32_bf16(w1, b, acc1, 0, 0, 0);
        }
        const size_t px = img + (size_t)y * W;
        const size_t o = (px + xs) * CH + 8 * kg;   // the lane's eight channels
        uint4 g = make_uint4(0, 0, 0, 0);
        if (zg) g = *reinterpret_cast<const uint4*>(zg + o);
        float zv[8];
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            zv[i] = acc0[i] + bs[i];
            zv[4 + i] = acc1[i] + bs[4 + i];
        }
        float ov[8];
        if (zg) {
            const uint32_t gw[4] = {g.x, g.y, g.z, g.w};
#pragma unroll
            for (int i = 0; i < 8; ++i) {
                const float zz = __uint_as_float(i & 1 ? gw[i >> 1] & 0xffff0000u : gw[i >> 1] << 16);
                ov[i] = zv[i] * silu_grad(zz);
            }
        } else {
#pragma unroll
            for (int i = 0; i < 8; ++i) ov[i] = act ? silu(zv[i]) : zv[i];
        }
        if (!xin) return;
        if (z) {
            *reinterpret_cast<float4*>(z + o) = make_float4(zv[0], zv[1], zv[2], zv[3]);
            *reinterpret_cast<float4*>(z + o + 4) = make_float4(zv[4], zv[5], zv[6], zv[7]);
        }
        if (zc && kg == 0) *reinterpret_cast<float4*>(zc + (px + xs) * KC) = make_float4(zv[0], zv[1], zv[2], zv[3]);
        if (a)
            *reinterpret_cast<uint4*>(a + o) =
                make_uint4(pack2(ov[0], ov[1]), pack2(ov[2], ov[3]), pack2(ov[4], ov[5]), pack2(ov[6], ov[7]));
        if (zb)
            *reinterpret_cast<uint4*>(zb + o) =
                make_uint4(pack2(zv[0], zv[1]), pack2(zv[2], zv[3]), pack2(zv[4], zv[5]), pack2(zv[6], zv[7]));
    };
    for (int y = ya; y < yb; y += 6) {
        step(y, F0, F1, F2, T0);
        if (y + 1 < yb) step(y + 1, F1, F2, F0, T1);
        if (y + 2 < yb) step(y + 2, F2, F0, F1, T0);
        if (y + 3 < yb) step(y + 3, F0, F1, F2, T1);
        if (y + 4 < yb) step(y + 4, F1, F2, F0, T0);
        if (y + 5 < yb) step(y + 5, F2, F0, F1, T1);
    }
}

// ---------------------------------------------------------------------------
// weight gradient: dW[u][v][co][ci] = sum over pixels p of gz[p][co] times
// a_in[p + (u - 1, v - 1)][ci], db[co] = sum_p gz[p][co].  Summed over the
// input pixel q = p + (u - 1, v - 1) instead, so that the input fragments are
// aligned.  Staging transposes channels-last rows to [channel][pixel] in LDS
// (2 pixels x 8 channels per thread); a gradient row is staged once, with one
// pixel beyond either end, and its fragments shifted by one pixel are made of
// two neighbouring words in registers.  A block owns 64 input columns of
// `rows` consecutive gradient rows; the input rows rotate through a ring of
// four and the gradient rows through two buffers, so one barrier per row
// separates staging row y + 1 from the MFMAs of row y; the reads run two rows
// ahead.  Wave w accumulates the input-channel half 16 (w & 1) and the pixel
// half 32 (w >> 1) of every tap; the two pixel halves are added in LDS at the
// end in a fixed order and the block writes one partial sum, reduced by the
// reduce kernels.
// ---------------------------------------------------------------------------
constexpr int WG_LA = 72;          // LDS row strides (u16), 16-byte aligned rows on distinct banks: input 64 + 8,
constexpr int WG_LG = 88;          // gradient 8 (the last one the pixel before) + 64 + 16 (the first the pixel after)
constexpr int WG_ROUND = 3 * 256;  // blocks the card holds at a time
constexpr int WG_SEG = 64;         // segments of the first reduction stage
// The partials of all layers are held for one reduction at the end (two
// launches instead of twelve) up to this many bytes: 170 MB at 16 states of
// 256 x 256 or more.  Small images in large batches have more blocks than one
// round, at least one per image; beyond the limit each layer is reduced before
// the next one takes its place.
constexpr size_t WG_HELD = (size_t)256 << 20;
constexpr int NWG = 9 * CH * CH;   // weight-gradient entries of one layer

// channels 8 cg .. 8 cg + 7 of pixel x of row y (zero outside the image)
__device__ inline uint4 load_px(const u16* __restrict__ src, size_t img, int H, int W, int y, int x, int cg) {
    if (y < 0 || y >= H || x < 0 || x >= W) return make_uint4(0, 0, 0, 0);
    return *reinterpret_cast<const uint4*>(src + (img + (size_t)y * W + x) * CH + 8 * cg);
}
// two pixels to dst[channel][pixel] (row stride ld, even place)
__device__ inline void store_pair(u16* dst, int ld, const uint4 (&v)[2], int cg) {
    const uint32_t a[4] = {v[0].x, v[0].y, v[0].z, v[0].w}, b[4] = {v[1].x, v[1].y, v[1].z, v[1].w};
#pragma unroll
    for (int k = 0; k < 4; ++k) {
        // word k of a pixel holds channels 2k (low half) and 2k + 1 (high half)
        *reinterpret_cast<uint32_t*>(dst + (8 * cg + 2 * k) * ld) = (a[k] & 0xffffu) | (b[k] << 16);
        *reinterpret_cast<uint32_t*>(dst + (8 * cg + 2 * k + 1) * ld) = (a[k] >> 16) | (b[k] & 0xffff0000u);
    }
}

__global__ __launch_bounds__(256, 3) void conv_wgrad_kernel(const u16* __restrict__ gz, const u16* __restrict__ ain,
                                                            float* __restrict__ part_w, float* __restrict__ part_b,
                                                            int H, int W, int rows) {
    // staging: gradient gT[2 buffers][32][88] and input aT[4 ring slots][32][72]
    // (29 KB); at the end the same memory holds the pixel-half exchange (36 KB)
    __shared__ __align__(16) unsigned char smem[2 * 72 * 64 * 4];
    __shared__ float bsum[2][CH];
    u16* gT = reinterpret_cast<u16*>(smem);
    u16* aT = gT + 2 * CH * WG_LG;
    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int col = lane % 16, kg = lane / 16;
    const int cih = wave & 1, kh = wave >> 1;
    const int n = blockIdx.z, x0 = blockIdx.x * 64;
    const int ya = blockIdx.y * rows, yb = min(ya + rows, H);
    const size_t img = (size_t)n * H * W;
    f32x4 acc[18];
#pragma unroll
    for (int i = 0; i < 18; ++i) acc[i] = (f32x4){0.f, 0.f, 0.f, 0.f};
    float bp[8];         // gradient threads: sums of channels 8 cg ..
#pragma unroll
    for (int i = 0; i < 8; ++i) bp[i] = 0.f;
    // threads of waves 0, 1 stage the gradient row, those of waves 2, 3 the
    // input row below it; the first eight threads also the two pixels beyond
    const bool grad = wave < 2;
    const int q = (tid >> 2) & 31, cg = tid & 3;
    struct Share {
        uint4 v[2], h;
    };
    auto load_share = [&](int y, Share& s) {     // gradient row y, input row y + 1
        const u16* src = grad ? gz : ain;
        const int yy = grad ? y : y + 1;
#pragma unroll
        for (int i = 0; i < 2; ++i) s.v[i] = load_px(src, img, H, W, yy, x0 + 2 * q + i, cg);
        if (tid < 8) s.h = load_px(gz, img, H, W, y, tid < 4 ? x0 - 1 : x0 + 64, cg);
    };
    auto store_share = [&](int y, const Share& s) {
        if (grad) {
            u16* g = gT + (y & 1) * CH * WG_LG;
            store_pair(g + 8 + 2 * q, WG_LG, s.v, cg);
            const uint32_t w[2][4] = {{s.v[0].x, s.v[0].y, s.v[0].z, s.v[0].w}, {s.v[1].x, s.v[1].y, s.v[1].z, s.v[1].w}};
#pragma unroll
            for (int i = 0; i < 2; ++i)
#pragma unroll
                for (int k = 0; k < 4; ++k) {
                    bp[2 * k] += __uint_as_float(w[i][k] << 16);
                    bp[2 * k + 1] += __uint_as_float(w[i][k] & 0xffff0000u);
                }
            if (tid < 8) {
                const uint32_t h[4] = {s.h.x, s.h.y, s.h.z, s.h.w};
                u16* d = g + (tid < 4 ? 7 : 72) + 8 * cg * WG_LG;
#pragma unroll
                for (int k = 0; k < 4; ++k) {
                    d[2 * k * WG_LG] = (u16)(h[k] & 0xffffu);
                    d[(2 * k + 1) * WG_LG] = (u16)(h[k] >> 16);
                }
            }
        } else {
            store_pair(aT + ((y + 1) & 3) * CH * WG_LA + 2 * q, WG_LA, s.v, cg);
        }
    };
    Share s0, s1;
    {
        // input rows ya - 1 and ya into their ring slots (row mod 4)
        uint4 v[2];
        const int r = grad ? ya - 1 : ya;
#pragma unroll
        for (int i = 0; i < 2; ++i) v[i] = load_px(ain, img, H, W, r, x0 + 2 * q + i, cg);
        load_share(ya, s0);
        if (ya + 1 < yb) load_share(ya + 1, s1);
        store_pair(aT + (r & 3) * CH * WG_LA + 2 * q, WG_LA, v, cg);
    }
    store_share(ya, s0);
    if (ya + 2 < yb) load_share(ya + 2, s0);
    __syncthreads();
    const int kc = 32 * kh + 8 * kg;
    // the MFMAs of row y, after the staging of row y + 1 (held in s, which
    // takes row y + 3)
    auto step = [&](int y, Share& s) {
        if (y + 1 < yb) store_share(y + 1, s);
        if (y + 3 < yb) load_share(y + 3, s);
        bf16x8 Bu[3];
#pragma unroll
        for (int u = 0; u < 3; ++u) Bu[u] = load8(aT + ((y + u - 1) & 3) * CH * WG_LA + (16 * cih + col) * WG_LA + kc);
#pragma unroll
        for (int coh = 0; coh < 2; ++coh) {
            const u16* g = gT + (y & 1) * CH * WG_LG + (16 * coh + col) * WG_LG + 8 + kc;
            const uint4 d = *reinterpret_cast<const uint4*>(g);
            const uint32_t before = *reinterpret_cast<const uint32_t*>(g - 2);
            const uint32_t after = *reinterpret_cast<const uint32_t*>(g + 8);
            // pixels one to the right (v = 0), in place, one to the left (v = 2)
            const uint32_t m = __builtin_amdgcn_alignbit(d.x, before, 16), a0 = __builtin_amdgcn_alignbit(d.y, d.x, 16),
                           a1 = __builtin_amdgcn_alignbit(d.z, d.y, 16), a2 = __builtin_amdgcn_alignbit(d.w, d.z, 16),
                           a3 = __builtin_amdgcn_alignbit(after, d.w, 16);
            const uint4 f[3] = {make_uint4(a0, a1, a2, a3), d, make_uint4(m, a0, a1, a2)};
#pragma unroll
            for (int v = 0; v < 3; ++v) {
                bf16x8 A;
                memcpy(&A, &f[v], 16);
#pragma unroll
                for (int u = 0; u < 3; ++u) {
                    f32x4& c = acc[(u * 3 + v) * 2 + coh];
                    c = __builtin_amdgcn_mfma_f32_16x16x32_bf16(A, Bu[u], c, 0, 0, 0);
                }
            }
        }
        __syncthreads();
    };
    for (int y = ya; y < yb; y += 2) {
        step(y, s1);
        if (y + 1 < yb) step(y + 1, s0);
    }
    // add the pixel halves: waves 2, 3 hand their sums to waves 0, 1
    float* red = reinterpret_cast<float*>(smem);
    if (kh == 1) {
#pragma unroll
        for (int i = 0; i < 18; ++i)
#pragma unroll
            for (int r = 0; r < 4; ++r) red[(cih * 72 + 4 * i + r) * 64 + lane] = acc[i][r];
    } else {
        // (waves 0 and 1 hold the gradient rows' sums) over the pixel pairs
#pragma unroll
        for (int i = 0; i < 8; ++i) {
            float b = bp[i];
            for (int off = 32; off >= 4; off >>= 1) b += __shfl_xor(b, off);
            if (lane < 4) bsum[wave][8 * lane + i] = b;
        }
    }
    __syncthreads();
    const int blk = (blockIdx.z * gridDim.y + blockIdx.y) * gridDim.x + blockIdx.x;
    if (kh == 0) {
        float* pw = part_w + (size_t)blk * NWG;
#pragma unroll
        for (int i = 0; i < 18; ++i) {
            const int tap = i / 2, coh = i % 2;
#pragma unroll
            for (int r = 0; r < 4; ++r) {
                const int co = 16 * coh + 4 * kg + r, ci = 16 * cih + col;
                pw[(tap * CH + co) * CH + ci] = acc[i][r] + red[(cih * 72 + 4 * i + r) * 64 + lane];
            }
        }
    }
    if (tid < CH) part_b[(size_t)blk * CH + tid] = bsum[0][tid] + bsum[1][tid];
}

// the layers of a launch over several of them (blockIdx.z)
struct LayerSet {
    int cin[NL], cout[NL];
    float *w[NL], *b[NL];            // weights [cout][cin][3][3] and biases (or their gradients)
    const float *gw[NL], *gb[NL];    // gradients (Adam)
    float *m1w[NL], *m1b[NL], *m2w[NL], *m2b[NL];
    u16 *wf[NL], *wtr[NL];           // bf16 forward and data-gradient weights
};

// first stage of the deterministic reduction: entry i (weights, then the 32
// bias entries) of a layer summed over segment blockIdx.y of the block
// partials, in block order
__global__ void wgrad_reduce1_kernel(const float* part_w, const float* part_b, int nblk, float* part2) {
    const int i = blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= NWG + CH) return;
    part_w += (size_t)blockIdx.z * nblk * NWG;
    part_b += (size_t)blockIdx.z * nblk * CH;
    part2 += (size_t)blockIdx.z * gridDim.y * (NWG + CH);
    const int per = (nblk + gridDim.y - 1) / gridDim.y;
    const int b0 = blockIdx.y * per, b1 = min(nblk, b0 + per);
    float s = 0.f;
    if (i < NWG) {
#pragma unroll 8
        for (int b = b0; b < b1; ++b) s += part_w[(size_t)b * NWG + i];
    } else {
#pragma unroll 8
        for (int b = b0; b < b1; ++b) s += part_b[(size_t)b * CH + i - NWG];
    }
    part2[(size_t)blockIdx.y * (NWG + CH) + i] = s;
}

// second stage: the segments in order, into the parameter layout
__global__ void wgrad_reduce2_kernel(const float* part2, int nseg, LayerSet ls) {
    const int i = blockIdx.x * blockDim.x + threadIdx.x, l = blockIdx.z;
    if (i >= NWG + CH) return;
    part2 += (size_t)l * nseg * (NWG + CH);
    float s = 0.f;
#pragma unroll 8
    for (int k = 0; k < nseg; ++k) s += part2[(size_t)k * (NWG + CH) + i];
    const int cin = ls.cin[l], cout = ls.cout[l];
    if (i < NWG) {
        const int tap = i / (CH * CH), co = (i / CH) % CH, ci = i % CH;
        if (co < cout && ci < cin) ls.w[l][(co * cin + ci) * 9 + tap] = s;
    } else if (i - NWG < cout) {
        ls.b[l][i - NWG] = s;
    }
}

// gz = g * silu'(z) (hidden layers) or g (last layer), as bf16
__global__ void act_bwd_kernel(const float* g, const float* z, u16* gz, size_t n, int act) {
    const size_t i = (size_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= n) return;
    const float v = act ? g[i] * silu_grad(z[i]) : g[i];
    gz[i] = f2bf(v);
}

// the 32 channels of the block's 256 pixels (first pixel p0 of npx) from
// the first NQ 16-byte quarters in LDS, the rest zero, so that consecutive
// lanes write consecutive 16 bytes
template <int NQ>
__device__ inline void write_pixels(u16* x, size_t p0, size_t npx, const uint4 (*q)[256]) {
    uint4* xo = reinterpret_cast<uint4*>(x) + 4 * p0;
#pragma unroll
    for (int it = 0; it < 4; ++it) {
        const int i = it * 256 + (int)threadIdx.x, px = i >> 2, k = i & 3;
        if (p0 + px < npx) xo[i] = k < NQ ? q[k < NQ ? k : 0][px] : make_uint4(0u, 0u, 0u, 0u);
    }
}

// x = (m, B / 50 mT, 0...) bf16 channels-last; m is [n][3][H][W] float,
// hw = H W; blockIdx.y: the state
__global__ __launch_bounds__(256) void make_input_kernel(const float* m, const float* B, u16* x, int hw) {
    __shared__ uint4 q[2][256];
    const int n = blockIdx.y;
    const size_t p0 = (size_t)blockIdx.x * 256, p = p0 + threadIdx.x;
    if (p < (size_t)hw) {
        // m as a BF16 pair: hi = bf16(m), lo = bf16(256 (m - hi)) (m - hi is
        // exact in FP32), so the first layer sees m to about 16 bits
        uint32_t ch[9];
        for (int c = 0; c < 3; ++c) {
            const float v = m[((size_t)n * 3 + c) * hw + p];
            const u16 hi = f2bf(v);
            ch[c] = hi;
            ch[3 + c] = f2bf((v - bf2f(hi)) * LO_SCALE);
        }
        for (int c = 0; c < 3; ++c) ch[6 + c] = f2bf(B[n * 3 + c] / B_SCALE);
        q[0][threadIdx.x] = make_uint4(ch[0] | ch[1] << 16, ch[2] | ch[3] << 16, ch[4] | ch[5] << 16, ch[6] | ch[7] << 16);
        q[1][threadIdx.x] = make_uint4(ch[8], 0u, 0u, 0u);
    }
    __syncthreads();
    write_pixels<2>(x + (size_t)n * hw * CH, p0, hw, q);
}

// loss gradient (bf16: the gradient at the last layer's pre-activation) of
// the mean squared error of the network output against
// (m_target - base) / scale, and per-block loss partials; blockIdx.y: the state
__global__ __launch_bounds__(256) void loss_kernel(const float* zout, const float* base, const float* mt, u16* gz,
                                                   float* part, int hw, float inv_scale) {
    __shared__ float red[256];
    __shared__ uint4 q[1][256];
    const int n = blockIdx.y;
    const size_t p0 = (size_t)blockIdx.x * 256, p = p0 + threadIdx.x;
    const float inv = 1.0f / (3.0f * (float)((size_t)gridDim.y * hw));
    float l = 0.f;
    if (p < (size_t)hw) {
        const float4 zo = *reinterpret_cast<const float4*>(zout + ((size_t)n * hw + p) * KC);
        const float zv[3] = {zo.x, zo.y, zo.z};
        uint32_t gb[3];
        for (int c = 0; c < 3; ++c) {
            const size_t i = ((size_t)n * 3 + c) * hw + p;
            const float d = zv[c] - (mt[i] - base[i]) * inv_scale;
            l += d * d;
            gb[c] = f2bf(2.0f * d * inv);
        }
        q[0][threadIdx.x] = make_uint4(gb[0] | gb[1] << 16, gb[2], 0u, 0u);
    }
    red[threadIdx.x] = l;
    __syncthreads();
    write_pixels<1>(gz + (size_t)n * hw * CH, p0, hw, q);
    for (int s = 128; s > 0; s >>= 1) {
        if (threadIdx.x < s) red[threadIdx.x] += red[threadIdx.x + s];
        __syncthreads();
    }
    if (threadIdx.x == 0) part[(size_t)blockIdx.y * gridDim.x + blockIdx.x] = red[0] * inv;
}

// one block of 256 threads: strided partial sums, then a fixed tree
__global__ void sum_kernel(const float* part, int n, float* out) {
    __shared__ float red[256];
    float s = 0.f;
    for (int i = threadIdx.x; i < n; i += 256) s += part[i];
    red[threadIdx.x] = s;
    __syncthreads();
    for (int st = 128; st > 0; st >>= 1) {
        if ((int)threadIdx.x < st) red[threadIdx.x] += red[threadIdx.x + st];
        __syncthreads();
    }
    if (threadIdx.x == 0) *out = red[0];
}

// proposals m' = normalize(base + scale * out)
__global__ void propose_kernel(const float* base, const float* zout, float* mo, int N, int H, int W, float scale) {
    const size_t i = (size_t)blockIdx.x * blockDim.x + threadIdx.x;
    const size_t npx = (size_t)N * H * W;
    if (i >= npx) return;
    const int n = (int)(i / ((size_t)H * W));
    const size_t p = i - (size_t)n * H * W;
    float v[3];
    for (int c = 0; c < 3; ++c) v[c] = base[((size_t)n * 3 + c) * H * W + p] + scale * zout[i * KC + c];
    const float inv = rsqrtf(v[0] * v[0] + v[1] * v[1] + v[2] * v[2]);
    for (int c = 0; c < 3; ++c) mo[((size_t)n * 3 + c) * H * W + p] = v[c] * inv;
}

// One Adam step of every layer (lr > 0), then the FP32 master weights to
// bf16 in the forward [tap][co][ci] and the data-gradient [tap'][ci][co]
// (tap' = 8 - tap) layouts, zero past the layer's channels
__global__ void update_pack_kernel(LayerSet ls, float lr, float c1, float c2) {
    const int i = blockIdx.x * blockDim.x + threadIdx.x, l = blockIdx.z;
    if (i >= NWG + CH) return;
    const int cin = ls.cin[l], cout = ls.cout[l];
    auto adam = [&](float& p, float g, float& m1, float& m2) {
        m1 = 0.9f * m1 + 0.1f * g;
        m2 = 0.999f * m2 + 0.001f * g * g;
        p -= lr * (m1 / c1) / (sqrtf(m2 / c2) + 1e-8f);
    };
    if (i < NWG) {
        const int tap = i / (CH * CH), co = (i / CH) % CH, ci = i % CH;
        float v = 0.f;
        if (co < cout && ci < cin) {
            const int o = (co * cin + ci) * 9 + tap;
            if (lr > 0.f) adam(ls.w[l][o], ls.gw[l][o], ls.m1w[l][o], ls.m2w[l][o]);
            v = ls.w[l][o];
        }
        ls.wf[l][i] = f2bf(v);
        ls.wtr[l][((8 - tap) * CH + ci) * CH + co] = f2bf(v);
    } else if (i - NWG < cout && lr > 0.f) {
        const int o = i - NWG;
        adam(ls.b[l][o], ls.gb[l][o], ls.m1b[l][o], ls.m2b[l][o]);
    }
}

// x (float, channels-last) -> bf16
__global__ void to_bf16_kernel(const float* x, u16* y, size_t n) {
    const size_t i = (size_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i < n) y[i] = f2bf(x[i]);
}

// out[j] = max over cells of |a_j - b_j| (Euclidean norm per cell), as the
// bits of a non-negative float (ordered like unsigned integers)
__global__ void maxdiff_kernel(const float* a, const float* b, int ncells, unsigned* out) {
    __shared__ float red[256];
    float m = 0.f;
    for (int i = blockIdx.x * blockDim.x + threadIdx.x; i < ncells; i += gridDim.x * blockDim.x) {
        const float dx = a[i] - b[i];
        const float dy = a[ncells + i] - b[ncells + i];
        const float dz = a[2 * ncells + i] - b[2 * ncells + i];
        float d = sqrtf(dx * dx + dy * dy + dz * dz);
        if (!(d <= 3.0e38f)) d = INFINITY;   // NaN or Inf: infinitely far
        m = fmaxf(m, d);
    }
    red[threadIdx.x] = m;
    __syncthreads();
    for (int st = 128; st > 0; st >>= 1) {
        if ((int)threadIdx.x < st) red[threadIdx.x] = fmaxf(red[threadIdx.x], red[threadIdx.x + st]);
        __syncthreads();
    }
    if (threadIdx.x == 0) atomicMax(out, __float_as_uint(red[0]));
}

__global__ void zero_u32_kernel(unsigned* p, int n) {
    const int i = blockIdx.x * blockDim.x + threadIdx.x;
    if (i < n) p[i] = 0u;
}

}  // namespace

// ============================================================================
// host side
// ============================================================================
struct llg_sur {
    int device = 0;
    hipStream_t stream = nullptr;
    int H = 0, W = 0, maxb = 0;
    std::string err;
    long long nparam = 0;
    std::vector<long long> woff, boff;        // offsets of each layer's weights / bias in params
    float* params = nullptr;                   // FP32 master, oracle layout
    float* grads = nullptr;
    float* mom1 = nullptr;
    float* mom2 = nullptr;
    u16* wf[NL] = {};                          // bf16 forward weights
    u16* wtr[NL] = {};                         // bf16 transposed/flipped weights
    u16* act[NL] = {};                         // layer inputs (bf16, 32 ch)
    float* z[NL] = {};                         // pre-activations: bf16 32 ch kept for the backward pass
                                               // (hidden layers), float 4 ch (network output) or float
                                               // 32 ch (parity checks)
    float* g = nullptr;                        // gradient w.r.t. a layer's output (float, 32 ch)
    u16* gz = nullptr;                         // gradient w.r.t. pre-activation (bf16)
    u16* gz2 = nullptr;                        // the same for the layer below (ping-pong)
    int wslots = NL;                           // layers whose per-block gradients are held at a time (NL or 1)
    float* part_w = nullptr;                   // per-block weight gradients
    float* part_b = nullptr;
    float* part2 = nullptr;                    // first-stage sums of the weight-gradient reduction
    float* part_l = nullptr;
    float* loss = nullptr;      // pinned host memory, written by the sum itself instead of a copy into
                                // pageable memory (a training step of 40 x 50 cells 206 -> 184 us)
    float* dm_in = nullptr;                    // staging for host inputs
    float* dm_t = nullptr;
    float* dB = nullptr;
    float* dm_out = nullptr;
    long long adam_t = 0;
    bool packed = false;
    float out_scale = 1.f;                     // dm = out_scale * network output
    // speculative verification
    std::vector<llg_batch*> vb;                // the plain segments of a round, in parts of kVerifyPart
    llg_batch* eb = nullptr;                   // one film: the coarse step of the proposals' base
    llg_film_desc vdesc = {};                  // the film the batch was built for
    int vwin = 0;
    float* props = nullptr;                    // proposals: window + 1 states
    unsigned* dmax = nullptr;                  // per-proposal max-cell distance (float bits)
};

namespace {

llg_status sfail(llg_sur* s, llg_status c, const char* fmt, ...) {
    char buf[512];
    va_list ap;
    va_start(ap, fmt);
    vsnprintf(buf, sizeof buf, fmt, ap);
    va_end(ap);
    if (s) s->err = buf;
    return c;
}

#define SCHK(s, x)                                                                                \
    do {                                                                                          \
        hipError_t e_ = (x);                                                                      \
        if (e_ != hipSuccess)                                                                     \
            return sfail(s, e_ == hipErrorOutOfMemory ? LLG_E_NOMEM : LLG_E_DEVICE, "%s: %s (%s:%d)", #x, \
                         hipGetErrorString(e_), __FILE__, __LINE__);                              \
    } while (0)

// gradient rows per weight-gradient block: at least 4, and as many as let
// one round of blocks cover the images
int wg_rows(const llg_sur* s, int N) {
    const long long rb = (long long)((s->W + 63) / 64) * s->H * N;
    return (int)std::min<long long>(s->H, std::max<long long>(4, (rb + WG_ROUND - 1) / WG_ROUND));
}
dim3 wg_grid(const llg_sur* s, int N) {
    const int r = wg_rows(s, N);
    return dim3((s->W + 63) / 64, (s->H + r - 1) / r, N);
}
int wg_blocks(const llg_sur* s, int N) {
    const dim3 g = wg_grid(s, N);
    return (int)(g.x * g.y * g.z);
}

// convolution rows per forward block: blocks of 64 pixels by `rows` rows,
// as many rows (at most 24) as let whole rounds of five blocks per compute
// unit cover the image (a partly filled last round costs a whole one), dealt
// evenly over each image's blocks (one pass of the network over 2344 images
// of 16 x 16: blocks of 15 rows and one 612 us, of 8 rows 398; 1042 of
// 24 x 24 437 -> 304; 16 of 256 x 256 keep their 13 rows)
void launch_conv(llg_sur* s, const u16* in, const u16* wt, const float* bias, float* z, float* zc, u16* zb, u16* a,
                 const u16* zg, int N, int act) {
    const long long rb = (long long)((s->W + 63) / 64) * s->H * N, round = 5 * 256;
    const long long rounds = (rb + round * 24 - 1) / (round * 24);
    const int most = (int)((rb + round * rounds - 1) / (round * rounds));
    const int parts = (s->H + most - 1) / most, rows = (s->H + parts - 1) / parts;
    hipLaunchKernelGGL(conv_fwd_kernel, dim3((s->W + 63) / 64, (s->H + rows - 1) / rows, N), dim3(256), 0,
                       s->stream, in, wt, bias, z, zc, zb, a, zg, s->H, s->W, act, rows);
}

// per-block weight and bias gradients of one layer from the pre-activation
// gradient gz and the layer input ain, into slot `slot` of the partials
void launch_wgrad(llg_sur* s, const u16* gz, const u16* ain, int N, int slot) {
    const dim3 grid = wg_grid(s, N);
    const size_t nblk = (size_t)grid.x * grid.y * grid.z;
    hipLaunchKernelGGL(conv_wgrad_kernel, grid, dim3(256), 0, s->stream, gz, ain, s->part_w + slot * nblk * NWG,
                       s->part_b + slot * nblk * CH, s->H, s->W, wg_rows(s, N));
}

// the partials of the first `layers` slots in two fixed-order stages into
// ls.w, ls.b
void launch_wgrad_reduce(llg_sur* s, int N, int layers, const LayerSet& ls) {
    const int nblk = wg_blocks(s, N), nseg = std::min(WG_SEG, nblk);
    hipLaunchKernelGGL(wgrad_reduce1_kernel, dim3((NWG + CH + 255) / 256, nseg, layers), dim3(256), 0, s->stream,
                       s->part_w, s->part_b, nblk, s->part2);
    hipLaunchKernelGGL(wgrad_reduce2_kernel, dim3((NWG + CH + 255) / 256, 1, layers), dim3(256), 0, s->stream,
                       s->part2, nseg, ls);
}

LayerSet layer_set(const llg_sur* s, float* w) {
    LayerSet ls = {};
    for (int l = 0; l < NL; ++l) {
        ls.cin[l] = CIN[l];
        ls.cout[l] = COUT[l];
        ls.w[l] = w + s->woff[l];
        ls.b[l] = w + s->boff[l];
        ls.gw[l] = s->grads + s->woff[l];
        ls.gb[l] = s->grads + s->boff[l];
        ls.m1w[l] = s->mom1 + s->woff[l];
        ls.m1b[l] = s->mom1 + s->boff[l];
        ls.m2w[l] = s->mom2 + s->woff[l];
        ls.m2b[l] = s->mom2 + s->boff[l];
        ls.wf[l] = s->wf[l];
        ls.wtr[l] = s->wtr[l];
    }
    return ls;
}

// layer l alone, as the first of a set to reduce into
LayerSet one_layer(int l, float* w, float* b) {
    LayerSet ls = {};
    ls.cin[0] = CIN[l];
    ls.cout[0] = COUT[l];
    ls.w[0] = w;
    ls.b[0] = b;
    return ls;
}

// an Adam step (lr > 0) and the bf16 weights
llg_status update_pack(llg_sur* s, float lr, float c1, float c2) {
    hipLaunchKernelGGL(update_pack_kernel, dim3((NWG + CH + 255) / 256, 1, NL), dim3(256), 0, s->stream,
                       layer_set(s, s->params), lr, c1, c2);
    SCHK(s, hipGetLastError());
    s->packed = true;
    return LLG_OK;
}

// keep_z: keep every hidden layer's pre-activation as bf16 for the backward
// pass (in the first half of its float buffer).  The last layer's (the
// network output) is written compact, four float channels per pixel, unless
// f32_layer asks for it; layer f32_layer's is written as float, 32 channels
llg_status forward(llg_sur* s, const float* m, const float* B, int N, bool keep_z, int f32_layer = -1) {
    const int hw = s->H * s->W;
    hipLaunchKernelGGL(make_input_kernel, dim3((hw + 255) / 256, N), dim3(256), 0, s->stream, m, B, s->act[0], hw);
    SCHK(s, hipGetLastError());
    for (int l = 0; l < NL; ++l) {
        const bool f32 = l == f32_layer, out = l == NL - 1 && !f32;
        launch_conv(s, s->act[l], s->wf[l], s->params + s->boff[l], f32 ? s->z[l] : nullptr, out ? s->z[l] : nullptr,
                    keep_z && l < NL - 1 && !f32 ? reinterpret_cast<u16*>(s->z[l]) : nullptr,
                    l < NL - 1 ? s->act[l + 1] : nullptr, nullptr, N, l < NL - 1 ? 1 : 0);
        SCHK(s, hipGetLastError());
    }
    return LLG_OK;
}

}  // namespace

extern "C" {

llg_status llg_mfma_selftest(int device, const float* A, const float* B, float* C) {
    if (!A || !B || !C) return LLG_E_ARG;
    if (hipSetDevice(device) != hipSuccess) return LLG_E_DEVICE;
    std::vector<u16> ha(16 * 32), hb(32 * 16);
    for (int i = 0; i < 16 * 32; ++i) ha[i] = f2bf(A[i]);
    for (int i = 0; i < 32 * 16; ++i) hb[i] = f2bf(B[i]);
    u16 *da = nullptr, *db = nullptr;
    float* dc = nullptr;
    if (hipMalloc(&da, 1024) != hipSuccess || hipMalloc(&db, 1024) != hipSuccess ||
        hipMalloc(&dc, 16 * 16 * 4) != hipSuccess)
        return LLG_E_DEVICE;
    (void)hipMemcpy(da, ha.data(), 1024, hipMemcpyHostToDevice);
    (void)hipMemcpy(db, hb.data(), 1024, hipMemcpyHostToDevice);
    hipLaunchKernelGGL(mfma_selftest_kernel, dim3(1), dim3(64), 0, 0, da, db, dc);
    hipError_t e = hipMemcpy(C, dc, 16 * 16 * 4, hipMemcpyDeviceToHost);
    (void)hipFree(da);
    (void)hipFree(db);
    (void)hipFree(dc);
    return e == hipSuccess ? LLG_OK : LLG_E_DEVICE;
}

llg_status llg_sur_create(int device, int H, int W, int max_batch, llg_sur** out) {
    if (!out || H < 1 || W < 1 || max_batch < 1) return LLG_E_ARG;
    *out = nullptr;
    if (hipSetDevice(device) != hipSuccess) return LLG_E_DEVICE;
    llg_sur* s = new llg_sur();
    *out = s;
    s->device = device;
    s->H = H;
    s->W = W;
    s->maxb = max_batch;
    SCHK(s, hipStreamCreateWithFlags(&s->stream, hipStreamNonBlocking));
    long long off = 0;
    for (int l = 0; l < NL; ++l) {
        s->woff.push_back(off);
        off += (long long)COUT[l] * CIN[l] * 9;
        s->boff.push_back(off);
        off += COUT[l];
    }
    s->nparam = off;
    // bias reads cover 32 entries: pad the parameter arrays at the end
    const size_t pbytes = sizeof(float) * (size_t)(off + CH);
    SCHK(s, hipMalloc(&s->params, pbytes));
    SCHK(s, hipMalloc(&s->grads, pbytes));
    SCHK(s, hipMalloc(&s->mom1, pbytes));
    SCHK(s, hipMalloc(&s->mom2, pbytes));
    SCHK(s, hipMemset(s->params, 0, pbytes));
    SCHK(s, hipMemset(s->grads, 0, pbytes));
    SCHK(s, hipMemset(s->mom1, 0, pbytes));
    SCHK(s, hipMemset(s->mom2, 0, pbytes));
    const size_t npx = (size_t)max_batch * H * W;
    for (int l = 0; l < NL; ++l) {
        SCHK(s, hipMalloc(&s->wf[l], 9 * CH * CH * 2));
        SCHK(s, hipMalloc(&s->wtr[l], 9 * CH * CH * 2));
        SCHK(s, hipMalloc(&s->z[l], npx * CH * 4));
    }
    for (int l = 0; l < NL; ++l) SCHK(s, hipMalloc(&s->act[l], npx * CH * 2));
    SCHK(s, hipMalloc(&s->g, npx * CH * 4));
    SCHK(s, hipMalloc(&s->gz, npx * CH * 2));
    SCHK(s, hipMalloc(&s->gz2, npx * CH * 2));
    int maxblk = 0;
    for (int n = 1; n <= max_batch; ++n) maxblk = std::max(maxblk, wg_blocks(s, n));
    s->wslots = (size_t)NL * maxblk * NWG * 4 <= WG_HELD ? NL : 1;
    SCHK(s, hipMalloc(&s->part_w, (size_t)s->wslots * maxblk * NWG * 4));
    SCHK(s, hipMalloc(&s->part_b, (size_t)s->wslots * maxblk * CH * 4));
    SCHK(s, hipMalloc(&s->part2, (size_t)s->wslots * WG_SEG * (NWG + CH) * 4));
    SCHK(s, hipMalloc(&s->part_l, ((size_t)H * W + 255) / 256 * max_batch * 4));
    SCHK(s, hipHostMalloc(&s->loss, sizeof(float)));
    SCHK(s, hipMalloc(&s->dm_in, npx * 3 * 4));
    SCHK(s, hipMalloc(&s->dm_t, npx * 3 * 4));
    SCHK(s, hipMalloc(&s->dm_out, npx * 3 * 4));
    SCHK(s, hipMalloc(&s->dB, (size_t)max_batch * 3 * 4));
    return LLG_OK;
}

void llg_sur_destroy(llg_sur* s) {
    if (!s) return;
    (void)hipSetDevice(s->device);
    if (s->stream) (void)hipStreamSynchronize(s->stream);
    void* ptrs[] = {s->params, s->grads, s->mom1, s->mom2, s->g, s->gz, s->gz2, s->part_w, s->part_b,
                    s->part2, s->part_l, s->dm_in, s->dm_t, s->dm_out, s->dB};
    for (void* p : ptrs)
        if (p) (void)hipFree(p);
    if (s->loss) (void)hipHostFree(s->loss);
    for (int l = 0; l < NL; ++l) {
        if (s->wf[l]) (void)hipFree(s->wf[l]);
        if (s->wtr[l]) (void)hipFree(s->wtr[l]);
        if (s->z[l]) (void)hipFree(s->z[l]);
    }
    for (int l = 0; l < NL; ++l)
        if (s->act[l]) (void)hipFree(s->act[l]);
    if (s->props) (void)hipFree(s->props);
    if (s->dmax) (void)hipFree(s->dmax);
    for (llg_batch* v : s->vb)
        if (v) llg_batch_destroy(v);
    s->vb.clear();
    if (s->eb) llg_batch_destroy(s->eb);
    if (s->stream) (void)hipStreamDestroy(s->stream);
    delete s;
}

const char* llg_sur_last_error(const llg_sur* s) { return s ? s->err.c_str() : "null surrogate"; }

int64_t llg_sur_num_params(void) {
    long long n = 0;
    for (int l = 0; l < NL; ++l) n += (long long)COUT[l] * CIN[l] * 9 + COUT[l];
    return n;
}

llg_status llg_sur_set_params(llg_sur* s, const float* params, int64_t n) {
    if (!s || !params) return LLG_E_ARG;
    if (n != s->nparam) return sfail(s, LLG_E_ARG, "expected %lld parameters", s->nparam);
    SCHK(s, hipSetDevice(s->device));
    SCHK(s, hipMemcpyAsync(s->params, params, sizeof(float) * n, hipMemcpyHostToDevice, s->stream));
    SCHK(s, hipMemsetAsync(s->mom1, 0, sizeof(float) * (n + CH), s->stream));
    SCHK(s, hipMemsetAsync(s->mom2, 0, sizeof(float) * (n + CH), s->stream));
    s->adam_t = 0;
    llg_status rc = update_pack(s, 0.f, 1.f, 1.f);
    if (rc != LLG_OK) return rc;
    SCHK(s, hipStreamSynchronize(s->stream));
    return LLG_OK;
}

llg_status llg_sur_set_output_scale(llg_sur* s, double scale) {
    if (!s || !(scale > 0) || !isfinite(scale) || scale > 1e30) return LLG_E_ARG;
    s->out_scale = (float)scale;
    return LLG_OK;
}

llg_status llg_sur_get_params(llg_sur* s, float* params, int64_t n) {
    if (!s || !params) return LLG_E_ARG;
    if (n != s->nparam) return sfail(s, LLG_E_ARG, "expected %lld parameters", s->nparam);
    SCHK(s, hipSetDevice(s->device));
    SCHK(s, hipMemcpyAsync(params, s->params, sizeof(float) * n, hipMemcpyDeviceToHost, s->stream));
    SCHK(s, hipStreamSynchronize(s->stream));
    return LLG_OK;
}

llg_status llg_sur_get_grads(llg_sur* s, float* grads, int64_t n) {
    if (!s || !grads) return LLG_E_ARG;
    if (n != s->nparam) return sfail(s, LLG_E_ARG, "expected %lld parameters", s->nparam);
    SCHK(s, hipSetDevice(s->device));
    SCHK(s, hipMemcpyAsync(grads, s->grads, sizeof(float) * n, hipMemcpyDeviceToHost, s->stream));
    SCHK(s, hipStreamSynchronize(s->stream));
    return LLG_OK;
}

// gradient of the loss (and optionally one Adam step) for a batch
llg_status llg_sur_train_step(llg_sur* s, const float* m_in, const float* m_target, const float* m_base,
                              const float* B, int batch, llg_mem where, float lr, float* loss) {
    llg::host::TraceRange trace_("llg_sur_train_step");
    if (!s || !m_in || !m_target || !B || batch < 1 || batch > s->maxb) return LLG_E_ARG;
    SCHK(s, hipSetDevice(s->device));
    if (!s->packed) return sfail(s, LLG_E_STATE, "parameters not set");
    const size_t npx = (size_t)batch * s->H * s->W;
    const float* mi = m_in;
    const float* mt = m_target;
    const float* mb = m_base;
    if (where != LLG_DEVICE) {
        SCHK(s, hipMemcpyAsync(s->dm_in, m_in, npx * 3 * 4, hipMemcpyHostToDevice, s->stream));
        SCHK(s, hipMemcpyAsync(s->dm_t, m_target, npx * 3 * 4, hipMemcpyHostToDevice, s->stream));
        mi = s->dm_in;
        mt = s->dm_t;
        if (m_base) {
            SCHK(s, hipMemcpyAsync(s->dm_out, m_base, npx * 3 * 4, hipMemcpyHostToDevice, s->stream));
            mb = s->dm_out;
        }
    }
    if (!mb) mb = mi;
    SCHK(s, hipMemcpyAsync(s->dB, B, (size_t)batch * 3 * 4, hipMemcpyHostToDevice, s->stream));
    llg_status rc = forward(s, mi, s->dB, batch, true);
    if (rc != LLG_OK) return rc;
    const int hw = s->H * s->W, lb = (hw + 255) / 256 * batch;
    hipLaunchKernelGGL(loss_kernel, dim3((hw + 255) / 256, batch), dim3(256), 0, s->stream, s->z[NL - 1], mb, mt, s->gz,
                       s->part_l, hw, 1.0f / s->out_scale);
    SCHK(s, hipGetLastError());
    hipLaunchKernelGGL(sum_kernel, dim3(1), dim3(256), 0, s->stream, s->part_l, lb, s->loss);
    SCHK(s, hipGetLastError());
    u16* gcur = s->gz;    // gradient at layer l's pre-activation
    u16* gnext = s->gz2;
    for (int l = NL - 1; l >= 0; --l) {
        launch_wgrad(s, gcur, s->act[l], batch, s->wslots > 1 ? l : 0);
        SCHK(s, hipGetLastError());
        if (s->wslots == 1) {
            launch_wgrad_reduce(s, batch, 1, one_layer(l, s->grads + s->woff[l], s->grads + s->boff[l]));
            SCHK(s, hipGetLastError());
        }
        if (l > 0) {
            // data gradient: the same convolution with flipped, transposed
            // weights, times SiLU'(z) of layer l - 1 (every hidden layer has
            // the activation)
            launch_conv(s, gcur, s->wtr[l], nullptr, nullptr, nullptr, nullptr, gnext,
                        reinterpret_cast<const u16*>(s->z[l - 1]), batch, 0);
            SCHK(s, hipGetLastError());
            std::swap(gcur, gnext);
        }
    }
    if (s->wslots > 1) {
        launch_wgrad_reduce(s, batch, NL, layer_set(s, s->grads));
        SCHK(s, hipGetLastError());
    }
    if (lr > 0.f) {
        s->adam_t += 1;
        const float c1 = 1.0f - powf(0.9f, (float)s->adam_t), c2 = 1.0f - powf(0.999f, (float)s->adam_t);
        rc = update_pack(s, lr, c1, c2);
        if (rc != LLG_OK) return rc;
    }
    SCHK(s, hipStreamSynchronize(s->stream));
    if (loss) *loss = *s->loss;
    return LLG_OK;
}

llg_status llg_sur_predict(llg_sur* s, const float* m_in, const float* m_base, const float* B, int batch,
                           llg_mem where, float* m_out) {
    if (!s || !m_in || !B || !m_out || batch < 1 || batch > s->maxb) return LLG_E_ARG;
    SCHK(s, hipSetDevice(s->device));
    if (!s->packed) return sfail(s, LLG_E_STATE, "parameters not set");
    const size_t npx = (size_t)batch * s->H * s->W;
    const float* mi = m_in;
    const float* mb = m_base;
    float* mo = m_out;
    if (where != LLG_DEVICE) {
        SCHK(s, hipMemcpyAsync(s->dm_in, m_in, npx * 3 * 4, hipMemcpyHostToDevice, s->stream));
        mi = s->dm_in;
        mo = s->dm_out;
        if (m_base) {
            SCHK(s, hipMemcpyAsync(s->dm_t, m_base, npx * 3 * 4, hipMemcpyHostToDevice, s->stream));
            mb = s->dm_t;
        }
    }
    if (!mb) mb = mi;
    SCHK(s, hipMemcpyAsync(s->dB, B, (size_t)batch * 3 * 4, hipMemcpyHostToDevice, s->stream));
    llg_status rc = forward(s, mi, s->dB, batch, false);
    if (rc != LLG_OK) return rc;
    hipLaunchKernelGGL(propose_kernel, dim3((unsigned)((npx + 255) / 256)), dim3(256), 0, s->stream, mb,
                       s->z[NL - 1], mo, batch, s->H, s->W, s->out_scale);
    SCHK(s, hipGetLastError());
    if (where != LLG_DEVICE) SCHK(s, hipMemcpyAsync(m_out, s->dm_out, npx * 3 * 4, hipMemcpyDeviceToHost, s->stream));
    SCHK(s, hipStreamSynchronize(s->stream));
    return LLG_OK;
}

// the pre-activation of layer `layer` (the last one: the net's dm before
// padding) for a batch, [batch][H][W][32] float into host memory; for parity
// checks
llg_status llg_sur_forward_raw(llg_sur* s, const float* m_in, const float* B, int batch, int layer, float* z_out) {
    if (!s || !m_in || !B || !z_out || batch < 1 || batch > s->maxb || layer < 0 || layer >= NL) return LLG_E_ARG;
    SCHK(s, hipSetDevice(s->device));
    if (!s->packed) return sfail(s, LLG_E_STATE, "parameters not set");
    const size_t npx = (size_t)batch * s->H * s->W;
    SCHK(s, hipMemcpyAsync(s->dm_in, m_in, npx * 3 * 4, hipMemcpyHostToDevice, s->stream));
    SCHK(s, hipMemcpyAsync(s->dB, B, (size_t)batch * 3 * 4, hipMemcpyHostToDevice, s->stream));
    llg_status rc = forward(s, s->dm_in, s->dB, batch, false, layer);
    if (rc != LLG_OK) return rc;
    SCHK(s, hipMemcpyAsync(z_out, s->z[layer], npx * CH * 4, hipMemcpyDeviceToHost, s->stream));
    SCHK(s, hipStreamSynchronize(s->stream));
    return LLG_OK;
}

// one convolution layer through the training kernels, for parity checks:
// x and gy are [batch][H][W][32] float (host) and are rounded to bf16 as the
// training path rounds activations and gradients; y = conv(x) + bias, and if
// gy is given gw [cout][cin][3][3], gb [cout] and gx [batch][H][W][32]
llg_status llg_sur_conv_check(llg_sur* s, int layer, const float* x, const float* gy, int batch, float* y,
                              float* gx, float* gw, float* gb) {
    if (!s || !x || !y || batch < 1 || batch > s->maxb || layer < 0 || layer >= NL) return LLG_E_ARG;
    if (gy && (!gx || !gw || !gb)) return LLG_E_ARG;
    SCHK(s, hipSetDevice(s->device));
    if (!s->packed) return sfail(s, LLG_E_STATE, "parameters not set");
    const size_t n = (size_t)batch * s->H * s->W * CH;
    const unsigned nb = (unsigned)((n + 255) / 256);
    SCHK(s, hipMemcpyAsync(s->g, x, n * 4, hipMemcpyHostToDevice, s->stream));
    hipLaunchKernelGGL(to_bf16_kernel, dim3(nb), dim3(256), 0, s->stream, s->g, s->act[0], n);
    SCHK(s, hipGetLastError());
    launch_conv(s, s->act[0], s->wf[layer], s->params + s->boff[layer], s->z[0], nullptr, nullptr, nullptr, nullptr,
                batch, 0);
    SCHK(s, hipGetLastError());
    SCHK(s, hipMemcpyAsync(y, s->z[0], n * 4, hipMemcpyDeviceToHost, s->stream));
    if (gy) {
        float *dgw = nullptr, *dgb = nullptr;
        SCHK(s, hipMalloc(&dgw, sizeof(float) * COUT[layer] * CIN[layer] * 9));
        SCHK(s, hipMalloc(&dgb, sizeof(float) * CH));
        SCHK(s, hipMemcpyAsync(s->g, gy, n * 4, hipMemcpyHostToDevice, s->stream));
        hipLaunchKernelGGL(act_bwd_kernel, dim3(nb), dim3(256), 0, s->stream, s->g, (const float*)nullptr, s->gz, n, 0);
        SCHK(s, hipGetLastError());
        launch_wgrad(s, s->gz, s->act[0], batch, 0);
        SCHK(s, hipGetLastError());
        launch_wgrad_reduce(s, batch, 1, one_layer(layer, dgw, dgb));
        SCHK(s, hipGetLastError());
        launch_conv(s, s->gz, s->wtr[layer], nullptr, s->z[1], nullptr, nullptr, nullptr, nullptr, batch, 0);
        SCHK(s, hipGetLastError());
        SCHK(s, hipMemcpyAsync(gx, s->z[1], n * 4, hipMemcpyDeviceToHost, s->stream));
        SCHK(s, hipMemcpyAsync(gw, dgw, sizeof(float) * COUT[layer] * CIN[layer] * 9, hipMemcpyDeviceToHost,
                               s->stream));
        SCHK(s, hipMemcpyAsync(gb, dgb, sizeof(float) * COUT[layer], hipMemcpyDeviceToHost, s->stream));
        SCHK(s, hipStreamSynchronize(s->stream));
        (void)hipFree(dgw);
        (void)hipFree(dgb);
    }
    SCHK(s, hipStreamSynchronize(s->stream));
    return LLG_OK;
}

// ---------------------------------------------------------------------------
// speculative verification: the surrogate chains up to `window` proposals,
// one plain batched launch advances every start state by seg_steps RK4
// steps, the prefix of proposals within max_dm of their plain counterparts
// is accepted and the plain state at the end of the accepted prefix (or at
// the first rejected proposal) is committed
// ---------------------------------------------------------------------------
namespace {

bool same_film(const llg_film_desc& a, const llg_film_desc& b) {
    if (a.nx != b.nx || a.ny != b.ny || a.dx != b.dx || a.dy != b.dy || a.dz != b.dz || a.Ms != b.Ms ||
        a.Aex != b.Aex || a.alpha != b.alpha || a.Ku != b.Ku)
        return false;
    for (int i = 0; i < 3; ++i)
        if (a.u[i] != b.u[i] || a.B[i] != b.B[i]) return false;
    return true;
}

llg_status max_distance(llg_sur* s, const float* a, const float* b, int ncells, unsigned* out) {
    const int blocks = std::min(1024, (ncells + 255) / 256);
    hipLaunchKernelGGL(maxdiff_kernel, dim3(blocks), dim3(256), 0, s->stream, a, b, ncells, out);
    SCHK(s, hipGetLastError());
    return LLG_OK;
}

float bits_to_float(unsigned u) {
    float f;
    memcpy(&f, &u, 4);
    return f;
}

}  // namespace

llg_status llg_sur_advance(llg_sur* s, const llg_film_desc* film, int window, int64_t n_segments, int seg_steps,
                           double dt, int predictor, double max_dm, float* m, llg_mem where, llg_sur_stats* out) {
    llg::host::TraceRange trace_("llg_sur_advance");
    if (!s || !film || !m || window < 1 || window > 256 || n_segments < 0 || seg_steps < 1 || !(dt > 0) ||
        !(max_dm >= 0) ||
        (predictor != LLG_SUR_BASE_STATE && predictor != LLG_SUR_BASE_EULER && predictor != LLG_SUR_BASE_RK4))
        return LLG_E_ARG;
    s->err.clear();
    SCHK(s, hipSetDevice(s->device));
    if (!s->packed) return sfail(s, LLG_E_STATE, "parameters not set");
    if (film->nx != s->W || film->ny != s->H)
        return sfail(s, LLG_E_ARG, "film %d x %d does not match the surrogate's %d x %d", film->nx, film->ny, s->W,
                     s->H);
    const int ncells = s->H * s->W;
    const size_t vec = sizeof(float) * 3 * (size_t)ncells;
    llg_sur_stats st = {};
    // the verification batches (start states kVerifyPart p ... of a round)
    // and the coarse-step batch: copies of the film
    const int nparts = (window + kVerifyPart - 1) / kVerifyPart;
    if (s->vb.empty() || s->vwin != window || !same_film(s->vdesc, *film)) {
        for (llg_batch* v : s->vb)
            if (v) llg_batch_destroy(v);
        s->vb.assign(nparts, nullptr);
        if (s->eb) llg_batch_destroy(s->eb);
        s->eb = nullptr;
        if (s->props) (void)hipFree(s->props);
        if (s->dmax) (void)hipFree(s->dmax);
        s->props = nullptr;
        s->dmax = nullptr;
        std::vector<float> h0(3 * (size_t)ncells);
        SCHK(s, hipMemcpy(h0.data(), m, vec, where == LLG_DEVICE ? hipMemcpyDeviceToHost : hipMemcpyHostToHost));
        std::vector<llg_film_desc> fd(window, *film);
        for (auto& f : fd) f.m0 = h0.data();
        for (int i = 0; i <= nparts; ++i) {
            const int count = i < nparts ? std::min(kVerifyPart, window - i * kVerifyPart) : 1;
            llg_batch** dst = i < nparts ? &s->vb[i] : &s->eb;
            const llg_status rc = llg_batch_create(s->device, fd.data(), count, dst);
            if (rc != LLG_OK) {
                const std::string why = *dst ? llg_batch_last_error(*dst) : "batch creation failed";
                if (*dst) llg_batch_destroy(*dst);
                *dst = nullptr;
                for (llg_batch* v : s->vb)   // the others are rebuilt by the next call
                    if (v) llg_batch_destroy(v);
                s->vb.clear();
                return sfail(s, rc, "%s batch: %s", i < nparts ? "verification" : "predictor", why.c_str());
            }
        }
        s->vdesc = *film;
        s->vdesc.m0 = nullptr;
        s->vwin = window;
        SCHK(s, hipMalloc(&s->props, vec * (window + 1)));
        SCHK(s, hipMalloc(&s->dmax, sizeof(unsigned) * 2 * window));
    }
    const float Bf[3] = {(float)film->B[0], (float)film->B[1], (float)film->B[2]};
    SCHK(s, hipMemcpyAsync(s->dB, Bf, sizeof Bf, hipMemcpyHostToDevice, s->stream));
    SCHK(s, hipMemcpyAsync(s->props, m, vec, where == LLG_DEVICE ? hipMemcpyDeviceToDevice : hipMemcpyHostToDevice,
                           s->stream));
    // the start state is checked and renormalised as llg_set_m does
    {
        hipLaunchKernelGGL(zero_u32_kernel, dim3(1), dim3(64), 0, s->stream, s->dmax, 1);
        SCHK(s, hipGetLastError());
        SCHK(s, llg::launch_normalize_check(s->props, ncells, reinterpret_cast<int*>(s->dmax), s->stream));
        unsigned bad = 0;
        SCHK(s, hipMemcpyAsync(&bad, s->dmax, sizeof bad, hipMemcpyDeviceToHost, s->stream));
        SCHK(s, hipStreamSynchronize(s->stream));
        if (bad) return sfail(s, LLG_E_ARG, "m is not a field of unit vectors");
    }
    std::vector<float*> ptr(window);
    std::vector<unsigned> hd(2 * window);
    const llg_method coarse = predictor == LLG_SUR_BASE_EULER ? LLG_EULER : LLG_RK4;
    int64_t done = 0;
    while (done < n_segments) {
        const int w = (int)std::min<int64_t>(window, n_segments - done);
        const int parts = (w + kVerifyPart - 1) / kVerifyPart;   // parts this round
        float* P = s->props;
        const size_t stride = 3 * (size_t)ncells;
        // plain segments from the start states of part p, on the part's
        // batch stream, overlapping the proposals still to come
        auto verify = [&](int p) -> llg_status {
            const int first = p * kVerifyPart, count = std::min(kVerifyPart, w - first);
            const llg_status rc = llg_batch_fixed_async_(s->vb[p], LLG_RK4, dt, seg_steps, P + first * stride,
                                                         stride, count, s->stream, ptr.data() + first);
            if (rc != LLG_OK) return sfail(s, rc, "verification batch: %s", llg_batch_last_error(s->vb[p]));
            return LLG_OK;
        };
        // proposals 1..w, each from the previous one: normalize(base + dm)
        // with base the previous state or its one coarse step (Euler or
        // RK4) over the whole segment by the plain solver; a part starts as
        // soon as its last start state exists
        int launched = 0;
        for (int j = 1; j <= w; ++j) {
            llg_status rc = LLG_OK;
            while (launched < parts && std::min((launched + 1) * kVerifyPart, w) <= j)
                if ((rc = verify(launched++)) != LLG_OK) return rc;
            const float* prev = P + (size_t)(j - 1) * stride;
            const float* base = prev;
            // (the coarse step on its batch's stream, the network beside it)
            if (predictor != LLG_SUR_BASE_STATE) {
                float* em = nullptr;
                rc = llg_batch_fixed_async_(s->eb, coarse, dt * seg_steps, 1, prev, 0, 1, s->stream, &em);
                if (rc != LLG_OK) return sfail(s, rc, "predictor batch: %s", llg_batch_last_error(s->eb));
                base = em;
            }
            rc = forward(s, prev, s->dB, 1, false);
            if (rc != LLG_OK) return rc;
            if (predictor != LLG_SUR_BASE_STATE) {
                rc = llg_batch_then_(s->eb, s->stream);
                if (rc != LLG_OK) return sfail(s, rc, "predictor batch: %s", llg_batch_last_error(s->eb));
            }
            hipLaunchKernelGGL(propose_kernel, dim3((ncells + 255) / 256), dim3(256), 0, s->stream, base,
                               s->z[NL - 1], P + (size_t)j * stride, 1, s->H, s->W, s->out_scale);
            SCHK(s, hipGetLastError());
        }
        for (int p = 0; p < parts; ++p) {
            const llg_status rc = llg_batch_then_(s->vb[p], s->stream);
            if (rc != LLG_OK) return sfail(s, rc, "verification batch: %s", llg_batch_last_error(s->vb[p]));
        }
        // d_j = distance of proposal j to the plain result from its
        // predecessor (non-finite: infinite), and whether each plain result
        // is finite (0) or not
        hipLaunchKernelGGL(zero_u32_kernel, dim3((2 * window + 255) / 256), dim3(256), 0, s->stream, s->dmax,
                           2 * window);
        SCHK(s, hipGetLastError());
        for (int j = 1; j <= w; ++j) {
            llg_status rc = max_distance(s, P + (size_t)j * stride, ptr[j - 1], ncells, s->dmax + j - 1);
            if (rc == LLG_OK) rc = max_distance(s, ptr[j - 1], ptr[j - 1], ncells, s->dmax + window + j - 1);
            if (rc != LLG_OK) return rc;
        }
        SCHK(s, hipMemcpyAsync(hd.data(), s->dmax, sizeof(unsigned) * 2 * window, hipMemcpyDeviceToHost, s->stream));
        SCHK(s, hipStreamSynchronize(s->stream));
        int k = w;       // segments this round commits
        int acc = w;     // proposals accepted
        for (int j = 1; j <= w; ++j) {
            const float d = bits_to_float(hd[j - 1]);
            st.max_dm_seen = std::max(st.max_dm_seen, (double)d);
            if (!((double)d <= max_dm)) { k = j; acc = j - 1; break; }
            st.max_dm_accepted = std::max(st.max_dm_accepted, (double)d);
        }
        if (hd[window + k - 1] != 0u)
            return sfail(s, LLG_E_DIVERGED, "plain segment %lld: non-finite field or torque", (long long)(done + k - 1));
        st.proposals += w;
        st.accepted += acc;
        st.rounds += 1;
        st.segments += k;
        SCHK(s, hipMemcpyAsync(P, ptr[k - 1], vec, hipMemcpyDeviceToDevice, s->stream));
        done += k;
    }
    SCHK(s, hipMemcpyAsync(m, s->props, vec, where == LLG_DEVICE ? hipMemcpyDeviceToDevice : hipMemcpyDeviceToHost,
                           s->stream));
    SCHK(s, hipStreamSynchronize(s->stream));
    if (out) *out = st;
    return LLG_OK;
}

}  // extern "C"
