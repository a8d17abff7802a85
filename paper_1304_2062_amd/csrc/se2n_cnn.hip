// BF16 MFMA kernels of the learned corrector: 3x3 circular convolutions as
// implicit GEMMs on v_mfma_f32_16x16x32_bf16 (bfloat16 operands, FP32
// accumulation), their input and weight gradients, the loss and Adam.
//
// Product shape of one MFMA: D[16 x 16] += A[16 x 32] B[32 x 16] with
//   A[row][k]: lane l holds row l%16, k = 8*(l/16) .. 8*(l/16)+7
//   B[k][col]: lane l holds col l%16, the same 8 k
//   D[row][col]: lane l holds col l%16, rows 4*(l/16) .. 4*(l/16)+3
// For a conv, rows are output channels, columns pixels and k input
// channels (one tap at a time); for the weight gradient rows are output
// channels, columns input channels and k pixels.
#include <hip/hip_runtime.h>

#include <cmath>
#include <cstdint>

#include "se2n_cnn.hpp"
#include "se2n_passes.hpp"

namespace se2n {

namespace {

typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef __bf16 bf16x4 __attribute__((ext_vector_type(4)));
typedef float f32x4 __attribute__((ext_vector_type(4)));

constexpr int C = kCnnC;
constexpr int T = kCnnTile;    // 16 x 16 output pixels per workgroup
constexpr int HT = T + 2;      // with a one-pixel halo
// LDS elements per pixel (32 channels + 8): an odd multiple of 16 bytes, so
// that the 8 lanes served together by a 128-byte LDS cycle hit distinct banks.
constexpr int PS = 40;

__device__ __forceinline__ int wrap(int i, int M) { return i < 0 ? i + M : (i >= M ? i - M : i); }

__device__ __forceinline__ f32x4 mfma(bf16x8 a, bf16x8 b, f32x4 c) {
    return __builtin_amdgcn_mfma_f32_16x16x32_bf16(a, b, c, 0, 0, 0);
}

// Per-image root mean square of the input volume: partial sums of squares
// over kScaleBlocks contiguous chunks, then their sum in a fixed order.
constexpr int kScaleBlocks = kCnnScaleBlocks;

__global__ __launch_bounds__(256) void k_cnn_sumsq(const float* __restrict__ psi, long n, float* __restrict__ parts);
__global__ __launch_bounds__(256) void k_cnn_scale(const float* __restrict__ parts, long n, float* __restrict__ scale);

__global__ __launch_bounds__(256) void k_cnn_pack(const float* __restrict__ psi, const float* __restrict__ scale,
                                                  bf16* __restrict__ act, int N, int M, int B) {
    const long MM = (long)M * M;
    const long t = (long)blockIdx.x * blockDim.x + threadIdx.x;
    if (t >= (long)B * 4 * MM) return;
    const long p = t % MM;
    const long q = t / MM;
    const int cb = (int)(q & 3);
    const long b = q >> 2;
    const float inv = 1.0f / scale[b];
    bf16x8 v;
#pragma unroll
    for (int j = 0; j < 8; ++j) {
        const int c = cb * 8 + j;
        v[j] = (bf16)(c < N ? psi[(b * N + c) * MM + p] * inv : 0.0f);
    }
    *reinterpret_cast<bf16x8*>(act + (b * MM + p) * C + cb * 8) = v;
}

// The sum over a workgroup of W waves, on thread 0 (after a barrier).
template <int W>
__device__ __forceinline__ float block_sum(float v, float* red) {
#pragma unroll
    for (int off = 32; off >= 1; off >>= 1) v += __shfl_xor(v, off, 64);
    const int w = threadIdx.x >> 6;
    if ((threadIdx.x & 63) == 0) red[w] = v;
    __syncthreads();
    float s = 0.0f;
    if (threadIdx.x == 0) {
#pragma unroll
        for (int i = 0; i < W; i += 2) s += red[i] + red[i + 1];
    }
    return s;
}

// A layer's weights as MFMA operands, NB blocks of 16 output channels: 36 NB
// registers.
template <int NB>
struct NetW {
    bf16x8 a[9][NB];
    // (the empty asm keeps a loop's loads in the loop: three layers' weights
    // together do not fit in the registers)
    __device__ __forceinline__ void load(const bf16* __restrict__ wA, int col, int kg) {
        int base = 0;
        asm volatile("" : "+s"(base));
        wA += base;
#pragma unroll
        for (int tap = 0; tap < 9; ++tap)
#pragma unroll
            for (int mb = 0; mb < NB; ++mb)
                a[tap][mb] = *reinterpret_cast<const bf16x8*>(wA + (tap * C + 16 * mb + col) * C + kg * 8);
    }
};

// One layer of k_cnn_net between LDS tiles: the input tile of side HS at `in`,
// output side OS = HS - 2.  Of the first 16 columns a wave takes RW rows, so
// that an operand read from LDS serves up to three rows (3 (RW + 2) reads for
// 18 RW MFMAs; 9 for 18 where every group of 16 pixels reads its own, which
// made LDS the bound); the columns beyond go in groups of 16 / REM rows.  The
// last wave's rows may overlap its neighbour's (the same values twice).
// put(pix, c0, v): the products of channels c0 .. c0 + 3 of output pixel pix.
template <int HS, int NB, class Put>
__device__ __forceinline__ void net_layer(const bf16* in, const NetW<NB>& wt, int w, int col, int kg, Put&& put) {
    constexpr int OS = HS - 2, RW = (OS + 3) / 4, REM = OS - 16;
    {
        const int y = min(RW * w, OS - RW);
        const bf16* src = in + (y * HS + col) * PS + kg * 8;
        f32x4 acc[RW][NB];
#pragma unroll
        for (int r = 0; r < RW; ++r)
#pragma unroll
            for (int mb = 0; mb < NB; ++mb) acc[r][mb] = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
        for (int q = 0; q < RW + 2; ++q) {
            bf16x8 bv[3];
#pragma unroll
            for (int dx = 0; dx < 3; ++dx) bv[dx] = *reinterpret_cast<const bf16x8*>(src + (q * HS + dx) * PS);
#pragma unroll
            for (int dx = 0; dx < 3; ++dx)
#pragma unroll
                for (int r = 0; r < RW; ++r) {
                    const int dy = q - r;
                    if (dy >= 0 && dy < 3) {
#pragma unroll
                        for (int mb = 0; mb < NB; ++mb)
                            acc[r][mb] = mfma(wt.a[3 * dy + dx][mb], bv[dx], acc[r][mb]);
                    }
                }
            if (q >= 2) {
                const int r = q - 2;
#pragma unroll
                for (int mb = 0; mb < NB; ++mb) put((y + r) * OS + col, 16 * mb + 4 * kg, acc[r][mb]);
            }
        }
    }
    if constexpr (REM > 0) {
        constexpr int RG = 16 / REM, G = (OS + RG - 1) / RG;
#pragma unroll 1
        for (int g = w; g < G; g += 4) {
            const int oy = g * RG + col / REM, ox = 16 + col % REM;
            const bf16* src = in + (min(oy, OS - 1) * HS + ox) * PS + kg * 8;
            f32x4 acc[NB];
#pragma unroll
            for (int mb = 0; mb < NB; ++mb) acc[mb] = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
            for (int tap = 0; tap < 9; ++tap) {
                const bf16x8 bv = *reinterpret_cast<const bf16x8*>(src + (tap / 3 * HS + tap % 3) * PS);
#pragma unroll
                for (int mb = 0; mb < NB; ++mb) acc[mb] = mfma(wt.a[tap][mb], bv, acc[mb]);
            }
            if (oy < OS)
#pragma unroll
                for (int mb = 0; mb < NB; ++mb) put(oy * OS + ox, 16 * mb + 4 * kg, acc[mb]);
        }
    }
}

// The whole network on a 16 x 16 pixel tile: the input with a halo of three
// pixels, layer 1 on 20 x 20 pixels, layer 2 on 18 x 18, layer 3 on the tile,
// the activations between them in LDS only (28 % more products than one layer
// at a time, for 268 MB of activations less at 2^20 pixels).  Layer 3 takes
// its operands the other way round, pixels as rows: a lane then holds four
// pixels of one channel, 16 bytes of the planar volume.
//   PACKED  the input is a0; otherwise coarse / scale, packed on the way
//   !TRAIN  out = coarse + scale (net + bias).  out may be coarse if PACKED: a
//           tile's halo is then not its neighbour's result.
//   TRAIN   the tile's inputs and activations a0, a1, a2 to memory for the
//           weight gradients; d = (out - target) / scale, g = gscale d (bf16,
//           channels last), per-tile sums of d^2
// A wave takes NB blocks of 16 output channels.  Two workgroups share a
// compute unit's LDS; a layer's weights and the values that layer 3 adds to are
// fetched one layer ahead.  At 2^20 pixels no unit is saturated: matrix cores
// 28 %, vector instructions 38 %, LDS 42 % of the time (202 MB read with the
// halos, 135 MB written, 2.5 TB/s).  Waves of one block each hide more of that
// where the registers allow it (inference 138 -> 127 us; training spills,
// 185 -> 245 us).
// Layer by layer, with the packing, 43 + 41 + 41 + 115 us before.
template <bool TRAIN, bool PACKED, int NB>
__global__ __launch_bounds__(512 / NB, 4 / NB) void k_cnn_net(bf16* __restrict__ a0, const bf16* __restrict__ wf,
                                                    const float* __restrict__ params, const float* coarse, float* out,
                                                    const float* __restrict__ scale, bf16* __restrict__ a1,
                                                    bf16* __restrict__ a2, const float* __restrict__ target,
                                                    bf16* __restrict__ gout, float* __restrict__ lparts, float gscale,
                                                    int N, int M) {
    constexpr int S0 = T + 6, S1 = T + 4, S2 = T + 2;
    __shared__ __attribute__((aligned(16))) bf16 s_a[S0 * S0 * PS];
    __shared__ __attribute__((aligned(16))) bf16 s_b[S1 * S1 * PS];
    __shared__ float s_bias[2 * C];
    __shared__ float red[8];
    typedef float f32x4u __attribute__((ext_vector_type(4), aligned(4)));
    const int tid = threadIdx.x;
    constexpr int NTHR = 512 / NB;
    const int lane = tid & 63, w = tid >> (NB == 1 ? 7 : 6);  // row group
    const int mo = NB == 1 ? (tid >> 2) & 16 : 0;             // first output channel of the wave
    const int col = lane & 15, kg = lane >> 4;
    const int tiles = M / T;
    const long MM = (long)M * M;
    const float* bias3 = params + 2 * kCnnL + kCnnW;

    const int blk = xcd_contiguous(blockIdx.x, gridDim.x);
    const int x0 = blk % tiles * T, y0 = blk / tiles % tiles * T;
    const long b = blk / (tiles * tiles);
    const float sc = scale[b];
    const float inv = 1.0f / sc;
    if (tid < 2 * C) s_bias[tid] = params[(tid / C) * kCnnL + kCnnW + tid % C];
    NetW<NB> w1, w2, w3;
    if constexpr (PACKED) {
        constexpr int L = (S0 * S0 * 4 + NTHR - 1) / NTHR;
        const bf16* inb = a0 + b * MM * C;
        bf16x8 in[L];
#pragma unroll
        for (int j = 0; j < L; ++j) {
            const int e = tid + NTHR * j;
            if (e < S0 * S0 * 4) {
                const int pix = e >> 2;
                const int hy = pix / S0, hx = pix - hy * S0;
                const int gy = wrap(y0 + hy - 3, M), gx = wrap(x0 + hx - 3, M);
                in[j] = *reinterpret_cast<const bf16x8*>(inb + ((long)gy * M + gx) * C + (e & 3) * 8);
            }
        }
        w1.load(wf + mo * C, col, kg);
#pragma unroll
        for (int j = 0; j < L; ++j) {
            const int e = tid + NTHR * j;
            if (e < S0 * S0 * 4) *reinterpret_cast<bf16x8*>(s_a + (e >> 2) * PS + (e & 3) * 8) = in[j];
        }
    } else {
        // a task: four pixels from x0 - 4 + 4 xq of a row, 8 channels; row runs
        // of 96 bytes across the lanes
        constexpr int XQ = 6, NT = S0 * XQ * 4, L = (NT + NTHR - 1) / NTHR;
        // (every lane loads, from the last task or channel where its own is
        // beyond: no branch, all loads in flight at once)
        f32x4u v[L][8];
#pragma unroll
        for (int h = 0; h < L; ++h) {
            const int e = min(NTHR * h + tid, NT - 1);
            const int cb = e / (S0 * XQ), q = e - cb * (S0 * XQ);
            const int hy = q / XQ, xq = q - hy * XQ;
            const int gy = wrap(y0 + hy - 3, M), gx = wrap(x0 - 4 + 4 * xq, M);
            const float* p = coarse + b * N * MM + (long)gy * M + gx;
#pragma unroll
            for (int k = 0; k < 8; ++k) v[h][k] = *reinterpret_cast<const f32x4u*>(p + min(cb * 8 + k, N - 1) * MM);
        }
        w1.load(wf + mo * C, col, kg);
        __builtin_amdgcn_sched_barrier(0);
#pragma unroll
        for (int h = 0; h < L; ++h) {
            const int e = NTHR * h + tid;
            if (e < NT) {
                const int cb = e / (S0 * XQ), q = e - cb * (S0 * XQ);
                const int hy = q / XQ, xq = q - hy * XQ;
#pragma unroll
                for (int x = 0; x < 4; ++x) {
                    const int hx = 4 * xq - 1 + x;
                    bf16x8 t;
#pragma unroll
                    for (int k = 0; k < 8; ++k) t[k] = (bf16)(cb * 8 + k < N ? v[h][k][x] * inv : 0.0f);
                    if ((unsigned)hx < (unsigned)S0)
                        *reinterpret_cast<bf16x8*>(s_a + (hy * S0 + hx) * PS + cb * 8) = t;
                }
            }
        }
    }
    {
        __syncthreads();
        // a hidden layer's bias and rectifier; dst: its LDS tile
        auto hidden = [&](int l, bf16* dst) {
            return [=](int pix, int cw, f32x4 v) {
                const int c0 = mo + cw;
                const f32x4 bs = *reinterpret_cast<const f32x4*>(s_bias + l * C + c0);
                bf16x4 s;
#pragma unroll
                for (int k = 0; k < 4; ++k) s[k] = (bf16)fmaxf(v[k] + bs[k], 0.0f);
                *reinterpret_cast<bf16x4*>(dst + pix * PS + c0) = s;
            };
        };
        // the tile's own pixels of an LDS tile of side S with this halo
        auto keep = [&](bf16* act, const bf16* src, int S, int halo) {
#pragma unroll
            for (int j = 0; j < T * T * 4 / NTHR; ++j) {
                const int e = tid + NTHR * j;
                const int y = e >> 6, x = (e >> 2) & 15;
                *reinterpret_cast<bf16x8*>(act + (b * MM + (long)(y0 + y) * M + x0 + x) * C + (e & 3) * 8) =
                    *reinterpret_cast<const bf16x8*>(src + ((y + halo) * S + x + halo) * PS + (e & 3) * 8);
            }
        };
        w2.load(wf + kCnnW + mo * C, col, kg);
        if (TRAIN) keep(a0, s_a, S0, 3);
        net_layer<S0>(s_a, w1, w, col, kg, hidden(0, s_b));
        __syncthreads();

        // layer 3: tile rows 4w .. 4w + 3, pixels 4 kg .. 4 kg + 3 of channels
        // 16 mb + col
        w3.load(wf + 2 * kCnnW + mo * C, col, kg);
        const long o0 = b * N * MM + (long)(y0 + 4 * w) * M + x0 + 4 * kg;
        long oc[NB];
        f32x4u pre[4][NB], tgt[TRAIN ? 4 : 1][NB];
#pragma unroll
        for (int mb = 0; mb < NB; ++mb) {
            oc[mb] = o0 + min(mo + 16 * mb + col, N - 1) * MM;
#pragma unroll
            for (int r = 0; r < 4; ++r) pre[r][mb] = *reinterpret_cast<const f32x4u*>(coarse + oc[mb] + (long)r * M);
        }
        if (TRAIN) keep(a1, s_b, S1, 2);
        net_layer<S1>(s_b, w2, w, col, kg, hidden(1, s_a));
        __syncthreads();
        if (TRAIN) {
            keep(a2, s_a, S2, 1);
#pragma unroll
            for (int r = 0; r < 4; ++r)
#pragma unroll
                for (int mb = 0; mb < NB; ++mb)
                    tgt[r][mb] = *reinterpret_cast<const f32x4u*>(target + oc[mb] + (long)r * M);
        }
        float s = 0.0f;
#pragma unroll
        for (int r = 0; r < 4; ++r) {
            f32x4 acc[NB];
#pragma unroll
            for (int mb = 0; mb < NB; ++mb) acc[mb] = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
            for (int tap = 0; tap < 9; ++tap) {
                const bf16x8 bv =
                    *reinterpret_cast<const bf16x8*>(s_a + ((4 * w + r + tap / 3) * S2 + col + tap % 3) * PS + kg * 8);
#pragma unroll
                for (int mb = 0; mb < NB; ++mb) acc[mb] = mfma(bv, w3.a[tap][mb], acc[mb]);
            }
#pragma unroll
            for (int mb = 0; mb < NB; ++mb) {
                const int c = mo + 16 * mb + col;
                const float bc = bias3[min(c, N - 1)];
                f32x4u o;
#pragma unroll
                for (int i = 0; i < 4; ++i) o[i] = pre[r][mb][i] + sc * (acc[mb][i] + bc);
                if (TRAIN) {
                    // s_b is free: the gradient tile, pixel-major
#pragma unroll
                    for (int i = 0; i < 4; ++i) {
                        const float d = c < N ? (o[i] - tgt[r][mb][i]) * inv : 0.0f;
                        s += d * d;
                        s_b[((4 * w + r) * T + 4 * kg + i) * PS + c] = (bf16)(gscale * d);
                    }
                } else if (c < N) {
                    *reinterpret_cast<f32x4u*>(out + oc[mb] + (long)r * M) = o;
                }
            }
        }
        if (TRAIN) {
            const float tot = block_sum<8 / NB>(s, red);  // a barrier: the gradient tile is complete
            if (tid == 0) lparts[blk] = tot;
            keep(gout, s_b, T, 0);
        }
    }
}

// Input gradient of a layer: act_out = conv(in) [mask > 0].  One workgroup: a
// 16 x 16 pixel tile of one image, 4 waves of 4 rows each.
__global__ __launch_bounds__(256) void k_cnn_dgrad(const bf16* __restrict__ in, const bf16* __restrict__ wA,
                                                   const bf16* __restrict__ mask, bf16* __restrict__ act_out, int M) {
    __shared__ __attribute__((aligned(16))) bf16 s_in[HT * HT * PS];
    const int tid = threadIdx.x;
    const int tiles = M / T;
    const int blk = xcd_contiguous(blockIdx.x, gridDim.x);
    const int tx = blk % tiles;
    const int ty = (blk / tiles) % tiles;
    const long b = blk / (tiles * tiles);
    const int x0 = tx * T, y0 = ty * T;
    const long MM = (long)M * M;
    const bf16* inb = in + b * MM * C;
    constexpr int L = (HT * HT * 4 + 255) / 256;
    bf16x8 v[L];
#pragma unroll
    for (int j = 0; j < L; ++j) {
        const int i = tid + 256 * j;
        if (i < HT * HT * 4) {
            const int pix = i >> 2;
            const int hy = pix / HT, hx = pix - hy * HT;
            const int gy = wrap(y0 + hy - 1, M), gx = wrap(x0 + hx - 1, M);
            v[j] = *reinterpret_cast<const bf16x8*>(inb + ((long)gy * M + gx) * C + (i & 3) * 8);
        }
    }
    NetW<2> wt;
    wt.load(wA, tid & 15, (tid & 63) >> 4);
#pragma unroll
    for (int j = 0; j < L; ++j) {
        const int i = tid + 256 * j;
        if (i < HT * HT * 4) *reinterpret_cast<bf16x8*>(s_in + (i >> 2) * PS + (i & 3) * 8) = v[j];
    }
    __syncthreads();
    const int lane = tid & 63, w = tid >> 6;
    net_layer<HT>(s_in, wt, w, lane & 15, lane >> 4, [&](int pix, int c0, f32x4 v) {
        const long p = (b * MM + (long)(y0 + (pix >> 4)) * M + x0 + (pix & 15)) * C + c0;
        const bf16x4 mk = *reinterpret_cast<const bf16x4*>(mask + p);
        bf16x4 s;
#pragma unroll
        for (int i = 0; i < 4; ++i) s[i] = (bf16)((float)mk[i] > 0.0f ? v[i] : 0.0f);
        *reinterpret_cast<bf16x4*>(act_out + p) = s;
    });
}

// Eight consecutive pixels of one channel out of a channels-last LDS tile, an
// operand of the weight gradient's products: ds_read_b64_tr_b16 takes four
// pixels by 16 channels per 16 lanes, lane i addressing channels 4 (i % 4) ..
// of pixel i / 4, and returns channel i of the four pixels.
__device__ __forceinline__ bf16x8 tr_read(const bf16* p) {
    typedef __bf16 v4 __attribute__((ext_vector_type(4)));
    typedef v4 __attribute__((address_space(3))) * lds_t;
    const v4 a = __builtin_amdgcn_ds_read_tr16_b64_v4bf16((lds_t)(p));
    const v4 b = __builtin_amdgcn_ds_read_tr16_b64_v4bf16((lds_t)(p + 4 * PS));
    return __builtin_shufflevector(a, b, 0, 1, 2, 3, 4, 5, 6, 7);
}

// Weight and bias gradient partials: each workgroup sums `tpw` consecutive
// 16 x 16 tiles.  A product has 32 pixels (two tile rows) as its inner
// dimension.  A wave takes four rows of the tile and all 36 blocks of the
// gradient: its five row pairs of the input, at three column shifts, are read
// once each and serve both products that they belong to.  The tiles are in LDS
// as they are in memory, channels last, and transposed by the reads; the next
// tile is fetched into registers meanwhile.  2^20 pixels: 91 -> 41 us (166 MB,
// a fifth of it halos and partials, 4.0 TB/s) against channel-major tiles with
// three shifted copies written two bytes at a time.
__global__ __launch_bounds__(256, 2) void k_cnn_wgrad(const bf16* __restrict__ g, const bf16* __restrict__ a,
                                                      float* __restrict__ parts, int M, int ntiles, int tpw) {
    constexpr int NG = T * T * PS, NA = HT * HT * PS;
    constexpr int LDS = (NG + NA) * 2 > kCnnPart * 4 ? (NG + NA) * 2 : kCnnPart * 4;
    __shared__ __attribute__((aligned(16))) unsigned char smem[LDS];
    bf16* s_g = reinterpret_cast<bf16*>(smem);
    bf16* s_a = s_g + NG;
    const int tid = threadIdx.x;
    const int lane = tid & 63, w = tid >> 6;
    const int col = lane & 15, kg = lane >> 4;
    const int tiles = M / T;
    const long MM = (long)M * M;
    constexpr int LG = T * T * 4 / 256, LA = (HT * HT * 4 + 255) / 256;
    bf16x8 vg[LG], va[LA];
    auto fetch = [&](int tile) {
        const int x0 = tile % tiles * T, y0 = tile / tiles % tiles * T;
        const long b = tile / (tiles * tiles);
#pragma unroll
        for (int j = 0; j < LG; ++j) {
            const int e = tid + 256 * j;
            vg[j] = *reinterpret_cast<const bf16x8*>(g + (b * MM + (long)(y0 + (e >> 6)) * M + x0 + ((e >> 2) & 15)) * C +
                                                     (e & 3) * 8);
        }
#pragma unroll
        for (int j = 0; j < LA; ++j) {
            const int e = tid + 256 * j;
            if (e < HT * HT * 4) {
                const int hy = (e >> 2) / HT, hx = (e >> 2) - hy * HT;
                va[j] = *reinterpret_cast<const bf16x8*>(
                    a + (b * MM + (long)wrap(y0 + hy - 1, M) * M + wrap(x0 + hx - 1, M)) * C + (e & 3) * 8);
            }
        }
    };
    f32x4 acc[9][2][2], accb[2];
#pragma unroll
    for (int t = 0; t < 9; ++t)
#pragma unroll
        for (int mb = 0; mb < 2; ++mb) acc[t][mb][0] = acc[t][mb][1] = f32x4{0.f, 0.f, 0.f, 0.f};
    accb[0] = accb[1] = f32x4{0.f, 0.f, 0.f, 0.f};
    bf16x8 ones;
#pragma unroll
    for (int k = 0; k < 8; ++k) ones[k] = (bf16)1.0f;
    // this lane's part of an operand: row kg / 2 of the pair, pixel 8 (kg % 2)
    // + col / 4 on, channels 4 (col % 4) on
    const int gy = kg >> 1, gx = 8 * (kg & 1) + (col >> 2), gc = 4 * (col & 3);

    const int first = blockIdx.x * tpw, last = min(ntiles, first + tpw);
    fetch(first);
    for (int tile = first; tile < last; ++tile) {
#pragma unroll
        for (int j = 0; j < LG; ++j) {
            const int e = tid + 256 * j;
            *reinterpret_cast<bf16x8*>(s_g + (e >> 2) * PS + (e & 3) * 8) = vg[j];
        }
#pragma unroll
        for (int j = 0; j < LA; ++j) {
            const int e = tid + 256 * j;
            if (e < HT * HT * 4) *reinterpret_cast<bf16x8*>(s_a + (e >> 2) * PS + (e & 3) * 8) = va[j];
        }
        __syncthreads();
        if (tile + 1 < last) fetch(tile + 1);
        bf16x8 A[2][2];
#pragma unroll
        for (int c = 0; c < 2; ++c)
#pragma unroll
            for (int mb = 0; mb < 2; ++mb) {
                A[c][mb] = tr_read(s_g + ((4 * w + 2 * c + gy) * T + gx) * PS + 16 * mb + gc);
                accb[mb] = mfma(A[c][mb], ones, accb[mb]);
            }
#pragma unroll
        for (int s = 0; s < 5; ++s)  // halo rows 4w + s, 4w + s + 1: tap row s of the first product, s - 2 of the second
#pragma unroll
            for (int dx = 0; dx < 3; ++dx)
#pragma unroll
                for (int nb = 0; nb < 2; ++nb) {
                    const bf16x8 B = tr_read(s_a + ((4 * w + s + gy) * HT + gx + dx) * PS + 16 * nb + gc);
#pragma unroll
                    for (int mb = 0; mb < 2; ++mb) {
                        if (s < 3) acc[3 * s + dx][mb][nb] = mfma(A[0][mb], B, acc[3 * s + dx][mb][nb]);
                        if (s >= 2) acc[3 * (s - 2) + dx][mb][nb] = mfma(A[1][mb], B, acc[3 * (s - 2) + dx][mb][nb]);
                    }
                }
        __syncthreads();
    }

    // the four waves' sums, one after the other
    float* red = reinterpret_cast<float*>(smem);
    for (int v = 0; v < 4; ++v) {
        if (w == v) {
#pragma unroll
            for (int t = 0; t < 9; ++t)
#pragma unroll
                for (int mb = 0; mb < 2; ++mb)
#pragma unroll
                    for (int nb = 0; nb < 2; ++nb)
#pragma unroll
                        for (int i = 0; i < 4; ++i) {
                            float* q = red + (t * C + 16 * mb + 4 * kg + i) * C + 16 * nb + col;
                            *q = acc[t][mb][nb][i] + (v ? *q : 0.0f);
                        }
            if (col == 0)
#pragma unroll
                for (int mb = 0; mb < 2; ++mb)
#pragma unroll
                    for (int i = 0; i < 4; ++i) {
                        float* q = red + kCnnW + 16 * mb + 4 * kg + i;
                        *q = accb[mb][i] + (v ? *q : 0.0f);
                    }
        }
        __syncthreads();
    }
    float* part = parts + (long)blockIdx.x * kCnnPart;
    for (int e = tid; e < kCnnPart; e += 256) part[e] = red[e];
}

// The gradient vector: the sums of each layer's partials (layer l's at parts +
// l stride), in a fixed order, in the parameter order W[o][c][tap], b[o].  A
// workgroup takes 32 columns, eight rows at a time.  12 us for 57 MB of
// partials; a sum in two launches per layer of twice as many took 90 us.
__global__ __launch_bounds__(256) void k_cnn_grad_sum(const float* __restrict__ parts, long stride, int rows,
                                                      float* __restrict__ grads) {
    __shared__ float red[8][32];
    const int c = threadIdx.x & 31, r0 = threadIdx.x >> 5;
    const int e = blockIdx.x * 32 + c;
    const float* src = parts + blockIdx.y * stride + e;
    float s = 0.0f;
#pragma unroll 8
    for (int r = r0; r < rows; r += 8) s += src[(long)r * kCnnPart];
    red[r0][c] = s;
    __syncthreads();
    if (r0 == 0) {
        float t = red[0][c];
#pragma unroll
        for (int r = 1; r < 8; ++r) t += red[r][c];
        float* grad = grads + (long)blockIdx.y * kCnnL;
        if (e < kCnnW) {
            const int tap = e / (C * C), o = (e / C) % C, k = e % C;
            grad[(o * C + k) * 9 + tap] = t;
        } else {
            grad[e] = t;  // biases follow the weights in both layouts
        }
    }
}
static_assert(kCnnPart % 32 == 0, "whole workgroups of columns");

__global__ __launch_bounds__(256) void k_cnn_sumsq(const float* __restrict__ psi, long n, float* __restrict__ parts) {
    __shared__ float red[4];
    const long b = blockIdx.y;
    const long chunk = (n + kScaleBlocks - 1) / kScaleBlocks;
    const long e0 = blockIdx.x * chunk, e1 = min(n, e0 + chunk);
    const float* x = psi + b * n;
    float s = 0.0f;
#pragma unroll 4
    for (long e = e0 + threadIdx.x; e < e1; e += 256) s += x[e] * x[e];
    const float tot = block_sum<4>(s, red);
    if (threadIdx.x == 0) parts[b * kScaleBlocks + blockIdx.x] = tot;
}

__global__ __launch_bounds__(256) void k_cnn_scale(const float* __restrict__ parts, long n, float* __restrict__ scale) {
    __shared__ float red[4];
    const int b = blockIdx.x;
    float s = 0.0f;
    for (int i = threadIdx.x; i < kScaleBlocks; i += 256) s += parts[b * kScaleBlocks + i];
    const float tot = block_sum<4>(s, red);
    if (threadIdx.x == 0) {
        const float r = sqrtf(tot / (float)n);
        scale[b] = r > 0.0f ? r : 1.0f;
    }
}

__global__ __launch_bounds__(256) void k_cnn_loss_reduce(const float* __restrict__ parts, int n, float inv_numel,
                                                         float* __restrict__ loss) {
    __shared__ float red[4];
    float s = 0.0f;
    for (int i = threadIdx.x; i < n; i += 256) s += parts[i];
    const float tot = block_sum<4>(s, red);
    if (threadIdx.x == 0) loss[0] = tot * inv_numel;
}

__global__ __launch_bounds__(256) void k_cnn_adam(float* __restrict__ p, const float* __restrict__ g,
                                                  float* __restrict__ m, float* __restrict__ v, int n, float lr,
                                                  float b1, float b2, float eps, float c1, float c2) {
    const int i = blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= n) return;
    const float gi = g[i];
    const float mi = b1 * m[i] + (1.0f - b1) * gi;
    const float vi = b2 * v[i] + (1.0f - b2) * gi * gi;
    m[i] = mi;
    v[i] = vi;
    p[i] -= lr * (mi * c1) / (sqrtf(vi * c2) + eps);
}

// MFMA weights of the three layers: forward A[l][tap][o][c] = W_l[o][c][tap];
// input gradient A[l][tap][c][o] = W_l[o][c][8 - tap] (the mirrored offset).
__global__ __launch_bounds__(256) void k_cnn_prep(const float* __restrict__ params, bf16* __restrict__ wf,
                                                  bf16* __restrict__ wd) {
    const int i = blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= 3 * kCnnW) return;
    const int l = i / kCnnW;
    const int e = i - l * kCnnW;
    const int tap = e / (C * C), r = (e / C) % C, k = e % C;  // A[l][tap][r][k]
    const float* W = params + (long)l * kCnnL;
    wf[i] = (bf16)W[(r * C + k) * 9 + tap];
    wd[i] = (bf16)W[(k * C + r) * 9 + (8 - tap)];
}

}  // namespace

hipError_t cnn_rms(const float* psi, float* parts, float* scale, int N, int M, int B, hipStream_t st) {
    const long n = (long)N * M * M;
    hipLaunchKernelGGL(k_cnn_sumsq, dim3(kScaleBlocks, (unsigned)B), dim3(256), 0, st, psi, n, parts);
    hipLaunchKernelGGL(k_cnn_scale, dim3((unsigned)B), dim3(256), 0, st, parts, n, scale);
    return hipGetLastError();
}

hipError_t cnn_pack(const float* psi, const float* scale, bf16* act, int N, int M, int B, hipStream_t st) {
    const long n = (long)B * 4 * M * M;
    hipLaunchKernelGGL(k_cnn_pack, dim3((unsigned)((n + 255) / 256)), dim3(256), 0, st, psi, scale, act, N, M, B);
    return hipGetLastError();
}

hipError_t cnn_forward(const bf16* a0, const bf16* wf, const float* params, const float* coarse, float* out,
                       const float* scale, int N, int M, int B, hipStream_t st) {
    const dim3 grid((unsigned)((M / T) * (M / T) * B));
    if (a0)
        hipLaunchKernelGGL((k_cnn_net<false, true, 1>), grid, dim3(512), 0, st, const_cast<bf16*>(a0), wf, params, coarse,
                           out, scale, (bf16*)nullptr, (bf16*)nullptr, (const float*)nullptr, (bf16*)nullptr,
                           (float*)nullptr, 0.0f, N, M);
    else
        hipLaunchKernelGGL((k_cnn_net<false, false, 1>), grid, dim3(512), 0, st, (bf16*)nullptr, wf, params, coarse, out,
                           scale, (bf16*)nullptr, (bf16*)nullptr, (const float*)nullptr, (bf16*)nullptr,
                           (float*)nullptr, 0.0f, N, M);
    return hipGetLastError();
}

hipError_t cnn_forward_loss(const bf16* wf, const float* params, const float* coarse, const float* target,
                            const float* scale, bf16* a0, bf16* a1, bf16* a2, bf16* g, float* loss_parts, float gscale,
                            int N, int M, int B, hipStream_t st) {
    const dim3 grid((unsigned)((M / T) * (M / T) * B));
    hipLaunchKernelGGL((k_cnn_net<true, false, 2>), grid, dim3(256), 0, st, a0, wf, params, coarse, (float*)nullptr, scale,
                       a1, a2, target, g, loss_parts, gscale, N, M);
    return hipGetLastError();
}

hipError_t cnn_dgrad(const bf16* g, const bf16* wd, const bf16* mask, bf16* out, int M, int B, hipStream_t st) {
    hipLaunchKernelGGL(k_cnn_dgrad, dim3((unsigned)((M / T) * (M / T) * B)), dim3(256), 0, st, g, wd, mask, out, M);
    return hipGetLastError();
}

namespace {
// Tiles per workgroup of the weight gradient: two workgroups per compute unit
int wgrad_tiles(int ntiles) { return (ntiles + kCnnWgradParts - 1) / kCnnWgradParts; }
}  // namespace

int cnn_wgrad_parts(int M, int B) {
    const int ntiles = (M / T) * (M / T) * B, tpw = wgrad_tiles(ntiles);
    return (ntiles + tpw - 1) / tpw;
}

hipError_t cnn_wgrad(const bf16* g, const bf16* a, float* parts, int M, int B, hipStream_t st) {
    const int ntiles = (M / T) * (M / T) * B;
    hipLaunchKernelGGL(k_cnn_wgrad, dim3((unsigned)cnn_wgrad_parts(M, B)), dim3(256), 0, st, g, a, parts, M, ntiles,
                       wgrad_tiles(ntiles));
    return hipGetLastError();
}

hipError_t cnn_wgrad_reduce(const float* parts, int nparts, float* grads, hipStream_t st) {
    hipLaunchKernelGGL(k_cnn_grad_sum, dim3((unsigned)(kCnnPart / 32), 3), dim3(256), 0, st, parts,
                       (long)nparts * kCnnPart, nparts, grads);
    return hipGetLastError();
}

int cnn_loss_blocks(int M, int B) { return (M / T) * (M / T) * B; }

hipError_t cnn_loss_reduce(const float* parts, int nparts, float inv_numel, float* loss, hipStream_t st) {
    hipLaunchKernelGGL(k_cnn_loss_reduce, dim3(1), dim3(256), 0, st, parts, nparts, inv_numel, loss);
    return hipGetLastError();
}

hipError_t cnn_adam(float* params, const float* grads, float* m, float* v, int t, float lr, float beta1, float beta2,
                    float eps, hipStream_t st) {
    const double c1 = 1.0 / (1.0 - std::pow((double)beta1, (double)t));
    const double c2 = 1.0 / (1.0 - std::pow((double)beta2, (double)t));
    hipLaunchKernelGGL(k_cnn_adam, dim3((kCnnP + 255) / 256), dim3(256), 0, st, params, grads, m, v, kCnnP, lr, beta1,
                       beta2, eps, (float)c1, (float)c2);
    return hipGetLastError();
}

hipError_t cnn_prep(const float* params, bf16* wfwd, bf16* wdgrad, hipStream_t st) {
    hipLaunchKernelGGL(k_cnn_prep, dim3((3 * kCnnW + 255) / 256), dim3(256), 0, st, params, wfwd, wdgrad);
    return hipGetLastError();
}

}  // namespace se2n
