// Orientation map of the corrupted image by a separable periodic stencil:
// the tile body shared by the single-image and the batched kernels.
//
// The orientation step smooths f_c = f (1 - mask) with a Gaussian and takes
// central differences, both as Fourier multipliers on the periodic grid
// (Sec. "A final inpainting algorithm ...").  A Fourier multiplier is a
// circular convolution with its inverse DFT, and both multipliers here are
// products of an x factor and a y factor, so
//     g_x = d (*)_x g (*)_y f_c,     g_y = g (*)_x d (*)_y f_c
// with g the inverse DFT of the 1-D Gaussian factor and d that of the
// Gaussian times the central-difference symbol.  For widths where both
// kernels fall below the FP32 rounding level within a few dozen pixels the
// convolutions are short stencils; the host truncates them there (or keeps
// the whole circle for small M) and passes the taps as kernel arguments.
//
// One workgroup makes a tile of bins (128 x 32): a vertical pass (both kernels,
// 8 rows per thread from a register window over global memory) writes the
// two partial results for the tile's columns plus the horizontal halo to
// LDS; a horizontal pass (16 columns per thread) finishes g_x and g_y and
// bins the level-line angle atan2(g_y, g_x) + pi/2 into N orientations.
#pragma once

#include <hip/hip_runtime.h>

#include <cstdint>

#include "se2n_internal.hpp"

namespace se2n {

// A tile: TX columns by TY rows, CV rows per vertical item, CH columns per
// horizontal item, one horizontal item per thread.
template <int TX_, int TY_, int CV_, int CH_>
struct OrientTile {
    static constexpr int TX = TX_, TY = TY_, CV = CV_, CH = CH_, NT = TY_ * TX_ / CH_;
    static_assert(TY % CV == 0 && TX % CH == 0, "whole items");
    __host__ __device__ static constexpr int tiles(int M) { return ((M + TX - 1) / TX) * ((M + TY - 1) / TY); }
    // LDS row stride and size (floats) of each of the two partial results
    __host__ __device__ static constexpr int stride(int rad) { return TX + 2 * rad + 4; }
    __host__ __device__ static constexpr int lds_floats(int rad) { return TY * stride(rad); }
};
// The least work per pixel; and a tile whose two passes are an eighth as long,
// for images that do not fill the chip with the other (launch_orient_stencil).
using OrientLarge = OrientTile<128, 32, 8, 16>;
using OrientSmall = OrientTile<64, 8, 4, 2>;

inline int orient_tiles(int M) { return OrientLarge::tiles(M); }

__device__ __forceinline__ int orient_wrap(int i, int M) {
    i %= M;
    return i < 0 ? i + M : i;
}

// Bins of tile `tile` (row-major over the tiles of the image); sa and sb hold
// TL::lds_floats(RAD) floats each.  Every tile sums its taps in the same order.
template <int RAD, class TL = OrientLarge>
__device__ __forceinline__ void orient_stencil_tile(const float* __restrict__ f, const uint8_t* __restrict__ mask,
                                                    uint8_t* __restrict__ rmap, int M, int N, int tile,
                                                    const OrientTaps& taps, float* sa, float* sb, int tid) {
    constexpr int NTAP = 2 * RAD + 1;
    constexpr int TX = TL::TX, TY = TL::TY, CV = TL::CV, CH = TL::CH;
    constexpr int W = TX + 2 * RAD;  // columns of the vertical pass
    constexpr int WS = TL::stride(RAD);
    constexpr int NV = CV + 2 * RAD;
    constexpr int NH = CH + 2 * RAD;
    constexpr int VW = CH % 4 == 0 ? 4 : 2;  // floats per LDS read
    typedef float vec_t __attribute__((ext_vector_type(VW)));
    static_assert(W % VW == 0 && NH % VW == 0 && WS % VW == 0 && CH % VW == 0, "whole reads");
    const int tiles_x = (M + TX - 1) / TX;
    const int x0 = (tile % tiles_x) * TX;
    const int y0 = (tile / tiles_x) * TY;

    for (int it = tid; it < W * (TY / CV); it += TL::NT) {
        const int c = it % W, q = it / W;
        const int xx = orient_wrap(x0 - RAD + c, M);
        int yy = orient_wrap(y0 + q * CV - RAD, M);
        float v[NV];
#pragma unroll
        for (int k = 0; k < NV; ++k) {
            const size_t o = (size_t)yy * M + xx;
            const float fv = f[o];
            v[k] = mask[o] ? 0.f : fv;
            yy = (yy + 1 == M) ? 0 : yy + 1;
        }
#pragma unroll
        for (int i = 0; i < CV; ++i) {
            float a = 0.f, b = 0.f;
#pragma unroll
            for (int j = 0; j < NTAP; ++j) {
                a = fmaf(taps.g[j], v[i + j], a);
                if (j != RAD) b = fmaf(taps.d[j], v[i + j], b);  // d is odd: no centre tap
            }
            sa[(q * CV + i) * WS + c] = a;
            sb[(q * CV + i) * WS + c] = b;
        }
    }
    __syncthreads();

    const int y = tid / (TX / CH), cq = tid % (TX / CH);
    float gx[CH], gy[CH];
    {
        float u[NH];
        const float* row = sa + y * WS + cq * CH;
#pragma unroll
        for (int k = 0; k < NH; k += VW) {
            const vec_t t = *reinterpret_cast<const vec_t*>(row + k);
#pragma unroll
            for (int i = 0; i < VW; ++i) u[k + i] = t[i];
        }
#pragma unroll
        for (int i = 0; i < CH; ++i) {
            float s = 0.f;
#pragma unroll
            for (int j = 0; j < NTAP; ++j)
                if (j != RAD) s = fmaf(taps.d[j], u[i + j], s);
            gx[i] = s;
        }
    }
    {
        float u[NH];
        const float* row = sb + y * WS + cq * CH;
#pragma unroll
        for (int k = 0; k < NH; k += VW) {
            const vec_t t = *reinterpret_cast<const vec_t*>(row + k);
#pragma unroll
            for (int i = 0; i < VW; ++i) u[k + i] = t[i];
        }
#pragma unroll
        for (int i = 0; i < CH; ++i) {
            float s = 0.f;
#pragma unroll
            for (int j = 0; j < NTAP; ++j) s = fmaf(taps.g[j], u[i + j], s);
            gy[i] = s;
        }
    }

    const int py = y0 + y, px = x0 + cq * CH;
    if (py >= M || px >= M) return;
    const float two_pi = 6.283185307179586476925f;
    const float half_pi = 1.570796326794896619231f;
    uint32_t w[(CH + 3) / 4];
#pragma unroll
    for (int i = 0; i < (CH + 3) / 4; ++i) w[i] = 0;
#pragma unroll
    for (int i = 0; i < CH; ++i) {
        const float t = (atan2f(gy[i], gx[i]) + half_pi) * (float)N / two_pi + 0.5f;
        // atan2 lies in [-pi, pi], so floor(t) lies in [-N/4, 3N/4]: one
        // wrap of the negative values is the remainder mod N
        int b = (int)floorf(t);
        if (b < 0) b += N;
        w[i / 4] |= (uint32_t)b << (8 * (i % 4));
    }
    uint8_t* dst = rmap + (size_t)py * M + px;
    if constexpr (CH == 2) {  // M is even
        *reinterpret_cast<uint16_t*>(dst) = (uint16_t)w[0];
    } else if (px + CH <= M && (M & 7) == 0) {
        // M is a multiple of 8, so each half of the run is 8-byte aligned
        reinterpret_cast<uint2*>(dst)[0] = make_uint2(w[0], w[1]);
        reinterpret_cast<uint2*>(dst)[1] = make_uint2(w[2], w[3]);
    } else {
#pragma unroll
        for (int i = 0; i < CH; ++i)
            if (px + i < M) dst[i] = (uint8_t)(w[i / 4] >> (8 * (i % 4)));
    }
}

}  // namespace se2n
