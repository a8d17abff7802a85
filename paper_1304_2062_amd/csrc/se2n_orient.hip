// Orientation map of one image by the separable periodic stencil: one
// workgroup per tile of bins (the tile body and the reasoning behind it are in
// se2n_orient.hpp).
#include "se2n_orient.hpp"

namespace se2n {
namespace {

template <int RAD, class TL>
__global__ __launch_bounds__(TL::NT) void k_orient_stencil(const float* __restrict__ f,
                                                           const uint8_t* __restrict__ mask,
                                                           uint8_t* __restrict__ rmap, int M, int N, OrientTaps taps) {
    __shared__ __attribute__((aligned(16))) float sa[TL::lds_floats(RAD)];  // g (*)_y f_c
    __shared__ __attribute__((aligned(16))) float sb[TL::lds_floats(RAD)];  // d (*)_y f_c
    // each XCD takes one contiguous band of tiles: the halo rows two tiles
    // share are fetched through one L2
    const int tile = xcd_contiguous((int)blockIdx.x, (int)gridDim.x);
    orient_stencil_tile<RAD, TL>(f, mask, rmap, M, N, tile, taps, sa, sb, (int)threadIdx.x);
}

template <class TL>
hipError_t orient_go(const float* f, const uint8_t* mask, uint8_t* rmap, int M, int N, int radius,
                     const OrientTaps& taps, hipStream_t st) {
    const dim3 grid((unsigned)TL::tiles(M)), block(TL::NT);
    switch (radius) {
#define SE2N_ORIENT_CASE(RV)                                                                              \
    case RV:                                                                                              \
        hipLaunchKernelGGL((k_orient_stencil<RV, TL>), grid, block, 0, st, f, mask, rmap, M, N, taps);    \
        break;
        SE2N_ORIENT_CASE(8)
        SE2N_ORIENT_CASE(12)
        SE2N_ORIENT_CASE(16)
        SE2N_ORIENT_CASE(20)
        SE2N_ORIENT_CASE(24)
        SE2N_ORIENT_CASE(32)
#undef SE2N_ORIENT_CASE
        default:
            return hipErrorInvalidValue;
    }
    return hipGetLastError();
}

}  // namespace

// Small tiles where the large ones would not give every compute unit one (the
// pass then takes as long as one tile: 64^2 10.3 -> 4.5 us, 512^2 10.4 -> 5.8
// us, 768^2 10.5 -> 8 us, 1024^2 equal, 2048^2 29 -> 36 us at radius 12), and at
// radius 32, whose taps are too many for the scalar registers and are fetched
// again and again, over 16 columns per thread in large tiles (64^2 54 -> 18 us,
// 2048^2 166 -> 136 us).
hipError_t launch_orient_stencil(const float* f, const uint8_t* mask, uint8_t* rmap, int M, int N, int radius,
                                 const OrientTaps& taps, hipStream_t st) {
    return OrientLarge::tiles(M) <= 256 || radius > 24 ? orient_go<OrientSmall>(f, mask, rmap, M, N, radius, taps, st)
                                                       : orient_go<OrientLarge>(f, mask, rmap, M, N, radius, taps, st);
}

}  // namespace se2n
