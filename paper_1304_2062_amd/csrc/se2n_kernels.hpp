// gfx950 kernels of the semi-discrete SE(2,N) diffusion and their launchers,
// included once per data type (se2n_kernels_f32.hip, se2n_kernels_f64.hip).
//
// Spectral layout.  The half spectrum of an orientation volume is stored
// "column major": spec[r][kx][ky], kx in [0, M/2], ky in [0, M) contiguous.
// Every column (r, kx) is M contiguous complex values, so the column FFTs
// and the per-mode solve read and write whole cache lines; the row passes
// move 8 (float) or 4 (double) rows at a time so that each (r, kx) segment
// they touch is 64 contiguous bytes.
//
// Pass structure of one diffusion (Theorem 2 of the paper: FFT over (Z/MZ)^2,
// M^2 decoupled N-dimensional systems, inverse FFT):
//   k_row_fwd   lift (or read the real volume) + real-to-complex FFT along x
//   k_col_fft   complex FFT along y, forward
//   k_solve     psi_hat(kx,ky) <- P(kx,ky) psi_hat(kx,ky), P the per-mode propagator
//   k_col_fft   complex FFT along y, inverse
//   k_row_inv   complex-to-real FFT along x + projection (or write the volume)
// The 1/M^2 of the inverse transform is folded into the stored propagators.
#pragma once

#include <hip/hip_runtime.h>

#include <cstdint>

#include "se2n_fft.hpp"
#include "se2n_internal.hpp"
#include "se2n_passes.hpp"

namespace se2n {

// Workgroup -> (row block, slice group) of a row pass launched on a 1-D grid.
// The dispatcher hands consecutive workgroups to the 8 XCDs in turn.  With
// `pair` set, row blocks 2j and 2j+1 of one slice group go to two workgroups
// that the same XCD runs back to back, so both 64-byte halves of every
// 128-byte line of a (slice, kx) column run are fetched through one L2.
__device__ __forceinline__ void row_block_of(int nrb, int ngroups, bool pair, int& rb, int& g) {
    const int i = blockIdx.x;
    if (pair && (nrb & 1) == 0 && ((nrb * ngroups) & 15) == 0) {
        const int xcd = i & 7;
        const int slot = i >> 3;
        const int pr = (slot >> 1) * 8 + xcd;
        const int per_group = nrb >> 1;
        g = pr / per_group;
        rb = 2 * (pr - g * per_group) + (slot & 1);
    } else {
        g = i / nrb;
        rb = i - g * nrb;
    }
}

// ---------------------------------------------------------------------------
// Single-image kernels: one workgroup per tile; the tile bodies are shared
// with the batched kernels.
// ---------------------------------------------------------------------------
// Row passes: grid (M/rows row blocks) x (slice groups) on a 1-D grid;
// block: nthr threads; LDS: twiddles + rows x (H+2) (padded).
template <class R, int SRC, int EPT, bool TWF, int MS>
__global__ __launch_bounds__(sizeof(R) == 8 ? kRowThreadsF64 : 1024) void k_row_fwd(const R* __restrict__ f, const uint8_t* __restrict__ mask,
                          const uint8_t* __restrict__ rmap, const R* __restrict__ vol,
                          C2<R>* __restrict__ spec, int M_, int nslices, int slices_per_group,
                          int rows_, int xcd_pair, FftPlan planH, const C2<R>* __restrict__ twg) {
    constexpr GeomCore GC = geom_core<R>(MS ? MS : 16);
    const int M = MS ? MS : M_;
    const int rows = MS ? GC.rows : rows_;
    const int nthr = MS ? GC.row_threads : (int)blockDim.x;
    extern __shared__ unsigned char smem_raw[];
    C2<R>* tw = reinterpret_cast<C2<R>*>(smem_raw);
    C2<R>* buf = tw + tw_elems(M, TWF);
    int rb, grp;
    row_block_of(M / rows, (nslices + slices_per_group - 1) / slices_per_group, xcd_pair != 0, rb, grp);
    const int s_begin = grp * slices_per_group;
    const int s_end = min(nslices, s_begin + slices_per_group);
    load_twiddles<R>(tw, twg, M >> 2, TWF, threadIdx.x, nthr);
    row_fwd_tile<R, SRC, EPT, TWF, MS, true>(f, mask, rmap, vol, spec, M, rows, nthr, rb, s_begin, s_end, planH, tw,
                                       buf, threadIdx.x, MS ? buf + row_buf_elems(M, rows) : nullptr);
}

// Column pass: one tile of cols_per_block contiguous columns per workgroup.
template <class R, bool INV, int EPT, bool TWF, int MS>
__global__ void k_col_fft(C2<R>* __restrict__ spec, long ncols, int M_, int cols_per_block_,
                          FftPlan planM, const C2<R>* __restrict__ twg, const uint8_t* __restrict__ negf,
                          int FS) {
    constexpr GeomCore GC = geom_core<R>(MS ? MS : 16);
    const int M = MS ? MS : M_;
    const int cols_per_block = MS ? GC.cols : cols_per_block_;
    const int nthr = MS ? GC.col_threads : (int)blockDim.x;
    extern __shared__ unsigned char smem_raw[];
    C2<R>* tw = reinterpret_cast<C2<R>*>(smem_raw);
    C2<R>* buf = tw + tw_elems(M, TWF);
    // tiles from the last slice to the first: the row pass before this one
    // wrote the high slices last, and the memory-side cache still holds them
    const long tile = (long)gridDim.x - 1 - (long)blockIdx.x;
    // the tile issues its own loads first and fetches the twiddles meanwhile
    col_fft_tile<R, INV, EPT, TWF, MS>(spec, ncols, M, cols_per_block, nthr, tile * cols_per_block, planM, tw, buf,
                                      threadIdx.x, negf, FS,
                                      [&] { load_twiddles<R>(tw, twg, M >> 2, TWF, threadIdx.x, nthr); });
}

template <class R, int EPT, bool TWF>
__global__ void k_col_orient(C2<R>* __restrict__ spec, int M, int cols_per_block, FftPlan planM,
                             const C2<R>* __restrict__ twg, R neg_two_pi2_sigma2_over_M2, R scale) {
    extern __shared__ unsigned char smem_raw[];
    C2<R>* tw = reinterpret_cast<C2<R>*>(smem_raw);
    C2<R>* buf = tw + tw_elems(M, TWF);
    const int nthr = blockDim.x;
    load_twiddles<R>(tw, twg, M >> 2, TWF, threadIdx.x, nthr);
    col_orient_tile<R, EPT, TWF>(spec, M, cols_per_block, nthr, blockIdx.x * cols_per_block, planM, tw, buf,
                                 neg_two_pi2_sigma2_over_M2, scale, threadIdx.x);
}

template <class R, int DST, int EPT, bool TWF, int MS, bool PAIRED, bool BLK = false>
__global__ __launch_bounds__(sizeof(R) == 8 ? kRowThreadsF64 : 1024) void k_row_inv(const C2<R>* __restrict__ spec, R* __restrict__ out,
                          typename Enc<R>::U* __restrict__ enc, uint8_t* __restrict__ rmap,
                          int M_, int nslices, int slices_per_group, int rows_, int xcd_pair, int N,
                          R out_scale, FftPlan planH, const C2<R>* __restrict__ twg) {
    constexpr GeomCore GC = geom_core<R>(MS ? MS : 16);
    const int M = MS ? MS : M_;
    const int rows = MS ? GC.rows : rows_;
    const int nthr = MS ? GC.row_threads : (int)blockDim.x;
    extern __shared__ unsigned char smem_raw[];
    C2<R>* tw = reinterpret_cast<C2<R>*>(smem_raw);
    C2<R>* buf = tw + tw_elems(M, TWF);
    int rb, grp;
    row_block_of(M / rows, (nslices + slices_per_group - 1) / slices_per_group, xcd_pair != 0, rb, grp);
    const int s_begin = grp * slices_per_group;
    const int s_end = min(nslices, s_begin + slices_per_group);
    load_twiddles<R>(tw, twg, M >> 2, TWF, threadIdx.x, nthr);
    row_inv_tile<R, DST, EPT, TWF, MS, PAIRED, BLK, true>(spec, out, enc, rmap, M, rows, nthr, rb, s_begin, s_end, N,
                                               out_scale, planH, tw, buf, threadIdx.x,
                                               MS ? buf + row_buf_elems(M, rows) : nullptr);
}

// Paired inverse column pass: one tile of column pairs per workgroup.
// TWO: each workgroup transforms slices 2s and 2s + 1 of its pair block (grid
// N/2 x pair blocks), loading the flags and twiddles once for both.
// BLK: the result goes to blk in the row-blocked layout.
template <class R, int EPT, int MS, bool TWO = false, bool BLK = false>
__global__ __launch_bounds__(1024) void k_col_inv_paired(C2<R>* __restrict__ spec, int M_, int pcols_, FftPlan planM,
                                                         const C2<R>* __restrict__ twg,
                                                         const uint8_t* __restrict__ negf, int FS,
                                                         C2<R>* __restrict__ blk) {
    constexpr GeomCore GC = geom_core<R>(MS ? MS : 16);
    const int M = MS ? MS : M_;
    const int nthr = MS ? GC.pcol_threads : (int)blockDim.x;
    extern __shared__ unsigned char smem_raw[];
    C2<R>* tw = reinterpret_cast<C2<R>*>(smem_raw);
    C2<R>* buf = tw + tw_elems(M, false);
    const int P = (MS ? GC.pcols : pcols_) / 2;
    const int tps = (M / 4 + 1 + P - 1) / P;
    const int nslices = (TWO ? 2 : 1) * (int)gridDim.x / tps;  // grid: slices (or slice pairs) x pair blocks
    int tile = blockIdx.x, tile2 = -1;
    if (TWO) {
        const int s2 = blockIdx.x / tps;
        tile = 2 * s2 * tps + (blockIdx.x - s2 * tps);
        tile2 = tile + tps;
    }
    // the tile fetches the twiddles while its flag loads are in flight
    auto pre = [&] { load_twiddles<R>(tw, twg, M >> 2, false, threadIdx.x, nthr); };
    col_inv_paired_tile<R, EPT, MS, true, decltype(pre), BLK>(spec, M, pcols_, nthr, tile, planM, tw, buf, threadIdx.x,
                                                              nslices, negf, FS, pre, tile2, blk);
}

// ---------------------------------------------------------------------------
// Small elementwise kernels.
// ---------------------------------------------------------------------------
template <class R>
__global__ void k_fill_enc(typename Enc<R>::U* __restrict__ enc, long n) {
    const long i = (long)blockIdx.x * blockDim.x + threadIdx.x;
    if (i < n) enc[i] = 0;
}

template <class R>
__global__ void k_decode_enc(const typename Enc<R>::U* __restrict__ enc, R* __restrict__ out, long n) {
    const long i = (long)blockIdx.x * blockDim.x + threadIdx.x;
    if (i < n) out[i] = Enc<R>::decode(enc[i]);
}

template <class R>
__global__ void k_lift(const R* __restrict__ f, const uint8_t* __restrict__ mask,
                       const uint8_t* __restrict__ rmap, R* __restrict__ psi, long MM, int N) {
    const long i = (long)blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= MM) return;
    const R v = mask[i] ? R(0) : f[i];
    const int r = rmap[i];
    for (int s = 0; s < N; ++s) psi[(size_t)s * MM + i] = (s == r) ? v : R(0);
}

template <class R, bool MEAN>
__global__ void k_project(const R* __restrict__ psi, R* __restrict__ out, long MM, int N) {
    const long i = (long)blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= MM) return;
    R a = psi[i];
    for (int s = 1; s < N; ++s) {
        const R v = psi[(size_t)s * MM + i];
        a = MEAN ? a + v : fmax(a, v);
    }
    out[i] = MEAN ? a / (R)N : a;
}

// ---------------------------------------------------------------------------
// Launchers (host side, called by the runtime with validated arguments).
// ---------------------------------------------------------------------------
template <class R>
constexpr bool kStatic = sizeof(R) == 4;  // fixed-size kernels exist for FP32 only

// M of the kernels compiled for a fixed size that this plan can use (0: none):
// FP32, M in {512, 1024, 2048}, with the default geometry.
template <class R>
static int static_size(int M, const LaunchGeom& g) {
    if (sizeof(R) != 4 || !g.static_ok) return 0;
    if (M != 512 && M != 1024 && M != 2048) return 0;
    const GeomCore c = geom_core<R>(M);
    const bool same = g.rows == c.rows && g.row_threads == c.row_threads && g.row_ept == c.row_ept &&
                      g.cols == c.cols && g.col_threads == c.col_threads && g.col_ept == 8 && c.col_ept == 8 &&
                      g.tw_full == c.tw_full && g.tw_full_col == 0;
    return same ? M : 0;
}

// Elements per thread and twiddle table of the row kernels compiled for a fixed M.
template <int M>
constexpr int kRowEpt = geom_core<float>(M).row_ept;
template <int M>
constexpr bool kRowTwf = geom_core<float>(M).tw_full != 0;

template <class R>
static size_t tw_bytes(int M, bool full) {
    return (size_t)tw_elems(M, full) * sizeof(C2<R>);
}

template <class R>
hipError_t launch_row_fwd(int src, const R* f, const uint8_t* mask, const uint8_t* rmap, const R* vol,
                          C2<R>* spec, int M, int nslices, const LaunchGeom& g, const FftPlan& planH,
                          const C2<R>* tw, hipStream_t st) {
    const int groups = (nslices + g.row_slices - 1) / g.row_slices;
    dim3 grid((M / g.rows) * groups);
    // the kernels compiled for a fixed M run their stages between two row buffers
    const size_t lds = tw_bytes<R>(M, g.tw_full != 0) +
                       (size_t)row_buf_elems(M, g.rows) * sizeof(C2<R>) * (kStatic<R> && static_size<R>(M, g) ? 2 : 1);
#define SE2N_ROWFWD(S, E, W, MSV)                                                                          \
    hipLaunchKernelGGL((k_row_fwd<R, S, E, W, MSV>), grid, dim3(g.row_threads), lds, st, f, mask, rmap, vol,    \
                       spec, M, nslices, g.row_slices, g.rows, g.xcd_pair, planH, tw)
#define SE2N_ROWFWD_E(S)                                                    \
    if (static_size<R>(M, g) == 2048) SE2N_ROWFWD(S, kRowEpt<2048>, kRowTwf<2048>, kStatic<R> ? 2048 : 0);        \
    else if (static_size<R>(M, g) == 1024) SE2N_ROWFWD(S, kRowEpt<1024>, kRowTwf<1024>, kStatic<R> ? 1024 : 0);   \
    else if (static_size<R>(M, g) == 512) SE2N_ROWFWD(S, kRowEpt<512>, kRowTwf<512>, kStatic<R> ? 512 : 0);     \
    else if (g.tw_full) {                                                   \
        if (g.row_ept == 8) SE2N_ROWFWD(S, 8, true, 0);                     \
        else SE2N_ROWFWD(S, 16, true, 0);                                   \
    } else {                                                                \
        if (g.row_ept == 8) SE2N_ROWFWD(S, 8, false, 0);                    \
        else SE2N_ROWFWD(S, 16, false, 0);                                  \
    }
    if (src == SRC_LIFT) { SE2N_ROWFWD_E(SRC_LIFT) }
    else if (src == SRC_VOLUME) { SE2N_ROWFWD_E(SRC_VOLUME) }
    else { SE2N_ROWFWD_E(SRC_IMAGE) }
#undef SE2N_ROWFWD_E
#undef SE2N_ROWFWD
    return hipGetLastError();
}

template <class R>
hipError_t launch_col_fft(bool inverse, C2<R>* spec, long ncols, int M, const LaunchGeom& g,
                          const FftPlan& planM, const C2<R>* tw, hipStream_t st, const uint8_t* negf) {
    dim3 grid((unsigned)((ncols + g.cols - 1) / g.cols));
    const size_t lds = tw_bytes<R>(M, g.tw_full_col != 0) + (size_t)lds_padded_size(g.cols * M) * sizeof(C2<R>);
#define SE2N_COL(I, E, W, MSV)                                                                                 \
    hipLaunchKernelGGL((k_col_fft<R, I, E, W, MSV>), grid, dim3(g.col_threads), lds, st, spec, ncols, M, g.cols, planM, \
                       tw, negf, flag_stride(M))
#define SE2N_COL_E(I)                                                   \
    if (static_size<R>(M, g) == 2048) SE2N_COL(I, 8, false, kStatic<R> ? 2048 : 0);      \
    else if (static_size<R>(M, g) == 1024) SE2N_COL(I, 8, false, kStatic<R> ? 1024 : 0); \
    else if (static_size<R>(M, g) == 512) SE2N_COL(I, 8, false, kStatic<R> ? 512 : 0);   \
    else if (g.tw_full_col) {                                           \
        if (g.col_ept == 8) SE2N_COL(I, 8, true, 0);                    \
        else SE2N_COL(I, 16, true, 0);                                  \
    } else {                                                            \
        if (g.col_ept == 8) SE2N_COL(I, 8, false, 0);                   \
        else SE2N_COL(I, 16, false, 0);                                 \
    }
    if (inverse) { SE2N_COL_E(true) }
    else { SE2N_COL_E(false) }
#undef SE2N_COL_E
#undef SE2N_COL
    return hipGetLastError();
}

template <class R>
hipError_t launch_col_orient(C2<R>* spec, int M, const LaunchGeom& g, const FftPlan& planM,
                             const C2<R>* tw, double sigma, hipStream_t st) {
    const int K = M / 2 + 1;
    dim3 grid((K + g.ocols - 1) / g.ocols);
    const size_t lds = tw_bytes<R>(M, g.tw_full_col != 0) + (size_t)lds_padded_size(2 * g.ocols * M) * sizeof(C2<R>);
    const double c = -2.0 * 9.869604401089358619 * sigma * sigma / ((double)M * M);
    const double scale = sqrt((double)M) / ((double)M * M);
    if (g.ocol_ept == 8)
        hipLaunchKernelGGL((k_col_orient<R, 8, false>), grid, dim3(g.ocol_threads), lds, st, spec, M, g.ocols,
                           planM, tw, (R)c, (R)scale);
    else
        hipLaunchKernelGGL((k_col_orient<R, 16, false>), grid, dim3(g.ocol_threads), lds, st, spec, M, g.ocols,
                           planM, tw, (R)c, (R)scale);
    return hipGetLastError();
}

// The compiled size of the paired inverse kernel for M (0: the generic one).
template <class R>
static int col_inv_static(int M, const LaunchGeom& g) {
    const GeomCore c = geom_core<R>(M);
    const bool fixed = static_size<R>(M, g) != 0 && g.pcols == c.pcols && g.pcol_threads == c.pcol_threads &&
                       c.pcol_ept == 8;
    return kStatic<R> && fixed && (M == 2048 || M == 1024 || M == 512) ? M : 0;
}

template <class R>
bool col_inv_masks(int M, const LaunchGeom& g) {
    const int ms = col_inv_static<R>(M, g);
    return ms != 0 && col_skip_shape(ms, geom_core<R>(ms).pcol_threads);
}

template <class R>
bool row_blocked(int M, const LaunchGeom& g) {
    return kStatic<R> && col_inv_static<R>(M, g) != 0 && static_size<R>(M, g) == M && M % kRowBlk == 0;
}

template <class R>
hipError_t launch_col_inv_paired(C2<R>* spec, int M, int N, const LaunchGeom& g, const FftPlan& planM,
                                 const C2<R>* tw, hipStream_t st, const uint8_t* negf, C2<R>* blk) {
    if (blk != nullptr && !row_blocked<R>(M, g)) return hipErrorInvalidValue;
    const int P = g.pcols / 2;
    const int npair = M / 4 + 1;
    const size_t lds = tw_bytes<R>(M, false) + (size_t)lds_padded_size(g.pcols * M) * sizeof(C2<R>);
    const int ms = col_inv_static<R>(M, g);
    // two slices per workgroup where every tile takes the flag-reading fast
    // path (full tiles of a compiled size whose rows meet few class indices)
    // (compiled for M = 2048, whose tiles are single pairs)
    const bool two = negf != nullptr && ms == 2048 && col_inv_masks<R>(M, g) && npair % P == 0 && N % 2 == 0;
    const dim3 grid((unsigned)((two ? N / 2 : N) * ((npair + P - 1) / P)));
#define SE2N_PCOL(E, MSV, TWOV, BLKV)                                                                      \
    hipLaunchKernelGGL((k_col_inv_paired<R, E, MSV, TWOV, BLKV>), grid, dim3(g.pcol_threads), lds, st, spec, M, \
                       g.pcols, planM, tw, negf, flag_stride(M), blk)
    if constexpr (kStatic<R>) {
        if (blk != nullptr) {
            if (two) SE2N_PCOL(8, 2048, true, true);
            else if (ms == 2048) SE2N_PCOL(8, 2048, false, true);
            else if (ms == 1024) SE2N_PCOL(8, 1024, false, true);
            else SE2N_PCOL(8, 512, false, true);
            return hipGetLastError();
        }
    }
    if (two && ms == 2048) SE2N_PCOL(8, kStatic<R> ? 2048 : 0, true, false);
    else if (ms == 2048) SE2N_PCOL(8, kStatic<R> ? 2048 : 0, false, false);
    else if (ms == 1024) SE2N_PCOL(8, kStatic<R> ? 1024 : 0, false, false);
    else if (ms == 512) SE2N_PCOL(8, kStatic<R> ? 512 : 0, false, false);
    else if (g.pcol_ept == 8) SE2N_PCOL(8, 0, false, false);
    else SE2N_PCOL(16, 0, false, false);
#undef SE2N_PCOL
    return hipGetLastError();
}

template <class R>
hipError_t launch_row_inv(int dst, const C2<R>* spec, R* out, typename Enc<R>::U* enc, uint8_t* rmap,
                          int M, int nslices, int N, R out_scale, const LaunchGeom& g,
                          int slices_per_group, const FftPlan& planH, const C2<R>* tw, hipStream_t st,
                          bool paired, bool blocked) {
    if (blocked && !(paired && dst != DST_ORIENT && row_blocked<R>(M, g))) return hipErrorInvalidValue;
    const int groups = (nslices + slices_per_group - 1) / slices_per_group;
    dim3 grid((M / g.rows) * groups);
    // the kernels compiled for a fixed M run their stages between two row buffers
    const size_t lds = tw_bytes<R>(M, g.tw_full != 0) +
                       (size_t)row_buf_elems(M, g.rows) * sizeof(C2<R>) * (kStatic<R> && static_size<R>(M, g) ? 2 : 1);
#define SE2N_ROWINV(D, E, W, MSV)                                                                              \
    do {                                                                                                       \
        if (paired)                                                                                            \
            hipLaunchKernelGGL((k_row_inv<R, D, E, W, MSV, true>), grid, dim3(g.row_threads), lds, st, spec, out, \
                               enc, rmap, M, nslices, slices_per_group, g.rows, g.xcd_pair, N, out_scale, planH,  \
                               tw);                                                                            \
        else                                                                                                   \
            hipLaunchKernelGGL((k_row_inv<R, D, E, W, MSV, false>), grid, dim3(g.row_threads), lds, st, spec, out, \
                               enc, rmap, M, nslices, slices_per_group, g.rows, g.xcd_pair, N, out_scale, planH,  \
                               tw);                                                                            \
    } while (0)
#define SE2N_ROWINV_BLK(D, MSV)                                                                                 \
    hipLaunchKernelGGL((k_row_inv<R, D, kRowEpt<MSV>, kRowTwf<MSV>, MSV, true, true>), grid, dim3(g.row_threads), lds, \
                       st, spec, out, enc, rmap, M, nslices, slices_per_group, g.rows, g.xcd_pair, N, out_scale,       \
                       planH, tw)
    if constexpr (kStatic<R>) {
        if (blocked) {
            if (dst == DST_MAX) {
                if (M == 2048) SE2N_ROWINV_BLK(DST_MAX, 2048);
                else if (M == 1024) SE2N_ROWINV_BLK(DST_MAX, 1024);
                else SE2N_ROWINV_BLK(DST_MAX, 512);
            } else if (dst == DST_SUM) {
                if (M == 2048) SE2N_ROWINV_BLK(DST_SUM, 2048);
                else if (M == 1024) SE2N_ROWINV_BLK(DST_SUM, 1024);
                else SE2N_ROWINV_BLK(DST_SUM, 512);
            } else {
                if (M == 2048) SE2N_ROWINV_BLK(DST_VOLUME, 2048);
                else if (M == 1024) SE2N_ROWINV_BLK(DST_VOLUME, 1024);
                else SE2N_ROWINV_BLK(DST_VOLUME, 512);
            }
            return hipGetLastError();
        }
    }
#undef SE2N_ROWINV_BLK
#define SE2N_ROWINV_E(D)                                                    \
    if (static_size<R>(M, g) == 2048) SE2N_ROWINV(D, kRowEpt<2048>, kRowTwf<2048>, kStatic<R> ? 2048 : 0);        \
    else if (static_size<R>(M, g) == 1024) SE2N_ROWINV(D, kRowEpt<1024>, kRowTwf<1024>, kStatic<R> ? 1024 : 0);   \
    else if (static_size<R>(M, g) == 512) SE2N_ROWINV(D, kRowEpt<512>, kRowTwf<512>, kStatic<R> ? 512 : 0);     \
    else if (g.tw_full) {                                                   \
        if (g.row_ept == 8) SE2N_ROWINV(D, 8, true, 0);                     \
        else SE2N_ROWINV(D, 16, true, 0);                                   \
    } else {                                                                \
        if (g.row_ept == 8) SE2N_ROWINV(D, 8, false, 0);                    \
        else SE2N_ROWINV(D, 16, false, 0);                                  \
    }
    if (dst == DST_MAX) { SE2N_ROWINV_E(DST_MAX) }
    else if (dst == DST_SUM) { SE2N_ROWINV_E(DST_SUM) }
    else if (dst == DST_VOLUME) { SE2N_ROWINV_E(DST_VOLUME) }
    else { SE2N_ROWINV_E(DST_ORIENT) }
#undef SE2N_ROWINV_E
#undef SE2N_ROWINV
    return hipGetLastError();
}

template <class R>
hipError_t launch_fill_enc(typename Enc<R>::U* enc, long n, hipStream_t st) {
    hipLaunchKernelGGL((k_fill_enc<R>), dim3((unsigned)((n + 255) / 256)), dim3(256), 0, st, enc, n);
    return hipGetLastError();
}

template <class R>
hipError_t launch_decode_enc(const typename Enc<R>::U* enc, R* out, long n, hipStream_t st) {
    hipLaunchKernelGGL((k_decode_enc<R>), dim3((unsigned)((n + 255) / 256)), dim3(256), 0, st, enc, out, n);
    return hipGetLastError();
}

template <class R>
hipError_t launch_lift(const R* f, const uint8_t* mask, const uint8_t* rmap, R* psi, int M, int N,
                       hipStream_t st) {
    const long MM = (long)M * M;
    hipLaunchKernelGGL((k_lift<R>), dim3((unsigned)((MM + 255) / 256)), dim3(256), 0, st, f, mask, rmap,
                       psi, MM, N);
    return hipGetLastError();
}

template <class R>
hipError_t launch_project(const R* psi, R* out, int M, int N, bool mean, hipStream_t st) {
    const long MM = (long)M * M;
    dim3 grid((unsigned)((MM + 255) / 256));
    if (mean) hipLaunchKernelGGL((k_project<R, true>), grid, dim3(256), 0, st, psi, out, MM, N);
    else hipLaunchKernelGGL((k_project<R, false>), grid, dim3(256), 0, st, psi, out, MM, N);
    return hipGetLastError();
}

#define SE2N_KERNELS_INSTANTIATE(R)                                                                    \
    template hipError_t launch_row_fwd<R>(int, const R*, const uint8_t*, const uint8_t*, const R*,     \
                                          C2<R>*, int, int, const LaunchGeom&, const FftPlan&,         \
                                          const C2<R>*, hipStream_t);                                  \
    template hipError_t launch_col_fft<R>(bool, C2<R>*, long, int, const LaunchGeom&, const FftPlan&,  \
                                          const C2<R>*, hipStream_t, const uint8_t*);                  \
    template hipError_t launch_col_orient<R>(C2<R>*, int, const LaunchGeom&, const FftPlan&,           \
                                             const C2<R>*, double, hipStream_t);                       \
    template hipError_t launch_row_inv<R>(int, const C2<R>*, R*, typename Enc<R>::U*, uint8_t*, int,   \
                                          int, int, R, const LaunchGeom&, int, const FftPlan&,         \
                                          const C2<R>*, hipStream_t, bool, bool);                      \
    template hipError_t launch_col_inv_paired<R>(C2<R>*, int, int, const LaunchGeom&, const FftPlan&,  \
                                                 const C2<R>*, hipStream_t, const uint8_t*, C2<R>*);   \
    template bool row_blocked<R>(int, const LaunchGeom&);                                              \
    template bool col_inv_masks<R>(int, const LaunchGeom&);                                            \
    template hipError_t launch_fill_enc<R>(typename Enc<R>::U*, long, hipStream_t);                    \
    template hipError_t launch_decode_enc<R>(const typename Enc<R>::U*, R*, long, hipStream_t);        \
    template hipError_t launch_lift<R>(const R*, const uint8_t*, const uint8_t*, R*, int, int,         \
                                       hipStream_t);                                                   \
    template hipError_t launch_project<R>(const R*, R*, int, int, bool, hipStream_t);

}  // namespace se2n
