// Row kernels of the pair path and their launchers, included once per data
// type (se2n_pair_rows_f32.hip, se2n_pair_rows_f64.hip).
#pragma once

#include "se2n_pair.hpp"

namespace se2n {

namespace {

// HALF: halved columns (PairLay)
template <class R, int SRC, int MS, int EPT, bool HALF>
__global__ __launch_bounds__(pair_max_threads((int)sizeof(R))) void k_pair_fwd(const R* __restrict__ f, const uint8_t* __restrict__ mask,
                                                   const uint8_t* __restrict__ rmap, const R* __restrict__ vol,
                                                   C2<R>* __restrict__ spec, PairLay lay, int M_, int N, int rows, int ppw,
                                                   FftPlan planM, const C2<R>* __restrict__ twg) {
    const int M = MS ? MS : M_;
    extern __shared__ unsigned char smem_raw[];
    C2<R>* tw = reinterpret_cast<C2<R>*>(smem_raw);
    C2<R>* buf = tw + pair_tw_elems(M);
    const int tid = threadIdx.x, nthr = blockDim.x;
    pair_load_tw<R>(tw, twg, M, tid, nthr);
    if (MS != 0) __syncthreads();
    const int nrb = M / rows;
    const int w = xcd_contiguous(blockIdx.x, gridDim.x);
    // row blocks fastest: neighbours on one XCD complete each other's lines
    const int grp = w / nrb, rb = w - grp * nrb;
    const int t0 = grp * ppw;
    pair_fwd_tile<R, SRC, MS, EPT, HALF>(f, mask, rmap, vol, spec, lay, M, N, rows, rb * (HALF ? rows / 2 : rows), t0,
                                         min(pair_count(N), t0 + ppw), planM, tw, buf, tid, nthr);
}

template <class R, int DST, int MS, int EPT>
__global__ __launch_bounds__(pair_max_threads((int)sizeof(R))) void k_pair_inv(C2<R>* __restrict__ spec, PairLay lay, R* __restrict__ out, R* __restrict__ hmax,
                                                   const R* __restrict__ f, const uint8_t* __restrict__ mask, R eps,
                                                   int M_, int N, int rows, int G, int ppw, FftPlan planM,
                                                   const C2<R>* __restrict__ twg) {
    const int M = MS ? MS : M_;
    extern __shared__ unsigned char smem_raw[];
    C2<R>* tw = reinterpret_cast<C2<R>*>(smem_raw);
    C2<R>* buf = tw + pair_tw_elems(M);
    const int tid = threadIdx.x, nthr = blockDim.x;
    pair_load_tw<R>(tw, twg, M, tid, nthr);
    const int nrb = M / rows;
    const int w = xcd_contiguous(blockIdx.x, gridDim.x);
    const int grp = w / nrb, rb = w - grp * nrb;
    const int t0 = grp * ppw;
    pair_inv_tile<R, DST, MS, EPT>(spec, lay, out, hmax, f, mask, eps, M, N, rows, G, rb * rows, t0,
                                   min(pair_count(N), t0 + ppw), planM, tw, buf, tid, nthr);
}

template <class R, int DST, int MS, int EPT>
__global__ __launch_bounds__(pair_max_threads((int)sizeof(R))) void k_pair_inv_half(
    const C2<R>* __restrict__ spec, PairLay lay, R* __restrict__ out, int N, int rows, int ppw,
    const C2<R>* __restrict__ twg) {
    extern __shared__ unsigned char smem_raw[];
    C2<R>* tw = reinterpret_cast<C2<R>*>(smem_raw);
    C2<R>* buf = tw + pair_tw_elems(MS);
    const int tid = threadIdx.x, nthr = blockDim.x;
    pair_load_tw<R>(tw, twg, MS, tid, nthr);
    __syncthreads();
    const int nrb = MS / rows;
    const int w = xcd_contiguous(blockIdx.x, gridDim.x);
    const int grp = w / nrb, rb = w - grp * nrb;
    const int t0 = grp * ppw;
    pair_inv_half_tile<R, DST, MS, EPT>(spec, lay, out, N, rows, rb * (rows / 2), t0, min(pair_count(N), t0 + ppw), tw,
                                        buf, tid, nthr);
}

template <class R, int MS, int EPT>
__global__ __launch_bounds__(pair_max_threads((int)sizeof(R))) void k_pair_dr(const R* __restrict__ vol, const R* __restrict__ h,
                                                  int16_t* __restrict__ join, R* __restrict__ href,
                                                  C2<R>* __restrict__ spec, PairLay lay, R eps, int step, int M_, int N,
                                                  FftPlan planM, const C2<R>* __restrict__ twg) {
    const int M = MS ? MS : M_;
    extern __shared__ unsigned char smem_raw[];
    C2<R>* tw = reinterpret_cast<C2<R>*>(smem_raw);
    C2<R>* buf = tw + pair_tw_elems(M);
    const int tid = threadIdx.x, nthr = blockDim.x;
    pair_load_tw<R>(tw, twg, M, tid, nthr);
    pair_dr_tile<R, MS, EPT>(vol, h, join, href, spec, lay, eps, step, M, N, 1, xcd_contiguous(blockIdx.x, gridDim.x), planM,
                             tw, buf, tid, nthr);
}

// f(std::integral_constant<int, MS>) for the compiled side of M (pair_rows_compiled), or 0
template <class R, class F>
hipError_t by_side(int M, F&& f) {
    switch (M) {
#define SE2N_SIDE(m)                                                                                        \
    case m:                                                                                                 \
        if constexpr (pair_rows_compiled(m, (int)sizeof(R))) return f(std::integral_constant<int, m>{});    \
        break;
        SE2N_SIDE(64) SE2N_SIDE(128) SE2N_SIDE(256) SE2N_SIDE(384) SE2N_SIDE(512) SE2N_SIDE(768) SE2N_SIDE(1024)
#undef SE2N_SIDE
        default: break;
    }
    return f(std::integral_constant<int, 0>{});
}
// The sides whose columns may be halved (pair_halves).
template <class F>
hipError_t by_half_side(int M, F&& f) {
    if (M == 384) return f(std::integral_constant<int, 384>{});
    if (M == 512) return f(std::integral_constant<int, 512>{});
    if (M == 768) return f(std::integral_constant<int, 768>{});
    if (M == 1024) return f(std::integral_constant<int, 1024>{});
    return f(std::integral_constant<int, 2048>{});
}
template <class F>
hipError_t by_ept(int ept, F&& f) {
    return ept == 8 ? f(std::integral_constant<int, 8>{}) : f(std::integral_constant<int, 16>{});
}

}  // namespace

template <class R>
hipError_t launch_pair_fwd(int src, const R* f, const uint8_t* mask, const uint8_t* rmap, const R* vol, C2<R>* spec,
                           int M, int N, const PairGeom& g, const FftPlan& planM, const C2<R>* tw, hipStream_t st) {
    const int np = pair_count(N);
    const int ppw = src == PSRC_VOLUME ? g.vol_fwd_pairs : g.fwd_pairs;
    const dim3 grid((unsigned)(M / g.fwd_rows * ((np + ppw - 1) / ppw)));
    const size_t lds = pair_lds_bytes(M, g.fwd_rows, (int)sizeof(R));
    if constexpr (sizeof(R) == 8) {
        if (g.lay.halved) return by_half_side(M, [&](auto ms) {
            constexpr int MS = decltype(ms)::value;
            constexpr int EPT = pair_row_ept(pair_fwd_rows(MS, (int)sizeof(R)) * MS, (int)sizeof(R));
            if (src == PSRC_LIFT)
                hipLaunchKernelGGL((k_pair_fwd<R, PSRC_LIFT, MS, EPT, true>), grid, dim3(g.fwd_threads), lds, st, f,
                                   mask, rmap, vol, spec, g.lay, M, N, g.fwd_rows, ppw, planM, tw);
            else
                hipLaunchKernelGGL((k_pair_fwd<R, PSRC_VOLUME, MS, EPT, true>), grid, dim3(g.fwd_threads), lds, st, f,
                                   mask, rmap, vol, spec, g.lay, M, N, g.fwd_rows, ppw, planM, tw);
            return hipGetLastError();
        });
    }
    return by_side<R>(M, [&](auto ms) {
        return by_ept(g.fwd_ept, [&](auto ept) {
            constexpr int MS = decltype(ms)::value, EPT = decltype(ept)::value;
            constexpr int rs = (int)sizeof(R);
            if constexpr (MS == 0 || EPT == pair_row_ept(pair_fwd_rows(MS ? MS : 16, rs) * MS, rs)) {
                if (src == PSRC_LIFT)
                    hipLaunchKernelGGL((k_pair_fwd<R, PSRC_LIFT, MS, EPT, false>), grid, dim3(g.fwd_threads), lds, st, f, mask,
                                       rmap, vol, spec, g.lay, M, N, g.fwd_rows, ppw, planM, tw);
                else
                    hipLaunchKernelGGL((k_pair_fwd<R, PSRC_VOLUME, MS, EPT, false>), grid, dim3(g.fwd_threads), lds, st, f,
                                       mask, rmap, vol, spec, g.lay, M, N, g.fwd_rows, ppw, planM, tw);
                return hipGetLastError();
            } else {
                return hipErrorInvalidValue;
            }
        });
    });
}

template <class R>
hipError_t launch_pair_inv(int dst, C2<R>* spec, R* out, int M, int N, const PairGeom& g, const FftPlan& planM,
                           const C2<R>* tw, hipStream_t st) {
    const int np = pair_count(N);
    const bool vol = dst == PDST_VOLUME;
    const int rows = vol ? g.fwd_rows : g.inv_rows;
    const int G = vol ? 1 : g.inv_G;
    const int ppw = vol ? g.vol_pairs : np;
    const int threads = vol ? g.fwd_threads : g.inv_threads;
    const dim3 grid((unsigned)(M / rows * ((np + ppw - 1) / ppw)));
    if constexpr (sizeof(R) == 8) {
        if (g.lay.halved) return by_half_side(M, [&](auto ms) {
            constexpr int MS = decltype(ms)::value;
            constexpr int EPT = pair_row_ept(pair_fwd_rows(MS, (int)sizeof(R)) * MS, (int)sizeof(R));
            const size_t lds = pair_lds_bytes(MS, rows, (int)sizeof(R));
#define SE2N_INV(D) \
    hipLaunchKernelGGL((k_pair_inv_half<R, D, MS, EPT>), grid, dim3(threads), lds, st, spec, g.lay, out, N, rows, ppw, tw)
            if (dst == PDST_MAX) SE2N_INV(PDST_MAX);
            else if (dst == PDST_SUM) SE2N_INV(PDST_SUM);
            else SE2N_INV(PDST_VOLUME);
#undef SE2N_INV
            return hipGetLastError();
        });
    }
    // the transforms, and the pixels' running values between rounds
    const size_t lds = pair_lds_bytes(M, rows * G, (int)sizeof(R)) + (G < ppw ? (size_t)rows * M * sizeof(R) : 0);
    return by_side<R>(M, [&](auto ms) {
        return by_ept(vol ? g.fwd_ept : g.inv_ept, [&](auto ept) {
            constexpr int MS = decltype(ms)::value, EPT = decltype(ept)::value;
#define SE2N_INV(D)                                                                                                 \
    hipLaunchKernelGGL((k_pair_inv<R, D, MS, EPT>), grid, dim3(threads), lds, st, spec, g.lay, out, (R*)nullptr,          \
                       (const R*)nullptr, (const uint8_t*)nullptr, R(0), M, N, rows, G, ppw, planM, tw)
            if (dst == PDST_MAX) SE2N_INV(PDST_MAX);
            else if (dst == PDST_SUM) SE2N_INV(PDST_SUM);
            else SE2N_INV(PDST_VOLUME);
#undef SE2N_INV
            return hipGetLastError();
        });
    });
}

template <class R>
hipError_t launch_pair_sr(C2<R>* spec, const R* f, const uint8_t* mask, double eps, int M, int N, const PairGeom& g,
                          const FftPlan& planM, const C2<R>* tw, hipStream_t st) {
    const int np = pair_count(N);
    const size_t lds = pair_lds_bytes(M, np, (int)sizeof(R));
    return by_side<R>(M, [&](auto ms) {
        return by_ept(g.all_ept, [&](auto ept) {
            constexpr int MS = decltype(ms)::value, EPT = decltype(ept)::value;
            hipLaunchKernelGGL((k_pair_inv<R, PDST_SR, MS, EPT>), dim3((unsigned)M), dim3(g.all_threads), lds, st, spec,
                               g.lay, (R*)nullptr, (R*)nullptr, f, mask, (R)eps, M, N, 1, np, np, planM, tw);
            return hipGetLastError();
        });
    });
}

template <class R>
hipError_t launch_pair_dr(C2<R>* spec, R* vol, R* h, int16_t* join, R* href, double eps, int step, int M, int N,
                          const PairGeom& g, const FftPlan& planM, const C2<R>* tw, hipStream_t st) {
    const int np = pair_count(N);
    const size_t lds = pair_lds_bytes(M, np, (int)sizeof(R));
    return by_side<R>(M, [&](auto ms) {
        return by_ept(g.all_ept, [&](auto ept) {
            constexpr int MS = decltype(ms)::value, EPT = decltype(ept)::value;
            hipLaunchKernelGGL((k_pair_inv<R, PDST_VOLMAX, MS, EPT>), dim3((unsigned)M), dim3(g.all_threads), lds, st,
                               spec, g.lay, vol, h, (const R*)nullptr, (const uint8_t*)nullptr, R(0), M, N, 1, np, np, planM,
                               tw);
            hipError_t e = hipGetLastError();
            if (e != hipSuccess) return e;
            hipLaunchKernelGGL((k_pair_dr<R, MS, EPT>), dim3((unsigned)M), dim3(g.all_threads), lds, st, vol, h, join,
                               href, spec, g.lay, (R)eps, step, M, N, planM, tw);
            return hipGetLastError();
        });
    });
}

#define SE2N_PAIR_ROWS_INSTANTIATE(R)                                                                                  \
    template hipError_t launch_pair_fwd<R>(int, const R*, const uint8_t*, const uint8_t*, const R*, C2<R>*, int, int,  \
                                           const PairGeom&, const FftPlan&, const C2<R>*, hipStream_t);                \
    template hipError_t launch_pair_inv<R>(int, C2<R>*, R*, int, int, const PairGeom&, const FftPlan&, const C2<R>*,   \
                                           hipStream_t);                                                               \
    template hipError_t launch_pair_sr<R>(C2<R>*, const R*, const uint8_t*, double, int, int, const PairGeom&,         \
                                          const FftPlan&, const C2<R>*, hipStream_t);                                  \
    template hipError_t launch_pair_dr<R>(C2<R>*, R*, R*, int16_t*, R*, double, int, int, int, const PairGeom&,        \
                                          const FftPlan&, const C2<R>*, hipStream_t);

}  // namespace se2n
