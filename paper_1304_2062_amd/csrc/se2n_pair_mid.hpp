// Middle kernel of the pair path and its launcher, included once per data
// type (se2n_pair_mid_f32.hip, se2n_pair_mid_f64.hip).
#pragma once

#include "se2n_pair.hpp"

namespace se2n {

namespace {

// WALK: workgroups walk the column blocks with stride gridDim.x, and the next
// block's column is fetched while the current one is transformed back.  The walk pays where a workgroup has a compute unit to itself (more
// than half of its LDS): 1024^2, N = 32, FP32: 105 -> 98 us, 512^2, N = 32,
// FP64: 51 -> 46 us; smaller blocks share a unit and overlap by themselves
// (512^2, N = 30 with one resident walker per unit: 23 -> 33 us), and get a
// workgroup each.
template <class R, int MS, int EPT, bool WALK>
__global__ __launch_bounds__(pair_max_threads((int)sizeof(R))) void k_pair_mid(C2<R>* __restrict__ spec, PairLay lay,
                                                                               const R* __restrict__ T, int M_, int N,
                                                                               FftPlan planM,
                                                                               const C2<R>* __restrict__ twg) {
    const int M = MS ? MS : M_;
    extern __shared__ unsigned char smem_raw[];
    C2<R>* tw = reinterpret_cast<C2<R>*>(smem_raw);
    C2<R>* buf = tw + pair_tw_elems(M);
    const int tid = threadIdx.x, nthr = blockDim.x;
    const int H = M >> 1, nblk = pair_nblk(N);
    const int nt = H * nblk;
    int kx, blk;
    pair_mid_col(blockIdx.x, H, nblk, kx, blk);
    if constexpr (MS != 0) {
        const int hs = pair_hs(N);
        PairMidIn<R, MS, EPT> in;
        long step;
        C2<R>* col = pair_col<R>(spec, lay, M, N, kx, blk, step);
        in.load(col, step, lay, N, hs, tid, nthr);
        pair_load_tw<R>(tw, twg, M, tid, nthr);
        for (int i = blockIdx.x;; i += gridDim.x) {
            const bool more = WALK && i + (int)gridDim.x < nt;
            int kn = 0, bn = 0;
            C2<R>* cn = col;
            if (more) {
                pair_mid_col(i + gridDim.x, H, nblk, kn, bn);
                cn = pair_col<R>(spec, lay, M, N, kn, bn, step);
            }
            pair_mid_run<R, MS, EPT, false, pair_direct((int)sizeof(R)) && (EPT < 16)>(
                in, col, step, lay, T, N, kx, blk, tw, buf, tid, nthr, [&] {
                if (more) in.load(cn, step, lay, N, hs, tid, nthr);
            });
            if (!more) return;
            col = cn;
            kx = kn;
            blk = bn;
        }
    } else {
        pair_load_tw<R>(tw, twg, M, tid, nthr);
        for (int i = blockIdx.x; i < nt; i += gridDim.x) {
            pair_mid_col(i, H, nblk, kx, blk);
            __syncthreads();
            pair_mid_generic<R, EPT>(spec, lay, T, M, N, kx, blk, planM, tw, buf, tid, nthr);
        }
    }
}

// Half columns (PairLay), side 2 MS.  1024^2, N = 32, FP64: 355 -> 237 us
// against the two column passes and the solve (268 MB read and written and 152
// MB of propagators, 3 TB/s); a workgroup each instead of walkers: 509 against
// 483 us for the whole.
template <class R, int MS, int EPT, bool WALK>
__global__ __launch_bounds__(pair_max_threads((int)sizeof(R))) void k_pair_mid_half(
    C2<R>* __restrict__ spec, PairLay lay, const R* __restrict__ T, int N, const C2<R>* __restrict__ twg) {
    extern __shared__ unsigned char smem_raw[];
    C2<R>* tw = reinterpret_cast<C2<R>*>(smem_raw);
    C2<R>* buf = tw + pair_tw_elems(MS);
    const int tid = threadIdx.x, nthr = blockDim.x;
    const int nblk = pair_nblk(N);
    const int nt = 2 * MS * nblk;
    const int hs = pair_hs(N);
    PairMidIn<R, MS, EPT, MS> in;
    int kx, blk, par;
    long step;
    auto column = [&](int i) {
        pair_mid_half(i, MS, nblk, kx, blk, par);
        return pair_col<R>(spec, lay, 2 * MS, N, kx, blk, step) + par * (lay.rb / 2);
    };
    C2<R>* col = column(blockIdx.x);
    in.load(col, step, lay, N, hs, tid, nthr);
    // the table of length 2 MS, every other entry
    for (int m = tid; m < MS / 4; m += nthr) {
        const C2<R> w = twg[2 * m];
        tw[tw_pos(m)] = w;
        tw[tw_pos(m + MS / 4)] = cmk<R>(w.y, -w.x);
        tw[tw_pos(m + MS / 2)] = cmk<R>(-w.x, -w.y);
    }
    for (int i = blockIdx.x;; i += gridDim.x) {
        const bool more = WALK && i + (int)gridDim.x < nt;
        const int k0 = kx, b0 = blk, p0 = par;
        C2<R>* cn = col;
        if (more) cn = column(i + gridDim.x);
        pair_mid_run<R, MS, EPT, true, false>(
            in, col, step, lay, T, N, k0, b0, tw, buf, tid, nthr,
            [&] {
                if (more) in.load(cn, step, lay, N, hs, tid, nthr);
            },
            p0);
        if (!more) return;
        col = cn;
    }
}

template <class R, int MS, int EPT>
hipError_t mid_half_go(C2<R>* spec, const R* T, int N, const PairGeom& g, const C2<R>* tw, hipStream_t st) {
    const int tiles = 2 * MS * pair_nblk(N);
    const size_t lds = pair_lds_bytes(MS, pair_hs(N), (int)sizeof(R));
    if constexpr (EPT == 16) {
        if (g.mid_grid < tiles) {
            hipLaunchKernelGGL((k_pair_mid_half<R, MS, EPT, true>), dim3((unsigned)g.mid_grid), dim3(g.mid_threads),
                               lds, st, spec, g.lay, T, N, tw);
            return hipGetLastError();
        }
    }
    hipLaunchKernelGGL((k_pair_mid_half<R, MS, EPT, false>), dim3((unsigned)tiles), dim3(g.mid_threads), lds, st, spec,
                       g.lay, T, N, tw);
    return hipGetLastError();
}
template <class R, int MS>
hipError_t mid_half(C2<R>* spec, const R* T, int N, const PairGeom& g, const C2<R>* tw, hipStream_t st) {
    if (g.mid_ept == 8) return mid_half_go<R, MS, 8>(spec, T, N, g, tw, st);
    return mid_half_go<R, MS, 16>(spec, T, N, g, tw, st);
}

template <class R, int MS, int EPT>
hipError_t mid_go(C2<R>* spec, const R* T, int M, int N, const PairGeom& g, const FftPlan& planM, const C2<R>* tw,
                  hipStream_t st) {
    const int tiles = M / 2 * pair_nblk(N);
    const size_t lds = pair_lds_bytes(M, pair_hs(N), (int)sizeof(R));
    if constexpr (EPT == 16 && MS != 0) {
        if (g.mid_grid < tiles) {
            hipLaunchKernelGGL((k_pair_mid<R, MS, EPT, true>), dim3((unsigned)g.mid_grid), dim3(g.mid_threads), lds, st,
                               spec, g.lay, T, M, N, planM, tw);
            return hipGetLastError();
        }
    }
    hipLaunchKernelGGL((k_pair_mid<R, MS, EPT, false>), dim3((unsigned)tiles), dim3(g.mid_threads), lds, st, spec,
                       g.lay, T, M, N, planM, tw);
    return hipGetLastError();
}

template <class R, int MS>
hipError_t mid_side(C2<R>* spec, const R* T, int M, int N, const PairGeom& g, const FftPlan& planM, const C2<R>* tw,
                    hipStream_t st) {
    if (g.mid_ept == 4) return mid_go<R, MS, 4>(spec, T, M, N, g, planM, tw, st);
    if (g.mid_ept == 8) return mid_go<R, MS, 8>(spec, T, M, N, g, planM, tw, st);
    return mid_go<R, MS, 16>(spec, T, M, N, g, planM, tw, st);
}

}  // namespace

template <class R>
hipError_t launch_pair_mid(C2<R>* spec, const R* T, int M, int N, const PairGeom& g, const FftPlan& planM,
                           const C2<R>* tw, hipStream_t st) {
    if constexpr (sizeof(R) == 8) {
        if (g.lay.halved) {
            if (M == 384) return mid_half<R, 192>(spec, T, N, g, tw, st);
            if (M == 512) return mid_half<R, 256>(spec, T, N, g, tw, st);
            if (M == 768) return mid_half<R, 384>(spec, T, N, g, tw, st);
            if (M == 1024) return mid_half<R, 512>(spec, T, N, g, tw, st);
            return mid_half<R, 1024>(spec, T, N, g, tw, st);
        }
    }
    switch (M) {
#define SE2N_SIDE(m) \
    case m: return mid_side<R, m>(spec, T, M, N, g, planM, tw, st);
        SE2N_SIDE(64) SE2N_SIDE(128) SE2N_SIDE(192) SE2N_SIDE(256) SE2N_SIDE(384) SE2N_SIDE(512) SE2N_SIDE(768)
        SE2N_SIDE(1024)
#undef SE2N_SIDE
        default: return mid_side<R, 0>(spec, T, M, N, g, planM, tw, st);
    }
}

#define SE2N_PAIR_MID_INSTANTIATE(R)                                                                            \
    template hipError_t launch_pair_mid<R>(C2<R>*, const R*, int, int, const PairGeom&, const FftPlan&,         \
                                           const C2<R>*, hipStream_t);

}  // namespace se2n
