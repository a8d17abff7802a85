// Batched kernels of the pair path (se2n_pair.hpp), FP32, for the compiled
// sides: one launch per pass, side and (middle pass) block size over the tiles
// of all images; tile bodies and geometry are the single-image ones.
#include <hip/hip_runtime.h>

#include <cstdint>

#include "se2n_batch.hpp"
#include "se2n_pair.hpp"

namespace se2n {

namespace {

using C = C2<float>;

__device__ __forceinline__ const BItem& pair_item(const BItem* __restrict__ items, int idx) {
    return items[__builtin_amdgcn_readfirstlane(idx)];
}
// The thread index, hidden from loop-invariant code motion out of the tile loop.
__device__ __forceinline__ int pair_tid() {
    int t = threadIdx.x;
    asm volatile("" : "+v"(t));
    return t;
}

// Tile {item, row block, first pair, end pair}.
template <int MS>
__global__ __launch_bounds__(1024) void kb_pair_fwd(const BItem* __restrict__ items, const int4* __restrict__ tiles,
                                                    int ntiles) {
    constexpr int rows = pair_fwd_rows(MS, 4);
    constexpr int EPT = pair_row_ept(rows * MS, 4);
    extern __shared__ unsigned char smem_raw[];
    C* tw = reinterpret_cast<C*>(smem_raw);
    C* buf = tw + pair_tw_elems(MS);
    // every image of a launch has the same side, hence the same twiddles
    pair_load_tw<float>(tw, pair_item(items, tiles[0].x).tw, MS, threadIdx.x, blockDim.x);
    __syncthreads();
    for (int t = blockIdx.x; t < ntiles; t += gridDim.x) {
        const int4 tl = tiles[t];
        const BItem& d = pair_item(items, tl.x);
        pair_fwd_tile<float, PSRC_LIFT, MS, EPT>(d.f, d.mask, d.rmap, nullptr, d.spec, d.lay, MS, d.N, rows,
                                                 tl.y * rows, tl.z, tl.w, d.planM, tw, buf, pair_tid(), blockDim.x);
    }
}

// Tile {item, row block, 0, pairs}: the maximum or the mean of every slice.
template <int DST, int MS, int EPT>
__global__ __launch_bounds__(1024) void kb_pair_inv(const BItem* __restrict__ items, const int4* __restrict__ tiles,
                                                    int ntiles) {
    extern __shared__ unsigned char smem_raw[];
    C* tw = reinterpret_cast<C*>(smem_raw);
    C* buf = tw + pair_tw_elems(MS);
    pair_load_tw<float>(tw, pair_item(items, tiles[0].x).tw, MS, threadIdx.x, blockDim.x);
    for (int t = blockIdx.x; t < ntiles; t += gridDim.x) {
        const int4 tl = tiles[t];
        const BItem& d = pair_item(items, tl.x);
        pair_inv_tile<float, DST, MS, EPT>(d.spec, d.lay, d.out, nullptr, nullptr, nullptr, 0.f, MS, d.N, d.inv_rows,
                                           d.inv_G, tl.y * d.inv_rows, tl.z, tl.w, d.planM, tw, buf, pair_tid(),
                                           blockDim.x);
    }
}

// Tile {item, column, block, 0}.  WALK as in k_pair_mid.
template <int MS, int EPT, bool WALK>
__global__ __launch_bounds__(1024) void kb_pair_mid(const BItem* __restrict__ items, const int4* __restrict__ tiles,
                                                    int ntiles) {
    extern __shared__ unsigned char smem_raw[];
    C* tw = reinterpret_cast<C*>(smem_raw);
    C* buf = tw + pair_tw_elems(MS);
    const int nthr = blockDim.x;
    PairMidIn<float, MS, EPT> in;
    auto fetch = [&](int t, int tid) {
        const int4 tl = tiles[t];
        const BItem& d = pair_item(items, tl.x);
        long step;
        const C* col = pair_col<float>(d.spec, d.lay, MS, d.N, tl.y, tl.z, step);
        in.load(col, step, d.lay, d.N, pair_hs(d.N), tid, nthr);
    };
    if (WALK && (int)blockIdx.x < ntiles) fetch(blockIdx.x, threadIdx.x);
    pair_load_tw<float>(tw, pair_item(items, tiles[0].x).tw, MS, threadIdx.x, nthr);
    for (int t = blockIdx.x; t < ntiles; t += gridDim.x) {
        const int4 tl = tiles[t];
        const BItem& d = pair_item(items, tl.x);
        const int tid = pair_tid();
        long step;
        C* col = pair_col<float>(d.spec, d.lay, MS, d.N, tl.y, tl.z, step);
        if (!WALK) in.load(col, step, d.lay, d.N, pair_hs(d.N), tid, nthr);
        pair_mid_run<float, MS, EPT, false, false>(in, col, step, d.lay, d.P, d.N, tl.y, tl.z, tw, buf, tid, nthr, [&] {
            if (WALK && t + (int)gridDim.x < ntiles) fetch(t + gridDim.x, tid);
        });
    }
}

// Calls f(kernel pointer) for the kernel of a pass.
template <int MS, class F>
hipError_t pair_kernel(int kind, int ept, bool walk, F&& f) {
    switch (kind) {
        case BK_PAIR_FWD: return f((const void*)kb_pair_fwd<MS>);
        case BK_PAIR_MAX:
            return ept == 8 ? f((const void*)kb_pair_inv<PDST_MAX, MS, 8>)
                            : f((const void*)kb_pair_inv<PDST_MAX, MS, 16>);
        case BK_PAIR_MEAN:
            return ept == 8 ? f((const void*)kb_pair_inv<PDST_SUM, MS, 8>)
                            : f((const void*)kb_pair_inv<PDST_SUM, MS, 16>);
        case BK_PAIR_MID:
            if (ept == 4) return f((const void*)kb_pair_mid<MS, 4, false>);
            if (ept == 8) return f((const void*)kb_pair_mid<MS, 8, false>);
            return walk ? f((const void*)kb_pair_mid<MS, 16, true>) : f((const void*)kb_pair_mid<MS, 16, false>);
        default: return hipErrorInvalidValue;
    }
}

template <class F>
hipError_t with_pair_kernel(int kind, int M, int ept, bool walk, F&& f) {
    switch (M) {
        case 128: return pair_kernel<128>(kind, ept, walk, f);
        case 192: return pair_kernel<192>(kind, ept, walk, f);
        case 256: return pair_kernel<256>(kind, ept, walk, f);
        case 384: return pair_kernel<384>(kind, ept, walk, f);
        case 512: return pair_kernel<512>(kind, ept, walk, f);
        case 768: return pair_kernel<768>(kind, ept, walk, f);
        case 1024: return pair_kernel<1024>(kind, ept, walk, f);
        default: return hipErrorInvalidValue;
    }
}

}  // namespace

hipError_t launch_batch_pair(int kind, int M, int ept, bool walk, int threads, const BItem* items, const int4* tiles,
                             int ntiles, int grid, size_t lds, hipStream_t st) {
    if (ntiles <= 0) return hipSuccess;
    return with_pair_kernel(kind, M, ept, walk, [&](const void* fn) {
        void* args[] = {(void*)&items, (void*)&tiles, (void*)&ntiles};
        return hipLaunchKernel(fn, dim3((unsigned)grid), dim3((unsigned)threads), args, lds, st);
    });
}

}  // namespace se2n
