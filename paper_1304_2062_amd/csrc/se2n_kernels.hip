// gfx950 kernels of the semi-discrete SE(2,N) diffusion.
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
#include <hip/hip_runtime.h>

#include <cstdint>
#include <cstdlib>

#include "se2n_fft.hpp"
#include "se2n_internal.hpp"
#include "se2n_pair.hpp"
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
// Propagator precompute, FP64: one 64-thread workgroup per frequency class.
// ---------------------------------------------------------------------------
// For class (lx, ly) and each block (periodic +, antiperiodic -) of size
// h = N/2:  A = beta L_h^{+-} - diag(pot_j), pot_j = M (cos e_j s_x + sin e_j s_y)^2.
// Odd N: one periodic block of size h = N, the whole propagator.
//   CN:    C = (I - tau A/2)^{-1} (I + tau A/2) by Gauss-Jordan (the left
//          matrix is symmetric, diagonally dominant: no pivoting), P = C^n by
//          binary powering.
//   EXACT: P = e^{T A} by scaling and squaring of a degree-16 Taylor sum.
__device__ void lds_matmul(const double* A, const double* B, double* Cm, int h, int tid) {
    for (int idx = tid; idx < h * h; idx += 64) {
        const int i = idx / h;
        const int j = idx - i * h;
        double s = 0.0;
        for (int k = 0; k < h; ++k) s += A[i * h + k] * B[k * h + j];
        Cm[idx] = s;
    }
    __syncthreads();
}

__device__ void lds_copy(const double* A, double* B, int n, int tid) {
    for (int idx = tid; idx < n; idx += 64) B[idx] = A[idx];
    __syncthreads();
}

// Negligible-class flag of a slot's class, under both orders when the slot
// is shared (the column passes look flags up by (lx, ly) as they come), and
// the padding of the flag rows the slot ends (by the thread group of one
// workgroup; tid < 64).
template <class R>
__device__ void store_class_flags(R* Ptab, int M, int N, int Q, int FS, int lx, int ly, bool negligible, int tid,
                                  int pair) {
    uint8_t* flags = reinterpret_cast<uint8_t*>(
        Ptab + (pair ? pair_table_entries(M, N, pair == 2) : table_slots(M, N) * (size_t)table_class_stride(N, (int)sizeof(R))));
    if (tid == 0) {
        flags[(size_t)lx * FS + ly] = negligible ? 1 : 0;
        if (table_sym(N)) flags[(size_t)ly * FS + lx] = negligible ? 1 : 0;
    }
    if (ly == Q - 1)  // row padding (every row lx has the slot (lx, Q - 1))
        for (int j = Q + tid; j < FS; j += 64) flags[(size_t)lx * FS + j] = 0;
}

// The element-major table of the pair path: block b of class (lx, ly), and
// with 4 | N of class (ly, lx), whose block is the same one conjugated by the
// reflection r -> N/4 - r (an index that wraps around turns the sign of an
// antiperiodic slice).  at(i, j) is the symmetrised entry of this class.
template <class R, class F>
__device__ void store_pair_block(R* Ptab, int M, int N, int halved, int b, int lx, int ly, int h, double scale, int tid,
                                 F&& at) {
    const int Eh = h * (h + 1) / 2;
    const int QP = pair_qp(M, halved);
    const int nblk = pair_nblk(N);
    R* d0 = Ptab + ((size_t)(lx * nblk + b) * Eh) * QP + pair_class_pos(M, halved, ly);
    R* d1 = Ptab + ((size_t)(ly * nblk + b) * Eh) * QP + pair_class_pos(M, halved, lx);
    const bool both = table_sym(N) && lx != ly;
    const int g = N / 4;
    const float inv_h = 1.0f / (float)h;
    for (int idx = tid; idx < h * h; idx += 64) {
        const int i = fdiv(idx, inv_h);
        const int j = idx - i * h;
        if (j < i) continue;
        const size_t e = (size_t)(i * h - i * (i - 1) / 2 + (j - i)) * QP;
        d0[e] = (R)(at(i, j) * scale);
        if (both) {
            const int a = i > g ? g - i + h : g - i, c = j > g ? g - j + h : g - j;
            const double u = at(a, c) * scale;
            d1[e] = (R)(b == 1 && (i > g) != (j > g) ? -u : u);
        }
    }
}

template <class R>
__global__ __launch_bounds__(64) void k_precompute(R* __restrict__ Ptab, int M, int N, int Q, int FS,
                                                   double beta, double T, int nsteps, int scheme,
                                                   double scale, int keep_all, int pair) {
    extern __shared__ double sm[];
    const bool odd = (N & 1) != 0;
    const int h = odd ? N : N / 2;
    const int nblk = odd ? 1 : 2;
    const int hh = h * h;
    // LDS: W (2hh) | Rs (hh) | Ts (hh) | pot (h).  CN builds the generator A
    // in Ts, fills the augmented matrix W from it, eliminates (Ts then holds
    // the pivot column), and compacts the right half of W (the one-step
    // propagator) into W's first hh entries, Bs.  EXACT keeps A in W.
    double* W = sm;          // h x 2h augmented matrix
    double* Bs = W;          // base of the powering (CN)
    double* Rs = W + 2 * hh; // running product
    double* Ts = Rs + hh;    // temporary
    double* pot = Ts + hh;
    double* A = scheme == 0 ? Ts : W;  // generator block
    const int tid = threadIdx.x;
    int lx, ly;  // the class of this workgroup's slot
    table_slot_class(blockIdx.x, Q, N, lx, ly);
    const double two_pi = 6.283185307179586476925;
    const double sx = sin(two_pi * lx / M);
    const double sy = sin(two_pi * ly / M);
    for (int j = tid; j < h; j += 64) {
        const double e = two_pi * j / N;
        const double a = cos(e) * sx + sin(e) * sy;
        pot[j] = (double)M * a * a;
    }
    __syncthreads();
    const int Eh = h * (h + 1) / 2;
    const int E = nblk * Eh;
    const int CS = table_class_stride(N, (int)sizeof(R));
    double pmax = 0.0;  // largest entry of the unscaled propagator, this thread's share
    for (int blk = 0; blk < nblk; ++blk) {
        const double wrap = blk == 0 ? 1.0 : -1.0;
        for (int idx = tid; idx < hh; idx += 64) {
            const int i = idx / h;
            const int j = idx - i * h;
            double v = (i == j) ? (-2.0 * beta - pot[i]) : 0.0;
            // neighbours i+1 and i-1 with wrap-around sign
            if (j == (i + 1) % h) v += (i + 1 < h) ? beta : wrap * beta;
            if (j == (i + h - 1) % h) v += (i >= 1) ? beta : wrap * beta;
            A[idx] = v;
        }
        __syncthreads();
        if (scheme == 0) {
            const double tau = T / nsteps;
            for (int idx = tid; idx < 2 * hh; idx += 64) {
                const int i = idx / (2 * h);
                const int j = idx - i * 2 * h;
                const double a = A[i * h + (j % h)];
                const double id = (i == (j % h)) ? 1.0 : 0.0;
                W[idx] = (j < h) ? (id - 0.5 * tau * a) : (id + 0.5 * tau * a);
            }
            __syncthreads();
            for (int piv = 0; piv < h; ++piv) {
                const double inv = 1.0 / W[piv * 2 * h + piv];
                __syncthreads();  // every thread has read the pivot
                for (int j = tid; j < 2 * h; j += 64) W[piv * 2 * h + j] *= inv;
                for (int i = tid; i < h; i += 64) Ts[i] = W[i * 2 * h + piv];
                __syncthreads();
                for (int idx = tid; idx < 2 * hh; idx += 64) {
                    const int i = idx / (2 * h);
                    const int j = idx - i * 2 * h;
                    if (i != piv) W[idx] -= Ts[i] * W[piv * 2 * h + j];
                }
                __syncthreads();
            }
            // compact the right half of W into its first hh entries, row by
            // row: row i's destination [i h, i h + h) holds only entries of
            // rows already copied (and left halves, no longer needed)
            for (int i = 0; i < h; ++i) {
                double v = 0.0;
                if (tid < h) v = W[i * 2 * h + h + tid];
                __syncthreads();
                if (tid < h) Bs[i * h + tid] = v;
                __syncthreads();
            }
            for (int idx = tid; idx < hh; idx += 64) {
                const int i = idx / h;
                const int j = idx - i * h;
                Rs[idx] = (i == j) ? 1.0 : 0.0;
            }
            __syncthreads();
            int n = nsteps;
            while (n > 0) {
                if (n & 1) {
                    lds_matmul(Rs, Bs, Ts, h, tid);
                    lds_copy(Ts, Rs, hh, tid);
                }
                n >>= 1;
                if (n) {
                    lds_matmul(Bs, Bs, Ts, h, tid);
                    lds_copy(Ts, Bs, hh, tid);
                }
            }
        } else {
            // X = T A / 2^s with ||X||_inf <= 1/2
            double nrm = 0.0;
            for (int i = 0; i < h; ++i) {
                double rs = 0.0;
                for (int j = 0; j < h; ++j) rs += fabs(A[i * h + j]);
                nrm = fmax(nrm, rs);
            }
            nrm *= T;
            __syncthreads();  // all norms read before A is scaled in place
            int sq = 0;
            while (nrm > 0.5) {
                nrm *= 0.5;
                ++sq;
            }
            const double xs = T * ldexp(1.0, -sq);
            for (int idx = tid; idx < hh; idx += 64) {
                A[idx] *= xs;
                const int i = idx / h;
                const int j = idx - i * h;
                Rs[idx] = (i == j) ? 1.0 : 0.0;
            }
            __syncthreads();
            // Horner: E = I + X (I + X/2 (I + X/3 (... (I + X/16))))
            for (int k = 16; k >= 1; --k) {
                lds_matmul(A, Rs, Ts, h, tid);
                for (int idx = tid; idx < hh; idx += 64) {
                    const int i = idx / h;
                    const int j = idx - i * h;
                    Rs[idx] = ((i == j) ? 1.0 : 0.0) + Ts[idx] / k;
                }
                __syncthreads();
            }
            for (int s = 0; s < sq; ++s) {
                lds_matmul(Rs, Rs, Ts, h, tid);
                lds_copy(Ts, Rs, hh, tid);
            }
        }
        // packed upper triangle, symmetrised, scaled, stored as R
        R* dst = Ptab + (size_t)blockIdx.x * CS;
        for (int idx = tid; idx < hh; idx += 64) {
            const int i = idx / h;
            const int j = idx - i * h;
            if (j >= i) {
                const int e = blk * Eh + i * h - i * (i - 1) / 2 + (j - i);
                const double u = 0.5 * (Rs[i * h + j] + Rs[j * h + i]);
                pmax = fmax(pmax, fabs(u));
                if (!pair) dst[e] = (R)(u * scale);
            }
        }
        if (pair)
            store_pair_block<R>(Ptab, M, N, pair == 2, blk, lx, ly, h, scale, tid,
                                [&](int i, int j) { return 0.5 * (Rs[i * h + j] + Rs[j * h + i]); });
        __syncthreads();
    }
    // negligible-class flag (the workgroup is one wavefront): set when every
    // entry of both blocks is below 2^-30 (FP32) or 2^-60 (FP64); the solve
    // then writes zeros for the class's modes without reading them
    for (int off = 32; off >= 1; off >>= 1) pmax = fmax(pmax, __shfl_xor(pmax, off, 64));
    store_class_flags<R>(Ptab, M, N, Q, FS, lx, ly, !keep_all && pmax < (sizeof(R) == 4 ? 0x1p-30 : 0x1p-60), tid, pair);
    // the class's line padding
    if (!pair) for (int e = E + tid; e < CS; e += 64) Ptab[(size_t)blockIdx.x * CS + e] = R(0);
}

// ---------------------------------------------------------------------------
// Propagator precompute on the FP64 matrix cores, for blocks of at most
// 32 x 32 (even N; odd N up to 32, whose one block is the whole propagator):
// one wavefront per frequency class.
// ---------------------------------------------------------------------------
// A block is embedded in TILES x TILES tiles of 16 x 16 (zero padding).  The
// result D[i][j] of v_mfma_f64_16x16x4 lies in lane j + 16 (i mod 4), element
// i div 4; its operands are A[i][k] in lane i + 16 k and B[k][j] in lane
// j + 16 k.  So element kk of a result is, as it stands, the B operand of
// k-step kk, and for a symmetric matrix also the A operand: every matrix here
// is a polynomial of the symmetric generator, so products feed products from
// registers, with no LDS and no barrier in the powering.  Bound by the chain
// of dependent products of each wavefront (FP32 tables, against operands
// through LDS for blocks of 9..16 and scalar products for the others):
// 1024^2, N = 32, 200 steps 278 -> 200 us, 384^2, N = 48, 100 steps 900 -> 152,
// N = 64 3276 -> 185, 256^2, N = 31, 200 steps 1325 -> 108.  Rounding leaves
// R = C^n asymmetric by a few ulps; the stored entries are symmetrised.
//   CN:    the left matrix I - tau A / 2 is cyclic tridiagonal: one lane per
//          block factors it (Thomas elimination with a Sherman-Morrison
//          correction for the corners, as the paper's remark 2 suggests for
//          the time steps themselves), and lane c solves for the unit vector e_c.
//          P = C^n by binary powering of C = G (I + tau A/2), G the inverse.  The
//          powering multiplies the rounding of C by n, so what is held is
//          E = C - I = G tau A, whose rounding is relative to the step:
//          (I + X)(I + Y) = I + (X + Y + X Y).  I is added at the end, or once
//          every mode has decayed below one half (the diagonal of E below -1/2:
//          the sum is exact there, and what has decayed keeps its own relative
//          rounding).  With a strong coupling (tau beta > 1/8) E is no smaller
//          than C and its products cancel: C = 2 G - I itself is held then, after
//          one step of refinement.  Relative error of an FP64 diffusion at 24^2
//          and 96^2, T = 2, beta = 1, 200 steps, N = 4 .. 64: 0.7e-14 .. 2.4e-14 with the
//          scalar build, 0.4e-15 .. 1.9e-15 here (powering 2 G - I: up to 5.5e-14).
//   EXACT: P = e^{T A} by scaling and squaring of a degree-16 Taylor sum.
typedef double mf64x4 __attribute__((ext_vector_type(4)));

template <int TILES>
struct RegMat {
    mf64x4 t[TILES][TILES];
    __device__ __forceinline__ void zero() {
#pragma unroll
        for (int a = 0; a < TILES; ++a)
#pragma unroll
            for (int b = 0; b < TILES; ++b) t[a][b] = mf64x4{0.0, 0.0, 0.0, 0.0};
    }
};

// Out of the accumulators.  A v_mfma_f64_16x16x4 (16 passes) may be read 19 wait
// states after its issue.  Left to itself the compiler puts that wait in front of
// the first read, and where a loop's branch lies between the two it counted too
// little: in the squaring loop of the powering, on the way round that skips the
// multiplication, it read the last register 6 states after the MFMA that writes
// it (element 3 came back stale from the second squaring on).  So the wait stands
// here, on the accumulators themselves, and so do the reads, which the compiler
// would otherwise give a wait of their own; the last two states are those that an
// MFMA needs after a vector instruction has written its operand.
template <int TILES>
__device__ __forceinline__ void accumulators_out(RegMat<TILES>& D) {
    typedef int i32x8 __attribute__((ext_vector_type(8)));
    if constexpr (TILES == 1)
        asm volatile("s_nop 15\n\ts_nop 2" : "+a"(D.t[0][0]));
    else
        asm volatile("s_nop 15\n\ts_nop 2"
                     : "+a"(D.t[0][0]), "+a"(D.t[0][1]), "+a"(D.t[1][0]), "+a"(D.t[1][1]));
#pragma unroll
    for (int a = 0; a < TILES; ++a)
#pragma unroll
        for (int b = 0; b < TILES; ++b) {
            const i32x8 x = __builtin_bit_cast(i32x8, D.t[a][b]);
            int y0, y1, y2, y3, y4, y5, y6, y7;
            asm volatile("v_accvgpr_read_b32 %0, %8\n\tv_accvgpr_read_b32 %1, %9\n\t"
                         "v_accvgpr_read_b32 %2, %10\n\tv_accvgpr_read_b32 %3, %11\n\t"
                         "v_accvgpr_read_b32 %4, %12\n\tv_accvgpr_read_b32 %5, %13\n\t"
                         "v_accvgpr_read_b32 %6, %14\n\tv_accvgpr_read_b32 %7, %15\n\ts_nop 1"
                         : "=&v"(y0), "=&v"(y1), "=&v"(y2), "=&v"(y3), "=&v"(y4), "=&v"(y5), "=&v"(y6), "=&v"(y7)
                         : "a"(x[0]), "a"(x[1]), "a"(x[2]), "a"(x[3]), "a"(x[4]), "a"(x[5]), "a"(x[6]), "a"(x[7]));
            D.t[a][b] = __builtin_bit_cast(mf64x4, i32x8{y0, y1, y2, y3, y4, y5, y6, y7});
        }
}

// D = X Y, X symmetric.
template <int TILES>
__device__ __forceinline__ RegMat<TILES> reg_mul(const RegMat<TILES>& X, const RegMat<TILES>& Y) {
    RegMat<TILES> D;
    D.zero();
#pragma unroll
    for (int c = 0; c < TILES; ++c)
#pragma unroll
        for (int kk = 0; kk < 4; ++kk)
#pragma unroll
            for (int a = 0; a < TILES; ++a)
#pragma unroll
                for (int b = 0; b < TILES; ++b)
                    D.t[a][b] = __builtin_amdgcn_mfma_f64_16x16x4f64(X.t[c][a][kk], Y.t[c][b][kk], D.t[a][b], 0, 0, 0);
    accumulators_out<TILES>(D);
    return D;
}

// X, Y symmetric: X Y + less (X + Y) and X X + 2 less X, with less = 1 the
// products of I + X and I + Y less I.
template <int TILES>
__device__ __forceinline__ RegMat<TILES> reg_mul_add(const RegMat<TILES>& X, const RegMat<TILES>& Y, double less) {
    RegMat<TILES> D = reg_mul<TILES>(X, Y);
#pragma unroll
    for (int a = 0; a < TILES; ++a)
#pragma unroll
        for (int b = 0; b < TILES; ++b)
#pragma unroll
            for (int kk = 0; kk < 4; ++kk) D.t[a][b][kk] += less * (X.t[a][b][kk] + Y.t[a][b][kk]);
    return D;
}
template <int TILES>
__device__ __forceinline__ RegMat<TILES> reg_square_add(const RegMat<TILES>& X, double less) {
    RegMat<TILES> D = reg_mul<TILES>(X, X);
#pragma unroll
    for (int a = 0; a < TILES; ++a)
#pragma unroll
        for (int b = 0; b < TILES; ++b)
#pragma unroll
            for (int kk = 0; kk < 4; ++kk) D.t[a][b][kk] += 2.0 * less * X.t[a][b][kk];
    return D;
}

template <class R, int TILES>
__global__ __launch_bounds__(64) void k_precompute_mfma(R* __restrict__ Ptab, int M, int N, int Q, int FS,
                                                        double beta, double T, int nsteps, int scheme, double scale,
                                                        int keep_all, int pair) {
    constexpr int HM = 16 * TILES;  // padded block
    constexpr int LS = HM + 1;      // LDS row stride
    __shared__ double mat[2][HM * LS];
    __shared__ double fac[2][3][HM];  // per block: 1/pivot, eliminated off-diagonal, Sherman-Morrison vector
    __shared__ double spot[HM];
    const int l = threadIdx.x;
    const int nblk = (N & 1) ? 1 : 2;
    const int h = (N & 1) ? N : N / 2;
    int lx, ly;  // the class of this workgroup's slot
    table_slot_class(blockIdx.x, Q, N, lx, ly);
    const double two_pi = 6.283185307179586476925;
    const double sx = sin(two_pi * lx / M);
    const double sy = sin(two_pi * ly / M);
    // the potential pot_j = M (cos e_j s_x + sin e_j s_y)^2, j < h
    if (l < h) {
        const double e = two_pi * l / N;
        const double a = cos(e) * sx + sin(e) * sy;
        spot[l] = (double)M * a * a;
    }
    __syncthreads();
    const int jl = l & 15, q = l >> 4;
    // element (i, j) of tile (a, b), k-step kk, of this lane
    auto row_of = [&](int a, int kk) { return 16 * a + 4 * kk + q; };
    auto col_of = [&](int b) { return 16 * b + jl; };
    // CN: C - I is held first, or C (see above)
    const bool less_one = !((T / nsteps) * beta > 0.125);
    if (scheme == 0) {
        const double tau = T / nsteps;
        const double o = -0.5 * tau * beta;  // off-diagonal of I - tau A / 2
        if (l < nblk) {
            const double cr = l == 0 ? o : -o;  // corners: periodic (p) / antiperiodic (q)
            // Thomas factorisation of Tm (d with d_0 - g, d_{h-1} - cr^2/g) and
            // Tm z = u, u = (g, 0, .., 0, cr)
            double* iden = fac[l][0];
            double* cp = fac[l][1];
            double* z = fac[l][2];
            const double d0 = 1.0 + tau * beta + 0.5 * tau * spot[0];
            const double g = -d0;
            double pc = 0.0, pz = 0.0;
            for (int j = 0; j < h; ++j) {
                double tj = 1.0 + tau * beta + 0.5 * tau * spot[j];
                double u = 0.0;
                if (j == 0) {
                    tj -= g;
                    u += g;
                }
                if (j == h - 1) {
                    tj -= cr * cr / g;
                    u += cr;
                }
                const double id = 1.0 / (tj - o * pc);
                pc = o * id;
                pz = (u - o * pz) * id;
                iden[j] = id;
                cp[j] = pc;
                z[j] = pz;
            }
            for (int j = h - 2; j >= 0; --j) {
                pz = z[j] - cp[j] * pz;
                z[j] = pz;
            }
        }
        __syncthreads();
        const int b = TILES == 1 ? (l >> 4) & 1 : l >> 5;
        const int c = TILES == 1 ? l & 15 : l & 31;
        if (l < 2 * HM && b < nblk && c < h) {
            const double cr = b == 0 ? o : -o;
            const double g = -(1.0 + tau * beta + 0.5 * tau * spot[0]);
            const double* iden = fac[b][0];
            const double* cp = fac[b][1];
            const double* z = fac[b][2];
            double* w = mat[b] + c;
            const double den = 1.0 + z[0] + (cr / g) * z[h - 1];
            double p = 0.0;
            for (int j = 0; j < h; ++j) {
                p = ((j == c ? 1.0 : 0.0) - o * p) * iden[j];
                w[j * LS] = p;
            }
            double last = p;
            for (int j = h - 2; j >= 0; --j) {
                p = w[j * LS] - cp[j] * p;
                w[j * LS] = p;
            }
            double f = (p + (cr / g) * last) / den;
            for (int j = 0; j < h; ++j) w[j * LS] -= f * z[j];
            if (!less_one) {
                // C = 2 (I - tau A/2)^{-1} - I, and one step of refinement: the
                // correction solves (I - tau A/2) x = (I + tau A/2) e_c less
                // (I - tau A/2) C e_c
                for (int j = 0; j < h; ++j) w[j * LS] = 2.0 * w[j * LS] - (j == c ? 1.0 : 0.0);
                double y[HM];
                p = 0.0;
#pragma unroll
                for (int j = 0; j < HM; ++j)
                    if (j < h) {
                        const int jm = j >= 1 ? j - 1 : h - 1, jp = j + 1 < h ? j + 1 : 0;
                        const double om = j >= 1 ? o : cr, op = j + 1 < h ? o : cr;
                        const double d = tau * beta + 0.5 * tau * spot[j];
                        double r = (j == c ? 1.0 - d : 0.0) - (1.0 + d) * w[j * LS];
                        r -= om * ((jm == c ? 1.0 : 0.0) + w[jm * LS]);
                        r -= op * ((jp == c ? 1.0 : 0.0) + w[jp * LS]);
                        p = (r - o * p) * iden[j];
                        y[j] = p;
                        last = p;
                    }
#pragma unroll
                for (int j = HM - 1; j >= 0; --j)
                    if (j < h) {
                        if (j < h - 1) p = y[j] - cp[j] * p;
                        y[j] = p;
                    }
                f = (p + (cr / g) * last) / den;
#pragma unroll
                for (int j = 0; j < HM; ++j)
                    if (j < h) w[j * LS] += y[j] - f * z[j];
            }
        }
        __syncthreads();
    }
    // X = T A / 2^sq with ||X||_inf <= 1/2 (the larger of the blocks' norms; EXACT)
    int sq = 0;
    double xs = 0.0;
    if (scheme != 0) {
        double nrm = 0.0;
        for (int i = 0; i < h; ++i)  // row sums: |diagonal| plus at most 2 beta off the diagonal
            nrm = fmax(nrm, fabs(-2.0 * beta - spot[i]) + 2.0 * beta);
        nrm *= T;
        while (nrm > 0.5) {
            nrm *= 0.5;
            ++sq;
        }
        xs = T * ldexp(1.0, -sq);
    }
    for (int blk = 0; blk < nblk; ++blk) {
        RegMat<TILES> X, P;
        const double wrap = blk == 0 ? 1.0 : -1.0;
#pragma unroll
        for (int a = 0; a < TILES; ++a)
#pragma unroll
            for (int b = 0; b < TILES; ++b)
#pragma unroll
                for (int kk = 0; kk < 4; ++kk) {
                    const int i = row_of(a, kk), j = col_of(b);
                    double v = 0.0;
                    if (i < h && j < h) {
                        if (scheme == 0) {
                            const double* Gi = mat[blk] + i * LS;
                            v = Gi[j];
                            if (less_one) {
                                const double tau = T / nsteps;
                                const double up = j + 1 < h ? Gi[j + 1] : wrap * Gi[0], dn = j >= 1 ? Gi[j - 1] : wrap * Gi[h - 1];
                                v = tau * beta * (up + dn - 2.0 * v) - tau * spot[j] * v;
                            }
                        } else {
                            if (i == j) v = -2.0 * beta - spot[i];
                            if (j == (i + 1 < h ? i + 1 : 0)) v += (i + 1 < h) ? beta : wrap * beta;
                            if (j == (i >= 1 ? i - 1 : h - 1)) v += (i >= 1) ? beta : wrap * beta;
                            v *= xs;
                        }
                    }
                    X.t[a][b][kk] = v;
                }
        if (scheme == 0) {
            // binary powering from the lowest set bit of n on; the matrices held
            // are the propagators less `less` I
            double less = less_one ? 1.0 : 0.0;
            auto add_identity = [&](RegMat<TILES>& E) {
#pragma unroll
                for (int a = 0; a < TILES; ++a)
#pragma unroll
                    for (int kk = 0; kk < 4; ++kk)
                        if (row_of(a, kk) == col_of(a) && row_of(a, kk) < h) E.t[a][a][kk] += 1.0;
            };
            // every mode of X has decayed
            auto decayed = [&]() {
                bool slow = false;
#pragma unroll
                for (int a = 0; a < TILES; ++a)
#pragma unroll
                    for (int kk = 0; kk < 4; ++kk)
                        slow |= row_of(a, kk) == col_of(a) && row_of(a, kk) < h && !(X.t[a][a][kk] < -0.5);
                return less != 0.0 && !__any(slow);
            };
            if (decayed()) {
                add_identity(X);
                less = 0.0;
            }
            int n = nsteps;
            while ((n & 1) == 0) {
                X = reg_square_add<TILES>(X, less);
                n >>= 1;
                if (decayed()) {
                    add_identity(X);
                    less = 0.0;
                }
            }
            P = X;
            for (n >>= 1; n > 0; n >>= 1) {
                X = reg_square_add<TILES>(X, less);
                if (decayed()) {
                    add_identity(X);
                    add_identity(P);
                    less = 0.0;
                }
                if (n & 1) P = reg_mul_add<TILES>(X, P, less);
            }
            if (less != 0.0) add_identity(P);
        } else {
            auto plus_identity = [&](RegMat<TILES>& E, double s) {
#pragma unroll
                for (int a = 0; a < TILES; ++a)
#pragma unroll
                    for (int b = 0; b < TILES; ++b)
#pragma unroll
                        for (int kk = 0; kk < 4; ++kk)
                            E.t[a][b][kk] = s * E.t[a][b][kk] + (row_of(a, kk) == col_of(b) ? 1.0 : 0.0);
            };
            // Horner: E = I + X (I + X/2 (I + X/3 (... (I + X/16))))
            P = X;
            plus_identity(P, 1.0 / 16.0);
            for (int k = 15; k >= 1; --k) {
                P = reg_mul<TILES>(X, P);
                plus_identity(P, 1.0 / k);
            }
            for (int s2 = 0; s2 < sq; ++s2) P = reg_mul<TILES>(P, P);
        }
#pragma unroll
        for (int a = 0; a < TILES; ++a)
#pragma unroll
            for (int b = 0; b < TILES; ++b)
#pragma unroll
                for (int kk = 0; kk < 4; ++kk) mat[blk][row_of(a, kk) * LS + col_of(b)] = P.t[a][b][kk];
    }
    __syncthreads();
    // packed upper triangles of the blocks, symmetrised, scaled, stored as R
    const int Eh = h * (h + 1) / 2;
    const int CS = table_class_stride(N, (int)sizeof(R));
    R* dst = Ptab + (size_t)blockIdx.x * CS;
    const float inv_h = 1.0f / (float)h;
    double pmax = 0.0;
    for (int b = 0; b < nblk; ++b) {
        auto at = [&](int i, int j) { return 0.5 * (mat[b][i * LS + j] + mat[b][j * LS + i]); };
        for (int e = l; e < h * h; e += 64) {
            const int i = fdiv(e, inv_h), j = e - i * h;
            if (j >= i) {
                const double u = at(i, j);
                pmax = fmax(pmax, fabs(u));
                if (!pair) dst[b * Eh + i * h - i * (i - 1) / 2 + (j - i)] = (R)(u * scale);
            }
        }
        if (pair) store_pair_block<R>(Ptab, M, N, pair == 2, b, lx, ly, h, scale, l, at);
    }
    for (int off = 32; off >= 1; off >>= 1) pmax = fmax(pmax, __shfl_xor(pmax, off, 64));
    store_class_flags<R>(Ptab, M, N, Q, FS, lx, ly, !keep_all && pmax < (sizeof(R) == 4 ? 0x1p-30 : 0x1p-60), l, pair);
    if (!pair)
        for (int e = nblk * Eh + l; e < CS; e += 64) dst[e] = R(0);
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

template <class R>
hipError_t launch_precompute(R* Ptab, int M, int N, double beta, double T, int nsteps, int scheme,
                             hipStream_t st, bool keep_all, int pair) {
    const int Q = M / 4 + 1;
    const size_t slots = table_slots(M, N);  // one workgroup per stored class
    const int h = (N & 1) ? N : N / 2;
    const size_t lds = (size_t)(4 * h * h + h) * sizeof(double);
    // the inverse FFT's 1/M^2, and for even N the 1/2 of the p/q recombination
    const double scale = ((N & 1) ? 1.0 : 0.5) / ((double)M * (double)M);
    // Matrix cores for blocks of at most 32, except where many classes of the
    // smallest blocks, padded to 16, make the products the bound: 200 steps of
    // N = 4 / 6 / 8 / 10, matrix cores against scalar, 256^2 19.3 / 27.9 / 21.0 / 29.5
    // against 19.7 / 26.0 / 23.7 / 31.9 us, 384^2 28.5 / 48.6 / 30.2 / 50.7 against 25.2 /
    // 42.2 / 30.3 / 50.7, 1024^2 138 / 261 / 143 / 275 against 107 / 211 / 128 / 257; N = 5 as
    // N = 6; N = 7 and 9 (one block of N) 193 and 201 against 203 and 323 at 1024^2.
    // SE2N_SCALAR_PRECOMPUTE forces the scalar build, which odd N above 32 keeps.
    const bool small = N <= 6 ? M >= 384 : !(N & 1) && N <= 10 && M >= 768;
    if (h <= 32 && !small && std::getenv("SE2N_SCALAR_PRECOMPUTE") == nullptr) {
        if (h <= 16)
            hipLaunchKernelGGL((k_precompute_mfma<R, 1>), dim3((unsigned)slots), dim3(64), 0, st, Ptab, M, N, Q,
                               flag_stride(M), beta, T, nsteps, scheme, scale, keep_all ? 1 : 0, pair);
        else
            hipLaunchKernelGGL((k_precompute_mfma<R, 2>), dim3((unsigned)slots), dim3(64), 0, st, Ptab, M, N, Q,
                               flag_stride(M), beta, T, nsteps, scheme, scale, keep_all ? 1 : 0, pair);
        return hipGetLastError();
    }
    hipLaunchKernelGGL((k_precompute<R>), dim3((unsigned)slots), dim3(64), lds, st, Ptab, M, N, Q,
                       flag_stride(M), beta,
                       T, nsteps, scheme, scale, keep_all ? 1 : 0, pair);
    return hipGetLastError();
}

#define SE2N_INSTANTIATE(R)                                                                             \
    template hipError_t launch_row_fwd<R>(int, const R*, const uint8_t*, const uint8_t*, const R*,     \
                                          C2<R>*, int, int, const LaunchGeom&, const FftPlan&,         \
                                          const C2<R>*, hipStream_t);                                  \
    template hipError_t launch_col_fft<R>(bool, C2<R>*, long, int, const LaunchGeom&, const FftPlan&,  \
                                          const C2<R>*, hipStream_t, const uint8_t*);                  \
    template hipError_t launch_col_orient<R>(C2<R>*, int, const LaunchGeom&, const FftPlan&,           \
                                             const C2<R>*, double, hipStream_t);                       \
    template hipError_t launch_row_inv<R>(int, const C2<R>*, R*, typename Enc<R>::U*, uint8_t*, int,   \
                                          int, int, R, const LaunchGeom&, int, const FftPlan&,         \
                                          const C2<R>*, hipStream_t, bool, bool);                            \
    template hipError_t launch_col_inv_paired<R>(C2<R>*, int, int, const LaunchGeom&, const FftPlan&,  \
                                                 const C2<R>*, hipStream_t, const uint8_t*, C2<R>*);   \
    template bool row_blocked<R>(int, const LaunchGeom&);                                              \
    template bool col_inv_masks<R>(int, const LaunchGeom&);                                            \
    template hipError_t launch_fill_enc<R>(typename Enc<R>::U*, long, hipStream_t);                    \
    template hipError_t launch_decode_enc<R>(const typename Enc<R>::U*, R*, long, hipStream_t);        \
    template hipError_t launch_lift<R>(const R*, const uint8_t*, const uint8_t*, R*, int, int,         \
                                       hipStream_t);                                                   \
    template hipError_t launch_project<R>(const R*, R*, int, int, bool, hipStream_t);                  \
    template hipError_t launch_precompute<R>(R*, int, int, double, double, int, int, hipStream_t, bool, int);

SE2N_INSTANTIATE(float)
SE2N_INSTANTIATE(double)

}  // namespace se2n
