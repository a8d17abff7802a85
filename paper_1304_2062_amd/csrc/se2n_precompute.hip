// Propagator builds (FP64): one wavefront per stored frequency class, on the
// matrix cores or with scalar products in LDS.  A file of its own, because a
// program's first launch from a file loads all of that file's code, and plans on
// the pair path take nothing else from the five passes: a program's first 512^2,
// N = 30 inpaint 19.6 -> 10.3 ms, first batch of 64 images 39.3 -> 29.4 ms.
#include <hip/hip_runtime.h>

#include <cstdint>
#include <cstdlib>

#include "se2n_internal.hpp"
#include "se2n_pair.hpp"

namespace se2n {

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
template hipError_t launch_precompute<float>(float*, int, int, double, double, int, int, hipStream_t, bool, int);
template hipError_t launch_precompute<double>(double*, int, int, double, double, int, int, hipStream_t, bool, int);

}  // namespace se2n
