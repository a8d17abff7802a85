// The pair path: one diffusion in three kernels instead of five, for every
// plan whose columns fit in LDS (pair_fits).
//
// The orientation slices are carried as N real images that pair up for the
// row transforms.  With even N = 2h pair t holds
//     p_t = x_t + x_{t+h}   and   q_t = x_t - x_{t+h},
// the basis in which every per-mode system splits into two h x h blocks (the
// potential has period h in the orientation); with odd N it holds the slices
// 2t and 2t + 1 (the last pair only 2t).  Row y of a pair is transformed as
// one complex sequence z = a + i b of length M, whose two half spectra come
// apart by additions alone:
//     A[k] = (Z[k] + conj Z[M-k]) / 2,   B[k] = (Z[k] - conj Z[M-k]) / (2i).
// Stored spectrum: rows y in blocks of rb (PairLay), within a block slice
// after slice, s = 2t (a) and 2t + 1 (b), within a slice the columns kx in
// [0, M/2), each holding its rb rows contiguously; rb = M is spec[s][kx][y].  A row's entries 0 and M/2 are real; column 0 holds
// both, A[0] + i A[M/2]: the two columns belong to the same frequency
// classes, so their packed column evolves by the same real propagators.
//
//   row pass, forward   lift (or a real volume) -> row FFTs -> spec
//   middle              per column kx and block (the h slices p, or the h
//                       slices q, or all N of odd N): column FFT, the per-mode
//                       products, inverse column FFT, all in LDS: the spectrum
//                       is read and written once
//   row pass, inverse   row FFTs -> x_t = p + q, x_{t+h} = p - q: maximum
//                       (p + |q| per pair), mean, real volume, or the
//                       restoration's mix followed by the forward row pass
#pragma once

#include <hip/hip_runtime.h>

#include <cstdint>

#include "se2n_fft.hpp"
#include "se2n_internal.hpp"
#include "se2n_passes.hpp"

namespace se2n {

// ---------------------------------------------------------------------------
// Geometry, shared by the host and the kernels
// ---------------------------------------------------------------------------
constexpr int kPairLds = 160 * 1024;

// Slices of one block of the middle pass, and the blocks of a column.
__host__ __device__ constexpr int pair_hs(int N) { return (N & 1) ? N : N / 2; }
__host__ __device__ constexpr int pair_nblk(int N) { return (N & 1) ? 1 : 2; }
__host__ __device__ constexpr int pair_count(int N) { return (N + 1) / 2; }
// LDS complex elements from one transform to the next: padded length, and two
// more so that equal positions of neighbouring transforms fall in other banks.
__host__ __device__ constexpr int pair_stride(int M) { return M + M / 32 + 2; }
__host__ __device__ constexpr int pair_buf_elems(int M, int ntrans) {
    const int a = ntrans * pair_stride(M), b = lds_padded_size(ntrans * (M + 2));
    return a > b ? a : b;
}
// The LDS twiddle table holds w_M^m, m < 3M/4: no stage reads beyond (radix R
// reads at most the exponents below (R - 4)/R of the period for R = 16, half
// of it for 8, 4 and 2, two thirds for 3).
__host__ __device__ constexpr int pair_tw_elems(int M) { return (tw_pos(3 * (M / 4) - 1) + 1 + 7) & ~7; }
__host__ __device__ constexpr size_t pair_lds_bytes(int M, int ntrans, int rsize) {
    return ((size_t)pair_tw_elems(M) + pair_buf_elems(M, ntrans)) * 2 * (size_t)rsize;
}


// Threads of a workgroup at most: FP64 kernels are bounded to 512, for 256
// registers each.
__host__ __device__ constexpr int pair_max_threads(int rsize) { return rsize == 4 ? 1024 : 512; }

// Middle pass: elements per thread, and threads: M/4 class positions times
// the row groups of the per-mode product (ept / 4 rows of the four modes of a
// class, see pair_solve).  8 elements, and twice the threads, up to 5120
// elements in FP32: over the plans of 4096 .. 5120 elements 1.03 .. 1.20 times as
// fast as 16 on runtime radices (324^2, N = 15 33.6 -> 28.1 us), 0.99 .. 1.13 on compiled
// sides (768^2, N = 12 28.5 -> 25.7).  Above, compiled sides from 256 on lose (768^2,
// N = 16 32.3 against 35.3 us), 128, 192 and runtime radices still gain up to 5800 and
// lose beyond (648^2, N = 18 57 against 72).  A side of 1024, which takes three stages
// with 16 and four with 8: N = 10 30.7 against 33.4 us.
__host__ __device__ constexpr int pair_mid_ept(int M, int hs, int rsize) {
    const int elems = hs * M;
    return elems <= 1024 ? 4 : elems <= (rsize == 4 && M < 1024 ? 5120 : 4096) ? 8 : 16;
}
__host__ __device__ constexpr int pair_mid_threads(int M, int hs, int rsize) {
    const int rpt = pair_mid_ept(M, hs, rsize) / 4;
    return (M / 4 * ((hs + rpt - 1) / rpt) + 63) / 64 * 64;
}

// The propagator table of the pair path: element-major, so that the lanes of
// consecutive classes ly read consecutive entries:
//     T[((lx nblk + blk) Eh + e) QP + ly],  Eh = hs (hs + 1) / 2,
// e over the packed upper triangle of the block, every class stored (no slot
// is shared), ly padded to QP.  The flags of negligible classes follow.
// With halved columns (PairLay) the even classes come first, then the odd ones.
__host__ __device__ constexpr int pair_qp(int M, bool halved) {
    return (M / 4 + 1 + 15) / 16 * 16 + (halved ? 16 : 0);
}
__host__ __device__ constexpr int pair_odd_pos(int M) { return (M / 8 + 1 + 15) / 16 * 16; }
__host__ __device__ constexpr int pair_class_pos(int M, bool halved, int ly) {
    return halved ? (ly >> 1) + ((ly & 1) ? pair_odd_pos(M) : 0) : ly;
}
__host__ __device__ constexpr size_t pair_table_entries(int M, int N, bool halved) {
    return (size_t)(M / 4 + 1) * table_class_entries(N) * pair_qp(M, halved);
}
__host__ __device__ constexpr size_t pair_table_bytes(int M, int N, int rsize, bool halved) {
    return pair_table_entries(M, N, halved) * (size_t)rsize + (size_t)(M / 4 + 1) * flag_stride(M) + 64;
}

// Whether a side and orientation count run on the pair path: a block of a
// column fits in the LDS of one workgroup, at most 16 elements per thread.
__host__ __device__ constexpr bool pair_block_fits(int M, int N, int rsize) {
    const int hs = pair_hs(N);
    return hs * M <= 16 * pair_max_threads(rsize) && pair_mid_threads(M, hs, rsize) <= pair_max_threads(rsize) &&
           pair_lds_bytes(M, hs, rsize) <= (size_t)kPairLds;
}
__host__ __device__ constexpr bool pair_fits(int M, int N, int rsize) {
    return M <= 1024 && pair_block_fits(M, N, rsize);
}
// Or half a column does: the row passes take the columns' first radix-2 step
// (PairLay).  FP64 on the sides with compiled transforms, 1024^2, N = 32 751
// -> 478 us against the five passes, 512^2, N = 40 308 -> 184 us, 768^2,
// N = 30 439 -> 303 us, 384^2, N = 44 212 -> 154 us, 2048^2, N = 16 1500 ->
// 1010 us.  Not FP32: its five passes run at the memory's rate
// (1024^2, N = 48 381 against 450 us this way, 2048^2, N = 32 755 against 1080).
__host__ __device__ constexpr bool pair_halves(int M, int N, int rsize) {
    return rsize == 8 && (M == 384 || M == 512 || M == 768 || M == 1024 || M == 2048) && !pair_fits(M, N, rsize) &&
           pair_block_fits(M / 2, N, rsize);
}

// ---------------------------------------------------------------------------
// Radix 16: one butterfly fills the 16 elements a thread stages, which takes
// 1024 = 16 8 8 in three stages instead of 8 8 4 4 in four
// ---------------------------------------------------------------------------
template <class R, bool INV>
__device__ __forceinline__ void dft16(C2<R>* v) {
    const R c1 = R(0.92387953251128675613), s1 = R(0.38268343236508977173), q = R(0.70710678118654752440);
    // w_16^m (conjugated for the inverse) times z
    auto rot = [&](C2<R> z, R c, R s) {
        return INV ? cmk<R>(c * z.x - s * z.y, c * z.y + s * z.x) : cmk<R>(c * z.x + s * z.y, c * z.y - s * z.x);
    };
    C2<R> a[4][4];
#pragma unroll
    for (int n = 0; n < 4; ++n) {
        C2<R> t[4] = {v[n], v[n + 4], v[n + 8], v[n + 12]};
        dft4<R, INV>(t);
#pragma unroll
        for (int k = 0; k < 4; ++k) a[n][k] = t[k];
    }
    // a[n][k] times w_16^{n k}
    a[1][1] = rot(a[1][1], c1, s1);
    a[1][2] = rot(a[1][2], q, q);
    a[1][3] = rot(a[1][3], s1, c1);
    a[2][1] = rot(a[2][1], q, q);
    a[2][2] = mul_mi<R, INV>(a[2][2]);
    a[2][3] = rot(a[2][3], -q, q);
    a[3][1] = rot(a[3][1], s1, c1);
    a[3][2] = rot(a[3][2], -q, q);
    a[3][3] = rot(a[3][3], -c1, -s1);
#pragma unroll
    for (int k = 0; k < 4; ++k) {
        C2<R> t[4] = {a[0][k], a[1][k], a[2][k], a[3][k]};
        dft4<R, INV>(t);
#pragma unroll
        for (int m = 0; m < 4; ++m) v[k + 4 * m] = t[m];
    }
}

template <class R, int RADIX, bool INV>
__device__ __forceinline__ void pair_dft(C2<R>* v) {
    if constexpr (RADIX == 16) dft16<R, INV>(v);
    else dft<R, RADIX, INV>(v);
}

// The twiddle table from the quarter table q in memory (callers synchronise).
template <class R>
__device__ __forceinline__ void pair_load_tw(C2<R>* tw, const C2<R>* __restrict__ q, int M, int tid, int nthr) {
    const int M4 = M >> 2;
    for (int m = tid; m < M4; m += nthr) {
        const C2<R> w = q[m];
        tw[tw_pos(m)] = w;
        tw[tw_pos(m + M4)] = cmk<R>(w.y, -w.x);
        tw[tw_pos(m + 2 * M4)] = cmk<R>(-w.x, -w.y);
    }
}

// Whether the transforms that a restoration repeats read every twiddle power.  A
// product of two powers has twice the rounding, and the same twiddles are applied
// at every mesh point, where their rounding adds up: 256^2, N = 30, 200 intervals of
// SR in FP32, error 5.5e-7 with every power read, 9.3e-7 with powers formed from three
// reads (8.0e-7 on the five passes), 5970 against 5958 us; 1024^2, N = 30 and 96^2, N = 30
// 1.13 and 1.1 times the five passes' error without, 1.0 and 0.9 with, within 1 % of
// the time.  In FP64 the error is the same either way (1.1e-15) and the reads cost 2 %.
// At 16 elements per thread the middle pass keeps the products (1024^2, N = 32 inpaint
// 240 -> 270 us), and so do the lift, volume and projecting rows, which meet an image
// once (768^2, N = 24 inpaint 115 -> 135 us).
__host__ __device__ constexpr bool pair_direct(int rsize) { return rsize == 4; }

// Inputs r of a butterfly times w^{r e} (see apply_twiddles); DIRECT: every power
// read.  Radix 16 reads six powers and forms the others by one product each.
template <class R, int RADIX, bool INV, bool DIRECT>
__device__ __forceinline__ void pair_twiddles(C2<R>* v, const C2<R>* tw, int e, int M4) {
    auto rd = [&](int m) {
        C2<R> w = tw[tw_pos(m)];
        if (INV) w.y = -w.y;
        return w;
    };
    if constexpr (RADIX == 16) {
        const C2<R> w1 = rd(e), w2 = rd(2 * e), w3 = rd(3 * e);
        v[1] = cmul<R>(v[1], w1);
        v[2] = cmul<R>(v[2], w2);
        v[3] = cmul<R>(v[3], w3);
#pragma unroll
        for (int g = 4; g < 16; g += 4) {
            const C2<R> wg = rd(g * e);
            v[g] = cmul<R>(v[g], wg);
            v[g + 1] = cmul<R>(v[g + 1], cmul<R>(wg, w1));
            v[g + 2] = cmul<R>(v[g + 2], cmul<R>(wg, w2));
            v[g + 3] = cmul<R>(v[g + 3], cmul<R>(wg, w3));
        }
    } else {
        apply_twiddles<R, RADIX, INV, true, DIRECT>(v, tw, e, M4);
    }
}

// Radix of stage s of a compiled length (0 past the last): 16s where a thread
// stages 16 elements, the factors 8, 4, 2 first, 3s last.
__host__ __device__ constexpr int pair_radix(int L, int EPT, int s) {
    if (EPT < 16) return static_radix(L, s);
    int a = 0, b = 0, m = L;
    while (m % 2 == 0) { m /= 2; ++a; }
    while (m % 3 == 0) { m /= 3; ++b; }
    int rad[16] = {};
    int n = 0;
    // 2^a as 16s, with one 8 (a = 3 mod 4), two 8s (a = 2), 8 8 8 (a = 1, from 9 on) or small factors
    if (a % 4 == 1 && a >= 9) { rad[n++] = 8; rad[n++] = 8; rad[n++] = 8; a -= 9; }
    else if (a % 4 == 1 && a >= 5) { rad[n++] = 8; rad[n++] = 4; a -= 5; }
    else if (a % 4 == 2 && a >= 6) { rad[n++] = 8; rad[n++] = 8; a -= 6; }
    else if (a % 4 == 3) { rad[n++] = 8; a -= 3; }
    else if (a % 4 != 0) { rad[n++] = 1 << (a % 4); a -= a % 4; }
    while (a > 0) { rad[n++] = 16; a -= 4; }
    for (int i = 0; i < b; ++i) rad[n++] = 3;
    return s < n ? rad[s] : 0;
}
__host__ __device__ constexpr int pair_last_radix(int L, int EPT) {
    int s = 0;
    while (pair_radix(L, EPT, s + 1) != 0) ++s;
    return pair_radix(L, EPT, s);
}

// ---------------------------------------------------------------------------
// Layout of the stored spectrum
// ---------------------------------------------------------------------------
// Halved columns: the first radix-2 step of a column's transform, by
// decimation in frequency, belongs to the row passes, which hold rows n and
// n + M/2 together.  With x the column of length M, the even frequencies are
// the transform of length M/2 of x[n] + x[n + M/2] and the odd ones that of
// (x[n] - x[n + M/2]) w_M^n.  A block then holds rb/2 rows n of the even half
// followed by the same rows of the odd half, and the middle pass takes the
// two halves of a column one by one: the classes of a column and of its
// mirror have the same parity.
struct PairLay {
    int rb;      // rows per block: a power of two, or M
    int lg;      // log2(rb), or 16 for rb = M (one block); of rb/2 with halved columns
    int halved;  // columns in halves
    // elements from one block to the next
    __host__ __device__ long block(int H, int N) const { return (long)N * H * rb; }
    // offset of row y (of row n of the even half) within the slice-and-column
    // grid of its block
    __host__ __device__ long row(int y, int H, int N) const {
        return (long)(y >> lg) * block(H, N) + (y - ((y >> lg) << lg));
    }
    // offset of column kx of slice s
    __host__ __device__ long col(int s, int kx, int H) const { return ((long)s * H + kx) * rb; }
};

// ---------------------------------------------------------------------------
// Transforms of a runtime number of sequences of a compiled length
// ---------------------------------------------------------------------------
// One Stockham stage over nt transforms of length L: in(t, j, v) fetches the
// inputs j + r L/RADIX of butterfly j of transform t, out(t, o, v, i) takes its
// outputs o + r NS (i: the thread's i-th butterfly).  `fence`: a barrier between the two, for stages that read
// and write the same LDS buffer.  nt L <= EPT nthr.
template <class R, int RADIX, bool INV, int L, int NS, int EPT, bool DIRECT, class In, class Out>
__device__ __forceinline__ void pair_stage(const C2<R>* tw, int nt, int tid, int nthr, In&& in, Out&& out,
                                           bool fence) {
    constexpr int NB = L / RADIX;
    constexpr int MAXB = (EPT + RADIX - 1) / RADIX;
    constexpr int TWSTEP = L / (NS * RADIX);
    const int total = NB * nt;
    C2<R> v[MAXB][RADIX];
#pragma unroll
    for (int i = 0; i < MAXB; ++i) {
        const int b = tid + i * nthr;
        if (b < total) {
            const int t = b / NB;
            in(t, b - t * NB, v[i]);
        }
    }
    if (fence) __syncthreads();
#pragma unroll
    for (int i = 0; i < MAXB; ++i) {
        const int b = tid + i * nthr;
        if (b < total) {
            const int t = b / NB;
            const int j = b - t * NB;
            const int q = j / NS;
            const int k = j - q * NS;
            if (NS > 1) pair_twiddles<R, RADIX, INV, DIRECT>(v[i], tw, k * TWSTEP, L / 4);
            pair_dft<R, RADIX, INV>(v[i]);
            out(t, q * NS * RADIX + k, v[i], i);
        }
    }
}

// Position i of transform t in LDS (the stages of a runtime length pad the
// whole buffer, those of a compiled one each transform).
template <int MS>
__device__ __forceinline__ int pair_pos(int M, int t, int i) {
    return MS ? t * pair_stride(MS) + lds_pad(i) : lds_pad(t * (M + 2) + i);
}

// Stages S .. of the transforms held in buf.  `first(t, j, v)` replaces the
// LDS read of stage 0 (Identity: read LDS), `last(t, o, v, i)` the LDS
// write of the last stage (Identity: write LDS).  Ends with a barrier exactly
// when the result is in LDS.
struct PairLds {};
template <class R, bool INV, int L, int EPT, int S, int NS, bool DIRECT, class First, class Last>
__device__ __forceinline__ void pair_fft_from(C2<R>* buf, const C2<R>* tw, int nt, int tid, int nthr, First&& first,
                                              Last&& last) {
    constexpr int RADIX = pair_radix(L, EPT, S);
    if constexpr (RADIX != 0) {
        constexpr int NB = L / RADIX;
        constexpr bool LASTST = pair_radix(L, EPT, S + 1) == 0;
        constexpr bool IN_LDS = S > 0 || std::is_same<typename std::decay<First>::type, PairLds>::value;
        constexpr bool OUT_LDS = !LASTST || std::is_same<typename std::decay<Last>::type, PairLds>::value;
        auto in = [&](int t, int j, C2<R>* v) {
            if constexpr (IN_LDS) {
                const C2<R>* pa = buf + t * pair_stride(L);
                if constexpr (pad_linear_read(NB)) {
                    pa += lds_pad(j);
#pragma unroll
                    for (int r = 0; r < RADIX; ++r) v[r] = pa[pad_offset(r, NB)];
                } else {
#pragma unroll
                    for (int r = 0; r < RADIX; ++r) v[r] = pa[lds_pad(j + r * NB)];
                }
            } else {
                first(t, j, v);
            }
        };
        auto out = [&](int t, int o, C2<R>* v, int i) {
            if constexpr (OUT_LDS) {
                C2<R>* pb = buf + t * pair_stride(L);
                if constexpr (pad_linear_write(NS, RADIX, 32)) {
                    pb += lds_pad(o);
#pragma unroll
                    for (int r = 0; r < RADIX; ++r) pb[pad_offset(r, NS)] = v[r];
                } else {
#pragma unroll
                    for (int r = 0; r < RADIX; ++r) pb[lds_pad(o + r * NS)] = v[r];
                }
            } else {
                last(t, o, v, i);
            }
        };
        pair_stage<R, RADIX, INV, L, NS, EPT, DIRECT>(tw, nt, tid, nthr, in, out, IN_LDS);
        if constexpr (OUT_LDS) __syncthreads();
        pair_fft_from<R, INV, L, EPT, S + 1, NS * RADIX, DIRECT>(buf, tw, nt, tid, nthr, first, last);
    }
}

// Transforms of nt sequences in LDS, in place (compiled length MS, or the
// runtime plan).
template <class R, bool INV, int MS, int EPT, bool DIRECT>
__device__ __forceinline__ void pair_fft(C2<R>* buf, const C2<R>* tw, int M, int nt, const FftPlan& plan, int tid,
                                         int nthr) {
    if constexpr (MS != 0) {
        pair_fft_from<R, INV, MS, EPT, 0, 1, DIRECT>(buf, tw, nt, tid, nthr, PairLds{}, PairLds{});
    } else {
        fft_lds<R, INV, EPT, true, DIRECT>(buf, plan, nt, M + 2, tw, M >> 2, tid, nthr);
    }
}

// ---------------------------------------------------------------------------
// Middle pass: column kx, block blk
// ---------------------------------------------------------------------------
// Per-mode products on the column spectra in LDS, slice t at pair_pos(t, ky).
// Class v holds the modes ky = v, M/2 - v and, where s_ky < 0, M/2 + v and
// M - v; at the latter two the propagator is the class one conjugated by
// r -> -r: slices j -> -j (mod hs), and in the block q the sign of slice 0
// turns (the common sign of the others cancels).  A thread takes RPT rows of
// the four modes of a class and walks the columns j: four vector entries from
// LDS and RPT propagator entries from memory (lanes are consecutive classes,
// so an entry's loads are consecutive words) for 8 RPT multiply-adds.  With
// RPT = 4 that is 1 byte of LDS and 1/2 byte of vector memory per
// multiply-add, both about half of what a compute unit delivers beside its
// 64 multiply-adds a cycle; whole rows of two modes with the vectors in
// registers read 1 byte per multiply-add and were bound by it (1024^2, N = 32:
// 64 us of the pass, 28 us this way).  Classes 0 and M/4 have two modes each
// and share the position v = 0.  Negligible classes give zeros unread.
//
// HALF: M is the length of the half columns of parity `par`, whose position k
// is the mode 2k + par of the column: the even half looks like a column of
// side M, in the odd half class 2v + 1 holds k = v, M/2 + v, M/2 - 1 - v and
// M - 1 - v.
template <class R, int RPT, int MS, bool HALF = false>
__device__ __forceinline__ void pair_solve(C2<R>* buf, const R* __restrict__ T, const uint8_t* __restrict__ flags,
                                           int M_, int N, int kx, int blk, int tid, int par = 0) {
    const int M = MS ? MS : M_;
    const int H = M >> 1, M4 = M >> 2;
    const int hs = pair_hs(N);
    const int Eh = hs * (hs + 1) / 2;
    const int MF = HALF ? 2 * M : M;  // the side
    const int QP = pair_qp(MF, HALF);
    const int lx = kx <= MF / 4 ? kx : MF / 2 - kx;
    const R* __restrict__ Tb =
        T + (size_t)(lx * pair_nblk(N) + blk) * Eh * QP + (HALF && par ? pair_odd_pos(MF) : 0);
    const uint8_t* __restrict__ fl = flags + (size_t)lx * flag_stride(MF);
    const bool odd_half = HALF && par;
    const bool flip0 = blk == 1;

    int part = tid / M4;
    const int v = tid - part * M4;
    if (MS != 0 && (MS / 4) % 64 == 0) part = __builtin_amdgcn_readfirstlane(part);
    const int i0 = part * RPT;
    const bool act = i0 < hs;
    // modes 0, 1: class v; modes 2, 3: class v again, or M/4 at v = 0
    const int lb = v == 0 && !odd_half ? M4 : v;
    const int down = odd_half ? v + 1 : lb;
    const int ky[4] = {v, H + v, H - down, v == 0 && !odd_half ? H + M4 : M - down};
    const bool live0 = act && !fl[HALF ? 2 * v + par : v], live1 = act && !fl[HALF ? 2 * lb + par : lb];
    C2<R> y[4][RPT];
#pragma unroll
    for (int m = 0; m < 4; ++m)
#pragma unroll
        for (int r = 0; r < RPT; ++r) y[m][r] = cmk<R>(R(0), R(0));
    auto slot = [&](bool mir, int j, int k) { return pair_pos<MS>(M, mir && j > 0 ? hs - j : j, k); };
    auto walk = [&](auto two) {
        constexpr bool TWO = decltype(two)::value;  // the lanes' second class differs from the first
        // entry (i, j) of the packed upper triangle, walked along j: below
        // the diagonal it is (j, i), one row down per step
        int off[RPT];
#pragma unroll
        for (int r = 0; r < RPT; ++r) off[r] = min(i0 + r, hs - 1);
#pragma unroll 2
        for (int j = 0; j < hs; ++j) {
            R w0[RPT], w1[RPT];
#pragma unroll
            for (int r = 0; r < RPT; ++r) {
                const R* p = Tb + (size_t)off[r] * QP;
                w0[r] = p[v];
                w1[r] = TWO ? p[lb] : w0[r];
                off[r] += j >= min(i0 + r, hs - 1) ? 1 : hs - 1 - j;
            }
            C2<R> x[4];
#pragma unroll
            for (int m = 0; m < 4; ++m) {
                x[m] = buf[slot(m & 1, j, ky[m])];
                if ((m & 1) && flip0 && j == 0) x[m] = cmk<R>(-x[m].x, -x[m].y);
            }
#pragma unroll
            for (int r = 0; r < RPT; ++r)
#pragma unroll
                for (int m = 0; m < 4; ++m) {
                    const R w = m < 2 ? w0[r] : w1[r];
                    y[m][r].x += w * x[m].x;
                    y[m][r].y += w * x[m].y;
                }
        }
    };
    if (live0 || live1) {
        if (!odd_half && __any(v == 0)) walk(std::true_type{});
        else walk(std::false_type{});
    }
    __syncthreads();  // every column is read before any row is replaced
    if (act) {
#pragma unroll
        for (int r = 0; r < RPT; ++r) {
            const int i = i0 + r;
            if (i < hs) {
#pragma unroll
                for (int m = 0; m < 4; ++m) {
                    C2<R> z = y[m][r];
                    if (!(m < 2 ? live0 : live1)) z = cmk<R>(R(0), R(0));
                    if ((m & 1) && flip0 && i == 0) z = cmk<R>(-z.x, -z.y);
                    buf[slot(m & 1, i, ky[m])] = z;
                }
            }
        }
    }
}

// Column kx of the slices of block blk, 2t + blk (even N) or t (odd N):
// slice t starts at base + t step, row y of it at lay.row(y).
template <class R>
__device__ __forceinline__ C2<R>* pair_col(C2<R>* spec, const PairLay& lay, int M, int N, int kx, int blk, long& step) {
    const int H = M >> 1;
    step = lay.col(pair_nblk(N), 0, H);
    return spec + lay.col(blk, kx, H);
}

// The stage-0 inputs of a column block of a compiled side, in registers.
// (H: columns; a half column's length MS is H, a column's 2H)
template <class R, int MS, int EPT, int H = MS / 2>
struct PairMidIn {
    static constexpr int R0 = pair_radix(MS, EPT, 0);
    static constexpr int NB = MS / R0;
    static constexpr int MAXB = (EPT + R0 - 1) / R0;
    C2<R> v[MAXB][R0];
    // rows j + r NB: NB is a multiple of every block's rows < M that a plan takes
    __device__ __forceinline__ void load(const C2<R>* __restrict__ col, long step, const PairLay& lay, int N, int hs,
                                         int tid, int nthr) {
        const int total = NB * hs;
        const long rstep = lay.row(NB, H, N);
#pragma unroll
        for (int i = 0; i < MAXB; ++i) {
            const int b = tid + i * nthr;
            if (b < total) {
                const int t = b / NB;
                const C2<R>* g = col + t * step + lay.row(b - t * NB, H, N);
#pragma unroll
                for (int r = 0; r < R0; ++r) v[i][r] = g[r * rstep];
            }
        }
    }
    // stage 0 into LDS (nobody reads the buffer any more)
    __device__ __forceinline__ void stage0(C2<R>* buf, int hs, int tid, int nthr) {
        const int total = NB * hs;
#pragma unroll
        for (int i = 0; i < MAXB; ++i) {
            const int b = tid + i * nthr;
            if (b < total) {
                const int t = b / NB;
                const int j = b - t * NB;
                pair_dft<R, R0, false>(v[i]);
                C2<R>* pb = buf + t * pair_stride(MS);
                if constexpr (pad_linear_write(1, R0, 32)) {
                    pb += lds_pad(j * R0);
#pragma unroll
                    for (int r = 0; r < R0; ++r) pb[pad_offset(r, 1)] = v[i][r];
                } else {
#pragma unroll
                    for (int r = 0; r < R0; ++r) pb[lds_pad(j * R0 + r)] = v[i][r];
                }
            }
        }
    }
};

// The rest of a column block of a compiled side, the stage-0 inputs in `in`:
// `next` runs before the inverse transform, whose last stage stores the
// column from registers (no LDS is read after its barrier).
template <class R, int MS, int EPT, bool HALF, bool DIRECT, class In, class Next>
__device__ __forceinline__ void pair_mid_run(In& in, C2<R>* __restrict__ col, long step,
                                             const PairLay& lay, const R* __restrict__ T, int N, int kx, int blk, const C2<R>* tw,
                                             C2<R>* buf, int tid, int nthr, Next&& next, int par = 0) {
    constexpr int RL = pair_last_radix(MS, EPT);
    constexpr int MF = HALF ? 2 * MS : MS;
    const int hs = pair_hs(N);
    const uint8_t* flags = reinterpret_cast<const uint8_t*>(T + pair_table_entries(MF, N, HALF));
    in.stage0(buf, hs, tid, nthr);
    __syncthreads();
    pair_fft_from<R, false, MS, EPT, 1, In::R0, DIRECT>(buf, tw, hs, tid, nthr, PairLds{}, PairLds{});
    pair_solve<R, EPT / 4, MS, HALF>(buf, T, flags, MS, N, kx, blk, tid, par);
    __syncthreads();
    next();
    const long rstep = lay.row(MS / RL, MF / 2, N);
    pair_fft_from<R, true, MS, EPT, 0, 1, DIRECT>(buf, tw, hs, tid, nthr, PairLds{}, [&](int t, int o, C2<R>* w, int) {
        C2<R>* g = col + t * step + lay.row(o, MF / 2, N);
#pragma unroll
        for (int r = 0; r < RL; ++r) g[r * rstep] = w[r];
    });
}

// One column block of a side without a compiled body (the twiddles are in LDS).
template <class R, int EPT>
__device__ __forceinline__ void pair_mid_generic(C2<R>* __restrict__ spec, const PairLay& lay, const R* __restrict__ T, int M,
                                                 int N, int kx, int blk, const FftPlan& planM, const C2<R>* tw, C2<R>* buf, int tid,
                                                 int nthr) {
    const int hs = pair_hs(N);
    long step;
    C2<R>* col = pair_col<R>(spec, lay, M, N, kx, blk, step);
    const uint8_t* flags = reinterpret_cast<const uint8_t*>(T + pair_table_entries(M, N, false));
    const float inv_M = 1.0f / (float)M;
    for (int e = tid; e < hs * M; e += nthr) {
        const int t = fdiv(e, inv_M);
        const int y = e - t * M;
        buf[pair_pos<0>(M, t, y)] = col[t * step + lay.row(y, M >> 1, N)];
    }
    __syncthreads();
    pair_fft<R, false, 0, EPT, pair_direct((int)sizeof(R)) && (EPT < 16)>(buf, tw, M, hs, planM, tid, nthr);
    pair_solve<R, EPT / 4, 0>(buf, T, flags, M, N, kx, blk, tid);
    __syncthreads();
    pair_fft<R, true, 0, EPT, pair_direct((int)sizeof(R)) && (EPT < 16)>(buf, tw, M, hs, planM, tid, nthr);
    for (int e = tid; e < hs * M; e += nthr) {
        const int t = fdiv(e, inv_M);
        const int y = e - t * M;
        col[t * step + lay.row(y, M >> 1, N)] = buf[pair_pos<0>(M, t, y)];
    }
}

// Column and block of workgroup i of the middle pass.  Each XCD (workgroups
// go to the 8 XCDs in turn) takes a contiguous range of class rows lx, and of
// each row the columns lx and M/2 - lx back to back, so that one L2 serves the
// second's propagators and sees neighbouring columns together; columns 0
// (with M/2) and M/4 are their own partners and pair up.  The two halves of a
// column (par) are neighbours: they share its lines.
__host__ __device__ inline void pair_mid_col(int i, int H, int nblk, int& kx, int& blk) {
    const int per = H / 2;
    const int w = xcd_contiguous(i, H * nblk);
    const int unit = w >> 1;
    const int lx = unit % per;
    blk = unit / per;
    kx = (w & 1) == 0 ? lx : (lx == 0 ? H / 2 : H - lx);
}
__host__ __device__ inline void pair_mid_half(int i, int H, int nblk, int& kx, int& blk, int& par) {
    const int per = H / 2;
    const int w = xcd_contiguous(i, 2 * H * nblk);
    const int unit = w >> 2;
    const int lx = unit % per;
    blk = unit / per;
    par = w & 1;
    kx = (w & 2) == 0 ? lx : (lx == 0 ? H / 2 : H - lx);
}

// ---------------------------------------------------------------------------
// Row passes
// ---------------------------------------------------------------------------
enum { PSRC_LIFT = 0, PSRC_VOLUME = 1 };
enum { PDST_MAX = 0, PDST_SUM = 1, PDST_VOLUME = 2, PDST_VOLMAX = 3, PDST_SR = 4 };

// Split rows of Z (LDS transform `base + row` holds row `row`) into the half
// spectra of slices 2t and 2t + 1 (below N) and store them: rows fastest across
// lanes, two rows per lane when there are several (one 16-byte store).  gain
// scales them.
template <class R, int MS>
__device__ __forceinline__ void pair_unpack(const C2<R>* buf, C2<R>* __restrict__ spec, const PairLay& lay, int M_, int N,
                                            int t, int base, int rows, int y0, int tid, int nthr, R gain = R(1)) {
    const int M = MS ? MS : M_;
    const int H = M >> 1;
    const bool has_b = 2 * t + 1 < N;
    const int rb = lay.rb;
    const R half = R(0.5) * gain;
    C2<R>* sa = spec + lay.row(y0, H, N) + lay.col(2 * t, 0, H);
    C2<R>* sb = sa + lay.col(1, 0, H);
    auto split = [&](int row, int k, C2<R>& a, C2<R>& b) {
        const C2<R> z = buf[pair_pos<MS>(M, base + row, k)];
        const C2<R> w = buf[pair_pos<MS>(M, base + row, k == 0 ? H : M - k)];
        if (k == 0) {
            // Z[0] = A[0] + i B[0], Z[M/2] = A[M/2] + i B[M/2]
            a = cmk<R>(gain * z.x, gain * w.x);
            b = cmk<R>(gain * z.y, gain * w.y);
        } else {
            a = cmk<R>(half * (z.x + w.x), half * (z.y - w.y));
            b = cmk<R>(half * (z.y + w.y), half * (w.x - z.x));
        }
    };
    if ((rows & 1) == 0) {
        typedef R v4_t __attribute__((ext_vector_type(4), aligned(2 * sizeof(R))));
        const int sh = __ffs(rows >> 1) - 1;
        const int rp = rows >> 1;
        for (int e = tid; e < rp * H; e += nthr) {
            const int r0 = 2 * (e & (rp - 1));
            const int k = e >> sh;
            C2<R> a0, b0, a1, b1;
            split(r0, k, a0, b0);
            split(r0 + 1, k, a1, b1);
            v4_t va, vb;
            va.x = a0.x; va.y = a0.y; va.z = a1.x; va.w = a1.y;
            vb.x = b0.x; vb.y = b0.y; vb.z = b1.x; vb.w = b1.y;
            *reinterpret_cast<v4_t*>(sa + (size_t)k * rb + r0) = va;
            if (has_b) *reinterpret_cast<v4_t*>(sb + (size_t)k * rb + r0) = vb;
        }
    } else {
        for (int e = tid; e < rows * H; e += nthr) {
            const int k = rows == 1 ? e : e / rows;
            const int row = rows == 1 ? 0 : e - k * rows;
            C2<R> a, b;
            split(row, k, a, b);
            sa[(size_t)k * rb + row] = a;
            if (has_b) sb[(size_t)k * rb + row] = b;
        }
    }
}

// The inverse of pair_unpack for np pairs from t0 on: rows y0 .. of their
// slices into LDS as Z.  Few registers: what hides the latency of the loads
// is other workgroups (a round's loads held in registers while the round
// before was transformed took 768^2, N = 24 volumes from 27 to 43 us).
template <class R, int MS>
__device__ __forceinline__ void pair_pack(C2<R>* buf, const C2<R>* __restrict__ spec, const PairLay& lay, int M_, int N,
                                          int t0, int np, int rows, int y0, int tid, int nthr) {
    const int M = MS ? MS : M_;
    const int H = M >> 1;
    const C2<R>* base = spec + lay.row(y0, H, N);
    const long plane = lay.col(1, 0, H);
    auto put = [&](int tr, int k, C2<R> a, C2<R> b) {
        C2<R> z, w;
        if (k == 0) {
            z = cmk<R>(a.x, b.x);
            w = cmk<R>(a.y, b.y);
        } else {
            z = cmk<R>(a.x - b.y, a.y + b.x);  // A + i B
            w = cmk<R>(a.x + b.y, b.x - a.y);  // conj A + i conj B
        }
        buf[pair_pos<MS>(M, tr, k)] = z;
        buf[pair_pos<MS>(M, tr, k == 0 ? H : M - k)] = w;
    };
    const float inv_H = 1.0f / (float)H;
    if ((rows & 1) == 0) {
        typedef R v4_t __attribute__((ext_vector_type(4), aligned(2 * sizeof(R))));
        const int rp = rows >> 1;
        const int sh = __ffs(rp) - 1;
        const int per = rp * H;
#pragma unroll 2
        for (int e = tid; e < np * per; e += nthr) {
            const int r0 = 2 * (e & (rp - 1));
            const int gk = e >> sh;
            const int g = MS ? gk / (MS ? MS / 2 : 1) : fdiv(gk, inv_H);
            const int k = gk - g * H;
            const int s = 2 * (t0 + g);
            const C2<R>* p = base + lay.col(s, k, H) + r0;
            const v4_t va = *reinterpret_cast<const v4_t*>(p);
            v4_t vb = v4_t(0);
            if (s + 1 < N) vb = *reinterpret_cast<const v4_t*>(p + plane);
            put(g * rows + r0, k, cmk<R>(va.x, va.y), cmk<R>(vb.x, vb.y));
            put(g * rows + r0 + 1, k, cmk<R>(va.z, va.w), cmk<R>(vb.z, vb.w));
        }
    } else {
        const float inv_r = 1.0f / (float)rows;
#pragma unroll 4
        for (int e = tid; e < np * rows * H; e += nthr) {
            const int gk = rows == 1 ? e : fdiv(e, inv_r);
            const int row = rows == 1 ? 0 : e - gk * rows;
            const int g = MS ? gk / (MS ? MS / 2 : 1) : fdiv(gk, inv_H);
            const int k = gk - g * H;
            const int s = 2 * (t0 + g);
            const C2<R>* p = base + lay.col(s, k, H) + row;
            const C2<R> a = *p;
            C2<R> b = cmk<R>(R(0), R(0));
            if (s + 1 < N) b = p[plane];
            put(g * rows + row, k, a, b);
        }
    }
}

// The tile's rows with halved columns: `rows` / 2 rows y0 .. and the same
// number from M/2 + y0 on.
template <bool HALF>
__device__ __forceinline__ int pair_image_row(int M, int rows, int y0, int row) {
    return y0 + row + (HALF && row >= (rows >> 1) ? (M >> 1) - (rows >> 1) : 0);
}

// pair_unpack with halved columns: a lane takes one row n and n + M/2, and its
// twiddle w_M^n serves every column.
template <class R, int MS>
__device__ __forceinline__ void pair_unpack_half(const C2<R>* buf, C2<R>* __restrict__ spec, const PairLay& lay, int N,
                                                 int t, int rows, int y0, const C2<R>* tw, int tid, int nthr) {
    constexpr int H = MS >> 1;
    const int r2 = rows >> 1;
    const int sh = __ffs(r2) - 1;
    const int r = tid & (r2 - 1);
    const bool has_b = 2 * t + 1 < N;
    const int odd = lay.rb / 2;  // from the even half's entry to the odd half's
    const R half = R(0.5);
    C2<R>* sa = spec + lay.row(y0, H, N) + lay.col(2 * t, 0, H) + r;
    const long plane = lay.col(1, 0, H);
    const C2<R> w = tw[tw_pos(y0 + r)];
    auto split = [&](int row, int k, C2<R>& a, C2<R>& b) {
        const C2<R> z = buf[pair_pos<MS>(MS, row, k)];
        const C2<R> u = buf[pair_pos<MS>(MS, row, k == 0 ? H : MS - k)];
        if (k == 0) {
            a = cmk<R>(z.x, u.x);
            b = cmk<R>(z.y, u.y);
        } else {
            a = cmk<R>(half * (z.x + u.x), half * (z.y - u.y));
            b = cmk<R>(half * (z.y + u.y), half * (u.x - z.x));
        }
    };
    for (int k = tid >> sh; k < H; k += nthr >> sh) {
        C2<R> a0, b0, a1, b1;
        split(r, k, a0, b0);
        split(r + r2, k, a1, b1);
        C2<R>* p = sa + (size_t)k * lay.rb;
        p[0] = cmk<R>(a0.x + a1.x, a0.y + a1.y);
        p[odd] = cmul<R>(cmk<R>(a0.x - a1.x, a0.y - a1.y), w);
        if (has_b) {
            p[plane] = cmk<R>(b0.x + b1.x, b0.y + b1.y);
            p[plane + odd] = cmul<R>(cmk<R>(b0.x - b1.x, b0.y - b1.y), w);
        }
    }
}

// The inverse of pair_unpack_half in two steps, so that the loads can be in
// flight behind a transform; rows MS <= EPT nthr.
template <class R, int MS, int EPT>
struct PairHalfIn {
    static constexpr int H = MS >> 1;
    static constexpr int NV = EPT / 4;  // columns per thread, four values each
    C2<R> a0[NV], a1[NV], b0[NV], b1[NV];
    __device__ __forceinline__ void load(const C2<R>* __restrict__ spec, const PairLay& lay, int N, int t, int rows,
                                         int y0, int tid, int nthr) {
        const int r2 = rows >> 1;
        const int sh = __ffs(r2) - 1;
        const C2<R>* base = spec + lay.row(y0, H, N) + lay.col(2 * t, 0, H) + (tid & (r2 - 1));
        const long plane = lay.col(1, 0, H);
        const bool has_b = 2 * t + 1 < N;
        const int odd = lay.rb / 2;
#pragma unroll
        for (int i = 0; i < NV; ++i) {
            const int k = (tid + i * nthr) >> sh;
            if (k < H) {
                const C2<R>* p = base + (size_t)k * lay.rb;
                a0[i] = p[0];
                a1[i] = p[odd];
                b0[i] = b1[i] = cmk<R>(R(0), R(0));
                if (has_b) {
                    b0[i] = p[plane];
                    b1[i] = p[plane + odd];
                }
            }
        }
    }
    __device__ __forceinline__ void store(C2<R>* buf, int rows, int y0, const C2<R>* tw, int tid, int nthr) {
        const int r2 = rows >> 1;
        const int sh = __ffs(r2) - 1;
        const int r = tid & (r2 - 1);
        auto put = [&](int tr, int k, C2<R> a, C2<R> b) {
            C2<R> z, w;
            if (k == 0) {
                z = cmk<R>(a.x, b.x);
                w = cmk<R>(a.y, b.y);
            } else {
                z = cmk<R>(a.x - b.y, a.y + b.x);
                w = cmk<R>(a.x + b.y, b.x - a.y);
            }
            buf[pair_pos<MS>(MS, tr, k)] = z;
            buf[pair_pos<MS>(MS, tr, k == 0 ? H : MS - k)] = w;
        };
        C2<R> w = tw[tw_pos(y0 + r)];
        w.y = -w.y;
#pragma unroll
        for (int i = 0; i < NV; ++i) {
            const int k = (tid + i * nthr) >> sh;
            if (k < H) {
                const C2<R> da = cmul<R>(a1[i], w), db = cmul<R>(b1[i], w);
                put(r, k, cmk<R>(a0[i].x + da.x, a0[i].y + da.y), cmk<R>(b0[i].x + db.x, b0[i].y + db.y));
                put(r + r2, k, cmk<R>(a0[i].x - da.x, a0[i].y - da.y), cmk<R>(b0[i].x - db.x, b0[i].y - db.y));
            }
        }
    }
};

// Forward row pass of pair t over rows y0 .. y0 + rows - 1.
//   PSRC_LIFT    f (1 - mask) at the pixel's orientation (rmap)
//   PSRC_VOLUME  real volume vol[N][M][M]
template <class R, int SRC, int MS, int EPT, bool HALF = false>
__device__ __forceinline__ void pair_fwd_tile(const R* __restrict__ f, const uint8_t* __restrict__ mask,
                                              const uint8_t* __restrict__ rmap, const R* __restrict__ vol,
                                              C2<R>* __restrict__ spec, const PairLay& lay, int M_, int N, int rows,
                                              int y0, int t_begin, int t_end, const FftPlan& planM, const C2<R>* tw, C2<R>* buf, int tid,
                                              int nthr) {
    const int M = MS ? MS : M_;
    const int h = N >> 1;
    const bool odd = N & 1;
    const size_t img = (size_t)M * M;
    // z of pixel (row, n) of pair t; `r`, `v`: its orientation and value (lift)
    auto lifted = [&](int t, int r, R v) {
        C2<R> z = cmk<R>(R(0), R(0));
        if (odd) {
            if (r == 2 * t) z.x = v;
            else if (r == 2 * t + 1 && r < N) z.y = v;
        } else {
            if (r == t) z = cmk<R>(v, v);
            else if (r == t + h) z = cmk<R>(v, -v);
        }
        return z;
    };
    auto from_volume = [&](int t, int row, int n) {
        const size_t p = (size_t)pair_image_row<HALF>(M, rows, y0, row) * M + n;
        if (odd) {
            const R a = vol[(size_t)(2 * t) * img + p];
            const R b = 2 * t + 1 < N ? vol[(size_t)(2 * t + 1) * img + p] : R(0);
            return cmk<R>(a, b);
        }
        const R a = vol[(size_t)t * img + p], b = vol[(size_t)(t + h) * img + p];
        return cmk<R>(a + b, a - b);
    };
    if constexpr (MS != 0) {
        constexpr int R0 = pair_radix(MS, EPT, 0);
        constexpr int NB = MS / R0;
        constexpr int MAXB = (EPT + R0 - 1) / R0;
        // the lift's sources stay in registers while the pairs go by
        R fv[MAXB][R0];
        uint32_t rv[MAXB][(R0 + 3) / 4];  // four orientations a word
        if constexpr (SRC == PSRC_LIFT) {
#pragma unroll
            for (int i = 0; i < MAXB; ++i) {
                const int b = tid + i * nthr;
#pragma unroll
                for (int r = 0; r < R0; ++r) fv[i][r] = R(0);
#pragma unroll
                for (int r = 0; r < (R0 + 3) / 4; ++r) rv[i][r] = 0;
                if (b < NB * rows) {
                    const int row = b / NB;
                    const size_t p = (size_t)pair_image_row<HALF>(M, rows, y0, row) * MS + (b - row * NB);
#pragma unroll
                    for (int r = 0; r < R0; ++r) {
                        const R v = f[p + r * NB];
                        fv[i][r] = mask[p + r * NB] ? R(0) : v;
                        rv[i][r / 4] |= (uint32_t)rmap[p + r * NB] << (8 * (r % 4));
                    }
                }
            }
        }
        C2<R> v[MAXB][R0];
        // stage-0 inputs of pair t; a volume's are fetched one pair ahead,
        // behind the transform of the pair before
        auto inputs = [&](int t) {
#pragma unroll
            for (int i = 0; i < MAXB; ++i) {
                const int b = tid + i * nthr;
                if (b < NB * rows) {
                    const int row = b / NB;
                    const int j = b - row * NB;
#pragma unroll
                    for (int r = 0; r < R0; ++r)
                        v[i][r] = SRC == PSRC_LIFT ? lifted(t, (int)((rv[i][r / 4] >> (8 * (r % 4))) & 0xff), fv[i][r])
                                                   : from_volume(t, row, j + r * NB);
                }
            }
        };
        if constexpr (SRC == PSRC_VOLUME) inputs(t_begin);
        for (int t = t_begin; t < t_end; ++t) {
            if constexpr (SRC == PSRC_LIFT) inputs(t);
#pragma unroll
            for (int i = 0; i < MAXB; ++i) {
                const int b = tid + i * nthr;
                if (b < NB * rows) {
                    const int row = b / NB;
                    const int j = b - row * NB;
                    pair_dft<R, R0, false>(v[i]);
                    C2<R>* pb = buf + row * pair_stride(MS);
                    if constexpr (pad_linear_write(1, R0, 32)) {
                        pb += lds_pad(j * R0);
#pragma unroll
                        for (int r = 0; r < R0; ++r) pb[pad_offset(r, 1)] = v[i][r];
                    } else {
#pragma unroll
                        for (int r = 0; r < R0; ++r) pb[lds_pad(j * R0 + r)] = v[i][r];
                    }
                }
            }
            __syncthreads();
            if constexpr (SRC == PSRC_VOLUME)
                if (t + 1 < t_end) inputs(t + 1);
            pair_fft_from<R, false, MS, EPT, 1, R0, false>(buf, tw, rows, tid, nthr, PairLds{}, PairLds{});
            if constexpr (HALF) pair_unpack_half<R, MS>(buf, spec, lay, N, t, rows, y0, tw, tid, nthr);
            else pair_unpack<R, MS>(buf, spec, lay, M, N, t, 0, rows, y0, tid, nthr);
            __syncthreads();
        }
    } else {
        const float inv_M = 1.0f / (float)M;
        for (int t = t_begin; t < t_end; ++t) {
            for (int e = tid; e < rows * M; e += nthr) {
                const int row = fdiv(e, inv_M);
                const int n = e - row * M;
                C2<R> z;
                if (SRC == PSRC_LIFT) {
                    const size_t p = (size_t)(y0 + row) * M + n;
                    z = lifted(t, rmap[p], mask[p] ? R(0) : f[p]);
                } else {
                    z = from_volume(t, row, n);
                }
                buf[pair_pos<0>(M, row, n)] = z;
            }
            __syncthreads();
            pair_fft<R, false, 0, EPT, false>(buf, tw, M, rows, planM, tid, nthr);
            pair_unpack<R, 0>(buf, spec, lay, M, N, t, 0, rows, y0, tid, nthr);
            __syncthreads();
        }
    }
}

// Inverse row pass of pairs [t_begin, t_end) over rows y0 .. y0 + rows - 1,
// G pairs at a time.
//   PDST_MAX     maximum over the slices (out; all pairs)
//   PDST_SUM     mean (out; all pairs)
//   PDST_VOLUME  the real volume (out[N][M][M])
//   PDST_VOLMAX  the real volume and the maximum (hmax); all pairs at once
//   PDST_SR      the static mix, then the forward row pass; all pairs at once
template <class R, int DST, int MS, int EPT>
__device__ __forceinline__ void pair_inv_tile(C2<R>* __restrict__ spec, const PairLay& lay, R* __restrict__ out, R* __restrict__ hmax,
                                              const R* __restrict__ f, const uint8_t* __restrict__ mask, R eps, int M_, int N, int rows, int G,
                                              int y0, int t_begin, int t_end, const FftPlan& planM, const C2<R>* tw,
                                              C2<R>* buf, int tid, int nthr) {
    const int M = MS ? MS : M_;
    const int h = N >> 1;
    const bool odd = N & 1;
    const size_t img = (size_t)M * M;
    const int npx = rows * M;
    const float inv_M = 1.0f / (float)M;
    // running maximum or sum of the tile's pixels between rounds, in LDS after
    // the transforms (a pixel belongs to one thread)
    R* acc = reinterpret_cast<R*>(buf + pair_buf_elems(M, rows * G));
    const int t_last = t_begin + (t_end - 1 - t_begin) / G * G;  // first pair of the last round
    for (int t0 = t_begin; t0 < t_end; t0 += G) {
        const int np = min(G, t_end - t0);
        pair_pack<R, MS>(buf, spec, lay, M, N, t0, np, rows, y0, tid, nthr);
        __syncthreads();
        constexpr bool DIRECT = pair_direct((int)sizeof(R)) && (DST == PDST_SR || DST == PDST_VOLMAX);
        pair_fft<R, true, MS, EPT, DIRECT>(buf, tw, M, np * rows, planM, tid, nthr);
#pragma unroll 1
        for (int e = tid; e < npx; e += nthr) {
            const int row = MS ? e / (MS ? MS : 1) : fdiv(e, inv_M);
            const int n = e - row * M;
            const size_t p = (size_t)(y0 + row) * M + n;
            R a = DST == PDST_SUM ? R(0) : -INFINITY;
            if (t0 != t_begin && (DST == PDST_MAX || DST == PDST_SUM)) a = acc[e];
#pragma unroll 4
            for (int g = 0; g < np; ++g) {
                const C2<R> z = buf[pair_pos<MS>(M, g * rows + row, n)];
                const int t = t0 + g;
                const bool two = !odd || 2 * t + 1 < N;
                if constexpr (DST == PDST_MAX || DST == PDST_SR || DST == PDST_VOLMAX)
                    a = vmax<R>(a, odd ? (two ? vmax<R>(z.x, z.y) : z.x) : z.x + fabs(z.y));
                if constexpr (DST == PDST_SUM) a += odd ? (two ? z.x + z.y : z.x) : R(2) * z.x;
                if constexpr (DST == PDST_VOLUME || DST == PDST_VOLMAX) {
                    if (odd) {
                        out[(size_t)(2 * t) * img + p] = z.x;
                        if (two) out[(size_t)(2 * t + 1) * img + p] = z.y;
                    } else {
                        out[(size_t)t * img + p] = z.x + z.y;
                        out[(size_t)(t + h) * img + p] = z.x - z.y;
                    }
                }
            }
            if constexpr (DST == PDST_MAX || DST == PDST_SUM) {
                if (t0 != t_last) acc[e] = a;
                else if (DST == PDST_SUM) out[p] = a * (R(1) / (R)N);
                else out[p] = a;
            }
            if constexpr (DST == PDST_VOLMAX) hmax[p] = a;
            if constexpr (DST == PDST_SR) {
                if (!mask[p] && a > R(0)) {
                    const R f0 = f[p];
                    const R href = f0 > R(0) ? f0 : R(0);
                    const R sg = (eps * href + (R(1) - eps) * a) / a;
#pragma unroll 4
                    for (int g = 0; g < np; ++g) {
                        C2<R>* q = buf + pair_pos<MS>(M, g * rows + row, n);
                        *q = cmk<R>(q->x * sg, q->y * sg);
                    }
                }
            }
        }
        __syncthreads();
        if constexpr (DST == PDST_SR) {
            pair_fft<R, false, MS, EPT, DIRECT>(buf, tw, M, np * rows, planM, tid, nthr);
            for (int g = 0; g < np; ++g)
                // the inverse pass leaves p/2 and q/2 (the propagators carry the
                // 1/2 of x = (p +- q) / 2)
                pair_unpack<R, MS>(buf, spec, lay, M, N, t0 + g, g * rows, rows, y0, tid, nthr,
                                   odd ? R(1) : R(2));
        }
    }
}

// The same with halved columns, one pair per round: PDST_MAX, PDST_SUM or
// PDST_VOLUME.  The next pair's rows are fetched while this one is transformed
// (there is a workgroup per compute unit, no other hides its latency), and a
// pixel's running value stays in the registers of the thread whose last
// butterfly produces it.  1024^2, N = 32, FP64: 212 -> 106 us against the five
// passes' kernel (268 MB, 2.5 TB/s); two workgroups per unit of half the rows
// each take as long.
template <class R, int DST, int MS, int EPT>
__device__ __forceinline__ void pair_inv_half_tile(const C2<R>* __restrict__ spec, const PairLay& lay,
                                                   R* __restrict__ out, int N, int rows, int y0, int t_begin,
                                                   int t_end, const C2<R>* tw, C2<R>* buf, int tid, int nthr) {
    constexpr int M = MS;
    constexpr int RL = pair_last_radix(MS, EPT);
    constexpr int NB = MS / RL;
    constexpr int MAXB = (EPT + RL - 1) / RL;
    const int h = N >> 1;
    const bool odd = N & 1;
    const size_t img = (size_t)M * M;
    PairHalfIn<R, MS, EPT> in;
    in.load(spec, lay, N, t_begin, rows, y0, tid, nthr);
    R acc[MAXB][RL];
#pragma unroll
    for (int i = 0; i < MAXB; ++i)
#pragma unroll
        for (int r = 0; r < RL; ++r) acc[i][r] = DST == PDST_SUM ? R(0) : -INFINITY;
    for (int t = t_begin; t < t_end; ++t) {
        in.store(buf, rows, y0, tw, tid, nthr);
        __syncthreads();
        if (t + 1 < t_end) in.load(spec, lay, N, t + 1, rows, y0, tid, nthr);
        const bool two = !odd || 2 * t + 1 < N;
        pair_fft_from<R, true, MS, EPT, 0, 1, false>(buf, tw, rows, tid, nthr, PairLds{}, [&](int row, int o, C2<R>* v, int i) {
            if constexpr (DST == PDST_VOLUME) {
                R* q = out + (size_t)pair_image_row<true>(M, rows, y0, row) * M + o;
                R* qa = q + (size_t)(odd ? 2 * t : t) * img;
                R* qb = q + (size_t)(odd ? 2 * t + 1 : t + h) * img;
#pragma unroll
                for (int r = 0; r < RL; ++r) {
                    qa[r * NB] = odd ? v[r].x : v[r].x + v[r].y;
                    if (two) qb[r * NB] = odd ? v[r].y : v[r].x - v[r].y;
                }
            } else {
#pragma unroll
                for (int r = 0; r < RL; ++r) {
                    if (DST == PDST_MAX)
                        acc[i][r] = vmax<R>(acc[i][r], odd ? (two ? vmax<R>(v[r].x, v[r].y) : v[r].x)
                                                           : v[r].x + fabs(v[r].y));
                    else acc[i][r] += odd ? (two ? v[r].x + v[r].y : v[r].x) : R(2) * v[r].x;
                }
            }
        });
        __syncthreads();
    }
    if constexpr (DST != PDST_VOLUME) {
#pragma unroll
        for (int i = 0; i < MAXB; ++i) {
            const int b = tid + i * nthr;
            if (b < NB * rows) {
                const int row = b / NB;
                R* q = out + (size_t)pair_image_row<true>(M, rows, y0, row) * M + (b - row * NB);
#pragma unroll
                for (int r = 0; r < RL; ++r) q[r * NB] = DST == PDST_SUM ? acc[i][r] * (R(1) / (R)N) : acc[i][r];
            }
        }
    }
}

// DR at mesh point `step` for the rows y0 .. y0 + rows - 1: grow the good set
// (see k_dr_grow_mix), mix the real volume and transform the rows forward.
// h, join and href are those of the whole image; a pixel's own entries are
// written by the thread that holds it.
template <class R, int MS, int EPT>
__device__ __forceinline__ void pair_dr_tile(const R* __restrict__ vol, const R* __restrict__ h,
                                             int16_t* __restrict__ join, R* __restrict__ href,
                                             C2<R>* __restrict__ spec, const PairLay& lay, R eps, int step, int M_,
                                             int N, int rows, int y0,
                                             const FftPlan& planM, const C2<R>* tw, C2<R>* buf, int tid, int nthr) {
    const int M = MS ? MS : M_;
    const int hn = N >> 1;
    const bool odd = N & 1;
    const size_t img = (size_t)M * M;
    const int np = pair_count(N);
    const float inv_M = 1.0f / (float)M;
    for (int e = tid; e < rows * M; e += nthr) {
        const int row = MS ? e / (MS ? MS : 1) : fdiv(e, inv_M);
        const int n = e - row * M;
        const int y = y0 + row;
        const size_t p = (size_t)y * M + n;
        const R hp = h[p];
        const int jp = join[p];
        bool good = jp >= 0 && jp < step;
        R hr = good ? href[p] : hp;  // a pixel that joins now is its own reference
        if (!good) {
            bool near_good = false;
            R s = R(0);
            int c = 0;
            for (int dy = -1; dy <= 1; ++dy) {
                const int yy = y + dy < 0 ? M - 1 : (y + dy >= M ? 0 : y + dy);
                for (int dx = -1; dx <= 1; ++dx) {
                    const int xx = n + dx < 0 ? M - 1 : (n + dx >= M ? 0 : n + dx);
                    const size_t q = (size_t)yy * M + xx;
                    const int jq = join[q];
                    if (jq >= 0 && jq < step) {
                        near_good = true;
                    } else {
                        s += h[q];
                        ++c;
                    }
                }
            }
            if (near_good && hp > s / (R)c) {
                join[p] = (int16_t)step;
                href[p] = hp;
                good = true;
            }
        }
        R sg = R(1);
        if (good && hp > R(0)) sg = (eps * hr + (R(1) - eps) * hp) / hp;
        for (int g = 0; g < np; ++g) {
            R a, b;
            if (odd) {
                a = vol[(size_t)(2 * g) * img + p];
                b = 2 * g + 1 < N ? vol[(size_t)(2 * g + 1) * img + p] : R(0);
                a *= sg;
                b *= sg;
                buf[pair_pos<MS>(M, g * rows + row, n)] = cmk<R>(a, b);
            } else {
                a = vol[(size_t)g * img + p] * sg;
                b = vol[(size_t)(g + hn) * img + p] * sg;
                buf[pair_pos<MS>(M, g * rows + row, n)] = cmk<R>(a + b, a - b);
            }
        }
    }
    __syncthreads();
    pair_fft<R, false, MS, EPT, pair_direct((int)sizeof(R))>(buf, tw, M, np * rows, planM, tid, nthr);
    for (int g = 0; g < np; ++g)
        pair_unpack<R, MS>(buf, spec, lay, M, N, g, g * rows, rows, y0, tid, nthr);
}

// ---------------------------------------------------------------------------
// Launch geometry of a plan
// ---------------------------------------------------------------------------
struct PairGeom {
    PairLay lay;
    int fwd_rows, fwd_threads, fwd_ept, fwd_pairs;  // forward rows: rows, threads, pairs per workgroup
    int vol_fwd_pairs, vol_pairs;                   // a volume's rows: the forward tile, pairs per workgroup each way
    int inv_rows, inv_G, inv_threads, inv_ept;      // projecting inverse rows: all pairs, G at a time
    int mid_threads, mid_ept, mid_grid;             // middle pass; column blocks, or walkers
    int all_threads, all_ept;                       // one row of all pairs (restoration)
    bool whole_sr, whole_dr;                        // a mesh point of a restoration runs on such rows
};

// Sides with compiled row bodies: in FP32 those of the batch and of the smallest
// images, in FP64 the powers of two from 256 on. (The halved columns have their own.)
// Every other side runs the runtime radices, in FP64 64^2, N = 32 82 -> 53 us against
// the five passes, 192^2, N = 32 124 -> 83, 768^2, N = 16 309 -> 209, in FP32 192^2,
// N = 32 72 -> 34; bodies for them have not been measured.
__host__ __device__ constexpr bool pair_rows_compiled(int M, int rsize) {
    return M == 256 || M == 512 || M == 1024 || (rsize == 4 && (M == 64 || M == 128 || M == 384 || M == 768));
}

// Elements per thread of a row workgroup: 8 while that fits in its threads
// (1024^2 forward rows, 8192 elements: 16 is faster, 46 -> 38 us).
__host__ __device__ constexpr int pair_row_ept(int elems, int rsize) {
    return elems <= (rsize == 4 ? 6144 : 4096) ? 8 : 16;
}
__host__ __device__ constexpr int pair_threads(int elems, int ept) { return ((elems + ept - 1) / ept + 63) / 64 * 64; }
// Rows of a forward tile: 64 bytes of a column.
__host__ __device__ constexpr int pair_fwd_rows(int M, int rsize) {
    int rows = 64 / (2 * rsize);
    while (M % rows) rows >>= 1;
    return rows;
}

// The spectrum is stored in blocks of 8 rows (4 where 8 does not divide M): a
// row pass then reads and writes runs of neighbouring columns, whole lines
// with 8 rows of a tile and a quarter of them with 2, instead of one piece
// per column, and the middle pass moves 64-byte pieces whose line-mates the
// same XCD handles at the same time.  FP32, against spec[s][kx][y]: inverse
// rows 512^2, N = 30 17.5 -> 12.6 us, 1024^2, N = 32 59 -> 48 us; SR rows 256^2,
// N = 30 16.1 -> 14.2 us; middle pass 23.9 -> 24.6, 103.6 -> 105.9 and 9.9 ->
// 10.0 us.  4 rows cost the middle pass more than the rows gain, 16 gain less.
//
// Forward and volume tiles take 8 rows (FP32) and few pairs each, so that
// there are many workgroups.  A projecting workgroup takes every pair of its
// rows: as few rows as give each compute unit a workgroup, without a last
// wave that is partly empty where halving the rows avoids it (768^2), and as
// many pairs per round as leave the workgroups of a unit resident together
// (768^2, N = 24: three of 6 pairs 24 us, two of 12 pairs 35 us).
//
// A volume's forward rows at 1024^2 take as many pairs per workgroup as leave one
// round of the two workgroups that a unit holds: N = 16 / 24 / 32 33 / 46 / 77 us; with
// up to four per unit in all, as the lift, 33 / 51 / 79 (768^2, N = 32, 64 us that way
// against 49, keeps the lift's).
//
// Halved columns (FP64): a tile's rows n and n + M/2 are half as many of each,
// one workgroup lifts every pair where the tiles fill the units (1024^2,
// N = 32: 104 -> 98 us), the projection halves its tiles until they do (512^2,
// N = 40: 193 -> 184 us).  Blocks of 4 or 16 rows: 482 -> 559 and 493 us for
// the whole of 1024^2, N = 32.
//
// A mesh point of a restoration on one row of every pair per workgroup saves the
// volume's way through memory, but where the rows outnumber the compute units it
// loses to the volume's own tiles once a row leaves a unit no second workgroup (DR,
// whose growth and mix stand between the two transforms) or, on runtime radices, has
// more than 16 pairs (DR in FP32: takes 16 elements per thread).  Interval, whole
// rows against volume: DR FP32 1024^2, N = 16 / 20 / 30 165 / 257 / 395 against 167 / 233 /
// 352 us, 648^2, N = 30 299 / 254, 864^2, N = 16 / 20 214 / 338 against 227 / 324, FP64
// 576^2, N = 16 222 / 193, 512^2, N = 20 120 / 113, FP32 512^2, N = 32 90 / 88 (two per
// unit), FP64 256^2, N = 48 76 / 89 (a unit each); SR FP32 288^2, N = 32 / 64 72 / 169
// against 74 / 147, 1024^2, N = 30 278 / 319.
inline PairGeom pair_geom(int M, int N, int rsize, int num_cu) {
    PairGeom g{};
    const int np = pair_count(N);
    g.lay.rb = M % 8 == 0 ? 8 : 4;
    g.lay.lg = M % 8 == 0 ? 3 : 2;
    const int most = pair_max_threads(rsize);
    g.lay.halved = pair_halves(M, N, rsize);
    g.lay.lg -= g.lay.halved;
    const int rows = pair_fwd_rows(M, rsize);
    g.fwd_rows = rows;
    g.fwd_ept = pair_row_ept(rows * M, rsize);
    g.fwd_threads = pair_threads(rows * M, g.fwd_ept);
    const int blocks = M / rows;
    int ppw = g.lay.halved && blocks >= num_cu ? np : 1;
    while (ppw < np && (long)blocks * ((np + ppw - 1) / ppw) > 4L * num_cu) ++ppw;
    g.fwd_pairs = ppw;
    g.vol_fwd_pairs = ppw;
    if (rsize == 4 && M == 1024)
        while (g.vol_fwd_pairs < np && (long)blocks * ((np + g.vol_fwd_pairs - 1) / g.vol_fwd_pairs) > 2L * num_cu)
            ++g.vol_fwd_pairs;
    // a halved volume's pairs share nothing and go to more workgroups than the
    // lift's (1024^2, N = 32, FP64: 184 -> 141 us)
    if (g.lay.halved && ppw > 4) g.vol_fwd_pairs = 4;
    g.vol_pairs = 1;
    if (g.lay.halved) {
        g.inv_rows = rows;
        while (g.inv_rows > 2 && M / g.inv_rows < num_cu) g.inv_rows >>= 1;
        g.inv_G = 1;
        g.inv_ept = g.fwd_ept;
        g.inv_threads = pair_threads(g.inv_rows * M, g.inv_ept);
        const int hs = pair_hs(N);
        g.mid_ept = pair_mid_ept(M / 2, hs, rsize);
        g.mid_threads = pair_mid_threads(M / 2, hs, rsize);
        g.mid_grid = M * pair_nblk(N);
        if (2 * pair_lds_bytes(M / 2, hs, rsize) > (size_t)kPairLds && g.mid_grid > num_cu) g.mid_grid = num_cu;
        return g;
    }
    int r = rows;
    while (r > 1 && M / r < num_cu) r >>= 1;
    while (r > 1 && M / r % num_cu != 0) r >>= 1;
    g.inv_rows = r;
    const int per_cu = (M / r + num_cu - 1) / num_cu;
    int G = 0;
    while (G < np && r * (G + 1) * M <= 16 * most &&
           pair_lds_bytes(M, r * (G + 1), rsize) + (size_t)r * M * rsize <= (size_t)kPairLds / (per_cu < 4 ? per_cu : 4))
        ++G;
    if (G < 1) G = 1;
    // as many rounds as needed, evenly filled
    const int rounds = (np + G - 1) / G;
    G = (np + rounds - 1) / rounds;
    g.inv_G = G;
    g.inv_ept = r * G * M <= 8 * most ? 8 : 16;
    g.inv_threads = pair_threads(r * G * M, g.inv_ept);
    const int hs = pair_hs(N);
    g.mid_ept = pair_mid_ept(M, hs, rsize);
    g.mid_threads = pair_mid_threads(M, hs, rsize);
    g.mid_grid = M / 2 * pair_nblk(N);
    if (2 * pair_lds_bytes(M, hs, rsize) > (size_t)kPairLds && g.mid_grid > num_cu) g.mid_grid = num_cu;
    // one row of every pair is no larger than a column block of the middle pass
    g.all_ept = np * M <= 8 * most ? 8 : 16;
    g.all_threads = pair_threads(np * M, g.all_ept);
    const bool many = !pair_rows_compiled(M, rsize) && rsize == 4 && g.all_ept == 16;
    g.whole_sr = M <= num_cu || pair_rows_compiled(M, rsize) || np <= 16;
    g.whole_dr = M <= num_cu || (g.whole_sr && !many && 2 * pair_lds_bytes(M, np, rsize) <= (size_t)kPairLds);
    return g;
}

// Launchers (se2n_pair_rows.hpp, se2n_pair_mid.hpp); spec holds N M/2 M
// complex values.
template <class R>
hipError_t launch_pair_fwd(int src, const R* f, const uint8_t* mask, const uint8_t* rmap, const R* vol, C2<R>* spec,
                           int M, int N, const PairGeom& g, const FftPlan& planM, const C2<R>* tw, hipStream_t st);
// dst: PDST_MAX, PDST_SUM (out an image) or PDST_VOLUME
template <class R>
hipError_t launch_pair_inv(int dst, C2<R>* spec, R* out, int M, int N, const PairGeom& g, const FftPlan& planM,
                           const C2<R>* tw, hipStream_t st);
// One mesh point of SR on the spectrum: inverse rows, mix, forward rows.
template <class R>
hipError_t launch_pair_sr(C2<R>* spec, const R* f, const uint8_t* mask, double eps, int M, int N, const PairGeom& g,
                          const FftPlan& planM, const C2<R>* tw, hipStream_t st);
// One mesh point of DR: inverse rows to vol and h, then growth, mix and forward rows.
template <class R>
hipError_t launch_pair_dr(C2<R>* spec, R* vol, R* h, int16_t* join, R* href, double eps, int step, int M, int N,
                          const PairGeom& g, const FftPlan& planM, const C2<R>* tw, hipStream_t st);
template <class R>
hipError_t launch_pair_mid(C2<R>* spec, const R* T, int M, int N, const PairGeom& g, const FftPlan& planM,
                           const C2<R>* tw, hipStream_t st);

}  // namespace se2n
