// Host-side checks of the halved columns (PairLay, FP64; no device code), over
// every side and N = 4 .. 64 that pair_halves accepts:
//  * the middle pass's workgroups cover every (column, block, half) once;
//  * the layout of the two halves is a bijection of (slice, column, row, half)
//    onto [0, N M/2 M);
//  * the class positions of a table row are distinct, within the row, the even
//    classes before the odd ones;
//  * every tile fits the threads, elements per thread and LDS it is launched
//    with, its rows lie inside one block, and the compiled first and last stages
//    step by whole blocks;
//  * the radix sequences of these and of every other pair plan's side multiply to
//    the length and read no twiddle beyond the 3M/4 entries held in LDS, also
//    where every power is read.
// Prints "plans <count> bad <count>" and exits with 1 when any check fails.
#include <cstdio>
#include <vector>

#include "se2n_pair.hpp"

using namespace se2n;

static long bad = 0, plans = 0;
static void check(bool ok, const char* what, int M, int N) {
    if (ok) return;
    if (++bad <= 20) printf("%s: M=%d N=%d\n", what, M, N);
}

static void radices(int L, int ept, int M, int N) {
    long prod = 1;
    for (int s = 0; pair_radix(L, ept, s) != 0; ++s) {
        const int r = pair_radix(L, ept, s);
        const long e = prod > 1 ? (long)(prod - 1) * (L / (prod * r)) : 0;
        const int reads = r == 16 ? 12 : r == 8 ? 6 : r - 1;
        check(reads * e < 3 * (L / 4) && (r != 8 || 7 * e - L / 2 < L / 2), "twiddle range", M, N);
        check(ept >= 16 || r <= 8, "radix", M, N);
        prod *= r;
    }
    check(prod == L, "radix product", M, N);
}

int main() {
    for (int M = 16; M <= 1024; M += 4) {
        int m = M;
        while (m % 2 == 0) m /= 2;
        while (m % 3 == 0) m /= 3;
        if (m == 1)
            for (int ept : {4, 8, 16}) radices(M, ept, M, ept);
    }
    for (int M = 16; M <= 4096; M += 4)
        for (int N = 4; N <= 64; ++N) {
            check(!pair_halves(M, N, 4), "FP32", M, N);
            if (!pair_halves(M, N, 8)) continue;
            ++plans;
            const int H = M / 2, nblk = pair_nblk(N), hs = pair_hs(N), most = pair_max_threads(8);
            const PairGeom g = pair_geom(M, N, 8, 256);
            check(g.lay.halved == 1 && !g.whole_sr && !g.whole_dr, "halved", M, N);
            std::vector<int> seen((size_t)2 * H * nblk, 0);
            for (int i = 0; i < 2 * H * nblk; ++i) {
                int kx = -1, blk = -1, par = -1;
                pair_mid_half(i, H, nblk, kx, blk, par);
                if (kx < 0 || kx >= H || blk < 0 || blk >= nblk || par < 0 || par > 1) {
                    check(false, "column range", M, N);
                    continue;
                }
                ++seen[((size_t)blk * H + kx) * 2 + par];
            }
            for (int v : seen) check(v == 1, "columns", M, N);
            const int rb2 = g.lay.rb / 2;
            check((1 << g.lay.lg) == rb2 && H % rb2 == 0, "half blocks", M, N);
            // the layout is periodic in the slice and column: the smallest N of a side and its largest
            if (M <= 768 && (N % 16 == 0 || N % 16 == 7)) {
                std::vector<char> at((size_t)N * H * M, 0);
                for (int s = 0; s < N; ++s)
                    for (int k = 0; k < H; ++k)
                        for (int n = 0; n < H; ++n)
                            for (int par = 0; par < 2; ++par) {
                                const long p = g.lay.col(s, k, H) + g.lay.row(n, H, N) + par * rb2;
                                if (p < 0 || p >= (long)at.size()) { check(false, "layout range", M, N); continue; }
                                check(!at[p], "layout", M, N);
                                at[p] = 1;
                            }
            }
            const int QP = pair_qp(M, true);
            std::vector<char> pos(QP, 0);
            for (int ly = 0; ly <= M / 4; ++ly) {
                const int p = pair_class_pos(M, true, ly);
                check(p >= 0 && p < QP && !pos[p], "class position", M, N);
                check((ly & 1) ? p == pair_odd_pos(M) + ly / 2 : p == ly / 2 && p < pair_odd_pos(M), "class order", M, N);
                if (p >= 0 && p < QP) pos[p] = 1;
            }
            check(pair_table_bytes(M, N, 8, true) >=
                      ((size_t)(M / 4) * nblk + nblk) * (hs * (hs + 1) / 2) * QP * 8 + (size_t)(M / 4 + 1) * flag_stride(M),
                  "table", M, N);
            for (int rows : {g.fwd_rows, g.inv_rows})
                check(rows >= 2 && (rows & (rows - 1)) == 0 && rb2 % (rows / 2) == 0 && H % (rows / 2) == 0, "rows", M, N);
            auto tile = [&](int elems, int threads, int ept, size_t lds, const char* what) {
                check(threads >= 64 && threads <= most && threads % 64 == 0 && elems <= ept * threads &&
                          lds <= (size_t)kPairLds, what, M, N);
            };
            tile(g.fwd_rows * M, g.fwd_threads, g.fwd_ept, pair_lds_bytes(M, g.fwd_rows, 8), "row tile");
            tile(g.inv_rows * M, g.inv_threads, g.inv_ept, pair_lds_bytes(M, g.inv_rows, 8), "projection tile");
            tile(hs * H, g.mid_threads, g.mid_ept, pair_lds_bytes(H, hs, 8), "middle tile");
            check(g.fwd_ept == pair_row_ept(pair_fwd_rows(M, 8) * M, 8) && g.inv_ept == g.fwd_ept, "compiled elements", M, N);
            check((long)g.inv_ept / 4 * g.inv_threads >= (long)H * (g.inv_rows / 2), "fetched columns", M, N);
            check(H / 4 * ((hs + g.mid_ept / 4 - 1) / (g.mid_ept / 4)) <= g.mid_threads, "product rows", M, N);
            check(g.mid_grid >= 1 && g.mid_grid <= 2 * H * nblk, "walkers", M, N);
            check(H / pair_radix(H, g.mid_ept, 0) % rb2 == 0 && H / pair_last_radix(H, g.mid_ept) % rb2 == 0, "stage step", M, N);
            radices(H, g.mid_ept, M, N);
            radices(M, g.fwd_ept, M, N);
        }
    printf("plans %ld bad %ld\n", plans, bad);
    return bad ? 1 : 0;
}
