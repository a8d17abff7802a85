// Host-side checks of the pair path's geometry and index maps (no device
// code), over every side 2^a 3^b (a >= 2) up to 1024, N = 4 .. 64 and both
// data types that pair_fits accepts:
//  * the middle pass's workgroups cover every (column, block) once;
//  * the spectrum layout is a bijection of (slice, column, row) onto [0, N M/2 M);
//  * every tile fits the threads, elements per thread and LDS it is launched
//    with, and row tiles lie inside one block of rows;
//  * the radix sequences multiply to the length and read no twiddle beyond
//    the 3M/4 entries held in LDS.
// Prints "bad <count>" and exits with 1 when any check fails.
#include <cstdio>
#include <vector>

#include "se2n_pair.hpp"

using namespace se2n;

static long bad = 0, plans = 0;
static void check(bool ok, const char* what, int M, int N, int rs) {
    if (ok) return;
    if (++bad <= 20) printf("%s: M=%d N=%d real=%d\n", what, M, N, rs);
}

int main() {
    for (int M = 16; M <= 1024; M += 4) {
        int m = M;
        while (m % 2 == 0) m /= 2;
        while (m % 3 == 0) m /= 3;
        if (m != 1) continue;
        for (int ept : {4, 8, 16}) {
            long prod = 1;
            for (int s = 0; pair_radix(M, ept, s) != 0; ++s) {
                const int r = pair_radix(M, ept, s);
                const long e = prod > 1 ? (long)(prod - 1) * (M / (prod * r)) : 0;  // largest k TWSTEP
                const int reads = r == 16 ? 12 : r == 8 ? 4 : r == 4 ? 2 : r == 3 ? 2 : 1;
                check(reads * e < 3 * (M / 4), "twiddle range", M, ept, 0);
                check(ept >= 16 || r <= 8, "radix", M, ept, 0);
                prod *= r;
            }
            check(prod == M, "radix product", M, ept, 0);
        }
        for (int N = 4; N <= 64; ++N)
            for (int rs : {4, 8}) {
                if (!pair_fits(M, N, rs)) continue;
                ++plans;
                const int H = M / 2, nblk = pair_nblk(N), np = pair_count(N), hs = pair_hs(N), most = pair_max_threads(rs);
                const PairGeom g = pair_geom(M, N, rs, 256);
                std::vector<int> seen((size_t)H * nblk, 0);
                for (int i = 0; i < H * nblk; ++i) {
                    int kx = -1, blk = -1;
                    pair_mid_col(i, H, nblk, kx, blk);
                    if (kx < 0 || kx >= H || blk < 0 || blk >= nblk) { check(false, "column range", M, N, rs); continue; }
                    ++seen[(size_t)blk * H + kx];
                }
                for (int v : seen) check(v == 1, "columns", M, N, rs);
                if (N <= 6 || N == 31) {
                    std::vector<char> at((size_t)N * H * M, 0);
                    for (int s = 0; s < N; ++s)
                        for (int k = 0; k < H; ++k)
                            for (int y = 0; y < M; ++y) {
                                const long p = g.lay.col(s, k, H) + g.lay.row(y, H, N);
                                if (p < 0 || p >= (long)at.size()) { check(false, "layout range", M, N, rs); continue; }
                                check(!at[p], "layout", M, N, rs);
                                at[p] = 1;
                            }
                }
                check(M % g.lay.rb == 0 && (1 << g.lay.lg) == g.lay.rb, "row blocks", M, N, rs);
                for (int rows : {g.fwd_rows, g.inv_rows})
                    check(rows >= 1 && M % rows == 0 && g.lay.rb % rows == 0 && (rows & (rows - 1)) == 0, "rows", M, N, rs);
                auto tile = [&](int elems, int threads, int ept, size_t lds, const char* what) {
                    check(threads >= 64 && threads <= most && threads % 64 == 0 && elems <= ept * threads &&
                              lds <= (size_t)kPairLds, what, M, N, rs);
                };
                tile(g.fwd_rows * M, g.fwd_threads, g.fwd_ept, pair_lds_bytes(M, g.fwd_rows, rs), "forward tile");
                tile(g.inv_rows * g.inv_G * M, g.inv_threads, g.inv_ept,
                     pair_lds_bytes(M, g.inv_rows * g.inv_G, rs) + (g.inv_G < np ? (size_t)g.inv_rows * M * rs : 0),
                     "inverse tile");
                tile(hs * M, g.mid_threads, g.mid_ept, pair_lds_bytes(M, hs, rs), "middle tile");
                check(M / 4 * ((hs + g.mid_ept / 4 - 1) / (g.mid_ept / 4)) <= g.mid_threads, "product rows", M, N, rs);
                tile(np * M, g.all_threads, g.all_ept, pair_lds_bytes(M, np, rs), "whole rows");
                // compiled first stages step by whole row blocks
                for (int ms : {64, 128, 192, 256, 384, 512, 768, 1024})
                    if (ms == M) check(M / pair_radix(M, g.mid_ept, 0) % g.lay.rb == 0, "stage step", M, N, rs);
            }
    }
    printf("plans %ld bad %ld\n", plans, bad);
    return bad ? 1 : 0;
}
