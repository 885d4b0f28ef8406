// Host check of csrc/cx_columns.hpp: on rows of P columns cut into segments, walked tile by tile as the mixing
// kernels do it, no lane reads a column outside [0, P) and every column of the row is stored exactly once.  Row
// lengths from the shortest that each count of slices per lane is launched for.
#include <algorithm>
#include <cstdio>
#include <cstdlib>
#include <vector>

#include "cx_columns.hpp"

static void fail(const char *what, int slice, int U, int64_t P, int64_t b, int64_t e, int64_t col)
{
    std::printf("%s: slices of %d columns, %d per lane, P = %lld, piece [%lld, %lld), column %lld\n", what, slice, U,
                static_cast<long long>(P), static_cast<long long>(b), static_cast<long long>(e), static_cast<long long>(col));
    std::exit(1);
}

// `cols` columns from `at` on: bit q of mask = column at + q is wanted; loaded whole as soon as one is
static void check_load(unsigned mask, int cols, int64_t at, int slice, int U, int64_t P, int64_t b, int64_t e)
{
    if ((mask & ((1u << cols) - 1u)) == 0) return;
    if (at < 0) fail("a load before the row", slice, U, P, b, e, at);
    if (at + cols > P) fail("a load beyond the row", slice, U, P, b, e, at + cols - 1);
}

int main()
{
    unsigned rng = 7u;
    auto next = [&rng](int64_t n) { rng = rng * 1664525u + 1013904223u; return static_cast<int64_t>(rng >> 8) % n; };
    long pieces = 0;
    for (int slice : {4, 8})
        for (int U : {1, 2, 4}) {
            const int tile_cols = 64 * slice * U;
            for (int64_t P = U == 1 ? slice : tile_cols; P <= 3 * tile_cols + 9; P = P < 20 || (P + 12) % tile_cols < 24 ? P + 1 : P + 5)
                for (int S : {1, 2, 9}) {
                    std::vector<int64_t> cut{0, P};
                    for (int k = 1; k < S; ++k) cut.push_back(next(3) ? next(P + 1) : std::max<int64_t>(0, P - next(6)));
                    for (int64_t c = 0; c < P; c += tile_cols) cut.push_back(c);          // tiles end pieces as well
                    std::sort(cut.begin(), cut.end());
                    std::vector<int> stored(static_cast<size_t>(P), 0);
                    for (size_t k = 0; k + 1 < cut.size(); ++k) {
                        const int64_t b = cut[k], e = cut[k + 1], c0 = b / tile_cols * tile_cols;
                        if (b >= e || (b == c0 && e == c0 + tile_cols)) {                 // empty, or a full tile
                            for (int64_t c = b; c < e; ++c) ++stored[static_cast<size_t>(c)];
                            continue;
                        }
                        ++pieces;
                        for (int lane = 0; lane < 64; ++lane)
                            for (int u = 0; u < U; ++u) {
                                const int64_t place = c0 + slice * lane;
                                const int64_t at = place - row_end_slide(P, c0, place, U, tile_cols, slice) + u * 64 * slice;
                                const unsigned mask = slice_mask(at, slice, wanted_from(b, place, U), e);
                                check_load(mask, slice, at, slice, U, P, b, e);
                                for (int hh = 0; slice == 8 && hh < 2; ++hh)              // fp32 rows beside 16-bit ones
                                    check_load(mask >> (4 * hh), 4, at + 4 * hh, slice, U, P, b, e);
                                for (int q = 0; q < slice; ++q)
                                    if ((mask >> q) & 1u) {
                                        if (at + q < b || at + q >= e) fail("a store outside the piece", slice, U, P, b, e, at + q);
                                        ++stored[static_cast<size_t>(at + q)];
                                    }
                            }
                    }
                    for (int64_t c = 0; c < P; ++c)
                        if (stored[static_cast<size_t>(c)] != 1) fail("a column not stored exactly once", slice, U, P, 0, P, c);
                }
        }
    std::printf("ok %ld pieces\n", pieces);
    return 0;
}
