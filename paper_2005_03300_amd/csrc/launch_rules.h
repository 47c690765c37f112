// Host-only rules of launches, free of HIP so that they can be tested by themselves.
#pragma once
#include <cstdint>

namespace gcn {

// Wavefronts of a workgroup of k_gemm_tall: eight or four, of up to eight strips of 16 rows per compute unit (with more the launch is capped),
// in `panels` columns of workgroups.  Each workgroup puts its part of op(B) into LDS, which eight share.  Four where the busiest
// compute unit then has fewer wavefronts: with one column of workgroups up to 16 K rows, where each has no more than one of either
// kind.  Not where the workgroups together read so much of op(B), more than 400 rows for each compute unit, that half as many
// wavefronts take longer for it; with three workgroups on the busiest up to 160 rows, with more never.  Microseconds with eight and four:
//   rows                  5000         10000        14000        16384        20000        32768
//   128 x 16           5.33  4.41   5.48  4.56   5.50  4.57   5.49  4.55
//   256 x 24           8.80  8.03   9.02  8.55   9.20  9.17  10.62 11.10  10.73 11.97  11.36 13.17
//   256 x 64           14.2  12.4   15.0  13.2   15.9  14.6   17.0  16.8   17.3  19.3   18.2  20.7
//   500 x 24           15.9  14.2   16.9  18.8   19.4  20.2   19.3  20.3   19.6  22.3   20.0  23.2
//   602 x 64           24.3  23.3   27.6  52.0   28.1  53.8   27.9  54.9   51.1  68.0   53.9  85.5
// (602 x 64 takes two columns of workgroups.)  On 3000 rows 1200 x 16 20.4 and 19.0, 1200 x 24, in two, 21.3 and 26.7.  Two columns: 100 x 100
// on 18 K 13.3 and 12.4, on 10 K, where both have eight wavefronts on the busiest, 128 x 128 9.8 and 10.3; four: 100 x 256 on 10 K
// 13.5 and 12.8, 200 x 256 22.1 and 27.1.  Of 2025 sizes, 256 to 1900 rows of op(B), 8 to 256 columns and 500 to 32768 rows, the slower is
// taken by more than 5 % for 63, by 16 % at the most (500 x 24 on 10 K is one of them; always eight 927, by 33 %).
inline int tall_waves(int64_t strips, int64_t panels, int64_t k, int64_t cus) {
    if (strips > 8 * cus) return 8;
    const int64_t of_four = (strips + 3) / 4 * panels, of_eight = (strips + 7) / 8 * panels;
    const int64_t each = (of_four + cus - 1) / cus;
    if (4 * each >= 8 * ((of_eight + cus - 1) / cus)) return 8;
    if (each > 1) return each <= 3 && k <= 160 ? 4 : 8;
    return k * of_four <= 400 * cus ? 4 : 8;
}

// Tiles of 16 columns per wavefront of a dense product whose columns go in equal shares of at most NT tiles, 80 as three and two and not as four and
// one; 0: as many as NT.  While operand and result are in the memory-side cache: 64 x 80 on 120 K rows 22.9 -> 19.6 us, 256 x 96 82.5 -> 69, 16 x 96 on
// 200 K 20.0 -> 19.4.  Beyond it the pieces of 48 columns, which are no whole lines, cost more (1 M rows of 16 x 96 148 and 164, of 128 x 67
// 327 and 384).  With a mask, which is read in the same pieces, while it and the result are in the L2s (32 MB; 16 x 80 on 20 K rows 0.92 of
// the time, on 120 K 16.9 and 19.4 us, 3 x 68 on 200 K 29.5 and 32.7, 41 x 80 on 326 K 63 and 77), and where the product takes longer than they do
// (128 x 68 to 96 on 65 K to 200 K 0.91 to 1.04, 256 x 80 on 120 K 0.82).
inline int equal_shares(int64_t M, int64_t N, int64_t K, bool mask, int NT) {
    const int tiles = (int)((N + 15) / 16), shares = (tiles + NT - 1) / NT, equal = (tiles + shares - 1) / shares;
    if (equal > 4 || M * (K + N) * 4 >= (192ll << 20)) return 0;
    return !mask || K >= 128 || M * N * 8 <= (32ll << 20) ? equal : 0;
}

// Whether rows of up to 15 columns, no whole 16 bytes, leave k_gemm_tall as single columns of four rows (SINGLE) and not four columns at a time: where
// every wavefront has one long strip and the busiest compute unit two workgroups of eight, 32 K to 64 K rows.  All of them read at the same time there, and
// that form of the loop puts fewer reads of op(B) together; with fewer workgroups, or a second strip for some wavefronts, it is the slower.  Microseconds
// with single columns and with four, 15 columns (30 K, 80 K and 200 K rows: as they were when all ragged rows left so):
//   rows              30 K          33 K          40 K          60 K          65 K          80 K          200 K
//   of 300 floats 10.9   9.0    12.0  11.6    13.3  13.8    15.1  16.3    15.8  17.1    22.7  20.4    48.9  44.7
//   of 409        13.7  12.2    15.5  17.1    16.9  17.9    19.2  20.5    20.1  21.6    29.4  26.2    80.0  73.3
//   of 602        18.3  16.0    21.1  23.3    23.2  24.5    26.3  28.4    27.8  29.9    41.3  36.5   116   111
//   of 700        20.8  18.2    23.5  26.1    25.8  27.4    29.5  31.9    31.0  33.8    46.5  41.1   133   123
// (Of 250 floats 36 K to 65 K rows take 0.92 to 1.02 with four; around 100 K rows of 409 and 602 single columns would be the faster too, by 6 to 8 %, of
// 300, 500 and 700 they are not.)
inline bool single_columns(int64_t strips, int64_t k, int64_t cus) { return k >= 300 && strips > 8 * cus && strips <= 16 * cus; }

// How many of the rows without entries a chunk of a product zeroes (zero_share), or 0: they take a launch of their own, which writes whole rows
// at the rate of the memory and costs a few microseconds.  A lane group of lpr lanes holds a row of a tile of lpr * vec columns.
// Microseconds with a launch and with shares, random matrices:
//  - No more than a chunk has entries.
//  - The stores of a wavefront one after another, and their list, 64 rows at a time, must be short beside the product: up to 20
//    stores of 240 rows they are (12.9 -> 12.0 with 139 rows of 16 floats, 21.9 -> 20.0 with 140 of 128; but masked 12.7 -> 13.9 with
//    274 of 16), more only where there are wavefronts enough to hide them, 25 to a store (3000 rows of 64 18.1 -> 19.2 with 32
//    stores on 16 wavefronts; of 31 35.4 -> 42.4 with 131 on 8, 41.9 -> 45.9 with 118 on 506, 57.2 -> 53.1 with 68 on 1755; of 41
//    70.4 -> 74.3 with 90 on 2195, 160.5 -> 149.6 with 138 on 5045; of 128 27.5 -> 25.1 with 30 on 796).
//  - Where a row is written tile by tile and the tiles are no whole lines, the pieces of a line must meet in a cache: results up to
//    the L2s' 32 MB (18.0 -> 16.3 with 100 floats, 12 MB), or up to the 256 MB behind them with few such rows (400 K of 36: 11
//    stores 68.4 -> 69.0, 17 73.1 -> 77.5).  1 M of 300, 0.3 to 0.8 of them empty, 1551 -> 1701 to 904 -> 1294, of 100 574 -> 595
//    to 334 -> 461; but of 128 356 -> 340 to 268 -> 234, of 160 466 -> 434 to 331 -> 283.
inline int share_of_empty_rows(int64_t rows, int64_t n_empty, int64_t nchunks, int64_t chunk, int lpr, int vec, int32_t f, int64_t ldz, uintptr_t Z) {
    if (n_empty <= 0 || n_empty > nchunks * chunk) return 0;
    const int64_t tiles = (f + lpr * vec - 1) / (lpr * vec), share = (n_empty + nchunks - 1) / nchunks;
    const int64_t at_once = 64 / lpr, stores = (share + at_once - 1) / at_once;
    if ((stores > 20 || share > 240) && 25 * stores > nchunks * tiles) return 0;
    const bool whole = tiles == 1 || (ldz % 32 == 0 && Z % 128 == 0);
    return whole || rows * ldz <= (8 << 20) || (stores <= 10 && rows * ldz <= (64 << 20)) ? (int)share : 0;
}

// Wavefronts of a workgroup that adds up 64 results (see sum_of_parts), for the sums of a launch with up to `parts` partial results each: one
// to a partial result, up to 16.  More of them only wait (16 always: layer calls with a bias, 602-256 on 64 vertices 34.3 us, so 29.1).
constexpr int sum_waves(int64_t parts) { return parts < 1 ? 1 : (parts < 16 ? (int)parts : 16); }

// Whether a matrix of short rows gets a copy at an equal pitch for k_spmm_short (see build_short).  Not where the copy is beyond the L2s (3 M
// places of 8 bytes), more than half padding, and rows of 16 entries and more are in most wavefronts of that kernel (32 rows at the
// widths that take so many), so that all of its lanes walk as far as these: rows of 0 to 64 entries of which most are
// short, 5 to 7 columns, against k_spmm_split: 60 K of mean 12.5 15.7 -> 13.1 us, of mean 21 18.0 -> 15.1, 52 K 13.8 -> 13.0; but 44 K
// (12.7 us) and 60 K of mean 5 with one long row (10.4) stay.
inline bool short_copy_pays(int64_t rows, int64_t pitch, int64_t nnz, int64_t rows_of_16) {
    return rows * pitch <= (3 << 20) || 2 * rows * pitch <= 5 * nnz || rows_of_16 * 32 < rows;
}

}  // namespace gcn
