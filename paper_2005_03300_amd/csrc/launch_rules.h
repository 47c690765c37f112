// Host-only rules of launches, free of HIP so that they can be tested by themselves.
#pragma once
#include <cstdint>

namespace gcn {

// Wavefronts of a workgroup of k_gemm_tall: each workgroup puts op(B) into LDS, so eight share it, unless the strips of 16 rows make so few
// workgroups that four leave every compute unit with no more than one, i.e. none reads op(B) twice.  Seven eighths of the compute units,
// half of them where op(B) has more than 400 rows, and never where it has more than 640: there the time it takes to put op(B)
// into LDS decides, and half as many wavefronts take twice as long.  Microseconds with eight and four:
//   rows                  5000         10000        14000        16384        20000        32768
//   128 x 16           5.33  4.41   5.48  4.56   5.50  4.57   5.49  4.55   6.34  5.40   6.52  5.62
//   256 x 24           8.80  8.03   9.02  8.55   9.20  9.17  10.62 11.10  10.73 11.97  11.36 13.17
//   256 x 64           14.2  12.4   15.0  13.2   15.9  14.6   17.0  16.8   17.3  19.3   18.2  20.7
//   500 x 24           15.9  14.2   16.9  18.8   19.4  20.2   19.3  20.3   19.6  22.3   20.0  23.2
//   602 x 64           24.3  23.3   27.6  52.0   28.1  53.8   27.9  54.9   51.1  68.0   53.9  85.5
// (602 x 64 takes two columns of workgroups, `panels`; 1200 x 24 on 3000 rows 21.5 and 26.0, 1900 x 24 31.7 and 43.6.  Narrow
// products gain up to twice as many rows, but not with 41 or 64 columns.)
inline int tall_waves(int64_t strips, int64_t panels, int64_t k, int64_t cus) {
    const int64_t workgroups = (strips + 3) / 4 * panels;
    return k <= 640 && workgroups <= (k > 400 ? cus / 2 : cus / 8 * 7) ? 4 : 8;
}

}  // namespace gcn
