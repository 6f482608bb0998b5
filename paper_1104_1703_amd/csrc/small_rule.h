// Where the one-workgroup call on small levels takes its deepest level as a
// matrix product (coarse_core.h).  No device code.
#pragma once

#include <cstddef>

namespace mg {
namespace small {

// The product takes 64 rows at a time, from registers for a level of up to 64
// cells, else from memory, some 3 us a time; a pass over the second of two levels
// in registers takes about 0.2 us.  Calls of two levels, matrix against 8, 32 and
// 64 passes, FP64: 8^3 + 4^3 8.4 us / 7.9 12.1 18.5, 10^3 + 5^3 11.5 / 9.0 13.6
// 20.4, 12^3 + 6^3 17.4 / 10.2 14.4 21.2, 8 x 16^2 + 4 x 8^2 18.8 / 11.0 14.5 21.3.
// Alone they meet at a pass for every five cells (FP64) or six and a half (FP32);
// within a solve the matrix comes from further away and 32 passes equal 130 to 150
// cells (a cycle of 80 x 96 x 96, 5 x 6 x 6 in the deepest: 142.1 us with the
// matrix, 134.1 relaxed, of 80^3, 5^3, 128.5 and 127.1, FP32 124.6 and 126.1).
// The second of two levels is relaxed up to a pass for every five.  Beyond two levels
// the relaxation is the general path's, 28 us at 4 passes and 34 at 32 where
// 16^3 + 8^3 + 4^3 takes 16.5.
constexpr int DEEP_MAX = 256;  // cells; a matrix of 512 KB
inline bool deep_product(int levels, size_t cells, long long passes) {
    return levels > 1 && cells <= (size_t)DEEP_MAX && !(levels == 2 && passes * 5 <= (long long)cells);
}

}  // namespace small
}  // namespace mg
