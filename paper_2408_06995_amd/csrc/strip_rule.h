// Which layers with results in rows the short-K kernel (gemm_strip_kernel.h) is the faster one for: plain arithmetic, for the choice of
// the kernel and the plan query.
#pragma once
#include <stdint.h>

namespace fpq {

// Against the 128 x 160, 128 x 64 and register-staged 64 x 64 tiles, 3400 layers of random sizes in the hardware's encodings and as halves:
//   - from 144 pairs of a strip and 128 rows on (1000 x 64 -> 2560 1.8, 16384 x 320 -> 960 1.3 times); below, layers are at the launch
//     floor, where the weights' way through LDS costs up to 1 us (500 x 256 -> 1000: 3.6 and 4.5 us);
//   - not strips that are mostly empty, and not long rows that share lines at K above 256 (33000 x 320 -> 1001: 49.7 and 52.9 us);
//   - K of at most 128 is one step of the tiles, which then lose nothing by walking in steps.  Above 64 codes results of less than 4 M
//     values stay with them (geometric mean of the times 0.95 to 1.02 of this kernel's, a third of the layers faster by more than 5 %;
//     above 4 M 1.05 to 1.19 of it), and with 4-bit weights, whose conversion the tiles hide as well, rows that share lines too (0.94 to
//     0.98, 3000 x 112 -> 1398 6.8 and 7.7 us).  From 20 M values on the stores decide, and the tiles' 4-bit forms store as fast (0.97 to
//     1.03; 20000 x 64 -> 2208 28.4 and 34.9 us).
constexpr bool strip_rows(int64_t M, int64_t N, int64_t K, bool hardware, bool four_bit)
{
    if (N < 64 || (N % 32 != 0 && N > 512 && K > 256) || ((M + 127) / 128) * ((N + 63) / 64) < 144) return false;
    if (!hardware || K > 128) return true;
    if (K > 64 && (M * N < 4000000 || (four_bit && N % 32 != 0))) return false;
    return !four_bit || M * N < 20000000;
}

}  // namespace fpq
