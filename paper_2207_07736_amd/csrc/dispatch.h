// dispatch.h -- which form of a kernel a call runs, as functions of its sizes and
// the device's compute units alone (plain C++: the library launches by them, and
// the probe library reports them).  All forms of a kernel give the same bits.
#pragma once

#include <stdint.h>

namespace rlsim_dev {

// Largest padding count of the register-resident (one thread per env) kernel;
// above it the two-phase wide kernel holds the words.  (262,144 envs x 500
// steps: D = 32 0.82-0.87 ms in registers; the wide kernel's eight-environment
// jump table, one word per lane, costs the same at every D up to 64, 0.88-0.94 ms
// at D = 48 and 64, where the register form, every thread updating all 64 words,
// takes 1.07-1.13 ms.)
constexpr uint32_t kMaxRegisterWords = 32u;

// Words of padding a thread of the register kernel holds, for D <= 32: 0, 4, 8 or
// 16, and above 16 in steps of four where the words set the pace, 32 elsewhere.
// An unused word costs three instructions a step.  A trajectory far past the
// 256 MB last-level cache (2^24 rows of 22 bytes: 369 MB) is bound by its stores
// instead, and those come out slower from the lighter kernels, unless no CU has
// more than one workgroup.  32 words / the fewest that hold D, us a launch:
//   envs x K          MB     D = 20       D = 24       D = 28
//   65,536 x 1,000   1,442   445 / 393    445 / 415    446 / 421
//   100,003 x 128      282    82 / 66      83 / 72      84 / 79
//   150,001 x 111      366   117 / 117    120 / 120    124 / 124
//   100,003 x 500    1,100   295 / 347    296 / 327    298 / 322
//   262,144 x 32       185    51 / 43      56 / 49      60 / 58
//   262,144 x 500    2,884   631 / 673    645 / 676    646 / 656
// More than four workgroups per CU:
//   300,000 x 40       264    84 / 84      85 / 88      89 / 87
//   1,048,576 x 4       92    77 / 75      99 / 88     121 / 114
//   1,048,576 x 128  2,953   687 / 745    709 / 761    759 / 739
// 12 words in 12 were no faster than in 16 (100,003 x 128: 76 / 68 us).
inline uint32_t register_words(uint32_t D, uint32_t n, uint32_t K, bool trajectory, uint32_t cus)
{
    if (D <= 8u) return (D + 3u) / 4u * 4u;
    if (D <= 16u) return 16u;
    const uint64_t rows = (uint64_t)n * K, per_cu = 256ull * cus;
    const bool light = !trajectory || n <= per_cu || rows < (n <= 4u * per_cu ? 1ull << 24 : 1ull << 23);
    return light ? (D + 3u) / 4u * 4u : 32u;
}

}  // namespace rlsim_dev
