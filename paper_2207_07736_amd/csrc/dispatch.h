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

// Words a lane of the wide kernel holds, for D > 32; a row is replayed in chunks of
// 64 lanes' words.
inline uint32_t wide_lane_words(uint32_t D)
{
    return D <= 64u ? 1u : D <= 128u ? 2u : D <= 256u ? 4u : D <= 512u ? 8u : 16u;
}

// Whether the wide kernel draws the padding parameters again instead of loading
// them, for rows of Dp words.  Short launches are bound by the bytes of the state,
// long ones by the replay's updates, to which the draw adds; a state that fits the
// 256 MB last-level cache between calls loads faster than it draws; and a draw
// costs the same for the unused words of a row's last chunk.  So what loading
// would bring is counted by the share of words in use.  Loaded / drawn, us a
// launch, by the megabytes of the three arrays and that share:
//          D x envs            K = 1        K = 32       K = 64       K = 96
//   101   128 x  65,536  1.00   23 / 20      38 / 39      55 / 59      75 / 79
//   201   128 x 131,072  1.00   42 / 30      62 / 63      97 / 101    140 / 139
//   240  1000 x  20,011  0.98   52 / 48      73 / 66      89 / 90     103 / 117
//   264  1100 x  20,011  0.54   67 / 85      84 / 109    105 / 148    146 / 189
//   307   512 x  50,000  1.00   68 / 47      82 / 69     102 / 94     129 / 120
//   472   300 x 131,072  0.59  129 / 85     156 / 127    187 / 183    226 / 238
//   420   700 x  50,000  0.68  111 / 85     129 / 112    153 / 151    185 / 193
//   604   192 x 262,144  0.75  164 / 93     213 / 157    267 / 226    321 / 300
//   660  1100 x  50,000  0.54  185 / 158    201 / 201    231 / 271    267 / 346
//   786  1000 x  65,536  0.98  213 / 99     230 / 138    244 / 183    262 / 234
// Over 68 such states at each of these K and at 8, the rule's choice is never more
// than 0.7 % slower than loading.
inline bool wide_draws(uint32_t n, uint32_t Dp, uint32_t K)
{
    const uint64_t chunk = 64ull * wide_lane_words(Dp), held = (Dp + chunk - 1u) / chunk * chunk;
    const uint64_t megabytes = 12ull * n * Dp / 1000000u * Dp / held;
    const uint64_t percent = 100ull * Dp / held;
    if (K <= 8u) return megabytes >= 160u;
    if (K <= 32u) return megabytes >= 220u;
    if (K <= 64u) return megabytes >= 250u && percent >= 60u;
    return K <= 96u && megabytes >= 300u && percent >= 70u;
}

// log2 of the environments in a block of the wide kernel: as few (down to the
// jump table's eight) as still give every block a resident workgroup of its
// own, 256 beyond that.  Blocks of 64 and more fill whole stepping waves and go
// two to a CU; smaller ones leave lanes empty, and two per CU would step twice
// the waves.  256 per block / this rule, us a launch: 1,024 envs D = 4,096
// K = 1 161 / 13, K = 500 2,490 / 262, D = 40 K = 500 302 / 246; 20,011 envs
// D = 400 K = 500 519 / 326; 65,536 envs D = 200 K = 500 412 / 387.  4,096 envs,
// D = 200, 512 blocks of 8 / 256 of 16: K = 1 9.9 / 7.8, K = 500 263 / 225.
inline uint32_t wide_log2(uint32_t n, uint32_t cus)
{
    uint32_t l = 3u;
    while (l < 8u && ((n - 1u) >> l) + 1u > (l < 6u ? cus : 2u * cus)) ++l;
    return l;
}

}  // namespace rlsim_dev
