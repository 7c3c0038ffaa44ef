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
//          D x envs             K = 1       K = 32       K = 64       K = 96
//   101   256 x  32,768  1.00      25 / 22      38 / 36      51 / 51      67 / 67
//   201   128 x 131,072  1.00      42 / 29      64 / 65    100 / 103    142 / 144
//   240  1000 x  20,011  0.98      52 / 50      74 / 69      90 / 95    105 / 121
//   264  1100 x  20,011  0.54      72 / 89     86 / 116    109 / 157    152 / 199
//   307   512 x  50,000  1.00      69 / 47      84 / 71     105 / 96    132 / 123
//   317   129 x 200,000  0.52      77 / 88    147 / 135    205 / 209    261 / 283
//   420   700 x  50,000  0.68     109 / 88    125 / 118    146 / 156    173 / 198
//   472   300 x 131,072  0.59     133 / 84    157 / 127    189 / 185    226 / 242
//   503   160 x 262,144  0.62     136 / 94    188 / 151    244 / 221    298 / 303
//   660  1100 x  50,000  0.54    187 / 168    194 / 210    221 / 276    299 / 353
//   786  1000 x  65,536  0.98    214 / 104    230 / 141    245 / 187    268 / 225
// Above 64 steps batches whose drawn blocks hold 64 environments (wide_log2) need
// more.  Over 2,144 calls (18 batch sizes, 23 row lengths, 8 values of K) the choice
// is at most 3.6 % slower than loading in blocks of 256, ten calls by 2 % or more.
inline bool wide_draws(uint32_t n, uint32_t Dp, uint32_t K, uint32_t cus)
{
    const uint64_t chunk = 64ull * wide_lane_words(Dp), held = (Dp + chunk - 1u) / chunk * chunk;
    const uint64_t megabytes = 12ull * n * Dp / 1000000u * Dp / held;
    const uint64_t percent = 100ull * Dp / held;
    if (K <= 8u) return megabytes >= 180u;
    if (K <= 32u) return megabytes >= 190u && (Dp <= 1024u || percent >= 55u);
    if (K <= 64u) return megabytes >= 300u && percent >= 60u;
    return K <= 96u && megabytes >= (n <= 192u * cus ? 410u : 250u) && percent >= 75u;
}

// Batches that may run the wide kernel in blocks of fewer than 256 environments.
inline bool wide_small_batch(uint32_t n, uint32_t cus) { return ((n - 1u) >> 7) + 1u <= 2u * cus; }

// log2 of the environments in a block of the wide kernel, for rows of Dp words: as
// few (down to the jump table's eight) as still give every block a resident
// workgroup of its own, 256 beyond that.  Blocks of 64 and more fill whole
// stepping waves and go two to a CU; smaller ones leave lanes empty, and two per CU
// would step twice the waves.  256 per block / this rule, us a launch: 1,024 envs
// D = 4,096 K = 1 161 / 13, K = 500 2,490 / 262, D = 40 K = 500 302 / 246; 20,011
// envs D = 400 K = 500 519 / 326.  4,096 envs, D = 200, 512 blocks of 8 / 256 of
// 16: K = 1 9.9 / 7.8, K = 500 263 / 225.
// Blocks of 128 put two workgroups on some CUs where blocks of 256 put one on
// fewer: loaded calls gain where the replay's steps weigh more than the row's bytes,
// and lose where the bytes do.  256 / 128 per block: 36,000 envs D = 300 K = 1 27 / 32,
// K = 64 80 / 73; D = 1,000 K = 97 179 / 213, K = 300 467 / 432.  With up to 128 words and
// a trajectory past 2^24 rows, where the stores set the pace, they lose too (57,000
// envs, D = 100: K = 256 even, K = 400 10 % slower).  Drawn calls are bound by the
// draws, which need every SIMD: up to three blocks of 64 per CU they stay with
// those (36,000 envs, D = 1,000, K = 8, 256 / 128 / 64 per block 87 / 91 / 72).
// One-step calls that stream more than 110 MB of loaded state through blocks of 64
// lose from three blocks for two CUs on: 32,768 envs D = 400 34 / 35, K = 8 36.6 / 38.3.
inline uint32_t wide_log2(uint32_t n, uint32_t Dp, uint32_t K, uint32_t cus)
{
    uint32_t l = 3u;
    while (l < 8u && ((n - 1u) >> l) + 1u > (l < 6u ? cus : 2u * cus)) ++l;
    if (l == 7u) {
        if (wide_draws(n, Dp, K, cus)) return n <= 192u * cus ? 6u : 7u;
        if (Dp <= 128u && (uint64_t)n * K >= 1ull << 24) return 8u;
        const uint32_t steps = Dp <= 64u ? 1u : Dp <= 128u ? 64u : Dp <= 960u ? Dp / 6u : 160u;
        return K >= steps ? 7u : 8u;
    }
    if (l == 6u && n > 96u * cus && K <= 8u && !wide_draws(n, Dp, K, cus) && 12ull * n * Dp >= 110000000ull) return 8u;
    return l;
}

// Environments of a wave of the policy kernel.  Small batches leave SIMDs idle, and
// fewer environments per wave shorten the step; large ones pay for the cart-pole
// steps that such waves repeat.  The lines lie where the smaller form fills three
// workgroups per CU; a fourth takes it past the next form.  K = 32 with learner
// outputs, us a launch with 16 / 32 / 64 environments per wave, 256 CUs:
//   bf16  4,096 envs 41 / - / 80; 49,152 81 / - / 84; 65,536 96 / - / 84
//   fp32  4,096 envs 65 / 101 / 183; 49,152 148 / 160 / 186; 65,536 177 / 169 /
//         186; 98,304 252 / 239 / 291; 131,072 337 / 317 / 315
// The fp32 form with 32 is the last one whose workgroups share rows of statistics.
inline uint32_t policy_envs(uint32_t n, bool bf16, uint32_t cus)
{
    if (n <= 192u * cus) return 16u;
    return !bf16 && n <= 384u * cus ? 32u : 64u;
}

}  // namespace rlsim_dev
