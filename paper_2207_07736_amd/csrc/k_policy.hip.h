// k_policy.hip.h -- the simulation/inference loop with an on-device MLP policy
// fused into the K-step kernel (the paper's Future Work: simulation/inference
// fusion).  Per step every environment evaluates
//     h1 = tanh(W1 obs + b1), h2 = tanh(W2 h1 + b2), logits = W3 h2 + b3,
//     p0 = softmax(logits)[0] = 1 / (1 + exp(l1 - l0)),
// samples action 0 when u < p0 (u from Philox stream POLICY), then takes the
// cart-pole step exactly as the random-action kernel does.  On request it also
// records what an actor-critic learner reads per step: log pi(a|obs) of the
// action taken and the value head v = Wv h2 + bv on the same trunk.
//
// Matrix layout.  The MLP runs as the transposed product  Z^T = W * H^T  on the
// matrix instructions (weights = A operand, activations = B operand,
// environments = columns).  Hidden units are summed in eight groups of eight:
// group g = 2 s + h (s 0..3, h 0..1) holds units 16 s + 4 h + {0..3, 8..11}, and
// one lane supplies one group's eight values of its column.  Three forms share the
// same tables, each laying its output rows out so that the lane that computes a
// group's units also supplies them to the next layer: activations never move
// between lanes.
//   WaveForm64: a wave owns 64 environments (lane = environment for the
//     cart-pole) and runs two 32-column tiles of 32x32 instructions; in the
//     accumulator (lane l, register i: row 8(i/4) + 4(l/32) + i%4 of column l%32)
//     lane half h holds groups (s, h).
//   WaveForm32: one such tile, both halves of the wave carrying the same 32
//     environments.
//   WaveForm16: a wave owns 16 environments, every quarter of the wave carrying
//     the same ones, and runs one 16-column tile of 16x16 instructions (lane l,
//     register i: row 4(l/16) + i); quarter q holds groups q and 4 + q.  A lane
//     evaluates 32 tanh per step instead of 128, which is what a step costs when
//     the batch is too small to fill the GPU.
// The matrix units sum a group's eight products at once and the groups in the
// order they are issued, so the forms give the same bits.
#pragma once

#include "k_cartpole.hip.h"

namespace rlsim_dev {

typedef float floatx16 __attribute__((ext_vector_type(16)));
typedef float floatx4 __attribute__((ext_vector_type(4)));
typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef uint32_t uintx4 __attribute__((ext_vector_type(4)));

struct PolicyArgs {
    const void* w1;     // [64][4]  f32 or bf16 bits
    const float* b1;    // [64] or null
    const void* w2;     // [64][64]
    const float* b2;    // [64] or null
    const void* w3;     // [2][64]
    const float* b3;    // [2] or null
    const void* wv;     // [1][64] value head or null
    const float* bv;    // [1] or null
    float* p0;          // [K][n] or null
    float* logp;        // [K][n] or null
    float* value;       // [K][n] or null
    uint32_t* stats_acc;    // [ceil(n/256)][8] accumulators of workgroups that share a row of stats, zero between calls
};

// log pi(a) for two logits, from d = l1 - l0: with z = l_other - l_a,
// log pi(a) = -softplus(z) = -(max(z, 0) + log(1 + e^-|z|)).  e^-|z| is in
// (0, 1], so the log term is in [0, ln 2] and neither part can overflow.
__device__ __forceinline__ float log_pi(float d, uint32_t act)
{
    const float z = act ? -d : d;
    const float e = __builtin_amdgcn_exp2f(-__builtin_fabsf(z) * 1.44269504088896340736f);
    const float l1p = __builtin_amdgcn_logf(1.0f + e) * 0.69314718055994530942f;
    return -(__builtin_fmaxf(z, 0.0f) + l1p);
}

__device__ __forceinline__ float tanh_fast(float x)
{
    // tanh x = 1 - 2 / (1 + e^(2x)); e^(2x) = 2^(2 x log2 e) on the exp2 unit
    const float e = __builtin_amdgcn_exp2f(x * 2.88539008177792681472f);
    return __builtin_fmaf(-2.0f, __builtin_amdgcn_rcpf(1.0f + e), 1.0f);
}

// softmax over two logits, from d = l1 - l0: p0 = 1 / (1 + e^d)
__device__ __forceinline__ float policy_p0(float d)
{
    return __builtin_amdgcn_rcpf(1.0f + __builtin_amdgcn_exp2f(d * 1.44269504088896340736f));
}

__device__ __forceinline__ __bf16 to_bf16(float x) { return (__bf16)x; }

// Eight consecutive weights from memory that is only aligned to the weight's
// own size (the ABI asks for no more).
struct __attribute__((packed, aligned(2))) Bf16Run { uint16_t v[8]; };
struct __attribute__((packed, aligned(4))) F32Run { float v[4]; };

// Group and element of hidden unit c (unit = 16 s + 8 (j / 4) + 4 h + j % 4).
__device__ __forceinline__ uint32_t unit_group(uint32_t c) { return 2u * (c / 16u) + (c % 8u) / 4u; }
__device__ __forceinline__ uint32_t unit_elem(uint32_t c) { return 4u * ((c % 16u) / 8u) + c % 4u; }

// How a wave's lanes map to the matrix tiles.
struct WaveForm64 {
    static constexpr int kEnvs = 64;        // environments of a wave
    static constexpr int kTileRows = 32;
    static constexpr int kCols = 2;         // column tiles of 32
    static constexpr int kTiles = 2;        // row tiles of 32 in 64 hidden units
    static constexpr int kRegs = 16;        // accumulator registers of a tile
    static constexpr int kSteps = 4;        // K steps of a 64-unit sum
    using Acc = floatx16;
    // row of A operand `tile` that this lane supplies, as a hidden unit: the
    // lane's part plus a_step(tile)
    __device__ static uint32_t a_row(uint32_t lane) { return lane % 32u; }
    static constexpr uint32_t a_step(int tile) { return 32u * (uint32_t)tile; }
    // the group this lane supplies in K step s (both operands), plus g_step(s)
    __device__ static uint32_t group(uint32_t lane) { return lane / 32u; }
    static constexpr uint32_t g_step(int s) { return 2u * (uint32_t)s; }
    // first hidden unit of accumulator registers 4 r .. 4 r + 3 of `tile`, plus
    // c_step(tile, r)
    __device__ static uint32_t c_unit(uint32_t lane) { return 4u * (lane / 32u); }
    static constexpr uint32_t c_step(int tile, int r) { return 32u * (uint32_t)tile + 8u * (uint32_t)r; }
    // accumulator tile and register of element j of the group of K step s
    static constexpr int tile_of(int s, int) { return s / 2; }
    static constexpr int reg_of(int s, int j) { return 8 * (s % 2) + j; }
    __device__ static Acc mfma(bf16x8 a, bf16x8 b, Acc c)
    {
        return __builtin_amdgcn_mfma_f32_32x32x16_bf16(a, b, c, 0, 0, 0);
    }
};

// One 32-column tile of WaveForm64's layout, both halves of the wave carrying
// the same 32 environments.
struct WaveForm32 : WaveForm64 {
    static constexpr int kEnvs = 32;
    static constexpr int kCols = 1;
};

struct WaveForm16 {
    static constexpr int kEnvs = 16;
    static constexpr int kCols = 1;
    static constexpr int kTileRows = 16;
    static constexpr int kTiles = 4;        // row tiles of 16
    static constexpr int kRegs = 4;
    static constexpr int kSteps = 2;
    using Acc = floatx4;
    __device__ static uint32_t a_row(uint32_t lane) { return 16u * ((lane % 16u) / 8u) + lane % 8u; }
    static constexpr uint32_t a_step(int tile) { return 32u * ((uint32_t)tile / 2u) + 8u * ((uint32_t)tile % 2u); }
    __device__ static uint32_t group(uint32_t lane) { return lane / 16u; }
    static constexpr uint32_t g_step(int s) { return 4u * (uint32_t)s; }
    __device__ static uint32_t c_unit(uint32_t lane) { return 16u * (lane / 32u) + 4u * ((lane / 16u) % 2u); }
    static constexpr uint32_t c_step(int tile, int) { return a_step(tile); }
    static constexpr int tile_of(int s, int j) { return 2 * s + j / 4; }
    static constexpr int reg_of(int, int j) { return j % 4; }
    __device__ static Acc mfma(bf16x8 a, bf16x8 b, Acc c)
    {
        return __builtin_amdgcn_mfma_f32_16x16x32_bf16(a, b, c, 0, 0, 0);
    }
};

// LDS tables of a workgroup, as vectors of eight bfloat16 (16 bytes):
//   hidden-layer weights W2 [piece][group 8][row 64]: element j of (g, r) is
//     W2[r][unit j of group g];
//   bf16 MLP: W1 [row 64] (four weights, four zeros) and the output layer
//     [group 8][row 8]: rows 0,1 and 4,5 the logits, 2 and 6 the value, 3 and 7
//     zero, so that every lane finds its environment's outputs in registers 0-2;
// then floats: biases b1, b2 [64]; fp32 MLP: the output layer [3][64].
// The workgroup reads each weight once, in 16-byte runs (a 2-byte load per
// weight made the prologue 40 us of a 1M-environment bf16 launch).
template <bool F32>
struct PolicyTables {
    static constexpr uint32_t kPieces = F32 ? 3u : 1u;
    static constexpr uint32_t kW2 = 0u, kPieceVecs = 8u * 64u;
    static constexpr uint32_t kW1 = kW2 + kPieces * kPieceVecs;
    static constexpr uint32_t kOut = kW1 + (F32 ? 0u : 64u);
    static constexpr uint32_t kVecs = kOut + (F32 ? 0u : 64u);
    bf16x8 vec[kVecs];
    alignas(16) float b1[64], b2[64];
    float w3[F32 ? 192 : 1];
    uint32_t bad[kBlock / 64];      // fp32: waves that saw a W2 past kSplitLimit
    // Largest |W2| that the split hidden layer takes.  The activations are within
    // [-1, 1], so below it 64 products sum to at most 2^126: no partial sum of any
    // order can overflow, and no piece of a weight either (a finite weight above
    // 3.3961e38 would round to an infinite first piece).
    static constexpr float kSplitLimit = 0x1.0p120f;

    __device__ void fill(const PolicyArgs& w)
    {
        const uint32_t tid = threadIdx.x;
        uint16_t* t = reinterpret_cast<uint16_t*>(vec);
        if (tid < 64u) {
            b1[tid] = w.b1 ? w.b1[tid] : 0.0f;
            b2[tid] = w.b2 ? w.b2[tid] : 0.0f;
        }
        if constexpr (F32) {
            bool fits = true;
#pragma unroll
            for (uint32_t it = 0; it < 4u; ++it) {
                const uint32_t q = tid + it * kBlock, r = q / 16u, c = 4u * (q % 16u);
                const F32Run run = *reinterpret_cast<const F32Run*>(reinterpret_cast<const float*>(w.w2) + 4u * q);
                const uint32_t slot = (unit_group(c) * 64u + r) * 8u + unit_elem(c);
                ushort4 piece[3];
#pragma unroll
                for (int i = 0; i < 4; ++i) {
                    // w = p0 + p1 + p2 exactly, each rounded to nearest
                    const float v = run.v[i];
                    fits = fits && __builtin_fabsf(v) <= kSplitLimit;      // NaN does not
                    const __bf16 p0 = to_bf16(v);
                    const float r1 = v - (float)p0;
                    const __bf16 p1 = to_bf16(r1);
                    const __bf16 p2 = to_bf16(r1 - (float)p1);
                    reinterpret_cast<uint16_t*>(&piece[0])[i] = __builtin_bit_cast(uint16_t, p0);
                    reinterpret_cast<uint16_t*>(&piece[1])[i] = __builtin_bit_cast(uint16_t, p1);
                    reinterpret_cast<uint16_t*>(&piece[2])[i] = __builtin_bit_cast(uint16_t, p2);
                }
#pragma unroll
                for (uint32_t p = 0; p < 3u; ++p)
                    *reinterpret_cast<ushort4*>(t + p * kPieceVecs * 8u + slot) = piece[p];
            }
            const bool wave_bad = __builtin_amdgcn_ballot_w64(!fits) != 0u;
            if (tid % 64u == 0u) bad[tid / 64u] = wave_bad ? 1u : 0u;
            if (tid < 192u) {
                const float* w3p = reinterpret_cast<const float*>(w.w3);
                const float* wvp = reinterpret_cast<const float*>(w.wv);
                w3[tid] = tid < 128u ? w3p[tid] : (wvp ? wvp[tid - 128u] : 0.0f);
            }
        } else {
#pragma unroll
            for (uint32_t it = 0; it < 2u; ++it) {
                const uint32_t q = tid + it * kBlock, r = q / 8u, c = 8u * (q % 8u);
                const Bf16Run run = *reinterpret_cast<const Bf16Run*>(reinterpret_cast<const uint16_t*>(w.w2) + 8u * q);
                const uint32_t slot = (unit_group(c) * 64u + r) * 8u + unit_elem(c);
                *reinterpret_cast<ushort4*>(t + slot) = make_ushort4(run.v[0], run.v[1], run.v[2], run.v[3]);
                *reinterpret_cast<ushort4*>(t + slot + 64u * 8u) = make_ushort4(run.v[4], run.v[5], run.v[6], run.v[7]);
            }
            const uint16_t* w1p = reinterpret_cast<const uint16_t*>(w.w1);
            const uint16_t* w3p = reinterpret_cast<const uint16_t*>(w.w3);
            const uint16_t* wvp = reinterpret_cast<const uint16_t*>(w.wv);
            if (tid < 64u) {
                uint16_t* d = t + (kW1 + tid) * 8u;
#pragma unroll
                for (uint32_t c = 0; c < 4u; ++c) {
                    d[c] = w1p[tid * 4u + c];
                    d[4u + c] = 0u;
                }
            }
            // output layer: thread (o, c) places weight c of output o (3: zeros)
            const uint32_t o = tid / 64u, c = tid % 64u;
            const uint16_t v = o < 2u ? w3p[o * 64u + c] : o == 2u && wvp ? wvp[c] : (uint16_t)0u;
            const uint32_t slot = (kOut + unit_group(c) * 8u + o) * 8u + unit_elem(c);
            t[slot] = v;
            t[slot + 4u * 8u] = v;
        }
    }
};

// Where a lane reads the tables, as byte offsets of its part of every index; the
// tile, step and piece are then constants in the read instructions.  hide()
// makes the offsets opaque, so that the tables are read where they are used
// instead of held in registers across the steps.
template <class F, class Tables>
struct LaneTables {
    const char* base;
    uint32_t w2, w1, out, unit;
    __device__ LaneTables(const Tables& tab, uint32_t lane)
        : base(reinterpret_cast<const char*>(&tab)),
          w2((F::group(lane) * 64u + F::a_row(lane)) * 16u),
          w1(F::a_row(lane) * 16u),
          out((F::group(lane) * 8u + lane % 8u) * 16u),
          unit(F::c_unit(lane) * 4u)
    {
    }
    __device__ void hide() { asm volatile("" : "+v"(w2), "+v"(w1), "+v"(out), "+v"(unit)); }
    __device__ bf16x8 vec(uint32_t off, uint32_t index) const
    {
        return *reinterpret_cast<const bf16x8*>(base + off + index * 16u);
    }
    __device__ bf16x8 hidden(int piece, int s, int tile) const
    {
        return vec(w2, Tables::kW2 + (uint32_t)piece * Tables::kPieceVecs + F::g_step(s) * 64u + F::a_step(tile));
    }
    __device__ bf16x8 first(int tile) const { return vec(w1, Tables::kW1 + F::a_step(tile)); }
    __device__ bf16x8 output(int s) const { return vec(out, Tables::kOut + F::g_step(s) * 8u); }
    // four consecutive units of one of the float tables, starting with the unit
    // of accumulator register 4 r of `tile`
    __device__ floatx4 units(size_t table, int tile, int r) const
    {
        return *reinterpret_cast<const floatx4*>(base + unit + table + F::c_step(tile, r) * 4u);
    }
    // accumulators of one row tile, initialised with the biases
    __device__ typename F::Acc bias(size_t table, int tile) const
    {
        typename F::Acc c;
#pragma unroll
        for (int r = 0; r < F::kRegs / 4; ++r) {
            const floatx4 v = units(table, tile, r);
#pragma unroll
            for (int i = 0; i < 4; ++i) c[4 * r + i] = v[i];
        }
        return c;
    }
};

// ---------------------------------------------------------------------------
// bf16 MLP: all three layers on the bf16 matrix instructions.
// ---------------------------------------------------------------------------
template <class F>
struct MlpBf16 {
    using Form = F;
    using Tables = PolicyTables<false>;
    using Lane = LaneTables<F, Tables>;
    static constexpr int kWaves = 2;     // waves per SIMD its registers are sized for
    // Held across the steps: the output layer's start value (left to itself the
    // compiler builds it again, eight 64-bit moves a step, for the second column
    // tile) and, in WaveForm64, layer 1's weights.  With the core's own stores in
    // WaveForm64, 262,144 environments, K = 128: 1,031 -> 1,010 us; 4,096
    // environments, K = 64, learner outputs: 79 -> 76 us.
    static constexpr bool kHoldFirst = F::kEnvs == 64;
    typename F::Acc out0;
    bf16x8 a1[kHoldFirst ? F::kTiles : 1];

    __device__ void load(const PolicyArgs& w, uint32_t)
    {
        out0 = typename F::Acc{};
        out0[0] = w.b3 ? w.b3[0] : 0.0f;
        out0[1] = w.b3 ? w.b3[1] : 0.0f;
        out0[2] = w.bv ? w.bv[0] : 0.0f;
        asm volatile("" : "+v"(out0));
    }
    __device__ void after_fill(const Tables&, const Lane& lane_tab)
    {
        if constexpr (kHoldFirst) {
#pragma unroll
            for (int M = 0; M < F::kTiles; ++M) a1[M] = lane_tab.first(M);
        }
    }

    // Logit difference d = l1 - l0 and value v of this lane's environment; obs
    // is this lane's pre-step state.  The value row rides in the output tile at
    // no extra cost, so VAL changes nothing here.
    template <bool VAL>
    __device__ void eval(const CartState& obs, Lane& tab, uint32_t lane, float& d, float& v) const
    {
        using Acc = typename F::Acc;
        bf16x8 own = {};
        own[0] = to_bf16(obs.x);
        own[1] = to_bf16(obs.xd);
        own[2] = to_bf16(obs.th);
        own[3] = to_bf16(obs.thd);
        const bf16x8 zero8 = {};
        float l0 = 0.0f, l1 = 0.0f, lv = 0.0f;
        tab.hide();
#pragma unroll
        for (uint32_t T = 0; T < (uint32_t)F::kCols; ++T) {
            // layer 1: the observations sit in one group, supplied by the lanes
            // that own the tile's environments (WaveForm16: the first quarter)
            const bool mine = F::group(lane) == T;
            const bf16x8 bin = mine ? own : zero8;
            Acc c1[F::kTiles];
#pragma unroll
            for (int M = 0; M < F::kTiles; ++M)
                c1[M] = F::mfma(kHoldFirst ? a1[M] : tab.first(M), bin, tab.bias(offsetof(Tables, b1), M));
            // layer 2
            Acc c2[F::kTiles];
#pragma unroll
            for (int M = 0; M < F::kTiles; ++M) c2[M] = tab.bias(offsetof(Tables, b2), M);
#pragma unroll
            for (int s = 0; s < F::kSteps; ++s) {
                bf16x8 b;
#pragma unroll
                for (int j = 0; j < 8; ++j) b[j] = to_bf16(tanh_fast(c1[F::tile_of(s, j)][F::reg_of(s, j)]));
#pragma unroll
                for (int M = 0; M < F::kTiles; ++M)
                    c2[M] = F::mfma(tab.hidden(0, s, M), b, c2[M]);
            }
            // layer 3: registers 0-2 of every lane are its column's outputs
            Acc c3 = out0;
#pragma unroll
            for (int s = 0; s < F::kSteps; ++s) {
                bf16x8 b;
#pragma unroll
                for (int j = 0; j < 8; ++j) b[j] = to_bf16(tanh_fast(c2[F::tile_of(s, j)][F::reg_of(s, j)]));
                c3 = F::mfma(tab.output(s), b, c3);
            }
            if (F::kCols == 1 || mine) {
                l0 = c3[0];
                l1 = c3[1];
                lv = c3[2];
            }
        }
        d = l1 - l0;
        v = lv;
    }
};

// ---------------------------------------------------------------------------
// fp32 MLP.  What bounds it is the vector work (tanh, the splits, layer 3: active for
// 82 % of a launch) beside matrix instructions that overlap it in part (50 %); fp32
// matrix instructions share the SIMD with fp32 vector ones and do not.  Layer 1 runs
// on the fp32 matrix instructions and layer 3 on the VALU; layer 2, nine
// tenths of the arithmetic, runs on the bf16 ones at 16 times the fp32 rate, with
// every operand split into three bfloat16 pieces (8 + 8 + 8 bits, each rounded to
// nearest: the split is exact).  Of the nine products of the pieces the one left
// out, of the two last pieces, is at most 2^-34 of the whole.  The seven small
// ones are within 2^-7 of it and are summed on their own, so that only the eight
// leading sums (one a group) and the last addition round at the result's scale,
// where 64 fp32 products summed one by one round 64 times.  Error against 64 bits over
// 24 random networks, 524,288 environments with swinging poles: the value head
// 1.04e-7 rms (6.7e-7 at most) with fp32 products, 7.6e-8 (4.3e-7) with these, p0 3.9e-8
// and 3.3e-8; one weight per row with a bias that cancels it: within 2^-30 of the
// product.  1,048,576 environments, K = 16, learner outputs: 1.51 ms with fp32
// products, 1.19 ms with these (102 -> 128 TFLOP/s of the network's own arithmetic);
// six products (the three left out reach 2^-24 together) took 1.04 ms.
// WaveForm64 takes its two column tiles one after the other: both at once need
// 256 registers, and four waves per SIMD spill.
// ---------------------------------------------------------------------------
template <class F>
struct MlpF32 {
    using Form = F;
    using Tables = PolicyTables<true>;
    using Lane = LaneTables<F, Tables>;
    static constexpr int kWaves = F::kEnvs == 16 ? 2 : 3;
    // layer 1: 32-row tiles [row tile][K step] W1[row][2 s + lane / 32];
    // WaveForm16 [row tile][0] W1[row][lane / 16]
    float a1[F::kTiles][F::kTileRows / 16];
    float b3_0, b3_1, bv;
    const float* w2;        // for the plain layer 2
    bool plain;             // some W2 is past the split's limit, or not a number

    __device__ void load(const PolicyArgs& w, uint32_t lane)
    {
        const float* w1 = reinterpret_cast<const float*>(w.w1);
#pragma unroll
        for (int M = 0; M < F::kTiles; ++M)
#pragma unroll
            for (int s = 0; s < F::kTileRows / 16; ++s)
                a1[M][s] = w1[(F::a_row(lane) + F::a_step(M)) * 4u + F::group(lane) + F::g_step(s)];
        b3_0 = w.b3 ? w.b3[0] : 0.0f;
        b3_1 = w.b3 ? w.b3[1] : 0.0f;
        bv = w.bv ? w.bv[0] : 0.0f;
        w2 = reinterpret_cast<const float*>(w.w2);
    }
    __device__ void after_fill(const Tables& tab, const Lane&)
    {
        uint32_t any = 0u;
#pragma unroll
        for (uint32_t i = 0; i < kBlock / 64u; ++i) any |= tab.bad[i];
        plain = __builtin_amdgcn_readfirstlane(any) != 0u;
    }

    // x = p0 + p1 + p2 for the eight values of a group, two values per
    // conversion (left to itself the compiler converts each value a second time,
    // alone, to take the difference)
    __device__ static void split(const float (&x)[8], bf16x8 (&p)[3])
    {
        float r[8];
        uintx4 out[3];
#pragma unroll
        for (int j = 0; j < 8; ++j) r[j] = x[j];
#pragma unroll
        for (int i = 0; i < 3; ++i)
#pragma unroll
            for (int j = 0; j < 8; j += 2) {
                typedef __bf16 bf16x2 __attribute__((ext_vector_type(2)));
                const bf16x2 pair = {to_bf16(r[j]), to_bf16(r[j + 1])};
                uint32_t bits = __builtin_bit_cast(uint32_t, pair);
                asm("" : "+v"(bits));       // one conversion for both uses
                out[i][j / 2] = bits;
                if (i < 2) {
                    r[j] -= __uint_as_float(bits << 16);
                    r[j + 1] -= __uint_as_float(bits & 0xFFFF0000u);
                }
            }
#pragma unroll
        for (int i = 0; i < 3; ++i) p[i] = __builtin_bit_cast(bf16x8, out[i]);
    }

    // one K step of layer 2 in plain fp32, eight units of every group in turn: the
    // sum runs over (s 0..3, j, h) in every form.  A K step of WaveForm16 covers
    // two s: the quarters of the wave that hold the other one supply zeros.
    __device__ void plain_step(int step, const float (&x)[8], uint32_t lane, typename F::Acc (&c2)[F::kTiles]) const
    {
        const uint32_t g = F::group(lane) + F::g_step(step);
        constexpr uint32_t kParts = F::kTileRows == 32 ? 1u : 2u;
#pragma unroll
        for (uint32_t part = 0; part < kParts; ++part) {
            const bool on = kParts == 1u || lane / 32u == part;
#pragma unroll
            for (int j = 0; j < 8; ++j) {
                const uint32_t unit = 16u * (g / 2u) + 8u * ((uint32_t)j / 4u) + 4u * (g % 2u) + (uint32_t)j % 4u;
                const float b = on ? x[j] : 0.0f;
#pragma unroll
                for (int M = 0; M < F::kTiles; ++M) {
                    const float w = w2[(F::a_row(lane) + F::a_step(M)) * 64u + unit], a = on ? w : 0.0f;
                    if constexpr (F::kTileRows == 32)
                        c2[M] = __builtin_amdgcn_mfma_f32_32x32x2f32(a, b, c2[M], 0, 0, 0);
                    else
                        c2[M] = __builtin_amdgcn_mfma_f32_16x16x4f32(a, b, c2[M], 0, 0, 0);
                }
            }
        }
    }

    // Logit difference d = l1 - l0 and (if VAL) value v of this lane's environment.
    template <bool VAL>
    __device__ void eval(const CartState& obs, Lane& tab, uint32_t lane, float& d, float& v) const
    {
        using Acc = typename F::Acc;
        // layer 1 operands: K slot k is observation component k.  WaveForm64
        // supplies components h and 2 + h of its own environment (tile h) and, for
        // the other tile, of the environment of lane ^ 32, exchanged once per step
        const uint32_t h = lane / 32u;
        float own[2], other[2] = {0.0f, 0.0f};
        if constexpr (F::kTileRows == 32) {
            own[0] = h ? obs.xd : obs.x;
            own[1] = h ? obs.thd : obs.th;
        }
        if constexpr (F::kCols == 2) {
            other[0] = __shfl_xor(h ? obs.x : obs.xd, 32, 64);
            other[1] = __shfl_xor(h ? obs.th : obs.thd, 32, 64);
        }
        if constexpr (F::kTileRows == 16) {
            const bool odd = (lane & 16u) != 0u;
            const float pos = odd ? obs.xd : obs.x, ang = odd ? obs.thd : obs.th;
            own[0] = h ? ang : pos;
            own[1] = 0.0f;
        }
        float mine[3] = {0.0f, 0.0f, 0.0f}, send[3] = {0.0f, 0.0f, 0.0f};
#pragma unroll 1
        for (uint32_t T = 0; T < (uint32_t)F::kCols; ++T) {
            tab.hide();
            const bool own_tile = F::kCols == 1 || h == T;
            Acc c1[F::kTiles];
#pragma unroll
            for (int M = 0; M < F::kTiles; ++M) {
                c1[M] = tab.bias(offsetof(Tables, b1), M);
                if constexpr (F::kTileRows == 32) {
                    const float x0 = own_tile ? own[0] : other[0], x1 = own_tile ? own[1] : other[1];
                    c1[M] = __builtin_amdgcn_mfma_f32_32x32x2f32(a1[M][0], x0, c1[M], 0, 0, 0);
                    c1[M] = __builtin_amdgcn_mfma_f32_32x32x2f32(a1[M][1], x1, c1[M], 0, 0, 0);
                } else {
                    c1[M] = __builtin_amdgcn_mfma_f32_16x16x4f32(a1[M][0], own[0], c1[M], 0, 0, 0);
                }
            }
            Acc c2[F::kTiles];
            if (__builtin_expect(plain, 0)) {
#pragma unroll
                for (int M = 0; M < F::kTiles; ++M) c2[M] = tab.bias(offsetof(Tables, b2), M);
                uint32_t at_lane = lane;
                asm volatile("" : "+v"(at_lane));       // no address of this path outside it
#pragma unroll
                for (int s = 0; s < F::kSteps; ++s) {
                    float x[8];
#pragma unroll
                    for (int j = 0; j < 8; ++j) x[j] = tanh_fast(c1[F::tile_of(s, j)][F::reg_of(s, j)]);
                    plain_step(s, x, at_lane, c2);
                }
            } else {
                // the small products, smallest first within four groups; the row
                // tiles' chains alternate
                constexpr int kHalf = F::kSteps / 2;
                constexpr int kW[7] = {2, 1, 2, 0, 1, 1, 0}, kX[7] = {1, 2, 0, 2, 1, 0, 1};
                bf16x8 lead[F::kSteps];
#pragma unroll
                for (int M = 0; M < F::kTiles; ++M) c2[M] = Acc{};
#pragma unroll
                for (int s0 = 0; s0 < F::kSteps; s0 += kHalf) {
                    bf16x8 p[kHalf][3];
#pragma unroll
                    for (int i = 0; i < kHalf; ++i) {
                        float x[8];
#pragma unroll
                        for (int j = 0; j < 8; ++j)
                            x[j] = tanh_fast(c1[F::tile_of(s0 + i, j)][F::reg_of(s0 + i, j)]);
                        split(x, p[i]);
                        lead[s0 + i] = p[i][0];
                    }
#pragma unroll
                    for (int pr = 0; pr < 7; ++pr)
#pragma unroll
                        for (int i = 0; i < kHalf; ++i)
#pragma unroll
                            for (int M = 0; M < F::kTiles; ++M)
                                c2[M] = F::mfma(tab.hidden(kW[pr], s0 + i, M), p[i][kX[pr]], c2[M]);
                }
                // 52 bytes of scratch in the two-tile form without it
                if constexpr (F::kCols == 2) __builtin_amdgcn_sched_barrier(0);
                // the leading products on the bias, and the small ones' sum
#pragma unroll
                for (int M = 0; M < F::kTiles; ++M) {
                    Acc c = tab.bias(offsetof(Tables, b2), M);
#pragma unroll
                    for (int s = 0; s < F::kSteps; ++s) c = F::mfma(tab.hidden(0, s, M), lead[s], c);
                    c2[M] += c;
                }
            }
            // layer 3 on the VALU: each group's units in order, then the groups
            // as (s 0 + s 2) + (s 1 + s 3) and last the two halves h
            float part[3][F::kSteps];
#pragma unroll
            for (int s = 0; s < F::kSteps; ++s) {
#pragma unroll
                for (int o = 0; o < 3; ++o) part[o][s] = 0.0f;
#pragma unroll
                for (int j4 = 0; j4 < 8; j4 += 4) {
                    const int M = F::tile_of(s, j4), r = F::reg_of(s, j4);
                    floatx4 w3[3];
#pragma unroll
                    for (int o = 0; o < (VAL ? 3 : 2); ++o)
                        w3[o] = tab.units(offsetof(Tables, w3) + 256 * o, M, r / 4);
#pragma unroll
                    for (int i = 0; i < 4; ++i) {
                        const float hv = tanh_fast(c2[M][r + i]);
#pragma unroll
                        for (int o = 0; o < (VAL ? 3 : 2); ++o) part[o][s] = __builtin_fmaf(w3[o][i], hv, part[o][s]);
                    }
                }
            }
#pragma unroll
            for (int o = 0; o < (VAL ? 3 : 2); ++o) {
                float sum;
                if constexpr (F::kTileRows == 32) {
                    sum = (part[o][0] + part[o][F::kSteps / 2]) + (part[o][1] + part[o][F::kSteps - 1]);
                } else {
                    sum = part[o][0] + part[o][1];
                    sum = sum + __shfl_xor(sum, 32, 64);
                }
                // the other tile's sum belongs to lane ^ 32
                if (own_tile) mine[o] = sum;
                else send[o] = sum;
            }
        }
        float out[3] = {0.0f, 0.0f, 0.0f};
#pragma unroll
        for (int o = 0; o < (VAL ? 3 : 2); ++o) {
            const float recv = F::kCols == 2 ? __shfl_xor(send[o], 32, 64) : __shfl_xor(mine[o], F::kTileRows, 64);
            out[o] = mine[o] + recv;
        }
        d = (out[1] + b3_1) - (out[0] + b3_0);
        v = VAL ? out[2] + bv : 0.0f;
    }
};

// CartCore hook of the policy kernel: stores the row of the lanes that own an
// environment's outputs.
template <bool REC>
struct PolicyRows {
    bool own;
    uint32_t off4, off1;
    size_t plane;
    float* obs;
    uint8_t* act_row;
    float* rew_row;
    uint8_t* done_row;
    __device__ __forceinline__ void record(const CartState& s, uint32_t act, uint32_t d)
    {
        if (REC && own) {
            *at(act_row, off1) = (uint8_t)act;
            *at(done_row, off1) = (uint8_t)d;
            *at(obs, off4) = s.x;
            *at(obs + plane, off4) = s.xd;
            *at(obs + 2 * plane, off4) = s.th;
            *at(obs + 3 * plane, off4) = s.thd;
            *at(rew_row, off4) = 1.0f;
        }
    }
    __device__ __forceinline__ void operator()(uint32_t, bool) {}
    __device__ __forceinline__ void advance()
    {
        obs += 4 * plane;
        act_row += plane;
        rew_row += plane;
        done_row += plane;
    }
};

// One row of the block statistics from the workgroups that share a
// 256-environment block.
__device__ __forceinline__ void share_block_stats(uint32_t* stats, uint32_t* acc, uint32_t blk, uint32_t parts,
                                                  uint32_t c0, uint32_t c1, uint32_t c2, uint32_t c3)
{
    __shared__ uint32_t part[kBlock / 64][4];
    const uint32_t v0 = wave_sum(c0), v1 = wave_sum(c1), v2 = wave_sum(c2), v3 = wave_sum(c3);
    const uint32_t wave = threadIdx.x / 64u;
    if (threadIdx.x % 64u == 0u) {
        part[wave][0] = v0;
        part[wave][1] = v1;
        part[wave][2] = v2;
        part[wave][3] = v3;
    }
    __syncthreads();
    if (threadIdx.x < 4u) {
        uint32_t sum = 0u;
#pragma unroll
        for (int w = 0; w < (int)(kBlock / 64); ++w) sum += part[w][threadIdx.x];
        add_shared_stats(stats, acc, blk, parts, threadIdx.x, sum);
    }
}

// Fused policy + cart-pole kernel.  Every lane takes part in the MLP (the
// matrix instructions need the whole wave); lanes past n_envs carry a zero
// state and store nothing.  OUT: some of the per-step policy outputs (p0,
// log pi, value) are recorded; each row pointer may still be null.
template <class Mlp, bool REC, bool STATS, bool OUT>
__global__ __launch_bounds__(kBlock) __attribute__((amdgpu_waves_per_eu(Mlp::kWaves)))
void k_policy_fused(StepArgs a, PolicyArgs w)
{
    using F = typename Mlp::Form;
    __shared__ __align__(16) typename Mlp::Tables tab;
    const uint32_t lane = threadIdx.x % 64u;
    tab.fill(w);
    Mlp mlp;
    mlp.load(w, lane);

    const uint32_t blk = xcd_block();
    const uint32_t env = (blk * (kBlock / 64u) + threadIdx.x / 64u) * (uint32_t)F::kEnvs + lane % (uint32_t)F::kEnvs;
    const bool live = env < a.n;
    const DevParams& p = a.p;
    // WaveForm64: every lane owns its environment, and the core stores the rows
    // itself (262,144 environments, K = 64: 519 -> 515 us against PolicyRows there)
    constexpr bool kWhole = F::kEnvs == 64;
    CartCore<REC && kWhole, STATS> core(p, env);
    if (live) {
        core.load(a);
    } else {
        core.s = CartState{0.0f, 0.0f, 0.0f, 0.0f};
        core.ep = 0u;
        core.ep_start = 0u;
    }
    const bool own = live && lane < (uint32_t)F::kEnvs;
    if (REC && kWhole) core.set_rows(a, 0);
    NoPad nopad;
    PolicyRows<REC && !kWhole> rows{own, env * 4u, env, a.n, a.obs, a.action, a.reward, a.done};
    __syncthreads();
    typename Mlp::Lane lane_tab(tab, lane);
    mlp.after_fill(tab, lane_tab);

    size_t out_row = 0u;        // wave-uniform, as the row pointers
    uint4 pw = make_uint4(0u, 0u, 0u, 0u);
    for (uint32_t k = 0; k < a.K; ++k) {
        const uint32_t t = a.t0 + k;
        if (k == 0u || ((t + 1u) & 7u) == 0u) core.draw_reset((t + 1u) >> 3);
        if (k == 0u || (t & 3u) == 0u) pw = philox(core.gid, t >> 2, STREAM_POLICY, p.key0, p.key1);
        const float u = u24(pick_word(pw, t & 3u));
        float d, v;
        mlp.template eval<OUT>(core.s, lane_tab, lane, d, v);
        const float p0 = policy_p0(d);
        const uint32_t act = (u < p0) ? 0u : 1u;
        if (OUT && own) {
            if (w.p0) *at(w.p0 + out_row, env * 4u) = p0;
            if (w.logp) *at(w.logp + out_row, env * 4u) = log_pi(d, act);
            if (w.value) *at(w.value + out_row, env * 4u) = v;
        }
        if constexpr (kWhole) {
            if (live) core.step_with(act, nopad);
            if (REC) core.advance_rows();
        } else {
            core.step_with(act, rows);
            if (REC) rows.advance();
        }
        if (OUT) out_row += a.n;
    }
    if (own) core.store(a);
    if (STATS) {
        const uint32_t c0 = own ? core.n_eps : 0u, c1 = own ? core.finished_length_sum(a.K) : 0u,
                       c2 = own ? core.n_term : 0u, c3 = own ? core.n_trunc : 0u;
        if constexpr (F::kEnvs == 64) {
            store_block_stats(a.stats, blk, c0, c1, c2, c3);
        } else {
            constexpr uint32_t kShare = (uint32_t)kBlock / (F::kEnvs * (kBlock / 64));     // workgroups per block
            const uint32_t groups = (a.n + kBlock / kShare - 1u) / (kBlock / kShare);
            const uint32_t b256 = blk / kShare;
            share_block_stats(a.stats, w.stats_acc, b256, min(kShare, groups - b256 * kShare), c0, c1, c2, c3);
        }
    }
}

}  // namespace rlsim_dev
