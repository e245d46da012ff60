// The DiT-block operations on either side of the attention core, for gfx950:
//
//   lp_qkv_projection   y = x W^T + b cut into q | k | v, with the per-head RMS normalisation
//                       and the 3-D rotary encoding of q and k done in the product's epilogue
//   lp_linear           y = x W^T + b (the block's output projection)
//   lp_qk_norm_rope     the normalisation + rotation alone, in place, for q / k that were
//                       projected elsewhere
//
// The paper leaves the block's internals open (Sec. 5.1: 30 DiT blocks whose atomic units are
// the patches of Sec. 3.1); the form taken is stated in include/lp.h.
//
// The product is computed TRANSPOSED, C^T[feature, token] = W . X^T with bf16 MFMA 16x16x32
// (A = rows of W, B = rows of x, both k-contiguous, both streamed global -> LDS without
// passing through registers): in the accumulator layout a lane then holds, for ONE token, four
// consecutive features of every 16-feature block, so the sum of squares of a head is an in-lane
// sum plus two exchanges inside the wavefront, and the two elements of a rotary pair sit in
// neighbouring registers.  16x16x32 and not 32x32x16: the part is limited by power, and a loop of
// nothing but products on N(0,1) operands sustains 2077 TFLOP/s with the former, 1837 with the
// latter (2480 and 2460 on zeros).
//
// Work decomposition.  A workgroup owns a tile of features x tokens (struct Tiling: the sizes, how
// its wavefronts share it, and the LDS stages); k advances in tiles of 64.  Which tiling a
// call runs, and how the tiles that do not fill a round of the compute units are cut, is chosen
// from the sizes in pick_plan.
#include <hip/hip_runtime.h>

#include <atomic>
#include <cmath>
#include <type_traits>

#include "lp_device.h"

namespace {

using namespace lp;

constexpr int kBK = 64;                  // k per LDS stage
constexpr int kRowBytes = kBK * 2;       // one tile row: 64 bf16
constexpr int kPanel = 8;                // token tiles per panel of the tile order
constexpr int kMaxPairs = 64;            // rotary pairs per head (head_dim <= 128)

// What the normalisation + rotation needs besides the data.
struct RopeArgs {
    float turns[kMaxPairs][4];   // pair p: turns (angle / 2 pi) per unit of the t, h, w coordinate; [3] unused
    FastDiv hw, w;               // grid_h * grid_w and grid_w
    int32_t grid_h;
    int32_t off[3];
    float eps;
};

struct GemmArgs {
    const __bf16 *x, *w;
    const float *bias;           // [d_out] or nullptr
    __bf16 *out[3];              // plain: out[0] = y [n, d_out]; qkv: q, k, v [n, heads, head_dim]
    const float *gain[2];        // qkv: gain_q, gain_k [heads, head_dim]
    int32_t n, d_in, d_out;
    int32_t heads;               // qkv: heads; d_out = 3 * heads * head_dim
    int32_t n_ftiles, n_ttiles;  // tiles of the call's tiling
    int32_t whole;               // workgroups [0, whole) take one tile each; the tiles from there on are cut in smaller ones
    RopeArgs rope;
};

// granule XOR mask of a tile row (reader and writer use the same function): with 128-byte rows
// the 16-byte granule g of row r lives at position g ^ swz(r), which makes the ds_read_b128 of
// 16 rows x 4 granules free of bank conflicts (SQ_LDS_BANK_CONFLICT: 1.6 % of the LDS cycles)
__device__ __forceinline__ int swz(int row) { return (row >> 1) & 7; }

// One matrix instruction, acc += a . b, as an assembly statement: such statements keep their
// program order, and the LDS reads written between them stay between them.  The compiler does
// not know what the statement is and adds no wait states after it: settle() stands between the
// last product and the first vector instruction that reads an accumulator.
__device__ __forceinline__ void mfma(f32x4 &acc, const bf16x8 &a, const bf16x8 &b) {
    asm volatile("v_mfma_f32_16x16x32_bf16 %0, %1, %2, %0" : "+v"(acc) : "v"(a), "v"(b));
}

// All of this wave's LDS reads have returned and at most PENDING of its global -> LDS loads are
// still in flight; then the workgroup's barrier.
template <int PENDING>
__device__ __forceinline__ void stage_barrier() {
    static_assert(PENDING >= 0 && PENDING < 64, "vmcnt range");
    asm volatile("s_waitcnt vmcnt(%0) lgkmcnt(0)\n\ts_barrier" ::"n"(PENDING) : "memory");
}

// The tile of one workgroup: WF x WT wavefronts, each with FB x TB blocks of 16 features x 16
// tokens, and S LDS stages of one k-tile (W rows, then x rows).  With SPLIT the wavefronts share k while they
// form the products (product_split_k) and the blocks from then on; kWide: one wavefront to a SIMD (product_wide).
enum How { kShared, kSplitK, kWide };    // product, product_split_k, product_wide
template <int WF_, int WT_, int FB_, int TB_, int S_, How HOW_ = kShared>
struct Tiling {
    static constexpr int WF = WF_, WT = WT_, FB = FB_, TB = TB_, S = S_;
    static constexpr How HOW = HOW_;
    static constexpr bool SPLIT = HOW == kSplitK;
    using Column = Tiling<WF_, WT_, FB_, 1, S_, HOW_>;                   // 16 of a wave's tokens
    static constexpr int kWaves = WF * WT, kThreads = 64 * kWaves;
    static constexpr int kF = WF * FB * 16, kT = WT * TB * 16;            // features and tokens of the tile
    static constexpr int kWBytes = kF * kRowBytes, kStage = kWBytes + kT * kRowBytes;
    static constexpr int kRing = S * kStage;
    static constexpr int kOut = kWaves * 16 * FB * 32;                    // result staging, see store_tile
    // + rotary table + sums of squares + per wave the bias and gain of its features
    static constexpr int kEpilogue = kOut + kMaxPairs * 16 + kWaves * TB * 16 * 4 + kWaves * FB * 16 * 8;
    static constexpr int kParts = SPLIT ? WF * WT * WF * WT * FB * TB * 1024 : 0;   // every wave's products of the whole tile
    static constexpr int kMost = kRing > kParts ? kRing : kParts, kLds = kMost > kEpilogue ? kMost : kEpilogue;
    static_assert(kLds <= 160 * 1024, "the LDS of a compute unit");
    static_assert(!SPLIT || (WF * WT == 4 && S % 2 == 0 && S >= 6), "one k-step of 32 of a pair of k-tiles per wave");
    static constexpr int FH = FB / 2;                                     // blocks in a lo (or hi) half of a wave's features
    // wave-wide loads (8 rows each) per wave and stage: X = x rows and the lo halves of W, Y = the hi halves
    static constexpr int kLoadsW = kF / 16 / kWaves, kLoadsX = kT / 8 / kWaves;
    static constexpr int X = kLoadsX + kLoadsW, Y = kLoadsW;
    static_assert(kWaves % 2 == 0 && kF % (16 * kWaves) == 0 && (kT % (8 * kWaves) == 0 || TB == 1) && FB % 2 == 0, "whole loads");
};

// acc[f][t] += W[f0 + ..] . x[t0 + ..]^T over all of k.
//
// What bounds it.  A k-tile is kStage bytes arriving in LDS against 2 kF kT 64 flop.  With a stage
// held until all its operands have been read and its successor sent for only then, a load had
// one tile's products to arrive in and did not make it (1131 TFLOP/s at 13230 x 5120 -> 15360; 1460
// without the loads).  Here a wave takes a stage's operands into registers half a tile ahead of
// their products, in two phases: while the products of the lo halves of its features run it reads
// the hi halves, while those of the hi halves run it reads the next tile's x and lo operands.
// Each half of a stage is refilled as soon as the barrier after its read has passed, so a load has one
// and a half tiles' products to arrive in and no wait ever drains the queue.  A barrier stands
// PRE products into its phase: the waves meet with products still in the pipeline.
// 1131 -> 1380 TFLOP/s (32x32x16 products: 1312; 256 x 256 tile, back to back on one box); matrix pipeline busy
// 76 % of the cycles, at a clock that the power limit holds to 1.65 GHz.  Among other kernels, with its epilogue, the
// projection runs at 1050 to 1370 by the clock the card has at the time (1.98 to 1.52 ms, 1.76 on average).
template <typename C>
__device__ __forceinline__ void product(uint32_t lds0, const GemmArgs &a, int f0, int t0, int wave, int lane,
                                        f32x4 (&acc)[C::FB][C::TB]) {
    constexpr int FB = C::FB, TB = C::TB, FH = C::FH, S = C::S, W = C::kWaves;
    const int col = lane % 16, quad = lane / 16;
    const int fw = wave / C::WT, tw = wave % C::WT;

    // raw buffers over the rows this tile can touch (rows past the end read as zeros)
    const int64_t w_rows = min(int64_t(C::kF), int64_t(a.d_out) - f0), x_rows = min(int64_t(C::kT), int64_t(a.n) - t0);
    const __amdgpu_buffer_rsrc_t w_rsrc = __builtin_amdgcn_make_buffer_rsrc(
        const_cast<__bf16 *>(a.w + int64_t(f0) * a.d_in), 0, int(w_rows * a.d_in * 2), 0x00020000);
    const __amdgpu_buffer_rsrc_t x_rsrc = __builtin_amdgcn_make_buffer_rsrc(
        const_cast<__bf16 *>(a.x + int64_t(t0) * a.d_in), 0, int(x_rows * a.d_in * 2), 0x00020000);

    // A wave-wide load moves a group of 8 rows x 128 bytes.  All of a wave's groups have the parity of the
    // wave, so one swizzled lane offset serves them all; the group and the k-tile are scalar offsets.
    const uint32_t row_bytes = uint32_t(a.d_in) * 2;
    const uint32_t voff = uint32_t(lane / 8) * row_bytes + 16 * ((lane % 8) ^ swz((wave & 1) * 8 + lane / 8));
    constexpr int kHalfGroups = FH * 2;                  // groups in the lo (or hi) half of a wave row's features
    auto lo_group = [&](int i) { const int g = wave + i * W; return (g / kHalfGroups) * 2 * kHalfGroups + g % kHalfGroups; };
    auto load = [&](const __amdgpu_buffer_rsrc_t &rsrc, int group, int kt, uint32_t lds) {
        load_to_lds_16(rsrc, __builtin_amdgcn_readfirstlane(lds0 + lds + group * 1024), voff,
                       __builtin_amdgcn_readfirstlane(uint32_t(kt) * kRowBytes + uint32_t(group) * 8 * row_bytes));
    };
    auto load_x = [&](int i, int kt, uint32_t stage) {
        if (i < C::kLoadsX) load(x_rsrc, wave + i * W, kt, stage + C::kWBytes);
        else load(w_rsrc, lo_group(i - C::kLoadsX), kt, stage);
    };
    auto load_y = [&](int i, int kt, uint32_t stage) { load(w_rsrc, lo_group(i) + kHalfGroups, kt, stage); };

    // operand addresses of the two k-steps of 32 in the stage being read
    uint32_t w_addr[2], x_addr[2];
#pragma unroll
    for (int s = 0; s < 2; ++s) {
        w_addr[s] = lds0 + (fw * FB * 16 + col) * kRowBytes + 16 * ((4 * s + quad) ^ swz(col));
        x_addr[s] = lds0 + C::kWBytes + (tw * TB * 16 + col) * kRowBytes + 16 * ((4 * s + quad) ^ swz(col));
    }
    bf16x8 lo[FH][2], hi[FH][2], xop[TB][2];
    auto read_lo = [&](int m, int s) { lo[m][s] = lds_load<bf16x8>(w_addr[s] + m * 16 * kRowBytes); };
    auto read_hi = [&](int m, int s) { hi[m][s] = lds_load<bf16x8>(w_addr[s] + (FH + m) * 16 * kRowBytes); };
    auto read_x = [&](int t, int s) { xop[t][s] = lds_load<bf16x8>(x_addr[s] + t * 16 * kRowBytes); };

    const int n_kt = a.d_in / kBK;
#pragma unroll
    for (int p = 0; p < S; ++p) {
        if (p < n_kt) {
#pragma unroll
            for (int i = 0; i < C::X; ++i) load_x(i, p, p * C::kStage);
#pragma unroll
            for (int i = 0; i < C::Y; ++i) load_y(i, p, p * C::kStage);
        }
    }
    // in registers from here on: zeroed right in front of the first products they would be read a wait state too early
#pragma unroll
    for (int f = 0; f < FB; ++f)
#pragma unroll
        for (int t = 0; t < TB; ++t) {
            acc[f][t] = f32x4{0.0f, 0.0f, 0.0f, 0.0f};
            asm volatile("" : "+v"(acc[f][t]));
        }
    if (n_kt >= S) stage_barrier<C::Y + (S - 1) * (C::X + C::Y)>();     // the first tile's X group has landed
    else stage_barrier<0>();
#pragma unroll
    for (int m = 0; m < FH; ++m) read_lo(m, 0);
#pragma unroll
    for (int t = 0; t < TB; ++t) read_x(t, 0);

    constexpr int PK = FH * TB;                          // products per k-step of a phase
    constexpr int PRE = PK >= 4 ? 3 * PK / 4 : PK / 2;   // products before a phase's barrier
    static_assert(PRE >= 1 && PRE < PK, "the lo operands are read between the barrier and the k-step's end");
    uint32_t cur = 0;                                    // stage of tile kt
    // LEFT = tiles after this one, as far as the code depends on it: with LEFT = S there is also a tile
    // to send for (kt + S); below that everything that is left is already under way.
    auto tile = [&](int kt, auto left_c) {
        constexpr int LEFT = decltype(left_c)::value;
        constexpr bool REFILL = LEFT >= S;
        constexpr int AHEAD = REFILL ? S - 1 : LEFT;     // later tiles whose loads are under way
        // products in an order in which neighbours share an operand
        auto tcol = [](int m, int i) constexpr { return (m & 1) ? TB - 1 - i % TB : i % TB; };
        // ---- phase 1: lo x x; meanwhile the rest of this tile's x and lo operands, then hi
        static_for<0, 2 * PK>([&](auto ic) {
            constexpr int i = decltype(ic)::value, s = i / PK, m = (i % PK) / TB, t = tcol(m, i);
            if constexpr (i == PRE) stage_barrier<AHEAD *(C::X + C::Y)>();
            mfma(acc[m][t], lo[m][s], xop[t][s]);
            if constexpr (i < PRE) {
                static_for<i *(FH + TB) / PRE, (i + 1) * (FH + TB) / PRE>([&](auto rc) {
                    constexpr int r = decltype(rc)::value;
                    if constexpr (r < FH) read_lo(r, 1);
                    else read_x(r - FH, 1);
                });
            } else {
                constexpr int j = i - PRE, rest = 2 * PK - PRE;
                if constexpr (j < PK)
                    static_for<j * 2 * FH / PK, (j + 1) * 2 * FH / PK>([&](auto rc) {
                        constexpr int r = decltype(rc)::value;
                        read_hi(r % FH, r / FH);
                    });
                if constexpr (REFILL)
                    static_for<j * C::X / rest, (j + 1) * C::X / rest>([&](auto rc) { load_x(decltype(rc)::value, kt + S, cur); });
            }
        });
        // ---- phase 2: hi x x; meanwhile the first k-step of the next tile's lo and x operands
        const uint32_t nxt = cur + C::kStage == C::kRing ? 0u : cur + C::kStage;
        const uint32_t delta = nxt - cur;
        static_for<0, 2 * PK>([&](auto ic) {
            constexpr int i = decltype(ic)::value, s = i / PK, m = (i % PK) / TB, t = tcol(m, i);
            if constexpr (i == PRE && LEFT > 0) stage_barrier<(AHEAD - 1) * (C::X + C::Y) + C::Y + (REFILL ? C::X : 0)>();
            mfma(acc[FH + m][t], hi[m][s], xop[t][s]);
            if constexpr (LEFT > 0) {
                if constexpr (i == 0) {
#pragma unroll
                    for (int q = 0; q < 2; ++q) { w_addr[q] += delta; x_addr[q] += delta; }
                }
                if constexpr (i >= PRE && i < PK) {
                    constexpr int j = i - PRE, slots = PK - PRE;
                    static_for<j * FH / slots, (j + 1) * FH / slots>([&](auto rc) { read_lo(decltype(rc)::value, 0); });
                }
                if constexpr (i >= PK && i < 2 * PK) {   // the first k-step's x operands have had their last product
                    constexpr int j = i - PK, slots = PK > TB ? PK / 2 : PK;
                    if constexpr (j < slots)
                        static_for<j * TB / slots, (j + 1) * TB / slots>([&](auto rc) { read_x(decltype(rc)::value, 0); });
                }
                if constexpr (REFILL && i >= PRE) {
                    constexpr int j = i - PRE, rest = 2 * PK - PRE;
                    static_for<j * C::Y / rest, (j + 1) * C::Y / rest>([&](auto rc) { load_y(decltype(rc)::value, kt + S, cur); });
                }
            }
        });
        cur = nxt;
    };
    int kt = 0;
    for (; kt + S < n_kt; ++kt) tile(kt, std::integral_constant<int, S>{});
    static_for<0, S>([&](auto lc) {
        constexpr int LEFT = S - 1 - decltype(lc)::value;
        if (kt + LEFT == n_kt - 1) tile(kt++, std::integral_constant<int, LEFT>{});
    });
    // products become readable by vector instructions
    asm volatile("s_nop 15\n\ts_nop 7");
#pragma unroll
    for (int f = 0; f < FB; ++f)
#pragma unroll
        for (int t = 0; t < TB; ++t) asm volatile("" : "+v"(acc[f][t]));
}

// acc += the same into an accumulation register.
__device__ __forceinline__ void mfma_acc(f32x4 &acc, const bf16x8 &a, const bf16x8 &b) {
    asm volatile("v_mfma_f32_16x16x32_bf16 %0, %1, %2, %0" : "+a"(acc) : "v"(a), "v"(b));
}
// M0 for the next load (base + off), then, an instruction or more later, the load.
__device__ __forceinline__ void set_m0(uint32_t base, uint32_t off) {
    asm volatile("s_add_u32 m0, %0, %1" ::"s"(base), "s"(off) : "memory", "m0", "scc");
}
__device__ __forceinline__ void load_at_m0(const __amdgpu_buffer_rsrc_t &rsrc, uint32_t voff, uint32_t soff) {
    asm volatile("buffer_load_dwordx4 %0, %1, %2 offen lds" ::"v"(voff), "s"(rsrc), "s"(soff) : "memory");
}

// The same with one wavefront to a SIMD (128 features x 128 or 64 tokens each), accumulators in the accumulation registers.
//
// With eight wavefronts of 128 x 64 a k-tile of 256 x 256 is 192 KB read from LDS and 64 KB written to it, as many cycles of its 128
// bytes as the products take; four of 128 x 128 read 128 KB, which is less power too.  Alone on its SIMD a wavefront keeps the
// matrix pipeline busy if no more than 8 cycles of other instructions (two) stand between two products, so that a load is a write of
// M0 before a product and the load behind it, and lane offsets hold what a scalar addition per load did.  Half as many
// wavefronts fill the stages and store the tile more slowly.  Four / eight, time: 1.06 to 1.10 at 8 k-tiles, 1.00 to 1.01 at 32, 0.99
// to 1.01 at 40, 0.97 to 0.99 at 64, 0.94 to 0.98 at 96; from 33 to 39 k-tiles seven calls of other sizes 0.98 to 1.00, so that
// the line (four_waves) lies where neither side gains.  13230 x 5120 -> 5120 466.6 / 460.5 us, 4096 x 6144 -> 1536 67.9 / 64.4.
// Not with the QKV epilogue, which one wavefront to a SIMD takes longer for, by what the products gain: 8192 x 2048 -> 6144 158.9 /
// 170.8, 8192 x 3072 -> 9216 355 / 369, and with 80 k-tiles 8192 x 5120 -> 15360 911.5 / 910.3, 13230 x 5120 1467 / 1438,
// 11340 x 5120 1273 / 1277, 4096 x 5120 468.4 / 468.4.  Nor for 128 x 128 (no change).
template <typename C>
__device__ __forceinline__ void product_wide(uint32_t lds0, const GemmArgs &a, int f0, int t0, int wave, int lane,
                                             f32x4 (&acc)[C::FB][C::TB]) {
    constexpr int FB = C::FB, TB = C::TB, FH = C::FH, S = C::S, W = C::kWaves;
    const int col = lane % 16, quad = lane / 16;
    const int fw = wave / C::WT, tw = wave % C::WT;
    const int64_t w_rows = min(int64_t(C::kF), int64_t(a.d_out) - f0), x_rows = min(int64_t(C::kT), int64_t(a.n) - t0);
    const __amdgpu_buffer_rsrc_t w_rsrc = __builtin_amdgcn_make_buffer_rsrc(
        const_cast<__bf16 *>(a.w + int64_t(f0) * a.d_in), 0, int(w_rows * a.d_in * 2), 0x00020000);
    const __amdgpu_buffer_rsrc_t x_rsrc = __builtin_amdgcn_make_buffer_rsrc(
        const_cast<__bf16 *>(a.x + int64_t(t0) * a.d_in), 0, int(x_rows * a.d_in * 2), 0x00020000);
    const uint32_t row_bytes = uint32_t(a.d_in) * 2;
    constexpr int kHalfGroups = FH * 2;
    auto lo_group = [&](int i) { const int g = wave + i * W; return (g / kHalfGroups) * 2 * kHalfGroups + g % kHalfGroups; };
    // load i of a stage: x rows, the lo halves of W, the hi halves; lane offsets with the group in them, the k-tile is the scalar offset
    constexpr int N = C::X + C::Y;
    uint32_t voff[N], dst[N];
    {
        const uint32_t v0 = uint32_t(lane / 8) * row_bytes + 16 * ((lane % 8) ^ swz((wave & 1) * 8 + lane / 8));
#pragma unroll
        for (int i = 0; i < N; ++i) {
            const int g = i < C::kLoadsX ? wave + i * W : i < C::X ? lo_group(i - C::kLoadsX) : lo_group(i - C::X) + kHalfGroups;
            voff[i] = v0 + uint32_t(g) * 8 * row_bytes;
            dst[i] = __builtin_amdgcn_readfirstlane(lds0 + (i < C::kLoadsX ? C::kWBytes : 0) + uint32_t(g) * 1024);
        }
    }
    uint32_t w_addr[2], x_addr[2];
#pragma unroll
    for (int s = 0; s < 2; ++s) {
        w_addr[s] = lds0 + (fw * FB * 16 + col) * kRowBytes + 16 * ((4 * s + quad) ^ swz(col));
        x_addr[s] = lds0 + C::kWBytes + (tw * TB * 16 + col) * kRowBytes + 16 * ((4 * s + quad) ^ swz(col));
    }
    bf16x8 lo[FH][2], hi[FH][2], xop[TB][2];
    auto read_lo = [&](int m, int s) { lo[m][s] = lds_load<bf16x8>(w_addr[s] + m * 16 * kRowBytes); };
    auto read_hi = [&](int m, int s) { hi[m][s] = lds_load<bf16x8>(w_addr[s] + (FH + m) * 16 * kRowBytes); };
    auto read_x = [&](int t, int s) { xop[t][s] = lds_load<bf16x8>(x_addr[s] + t * 16 * kRowBytes); };
#pragma unroll
    for (int f = 0; f < FB; ++f)
#pragma unroll
        for (int t = 0; t < TB; ++t) {
            acc[f][t] = f32x4{0.0f, 0.0f, 0.0f, 0.0f};
            asm volatile("" : "+a"(acc[f][t]));
        }
    const int n_kt = a.d_in / kBK;
#pragma unroll
    for (int p = 0; p < S; ++p)
        if (p < n_kt)
#pragma unroll
            for (int i = 0; i < N; ++i) {
                set_m0(dst[i], p * C::kStage);
                asm volatile("s_nop 0");
                load_at_m0(i < C::kLoadsX ? x_rsrc : w_rsrc, voff[i], uint32_t(p) * kRowBytes);
            }
    if (n_kt >= S) stage_barrier<C::Y + (S - 1) * N>();  // the first tile's X group has landed
    else stage_barrier<0>();
#pragma unroll
    for (int m = 0; m < FH; ++m) read_lo(m, 0);
#pragma unroll
    for (int t = 0; t < TB; ++t) read_x(t, 0);

    // Products per k-step of a phase; before a phase's barrier; and the windows over which a phase's loads are spread
    constexpr int PK = FH * TB, PRE = FH + TB + 3;
    constexpr int kRest = 2 * PK - PRE, kEveryX = kRest / C::X > 0 ? kRest / C::X : 1, kEveryY = kRest / C::Y > 0 ? kRest / C::Y : 1;
    static_assert(PRE < PK && kRest >= 2 * FH && C::X <= kRest && C::Y <= kRest && PK + TB <= 2 * PK, "everything has its window");
    uint32_t cur = 0;
    auto tile = [&](int kt, auto left_c) {
        constexpr int LEFT = decltype(left_c)::value;
        constexpr bool REFILL = LEFT >= S;
        constexpr int AHEAD = REFILL ? S - 1 : LEFT;
        const uint32_t soff = uint32_t(kt + S) * kRowBytes;
        auto tcol = [](int m, int i) constexpr { return (m & 1) ? TB - 1 - i % TB : i % TB; };
        // ---- phase 1: lo x x; meanwhile the rest of this tile's x and lo operands, then hi
        static_for<0, 2 * PK>([&](auto ic) {
            constexpr int i = decltype(ic)::value, s = i / PK, m = (i % PK) / TB, t = tcol(m, i), j = i - PRE;
            constexpr bool kLoad = REFILL && j >= 0 && j % kEveryX == 0 && j / kEveryX < C::X;
            if constexpr (i == PRE) stage_barrier<AHEAD * N>();
            if constexpr (kLoad) set_m0(dst[j / kEveryX], cur);
            mfma_acc(acc[m][t], lo[m][s], xop[t][s]);
            if constexpr (kLoad) load_at_m0(j / kEveryX < C::kLoadsX ? x_rsrc : w_rsrc, voff[j / kEveryX], soff);
            if constexpr (i < FH) read_lo(i, 1);
            else if constexpr (i < FH + TB) read_x(i - FH, 1);
            if constexpr (j >= 0 && j < 2 * FH) read_hi(j % FH, j / FH);
        });
        // ---- phase 2: hi x x; meanwhile the first k-step of the next tile's lo and x operands
        const uint32_t nxt = cur + C::kStage == C::kRing ? 0u : cur + C::kStage;
        const uint32_t delta = nxt - cur;
        static_for<0, 2 * PK>([&](auto ic) {
            constexpr int i = decltype(ic)::value, s = i / PK, m = (i % PK) / TB, t = tcol(m, i), j = i - PRE;
            constexpr bool kLoad = REFILL && j >= 0 && j % kEveryY == 0 && j / kEveryY < C::Y;
            if constexpr (i == PRE && LEFT > 0) stage_barrier<(AHEAD - 1) * N + C::Y + (REFILL ? C::X : 0)>();
            if constexpr (kLoad) set_m0(dst[C::X + j / kEveryY], cur);
            mfma_acc(acc[FH + m][t], hi[m][s], xop[t][s]);
            if constexpr (kLoad) load_at_m0(w_rsrc, voff[C::X + j / kEveryY], soff);
            if constexpr (LEFT > 0) {
                if constexpr (i < 2) { w_addr[i] += delta; x_addr[i] += delta; }
                if constexpr (j >= 0 && j < FH) read_lo(j, 0);
                if constexpr (i >= PK && i < PK + TB) read_x(i - PK, 0);      // the first k-step's have had their last product
            }
        });
        cur = nxt;
    };
    int kt = 0;
    for (; kt + S < n_kt; ++kt) tile(kt, std::integral_constant<int, S>{});
    static_for<0, S>([&](auto lc) {
        constexpr int LEFT = S - 1 - decltype(lc)::value;
        if (kt + LEFT == n_kt - 1) tile(kt++, std::integral_constant<int, LEFT>{});
    });
    asm volatile("s_nop 15\n\ts_nop 7");
#pragma unroll
    for (int f = 0; f < FB; ++f)
#pragma unroll
        for (int t = 0; t < TB; ++t) asm volatile("" : "+a"(acc[f][t]));
}

// The same for calls of few tiles and a long k: the four waves of a workgroup share k.
//
// What bounds it: what a compute unit takes in, and that depends on where the bytes are.  A k-tile of 12 KB takes 0.07 to 0.085 us
// (150 GB/s a compute unit) while the rows of W and x that an XCD's workgroups read fit its L2, and 0.13 to 0.17 us (72 to 92
// GB/s) where they come from behind it, with 30 workgroups as with 250.  Six, eight and twelve stages (72, 96, 144 KB sent for): 14.5,
// 13.5, 13.8 us at 520 x 5120 -> 640, so it is not what the stages have under way.  64 x 64 and 128 x 64 tiles take in 72 to 74
// GB/s with 160 to 256 workgroups, so with compute units to spare the tile with fewer bytes is the faster one.
// A 64 x 32 tile has too few products per k-tile to keep four waves that share its rows apart from LDS and the barrier
// (0.19 us with two such waves); here a wave takes all of the tile's rows for one k-step of 32 out of a pair of k-tiles, every
// byte is read from LDS once, and the four partial tiles are added up through LDS at the end.  A wave holds the operands of
// two pairs: behind the one barrier of a pair it fetches those of the next pair and sends for the pair S / 2 later, under
// the products of this one.  520 x 5120 -> 640: 17.3 to 13.7 us; 100 x 3072 -> 3072: 12.0 to 9.9.
// A 64 x 64 tile gains nothing from it (17.4), and operands fetched straight into registers are slower (30).
//
// Leaves the wave's own FB x TB blocks in acc, like product().
template <typename C>
__device__ __forceinline__ void product_split_k(uint32_t lds0, const GemmArgs &a, int f0, int t0, int wave, int lane,
                                                f32x4 (&acc)[C::FB][C::TB]) {
    constexpr int FB = C::WF * C::FB, TB = C::WT * C::TB, S = C::S, W = C::kWaves, kLoads = C::X + C::Y;
    const int col = lane % 16, quad = lane / 16;
    const int64_t w_rows = min(int64_t(C::kF), int64_t(a.d_out) - f0), x_rows = min(int64_t(C::kT), int64_t(a.n) - t0);
    const __amdgpu_buffer_rsrc_t w_rsrc = __builtin_amdgcn_make_buffer_rsrc(
        const_cast<__bf16 *>(a.w + int64_t(f0) * a.d_in), 0, int(w_rows * a.d_in * 2), 0x00020000);
    const __amdgpu_buffer_rsrc_t x_rsrc = __builtin_amdgcn_make_buffer_rsrc(
        const_cast<__bf16 *>(a.x + int64_t(t0) * a.d_in), 0, int(x_rows * a.d_in * 2), 0x00020000);
    const int n_kt = a.d_in / kBK;
    // As in product(): a load moves 8 rows, and all of a wave's groups of rows have the parity of the wave.  A k-tile
    // past the last is sent for outside the buffers (nothing is fetched, zeros arrive), which leaves one body
    // for every pair: behind the loads waited for there are always as many others.
    const uint32_t row_bytes = uint32_t(a.d_in) * 2;
    const uint32_t voff = uint32_t(lane / 8) * row_bytes + 16 * ((lane % 8) ^ swz((wave & 1) * 8 + lane / 8));
    auto load = [&](int i, int kt, uint32_t stage) {
        const bool is_x = i < C::kLoadsX;
        const int rows8 = wave + (is_x ? i : i - C::kLoadsX) * W;
        load_to_lds_16(is_x ? x_rsrc : w_rsrc, __builtin_amdgcn_readfirstlane(lds0 + stage + (is_x ? C::kWBytes : 0) + rows8 * 1024),
                       kt < n_kt ? voff : 0x80000000u,
                       __builtin_amdgcn_readfirstlane(uint32_t(kt) * kRowBytes + uint32_t(rows8) * 8 * row_bytes));
    };
    auto load_pair = [&](int i, int kt, uint32_t stage) { load(i % kLoads, kt + i / kLoads, stage + (i / kLoads) * C::kStage); };
    // operand addresses of this wave's k-step in the first pair of stages
    const uint32_t w_addr = lds0 + (wave / 2) * C::kStage + col * kRowBytes + 16 * ((4 * (wave % 2) + quad) ^ swz(col));
    const uint32_t x_addr = w_addr + C::kWBytes;
    struct Operands {
        bf16x8 w[FB], x[TB];
    };
    auto read = [&](Operands &o, uint32_t stage) {
#pragma unroll
        for (int t = 0; t < TB; ++t) o.x[t] = lds_load<bf16x8>(x_addr + stage + t * 16 * kRowBytes);
#pragma unroll
        for (int f = 0; f < FB; ++f) o.w[f] = lds_load<bf16x8>(w_addr + stage + f * 16 * kRowBytes);
    };
    f32x4 part[FB][TB];
#pragma unroll
    for (int f = 0; f < FB; ++f)
#pragma unroll
        for (int t = 0; t < TB; ++t) part[f][t] = f32x4{0.0f, 0.0f, 0.0f, 0.0f};
#pragma unroll
    for (int p = 0; p < S; p += 2)
#pragma unroll
        for (int i = 0; i < 2 * kLoads; ++i) load_pair(i, p, p * C::kStage);
    stage_barrier<(S - 2) * kLoads>();                   // the first pair has landed
    Operands even, odd;                                  // of the pairs of even and odd number
    read(even, 0);
    uint32_t cur = 0;                                    // first stage of the pair at kt
    auto pair = [&](int kt, const Operands &now, Operands &next) {
        const uint32_t nxt = cur + 2 * C::kStage == C::kRing ? 0u : cur + 2 * C::kStage;
        stage_barrier<(S - 4) * kLoads>();               // the next pair has landed; every wave has its operands of this one, whose stages are free
        read(next, nxt);
        static_for<0, FB>([&](auto fc) {
            constexpr int f = decltype(fc)::value;
#pragma unroll
            for (int t = 0; t < TB; ++t) part[f][t] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(now.w[f], now.x[t], part[f][t], 0, 0, 0);
            static_for<f * 2 * kLoads / FB, (f + 1) * 2 * kLoads / FB>([&](auto ic) { load_pair(decltype(ic)::value, kt + S, cur); });
        });
        cur = nxt;
    };
    for (int kt = 0;; kt += 4) {
        pair(kt, even, odd);
        if (kt + 2 >= n_kt) break;
        pair(kt + 2, odd, even);
        if (kt + 4 >= n_kt) break;
    }
    // every wave's partial tile through LDS; a wave adds up its own blocks, in the order of the waves
    stage_barrier<0>();
#pragma unroll
    for (int f = 0; f < FB; ++f)
#pragma unroll
        for (int t = 0; t < TB; ++t) *LP_LDS_PTR(f32x4, uintptr_t(lds0 + ((wave * FB + f) * TB + t) * 1024 + 16 * lane)) = part[f][t];
    __syncthreads();
    const int f_own = (wave / C::WT) * C::FB, t_own = (wave % C::WT) * C::TB;
#pragma unroll
    for (int f = 0; f < C::FB; ++f)
#pragma unroll
        for (int t = 0; t < C::TB; ++t) {
            f32x4 sum = lds_load<f32x4>(lds0 + ((f_own + f) * TB + t_own + t) * 1024 + 16 * lane);
#pragma unroll
            for (int w = 1; w < W; ++w) sum += lds_load<f32x4>(lds0 + ((w * FB + f_own + f) * TB + t_own + t) * 1024 + 16 * lane);
            acc[f][t] = sum;
        }
}

// Per-head RMS normalisation and rotary encoding, in place, of the features a wave holds in acc
// (those of one section of q or k): block f, token block t, element i of lane (col, quad) is
// feature 16 f + 4 quad + i of token 16 t + col.  sum_sq(t, h) is the sum of squares over the
// h-th head's features; gain_lds holds the gains of the wave's features; in_head is the first one's
// place in its head.  The rotary table sits in LDS at rope_lds, float4 per pair.
template <int HD, typename C, typename F>
__device__ __forceinline__ void norm_rope(f32x4 (&acc)[C::FB][C::TB], F &&sum_sq, uint32_t gain_lds, int in_head,
                                          const RopeArgs &r, uint32_t rope_lds, int tok_first, int n, int col, int quad) {
    constexpr int kHeads = C::FB * 16 > HD ? C::FB * 16 / HD : 1, kBlocks = C::FB / kHeads;
    float pt[C::TB], ph[C::TB], pw[C::TB];               // coordinates of this lane's tokens
#pragma unroll
    for (int t = 0; t < C::TB; ++t) {
        const uint32_t tk = uint32_t(min(tok_first + 16 * t + col, n - 1));
        const uint32_t ct = fastdiv(tk, r.hw), rem = tk - ct * r.hw.d, ch = fastdiv(rem, r.w);
        pt[t] = float(int32_t(ct) + r.off[0]);
        ph[t] = float(int32_t(ch) + r.off[1]);
        pw[t] = float(int32_t(rem - ch * r.w.d) + r.off[2]);
    }
#pragma unroll
    for (int hh = 0; hh < kHeads; ++hh) {
        float inv[C::TB];
#pragma unroll
        for (int t = 0; t < C::TB; ++t) inv[t] = 1.0f / sqrtf(sum_sq(t, hh) * (1.0f / float(HD)) + r.eps);
#pragma unroll
        for (int b = 0; b < kBlocks; ++b) {
            const int f = hh * kBlocks + b;
            const f32x4 gn = lds_load<f32x4>(gain_lds + 4 * (16 * f + 4 * quad));
            const int pair = ((in_head + 16 * f + 4 * quad) % HD) / 2;
#pragma unroll
            for (int pr = 0; pr < 2; ++pr) {
                const f32x4 tb = lds_load<f32x4>(rope_lds + 16 * (pair + pr));
#pragma unroll
                for (int t = 0; t < C::TB; ++t) {
                    float turns = pt[t] * tb.x + ph[t] * tb.y + pw[t] * tb.z;
                    turns = turns - floorf(turns);
                    const float c = __builtin_amdgcn_cosf(turns), s = __builtin_amdgcn_sinf(turns);
                    const float x = acc[f][t][2 * pr] * inv[t] * gn[2 * pr], y = acc[f][t][2 * pr + 1] * inv[t] * gn[2 * pr + 1];
                    acc[f][t][2 * pr] = x * c - y * s;
                    acc[f][t][2 * pr + 1] = x * s + y * c;
                }
            }
        }
    }
}

// Writes a wave's results, rounded to bf16, to dst + token * row_stride + feature: 16 tokens at
// a time pass through the wave's own LDS (16-byte granules XORed with the row) and leave as
// rows of FB * 32 bytes: two whole lines, one, or (the tilings of 64 and fewer tokens) half of one.
template <typename C>
__device__ __forceinline__ void store_tile(uint32_t out_lds, const f32x4 (&acc)[C::FB][C::TB], __bf16 *dst, int64_t row_stride,
                                           int tokens_valid, int lane) {
    constexpr int kGran = C::FB * 2, kRow = kGran * 16;  // granules and bytes of a staged row
    const int col = lane % 16, quad = lane / 16;
#pragma unroll
    for (int t = 0; t < C::TB; ++t) {
        if (16 * t >= tokens_valid) break;
#pragma unroll
        for (int f = 0; f < C::FB; ++f) {
            union { u32x2 u; bf16x2 p[2]; } ow;
            ow.p[0] = to_bf16x2(acc[f][t][0], acc[f][t][1]);
            ow.p[1] = to_bf16x2(acc[f][t][2], acc[f][t][3]);
            *LP_LDS_PTR(u32x2, uintptr_t(out_lds + col * kRow + 16 * ((2 * f + quad / 2) ^ (col % kGran)) + 8 * (quad % 2))) = ow.u;
        }
#pragma unroll
        for (int j = 0; j < 16 * kGran / 64; ++j) {
            const int r = (lane + 64 * j) / kGran, g = lane % kGran;
            const u32x4 u = lds_load<u32x4>(out_lds + r * kRow + 16 * (g ^ (r % kGran)));
            if (16 * t + r < tokens_valid) *reinterpret_cast<u32x4 *>(dst + int64_t(16 * t + r) * row_stride + 8 * g) = u;
        }
    }
}

// One tile from its first load to its last store.  QKV = true: the epilogue cuts the features into
// q | k | v sections of heads * HD, normalises and rotates q and k.  QKV = false: plain y = x W^T + b.
template <bool QKV, int HD, typename C>
__device__ __forceinline__ void run_tile(uint32_t lds0, const GemmArgs &a, int f0, int t0) {
    constexpr int FB = C::FB, TB = C::TB;
    const int tid = threadIdx.x;
    const int wave = __builtin_amdgcn_readfirstlane(tid / 64);
    const int lane = tid % 64, col = lane % 16, quad = lane / 16;
    const int fbase = f0 + (wave / C::WT) * FB * 16;     // first of this wave's features
    const bool live = fbase < a.d_out;                   // d_out is a multiple of FB * 16: all of them or none
    const int dm = QKV ? a.heads * HD : a.d_out;
    const int section = QKV ? min(fbase / dm, 2) : 0, f_in_section = fbase - section * dm;
    // what the epilogue needs from memory is fetched before the product starts: two features' bias
    // and gain per lane, one pair's rotary turns per thread
    const int f_pre = min(2 * lane, FB * 16 - 2);
    f32x2 bias_pre = {0.0f, 0.0f}, gain_pre = {0.0f, 0.0f};
    f32x4 turns_pre = {0.0f, 0.0f, 0.0f, 0.0f};
    if (live && a.bias != nullptr) bias_pre = *reinterpret_cast<const f32x2 *>(a.bias + fbase + f_pre);
    if (QKV) {
        if (live && section < 2) gain_pre = *reinterpret_cast<const f32x2 *>(a.gain[section] + f_in_section + f_pre);
        const float *tp = a.rope.turns[tid % kMaxPairs];
        turns_pre = f32x4{tp[0], tp[1], tp[2], 0.0f};
    }
    f32x4 acc[FB][TB];
    if constexpr (C::SPLIT) product_split_k<C>(lds0, a, f0, t0, wave, lane, acc);
    else if constexpr (C::HOW == kWide) product_wide<C>(lds0, a, f0, t0, wave, lane, acc);
    else product<C>(lds0, a, f0, t0, wave, lane, acc);

    stage_barrier<0>();                                  // the ring is free: every wave has read its last operand
    const uint32_t out_lds = lds0 + wave * (16 * FB * 32), rope_lds = lds0 + C::kOut, ss_lds = rope_lds + kMaxPairs * 16;
    const uint32_t bias_lds = ss_lds + C::kWaves * TB * 16 * 4 + wave * FB * 16 * 8, gain_lds = bias_lds + FB * 16 * 4;
    *LP_LDS_PTR(f32x2, uintptr_t(bias_lds + 4 * f_pre)) = bias_pre;
    if constexpr (C::HOW == kWide) {                     // 16 tokens at a time, out of the accumulation registers
        static_assert(!QKV, "lp_linear's");
        using One = typename C::Column;
        if (!live) return;
        const int tok_first = t0 + (wave % C::WT) * TB * 16;
        __bf16 *dst = a.out[0] + int64_t(tok_first) * dm + fbase;
#pragma unroll
        for (int t = 0; t < TB; ++t) {
            if (tok_first + 16 * t >= a.n) break;
            f32x4 y[FB][1];
#pragma unroll
            for (int f = 0; f < FB; ++f) y[f][0] = acc[f][t] + lds_load<f32x4>(bias_lds + 4 * (16 * f + 4 * quad));
            store_tile<One>(out_lds, y, dst + int64_t(16 * t) * dm, dm, a.n - tok_first - 16 * t, lane);
        }
        return;
    }
#pragma unroll
    for (int f = 0; f < FB; ++f) {
        const f32x4 b4 = lds_load<f32x4>(bias_lds + 4 * (16 * f + 4 * quad));
#pragma unroll
        for (int t = 0; t < TB; ++t)
#pragma unroll
            for (int i = 0; i < 4; ++i) acc[f][t][i] += b4[i];
    }
    const int tok_first = t0 + (wave % C::WT) * TB * 16;
    if (QKV) {
        // sums of squares over the features of a head that this wave holds
        constexpr int kHeads = FB * 16 > HD ? FB * 16 / HD : 1, kSharing = FB * 16 < HD ? HD / (FB * 16) : 1;
        float ss[TB][kHeads];
#pragma unroll
        for (int t = 0; t < TB; ++t)
#pragma unroll
            for (int hh = 0; hh < kHeads; ++hh) {
                float s = 0.0f;
#pragma unroll
                for (int b = 0; b < FB / kHeads; ++b)
#pragma unroll
                    for (int i = 0; i < 4; ++i) s += acc[hh * (FB / kHeads) + b][t][i] * acc[hh * (FB / kHeads) + b][t][i];
                ss[t][hh] = lp::over_quads(s, [](float x, float y) { return x + y; });
            }
        if (tid < kMaxPairs) *LP_LDS_PTR(f32x4, uintptr_t(rope_lds + 16 * tid)) = turns_pre;
        *LP_LDS_PTR(f32x2, uintptr_t(gain_lds + 4 * f_pre)) = gain_pre;
        if (kSharing > 1 && quad == 0) {
#pragma unroll
            for (int t = 0; t < TB; ++t)
                *LP_LDS_PTR(float, uintptr_t(ss_lds + 4 * (wave * TB * 16 + t * 16 + col))) = ss[t][0];
        }
        __syncthreads();
        if (!live) return;
        if (kSharing > 1) {                              // the head's other features are with the neighbouring wave rows
            const int first = (wave / (C::WT * kSharing)) * (C::WT * kSharing) + wave % C::WT;
#pragma unroll
            for (int t = 0; t < TB; ++t) {
                float s = 0.0f;
#pragma unroll
                for (int q = 0; q < kSharing; ++q)
                    s += lds_load<float>(ss_lds + 4 * ((first + q * C::WT) * TB * 16 + t * 16 + col));
                ss[t][0] = s;
            }
        }
        if (section < 2)
            norm_rope<HD, C>(acc, [&](int t, int hh) { return ss[t][hh]; }, gain_lds, f_in_section % HD, a.rope, rope_lds, tok_first,
                             a.n, col, quad);
    } else if (!live) {
        return;
    }
    store_tile<C>(out_lds, acc, a.out[section] + int64_t(tok_first) * dm + f_in_section, dm, a.n - tok_first, lane);
}

// Workgroups [0, whole) take one tile of tiling P each; every later tile is cut into tiles of R.
// P's tiles are ordered in panels of kPanel token tiles, feature tile by feature tile inside a
// panel: the workgroups an XCD runs at a time share their W and x rows through its L2.
template <bool QKV, int HD, typename P, typename R>
__global__ __launch_bounds__(P::kThreads, P::HOW == kShared ? 2 : 1) void gemm_kernel(const GemmArgs a) {
    static_assert(P::kThreads == R::kThreads && P::kF % R::kF == 0 && P::kT % R::kT == 0, "R cuts P");
    extern __shared__ __attribute__((aligned(1024))) unsigned char smem[];
    const uint32_t lds0 = uint32_t(uintptr_t(LP_LDS_PTR(unsigned char, smem)));
    constexpr int kCutF = P::kF / R::kF, kCut = kCutF * (P::kT / R::kT);
    const bool cut = std::is_same<P, R>::value ? false : int(blockIdx.x) >= a.whole;
    int tile, part = 0;
    if (!cut) {
        tile = int(logical_workgroup(blockIdx.x, std::is_same<P, R>::value ? gridDim.x : uint32_t(a.whole)));
    } else {
        const int j = int(logical_workgroup(blockIdx.x - uint32_t(a.whole), gridDim.x - uint32_t(a.whole)));
        tile = a.whole + j / kCut;
        part = j % kCut;
    }
    const int panel_tiles = kPanel * a.n_ftiles;
    const int panel = tile / panel_tiles, in_panel = tile - panel * panel_tiles;
    const int panel_h = min(kPanel, a.n_ttiles - panel * kPanel);
    const int ftile = in_panel / panel_h, ttile = panel * kPanel + in_panel - ftile * panel_h;
    const int f0 = ftile * P::kF, t0 = ttile * P::kT;
    if (!cut) {
        run_tile<QKV, HD, P>(lds0, a, f0, t0);
    } else {
        const int fr = f0 + (part % kCutF) * R::kF, tr = t0 + (part / kCutF) * R::kT;
        if (fr < a.d_out && tr < a.n) run_tile<QKV, HD, R>(lds0, a, fr, tr);
    }
}

// Normalisation + rotation alone, in place: one thread per 8 consecutive features of a
// (token, head) row, HD / 8 threads per row.
template <int HD>
__global__ __launch_bounds__(256) void norm_rope_kernel(__bf16 *x, const float *gain, int64_t n, int32_t heads,
                                                        int64_t stride_tok, int64_t stride_head, const RopeArgs r) {
    __shared__ float4 table[kMaxPairs];
    if (threadIdx.x < kMaxPairs)
        table[threadIdx.x] = make_float4(r.turns[threadIdx.x][0], r.turns[threadIdx.x][1], r.turns[threadIdx.x][2], 0.0f);
    __syncthreads();
    constexpr int kPer = HD / 8;                          // threads per row
    const int64_t row = (int64_t(blockIdx.x) * 256 + threadIdx.x) / kPer;
    const int part = threadIdx.x % kPer;
    const bool live = row < n * heads;
    const int64_t rc = live ? row : 0;
    const int64_t tk = rc / heads;
    const int head = int(rc - tk * heads);
    __bf16 *p = x + tk * stride_tok + int64_t(head) * stride_head + part * 8;
    union { uint4 u; bf16x2 p[4]; } in;
    in.u = *reinterpret_cast<const uint4 *>(p);
    float v[8];
    const uint32_t wds[4] = {in.u.x, in.u.y, in.u.z, in.u.w};
#pragma unroll
    for (int e = 0; e < 4; ++e) {      // a bf16 is the upper half of the binary32 with the same value
        v[2 * e] = __uint_as_float(wds[e] << 16);
        v[2 * e + 1] = __uint_as_float(wds[e] & 0xffff0000u);
    }
    float ss = 0.0f;
#pragma unroll
    for (int e = 0; e < 8; ++e) ss += v[e] * v[e];
#pragma unroll
    for (int m = 1; m < kPer; m *= 2) ss += __shfl_xor(ss, m, 64);
    const float inv = 1.0f / sqrtf(ss * (1.0f / float(HD)) + r.eps);
    const uint32_t t = fastdiv(uint32_t(tk), r.hw);
    const uint32_t rem = uint32_t(tk) - t * r.hw.d;
    const uint32_t h = fastdiv(rem, r.w);
    const float pt = float(int32_t(t) + r.off[0]), ph = float(int32_t(h) + r.off[1]), pw = float(int32_t(rem - h * r.w.d) + r.off[2]);
    const float *gr = gain + head * HD + part * 8;
    const float4 g0 = *reinterpret_cast<const float4 *>(gr), g1 = *reinterpret_cast<const float4 *>(gr + 4);
    const float gv[8] = {g0.x, g0.y, g0.z, g0.w, g1.x, g1.y, g1.z, g1.w};
    union { uint4 u; bf16x2 p[4]; } out;
#pragma unroll
    for (int e = 0; e < 4; ++e) {
        const float4 tb = table[part * 4 + e];
        float turns = pt * tb.x + ph * tb.y + pw * tb.z;
        turns = turns - floorf(turns);
        const float c = __builtin_amdgcn_cosf(turns), s = __builtin_amdgcn_sinf(turns);
        const float a = v[2 * e] * inv * gv[2 * e], b = v[2 * e + 1] * inv * gv[2 * e + 1];
        out.p[e] = to_bf16x2(a * c - b * s, a * s + b * c);
    }
    if (live) *reinterpret_cast<uint4 *>(p) = out.u;
}

// Fills the device-side rotary description; LP_OK or the error.
int make_rope_args(const lp_rope *rope, int64_t n, int32_t head_dim, float eps, RopeArgs *out) {
    if (rope == nullptr) return LP_ERR_INVALID_ARG;
    int64_t cells = 1;
    int32_t sum = 0;
    for (int ax = 0; ax < 3; ++ax) {
        if (rope->grid[ax] < 1 || rope->split[ax] < 0 || rope->split[ax] % 2 != 0) return LP_ERR_INVALID_ARG;
        cells *= rope->grid[ax];
        sum += rope->split[ax];
    }
    if (cells != n || sum != head_dim || !(rope->base > 0.0f) || !(eps >= 0.0f)) return LP_ERR_INVALID_ARG;
    if (n >= (int64_t(1) << 31)) return LP_ERR_UNSUPPORTED;
    RopeArgs r{};
    int pair = 0;
    for (int ax = 0; ax < 3; ++ax) {
        const int p = rope->split[ax];
        for (int j = 0; j < p / 2; ++j, ++pair) {
            // angle per unit coordinate base^(-2 j / p), stored in turns
            const double freq = std::pow(double(rope->base), -2.0 * double(j) / double(p));
            r.turns[pair][ax] = float(freq / (2.0 * M_PI));
        }
    }
    r.hw = make_fastdiv(uint32_t(rope->grid[1]) * uint32_t(rope->grid[2]));
    r.w = make_fastdiv(uint32_t(rope->grid[2]));
    r.grid_h = rope->grid[1];
    for (int ax = 0; ax < 3; ++ax) r.off[ax] = rope->offset[ax];
    r.eps = eps;
    *out = r;
    return LP_OK;
}

using Tile256x256 = Tiling<2, 4, 8, 4, 2>;
using Tile256x128 = Tiling<2, 4, 8, 2, 3>;
using Tile128x128 = Tiling<2, 4, 4, 2, 4>;
using Tile128x64 = Tiling<4, 2, 2, 2, 5>;
using Tile64x64 = Tiling<2, 2, 2, 2, 5>;
// The same sizes with four wavefronts, for lp_linear with a long k
using Wide256x256 = Tiling<2, 2, 8, 8, 2, kWide>;
using Wide256x128 = Tiling<2, 2, 8, 4, 3, kWide>;
using Four128x128 = Tiling<2, 2, 4, 4, 4>;
using Four128x64 = Tiling<2, 2, 4, 2, 5>;
using Split64x32 = Tiling<2, 2, 2, 1, 8, kSplitK>;

// How a call is cut.  The prices are those of the kernels of eight wavefronts; from 32 k-tiles on lp_linear runs the plan's tiles of
// 256 features with four (four_waves), which are up to 6 % faster and change no plan: of 160 products of 32 to 120 k-tiles, timed in
// every tiling with the wavefronts it would run with, none was more than 5 % off the fastest, 1.0 % on average with the spread of the times in it.
//
// A round is one tile on every compute unit (two of 64 x 64).  Per round, in us, fitted to 4004 calls (3133
// products of 1 .. 200000 tokens, d_in 64 .. 13824, d_out 128 .. 13824, and 871 QKV projections), each timed on every tiling,
// so that the tiling chosen is the fastest: a k-tile of 64, and `once`, what a tile costs besides (first loads, stores); `part`
// with at most half of the compute units busy, `full` with all of them, where the power limit lowers the clock and
// the stores of all tiles share the memory's rate.
struct TileCost {
    int f, t, threads, per_cu;
    float part, full, once_part, once_full;
};
constexpr TileCost kTileCost[] = {
    {256, 256, 512, 1, 1.198f, 1.252f, 3.22f, 5.24f}, {256, 128, 512, 1, 0.647f, 0.737f, 1.92f, 3.16f},
    {128, 128, 512, 1, 0.313f, 0.493f, 1.78f, 1.95f}, {128, 64, 512, 1, 0.207f, 0.304f, 1.10f, 1.16f},
    {64, 64, 256, 2, 0.164f, 0.340f, 0.80f, 1.54f},   {64, 32, 256, 1, 0.096f, 0.107f, 1.27f, 1.30f},
};
constexpr int kCutNone = -1;
template <typename C, int TILE>
constexpr bool describes() { return C::kF == kTileCost[TILE].f && C::kT == kTileCost[TILE].t && C::kThreads == kTileCost[TILE].threads; }
static_assert(describes<Tile256x256, 0>() && describes<Tile256x128, 1>() && describes<Tile128x128, 2>() && describes<Tile128x64, 3>() &&
              describes<Tile64x64, 4>() && describes<Split64x32, 5>(), "the table is in the order of the tilings");

// us for `tiles` tiles of one kind over n_kt k-tiles
float tiles_cost(const TileCost &c, int64_t tiles, int n_kt, int cus) {
    const int64_t slots = int64_t(cus) * c.per_cu, rounds = tiles / slots, rest = tiles - rounds * slots;
    float us = float(rounds) * (c.full * float(n_kt) + c.once_full);
    if (rest > 0) {
        const float u = float(rest) / float(slots);
        // from half to all of the compute units; with two tiles to a unit every tile beyond one each shares its unit
        const float f = u <= 0.5f ? 0.0f : c.per_cu > 1 ? 1.0f : (u - 0.5f) * 2.0f;
        us += (c.part + f * (c.full - c.part)) * float(n_kt) + c.once_part + f * (c.once_full - c.once_part);
    }
    return us;
}

struct Plan {
    int tile, cut;       // indexes of kTileCost; cut = kCutNone: every tile is taken whole
    int64_t whole;       // tiles taken whole
};

// Whole rounds run the largest tiling that fills them.  What is left of a last round is cut into
// tiles that fill the chip once: 13230 x 5120 -> 5120 is 4 rounds of 256 x 256 tiles and 16 tiles
// more, 546 us with them whole and 494 us with those 16 cut into 128 x 64; 3780 x 1536 -> 4608 (one
// round and 14 tiles) 67 and 48 us; 2737 x 1024 -> 1024 (44 tiles) 22 us whole, 10.3 us as 176 tiles of
// 128 x 128; 520 x 5120 -> 640 (9 tiles) 85 us, 17 us as 90 tiles of 64 x 64 and 14 us as 170 of 64 x 32.
// With a k of a few tiles a round is its first loads and its stores, and large tiles are the cheaper ones: 60000 x 64 -> 3840
// takes 96 us in 256 x 256 tiles and 219 in 128 x 64; in the kernel of two tilings such rounds take up to 20 %
// longer (24000 x 256 -> 5120: 87 us whole, 106 cut), so that a cut has to promise 5 % there.
// One round of 120 to 250 tiles of 128 x 64 is faster than one of half as many of 128 x 128: 1271 x 704 -> 1536 6.7 and 8.1 us.
// Over the calls above the choice is off the best tiling by 0.4 % on average, by more than 10 % in 20 of them.
Plan pick_plan(int64_t n, int32_t d_in, int32_t d_out, bool small_ok, int cus) {
    static constexpr int kCuts[][2] = {{0, 1}, {0, 2}, {0, 3}, {2, 3}};   // the pairs compiled below
    const int n_kt = d_in / kBK;
    auto count = [&](int k) { return ((n + kTileCost[k].t - 1) / kTileCost[k].t) * ((d_out + kTileCost[k].f - 1) / kTileCost[k].f); };
    Plan best{0, kCutNone, 0};
    float best_us = 0.0f;
    auto offer = [&](int tile, int cut, int64_t whole, int64_t workgroups, float us) {
        // the largest tiling, offered first, stands where a smaller one has more threads than a launch may
        if (best.whole != 0 && (us >= best_us || workgroups * kTileCost[tile].threads > lp::kMaxLaunchThreads)) return;
        best = Plan{tile, cut, whole};
        best_us = us;
    };
    for (int k = 0; k < (small_ok ? 6 : 4); ++k) offer(k, kCutNone, count(k), count(k), tiles_cost(kTileCost[k], count(k), n_kt, cus));
    for (const auto &p : kCuts) {
        const TileCost &big = kTileCost[p[0]], &small = kTileCost[p[1]];
        const int64_t tiles = count(p[0]), whole = tiles / cus * cus;
        if (whole == 0 || whole == tiles) continue;
        const int64_t parts = (tiles - whole) * (big.f / small.f) * (big.t / small.t);
        const float cut_us = tiles_cost(big, whole, n_kt, cus) + tiles_cost(small, parts, n_kt, cus);
        offer(p[0], p[1], whole, whole + parts, n_kt < 12 ? 1.05f * cut_us : cut_us);
    }
    return best;
}

template <bool QKV, int HD, typename P, typename R>
int launch_tiles(GemmArgs a, int64_t whole, hipStream_t stream) {
    constexpr int kLds = P::kLds > R::kLds ? P::kLds : R::kLds;
    static std::atomic<uint64_t> attr_set{0};
    const void *kern = reinterpret_cast<const void *>(&gemm_kernel<QKV, HD, P, R>);
    int dev = 0;
    const hipError_t e = hipGetDevice(&dev);
    if (e != hipSuccess) {
        lp::set_last_hip_error(int(e));
        return LP_ERR_HIP;
    }
    const int rc = allow_lds(kern, kLds, dev, attr_set);
    if (rc != LP_OK) return rc;
    a.n_ftiles = (a.d_out + P::kF - 1) / P::kF;
    a.n_ttiles = (a.n + P::kT - 1) / P::kT;
    const int64_t tiles = int64_t(a.n_ftiles) * a.n_ttiles;
    constexpr int64_t kCut = int64_t(P::kF / R::kF) * (P::kT / R::kT);
    const int64_t grid = whole + (tiles - whole) * kCut;
    if (grid >= (int64_t(1) << 31)) return LP_ERR_UNSUPPORTED;
    a.whole = int32_t(whole);
    return lp::launch_kernel(kern, dim3(uint32_t(grid)), dim3(P::kThreads), kLds, stream, a);
}

// head_dim 0: lp_linear; a head of 128 does not fit the smallest tiles' features
constexpr bool small_tilings(int head_dim) { return head_dim <= 64; }

// Whether lp_linear runs a plan's tiles of 256 features with four wavefronts: see product_wide.
bool four_waves(const Plan &p, int32_t d_in) { return p.tile <= 1 && d_in / kBK >= (p.tile == 0 && p.cut == kCutNone ? 64 : 32); }

template <bool QKV, int HD>
int launch_gemm(GemmArgs a, hipStream_t stream) {
    constexpr bool kSmall = small_tilings(QKV ? HD : 0);
    const int cus = lp::device_compute_units();
    if (cus <= 0) return LP_ERR_HIP;
    const Plan p = pick_plan(a.n, a.d_in, a.d_out, kSmall, cus);
    if constexpr (!QKV) {
        if (four_waves(p, a.d_in)) {
            switch (p.tile * 8 + p.cut + 1) {
                case 0 * 8: return launch_tiles<QKV, HD, Wide256x256, Wide256x256>(a, p.whole, stream);
                case 0 * 8 + 2: return launch_tiles<QKV, HD, Wide256x256, Wide256x128>(a, p.whole, stream);
                case 0 * 8 + 3: return launch_tiles<QKV, HD, Wide256x256, Four128x128>(a, p.whole, stream);
                case 0 * 8 + 4: return launch_tiles<QKV, HD, Wide256x256, Four128x64>(a, p.whole, stream);
                default: return launch_tiles<QKV, HD, Wide256x128, Wide256x128>(a, p.whole, stream);
            }
        }
    }
    switch (p.tile * 8 + p.cut + 1) {
        case 0 * 8 + 2: return launch_tiles<QKV, HD, Tile256x256, Tile256x128>(a, p.whole, stream);
        case 0 * 8 + 3: return launch_tiles<QKV, HD, Tile256x256, Tile128x128>(a, p.whole, stream);
        case 0 * 8 + 4: return launch_tiles<QKV, HD, Tile256x256, Tile128x64>(a, p.whole, stream);
        case 2 * 8 + 4: return launch_tiles<QKV, HD, Tile128x128, Tile128x64>(a, p.whole, stream);
        case 1 * 8: return launch_tiles<QKV, HD, Tile256x128, Tile256x128>(a, p.whole, stream);
        case 2 * 8: return launch_tiles<QKV, HD, Tile128x128, Tile128x128>(a, p.whole, stream);
        case 3 * 8: return launch_tiles<QKV, HD, Tile128x64, Tile128x64>(a, p.whole, stream);
        case 4 * 8:
            if constexpr (kSmall) return launch_tiles<QKV, HD, Tile64x64, Tile64x64>(a, p.whole, stream);
            [[fallthrough]];
        case 5 * 8:
            if constexpr (kSmall) return launch_tiles<QKV, HD, Split64x32, Split64x32>(a, p.whole, stream);
            [[fallthrough]];
        default: return launch_tiles<QKV, HD, Tile256x256, Tile256x256>(a, p.whole, stream);
    }
}

// shape limits of the product: k in whole tiles, 32-bit byte offsets inside a tile's rows
int check_gemm_shape(int64_t n, int32_t d_in, int32_t d_out) {
    if (n < 0 || d_in < 1 || d_out < 1) return LP_ERR_INVALID_ARG;
    if (d_in % kBK != 0 || d_out % 128 != 0) return LP_ERR_UNSUPPORTED;   // whole k-tiles; whole wave tiles of features (32, 64 or 128)
    if (int64_t(256) * d_in * 2 >= (int64_t(1) << 31) || n >= (int64_t(1) << 31)) return LP_ERR_UNSUPPORTED;
    return LP_OK;
}

}  // namespace

extern "C" int lp_internal_gemm_way(int64_t n, int32_t d_in, int32_t d_out, int32_t head_dim, int32_t cus, int64_t way[6]) {
    const Plan p = pick_plan(n, d_in, d_out, small_tilings(head_dim), cus);
    const TileCost &c = kTileCost[p.tile], &r = kTileCost[p.cut < 0 ? p.tile : p.cut];
    const int64_t tiles = ((n + c.t - 1) / c.t) * ((d_out + c.f - 1) / c.f);
    way[0] = c.f;
    way[1] = c.t;
    way[2] = p.cut < 0 ? 0 : r.f;
    way[3] = p.cut < 0 ? 0 : r.t;
    way[4] = p.whole + (tiles - p.whole) * (c.f / r.f) * (c.t / r.t);
    way[5] = head_dim == 0 && four_waves(p, d_in) ? Wide256x256::kThreads : c.threads;
    return LP_OK;
}

extern "C" int lp_linear(const void *x, const void *w, const float *bias, void *y, int64_t n, int32_t d_in, int32_t d_out,
                         void *stream) {
    const int chk = check_gemm_shape(n, d_in, d_out);
    if (chk != LP_OK) return chk;
    if (n == 0) return LP_OK;
    if (x == nullptr || w == nullptr || y == nullptr) return LP_ERR_INVALID_ARG;
    if (!aligned16(x) || !aligned16(w) || !aligned16(y) || !aligned16(bias) || y == x || y == w) return LP_ERR_INVALID_ARG;
    GemmArgs a{};
    a.x = static_cast<const __bf16 *>(x);
    a.w = static_cast<const __bf16 *>(w);
    a.bias = bias;
    a.out[0] = static_cast<__bf16 *>(y);
    a.n = int32_t(n);
    a.d_in = d_in;
    a.d_out = d_out;
    return launch_gemm<false, 128>(a, static_cast<hipStream_t>(stream));
}

extern "C" int lp_qkv_projection(const void *x, const void *w_qkv, const float *bias, const float *gain_q, const float *gain_k,
                                 float eps, const lp_rope *rope, void *q, void *k, void *v, int64_t n_tokens, int32_t heads,
                                 int32_t head_dim, void *stream) {
    if (heads < 1) return LP_ERR_INVALID_ARG;
    if (head_dim != 64 && head_dim != 128) return LP_ERR_UNSUPPORTED;
    const int64_t dm64 = int64_t(heads) * head_dim;
    if (3 * dm64 >= (int64_t(1) << 31)) return LP_ERR_UNSUPPORTED;
    const int32_t dm = int32_t(dm64);
    if (dm % 128 != 0) return LP_ERR_UNSUPPORTED;          // a wave's features (up to 128) must not straddle q | k | v
    const int chk = check_gemm_shape(n_tokens, dm, 3 * dm);
    if (chk != LP_OK) return chk;
    if (n_tokens == 0) return LP_OK;
    if (x == nullptr || w_qkv == nullptr || gain_q == nullptr || gain_k == nullptr || q == nullptr || k == nullptr || v == nullptr)
        return LP_ERR_INVALID_ARG;
    if (!aligned16(x) || !aligned16(w_qkv) || !aligned16(bias) || !aligned16(gain_q) || !aligned16(gain_k) || !aligned16(q) ||
        !aligned16(k) || !aligned16(v))
        return LP_ERR_INVALID_ARG;
    if (q == k || q == v || k == v || q == x || k == x || v == x) return LP_ERR_INVALID_ARG;
    GemmArgs a{};
    const int rc = make_rope_args(rope, n_tokens, head_dim, eps, &a.rope);
    if (rc != LP_OK) return rc;
    a.x = static_cast<const __bf16 *>(x);
    a.w = static_cast<const __bf16 *>(w_qkv);
    a.bias = bias;
    a.out[0] = static_cast<__bf16 *>(q);
    a.out[1] = static_cast<__bf16 *>(k);
    a.out[2] = static_cast<__bf16 *>(v);
    a.gain[0] = gain_q;
    a.gain[1] = gain_k;
    a.n = int32_t(n_tokens);
    a.d_in = dm;
    a.d_out = 3 * dm;
    a.heads = heads;
    hipStream_t st = static_cast<hipStream_t>(stream);
    return head_dim == 128 ? launch_gemm<true, 128>(a, st) : launch_gemm<true, 64>(a, st);
}

extern "C" int lp_qk_norm_rope(void *x, const float *gain, float eps, const lp_rope *rope, int64_t n_tokens, int32_t heads,
                               int32_t head_dim, int64_t stride_tok, int64_t stride_head, void *stream) {
    if (heads < 1 || n_tokens < 0) return LP_ERR_INVALID_ARG;
    if (head_dim != 64 && head_dim != 128) return LP_ERR_UNSUPPORTED;
    if (n_tokens == 0) return LP_OK;
    if (x == nullptr || gain == nullptr || !aligned16(x) || !aligned16(gain)) return LP_ERR_INVALID_ARG;
    if (stride_head < head_dim || stride_head % 8 != 0 || stride_tok % 8 != 0) return LP_ERR_INVALID_ARG;
    const bool token_major = stride_tok >= int64_t(heads) * stride_head;
    const bool head_major = stride_head >= n_tokens * stride_tok && stride_tok >= head_dim;
    if (!token_major && !head_major) return LP_ERR_INVALID_ARG;
    RopeArgs r;
    const int rc = make_rope_args(rope, n_tokens, head_dim, eps, &r);
    if (rc != LP_OK) return rc;
    const int64_t threads = n_tokens * heads * (head_dim / 8);
    const int64_t blocks = (threads + 255) / 256;
    if (blocks >= (int64_t(1) << 31)) return LP_ERR_UNSUPPORTED;
    hipStream_t st = static_cast<hipStream_t>(stream);
    const void *fn = head_dim == 128 ? reinterpret_cast<const void *>(&norm_rope_kernel<128>)
                                     : reinterpret_cast<const void *>(&norm_rope_kernel<64>);
    return lp::launch_kernel(fn, dim3(uint32_t(blocks)), dim3(256), 0, st, static_cast<__bf16 *>(x), gain, n_tokens, heads,
                             stride_tok, stride_head, r);
}
