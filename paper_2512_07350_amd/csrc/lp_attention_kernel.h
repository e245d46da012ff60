// attention_kernel, the kernel of lp_attention for all but short calls: non-causal multi-head self-attention over the patch tokens of one
// sub-latent (supplement, proof of Theorem 1, step 3: inside a sub-latent the DiT
// blocks attend globally over all of its positions), as a flash-style kernel for
// gfx950: bf16 MFMA 16x16x32 for both products, binary32 online softmax, K and V
// tiles streamed global -> LDS without passing through registers.
//
// Work decomposition.  One workgroup = 4 wavefronts = 256 query rows of one head, one
// wavefront per SIMD; each wavefront owns 64 query rows (QB = four 16-column MFMA blocks) and
// walks all keys in rounds of 32.  (Where 256 rows leave compute units idle or rows past the end of many heads, 192 or 128: QB =
// 3 or 2, see deal_finer in lp_attention.hip.  All that is said here of 64 rows holds for 48 and 32, with fewer products to an
// operand fetched.)  Per round it forms the TRANSPOSED scores
//     S^T[key, query] = K . Q^T            (A = K rows from LDS, B = Q in registers)
// so that in the MFMA accumulator layout a lane holds 8 scores of ONE query per block: the
// row maximum and row sum are in-lane reductions, the rescale factor of the running
// output is a per-lane scalar, and the bf16 probabilities are already laid out as
// the B operand of
//     O^T[d, query] += V^T . P^T           (A = V^T, read transposed from LDS).
// Every operand fetched from LDS feeds four products (one per 16-query block).  The 64 rows
// need more than 256 registers per lane: the O^T accumulators and the Q^T operands are kept in
// the accumulation registers (AGPRs) by writing the matrix instructions as assembly statements
// with the register file of every operand spelled out (see mfma_score / mfma_pv).
//
// The products are 16x16x32 and not 32x32x16: the part is limited by power, and a loop of nothing
// but products on N(0,1) operands sustains 2077 TFLOP/s with the former and 1837 with the latter.
// The kernel's own step on the same schedule: 1258 TFLOP/s with 32x32x16, 1373 with 16x16x32, 1408
// with four tiles unrolled (13230 tokens, 40 heads of 128).
//
// What a step costs follows from what a SIMD issues for its one wavefront (measured in loops of nothing else): a product
// 8 cycles of issue and 16 of the matrix pipeline, a vector instruction 4, an exponential 8; v_dot2c_f32_bf16 goes through
// the matrix pipeline and holds it 16 cycles.  With the row sums as 16 dots a step, and windows of unequal length, a step took 1450
// cycles at head_dim 128 (1024 of products); with the row sums as four products and the windows evened out 1120: 13230
// tokens, 40 heads of 128 2590 -> 2350 us, 2999 x 16 of 64 45.4 -> 40.4 us.  Without any row sums it would be 2.5 % less,
// with the probabilities added one by one in binary32 it is 4 % more (12 % at head_dim 64, where issue binds).
//
// Details that matter for speed:
//  * Q is multiplied by scale*log2(e) once and re-rounded to bf16, and the score
//    accumulators start at -m (m = running maximum, log2 units), so a probability
//    is a bare exp2 of the accumulator.
//  * A segment's rounds run first with the maximum fixed at what the segment's first round made
//    it and no look at the scores at all: exp2 of a score 100 log2 units above that maximum is
//    still an ordinary binary32 / bf16 number, and numerator and denominator of the final
//    division carry the same power of two.  Only if a row sum or an accumulator comes out
//    non-finite (a score about 2^7 log2 units above the first round's), or a row sum vanishes (nothing but -inf
//    in the first round), does the workgroup run the segment again, this time raising the maximum lazily: when some score exceeds it by
//    more than kRescaleThreshold, in a rarely taken, wave-uniform branch that rescales the
//    output accumulators.
//  * The score product of round r+1, the softmax of round r and the PV product of round
//    r-1 (with the row sums, the same probabilities times an operand of ones) share one step, and the step's vector and
//    LDS work is cut into one small window per matrix instruction (pipeline_step), so that the one wavefront of a
//    SIMD has its next product ready when the matrix pipeline takes it.
//  * The key order inside a 32-key round is permuted (MFMA row r of the round's block b is
//    key 8 (r / 4) + 4 b + r % 4) so that the 8 probabilities a lane feeds to one MFMA
//    belong to 8 consecutive keys; V^T operands then come from two ds_read_b64_tr_b16
//    (transposing LDS reads) of the row-major V tile.
//  * K/V tiles go global -> LDS with buffer_load_dwordx4 ... lds (kStages tiles
//    resident), with XOR swizzles of the 16-byte granules chosen so that the K
//    reads (ds_read_b128) and the V reads are free of bank conflicts.
//  * One persistent workgroup per compute unit.  Query tiles left over after whole rounds are taken whole, in tiles of 192
//    rows, or the (query tile, key tile) space is dealt so that every workgroup gets the same cost, and a
//    query tile shared by several workgroups is merged by combine_kernel (see AttnParams).
//  * A segment's results leave as whole 128-byte lines through per-wave LDS
//    staging, after the next segment's first tiles and Q rows have been sent for.
#pragma once
#include <hip/hip_runtime.h>

#include <atomic>
#include <type_traits>

#include "lp_attention.h"

namespace {

using namespace lp;

constexpr int kStages = 4;                    // LDS stages: three tiles in use plus one arriving
constexpr float kRescaleThreshold = 8.0f;     // log2 units the running max may lag behind

template <int D>
struct Tile : TileSwizzle<D> {
    static constexpr int kRowBytes = D * 2;
    static constexpr int kGran = kRowBytes / 16;            // 16-byte granules per row
    static constexpr int kTileBytes = kBN * kRowBytes;      // one K or one V tile
    static constexpr int kStageBytes = 2 * kTileBytes;      // K tile then V tile
    static constexpr int kRingBytes = kStages * kStageBytes;
    static constexpr int kOutBytes = 16 * kRowBytes;        // per wave: 16 result rows in bf16
    static constexpr int kBytes = kRingBytes + kWaves * kOutBytes;
    // Stages an LDS instruction reaches by its 16-bit offset from the first of them (power of two)
    static constexpr int kReach = kStages * kStageBytes <= 65536 ? kStages : 2;
    static constexpr int kRowsPerInstr = 1024 / kRowBytes;  // rows one wave-wide 16-byte load covers
    static constexpr int kInstrPerTile = kBN / kRowsPerInstr;
};

// Wait until at most `pending` of this wave's global->LDS loads are still in flight.
template <int PENDING>
__device__ __forceinline__ void wait_tile_loads() {
    static_assert(PENDING >= 0 && PENDING < 64, "vmcnt range");
    asm volatile("s_waitcnt vmcnt(%0)" ::"n"(PENDING) : "memory");
}

// At most N LDS operations of this wavefront still outstanding (the compiler sees this wait
// and leaves out its own for everything older).
template <int N>
__device__ __forceinline__ void lds_wait() {
    static_assert(N >= 0 && N < 16, "lgkmcnt range");
    __builtin_amdgcn_s_waitcnt(0xC07F | (N << 8));
}

// The same value, but not a loop invariant as far as the compiler can tell.
__device__ __forceinline__ int opaque(int x) {
    asm volatile("" : "+v"(x));
    return x;
}

// addr += delta, here and once (the compiler would otherwise form every address of an unrolled
// stretch anew from the first one).
__device__ __forceinline__ void move_address(uint32_t &addr, uint32_t delta) {
    addr += delta;
    asm volatile("" : "+v"(addr));
}

// What a lane needs to know to move tiles from global memory into LDS.
template <int D>
struct Lane {
    using T = Tile<D>;
    static constexpr int kLd = T::kInstrPerTile / kWaves;   // K (and V) load instructions per wave per tile
    __amdgpu_buffer_rsrc_t k_rsrc, v_rsrc;   // K and V of this head as raw buffers ending with token n-1
    uint32_t k_voff[kLd], v_voff[kLd];       // byte offset of this lane's 16 bytes in tile 0
    uint32_t ld_dst[kLd];                    // LDS offset of the 1024-byte block inside a K tile (wave-uniform)
    uint32_t ld_base[kLd];                   // lds0 + ld_dst
    uint32_t tile_bytes;                     // global byte distance between consecutive tiles
    uint32_t valid_bytes;                    // size of the K (and V) buffer of the current head: a load at or past it reads zeros and fetches nothing
    int quad;                                // lane / 16
    int key_end;                             // keys at and past this index do not exist for the current segment
    int t_end;                               // one past the segment's last tile
};

// The global -> LDS loads of a K and a V block (see load_to_lds_16): the waits that order them against the reads of their own
// stage are wait_tile_loads + barrier.  M0 belongs to these and to set_m0 / load_to_lds_16 below, whose value lives on from one window to
// the next: nothing may write it between a set_m0 and its load.  The compiler has no use for M0 in these kernels;
// tests/test_wait_states.py looks for one in the built library.
template <int V_LDS_OFFSET>
__device__ __forceinline__ void load_kv_to_lds_16(__amdgpu_buffer_rsrc_t k_rsrc, __amdgpu_buffer_rsrc_t v_rsrc, uint32_t k_lds,
                                                  uint32_t k_voff, uint32_t v_voff, uint32_t soff) {
    // K block, then the V block V_LDS_OFFSET bytes further on.  M0 must be written one
    // instruction before the load that uses it: the address of the V block is formed between
    // the first write and its use, an s_nop stands between the second write and its use.
    uint32_t v_lds;
    asm volatile("s_mov_b32 m0, %1\n\ts_add_u32 %0, %1, %2\n\tbuffer_load_dwordx4 %3, %5, %7 offen lds\n\t"
                 "s_mov_b32 m0, %0\n\ts_nop 0\n\tbuffer_load_dwordx4 %4, %6, %7 offen lds"
                 : "=&s"(v_lds)
                 : "s"(k_lds), "n"(V_LDS_OFFSET), "v"(k_voff), "v"(v_voff), "s"(k_rsrc), "s"(v_rsrc), "s"(soff)
                 : "memory", "m0", "scc");
}

// The same in two statements, one window apart: M0 for the next load (its LDS address, base + OFF), then the load.
template <int OFF>
__device__ __forceinline__ void set_m0(uint32_t base) {
    asm volatile("s_add_u32 m0, %0, %1" ::"s"(base), "n"(OFF) : "memory", "m0", "scc");
}
__device__ __forceinline__ void load_to_lds_16(__amdgpu_buffer_rsrc_t rsrc, uint32_t voff, uint32_t soff) {
    asm volatile("buffer_load_dwordx4 %0, %1, %2 offen lds" ::"v"(voff), "s"(rsrc), "s"(soff) : "memory");
}

// global -> LDS loads of one K/V tile into the stage at byte offset stage_off.  One
// wave-wide instruction moves 1024 bytes.  Rows past token n-1 lie outside the buffers
// and arrive as zeros.
template <int D>
__device__ __forceinline__ void issue_tile(uint32_t lds0, const Lane<D> &c, int tile, uint32_t stage_off) {
    using T = Tile<D>;
    const uint32_t soff = uint32_t(tile) * c.tile_bytes;
#pragma unroll
    for (int i = 0; i < Lane<D>::kLd; ++i) {
        const uint32_t dst_k = __builtin_amdgcn_readfirstlane(lds0 + stage_off + c.ld_dst[i]);
        load_kv_to_lds_16<T::kTileBytes>(c.k_rsrc, c.v_rsrc, dst_k, c.k_voff[i], c.v_voff[i], soff);
    }
}

// The I-th of a wave's kLd load statements of a tile (K block and V block), at scalar byte offset
// soff (which takes part in the buffer's range check, like the lane's own offset).
template <int D, int I>
__device__ __forceinline__ void issue_tile_part(uint32_t lds0, const Lane<D> &c, uint32_t soff, uint32_t stage_off) {
    using T = Tile<D>;
    const uint32_t dst_k = __builtin_amdgcn_readfirstlane(lds0 + stage_off + c.ld_dst[I]);
    load_kv_to_lds_16<T::kTileBytes>(c.k_rsrc, c.v_rsrc, dst_k, c.k_voff[I], c.v_voff[I], soff);
}

// Keys past the end get score -inf.  Element i of a lane's block b is key 32 r + 8 quad + 4 b + i.
template <int QB>
__device__ __forceinline__ void mask_scores(int r, int quad, int n, f32x4 (&s)[2][QB]) {
    const int kbase = r * 32 + quad * 8;
#pragma unroll
    for (int b = 0; b < 2; ++b)
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            const bool past = kbase + 4 * b + i >= n;
#pragma unroll
            for (int qb = 0; qb < QB; ++qb) s[b][qb][i] = past ? -INFINITY : s[b][qb][i];
        }
}

// ---- the matrix instructions, with the register file of every operand chosen here.
// A wavefront that owns 64 query rows needs more than 256 registers: the O^T accumulators
// (D / 16 * QB * 4) and the Q^T operands (QB * D / 32 * 4) live in the accumulation registers
// (AGPRs) and are touched by matrix instructions only; scores, probabilities and the LDS
// operands live in the ordinary ones, where the vector ALU works on them.  The compiler is
// not told what these statements are, so it neither moves operands between the two files
// nor inserts the wait states that separate a matrix instruction's result from a vector
// instruction reading it; settle_scores / settle_acc below do that where such a read follows.
__device__ __forceinline__ void mfma_score_init(f32x4 &d, const bf16x8 &k, const bf16x8 &q, const f32x4 &c) {
    asm volatile("v_mfma_f32_16x16x32_bf16 %0, %1, %2, %3" : "=&v"(d) : "v"(k), "a"(q), "v"(c));
}
__device__ __forceinline__ void mfma_score(f32x4 &d, const bf16x8 &k, const bf16x8 &q) {
    asm volatile("v_mfma_f32_16x16x32_bf16 %0, %1, %2, %0" : "+v"(d) : "v"(k), "a"(q));
}
__device__ __forceinline__ void mfma_pv(f32x4 &acc, const bf16x8 &vt, const bf16x8 &p) {
    asm volatile("v_mfma_f32_16x16x32_bf16 %0, %1, %2, %0" : "+a"(acc) : "v"(vt), "v"(p));
}

// The vector work between the products, likewise as assembly statements: they keep their program
// order, so every instruction stays in the window it is written in.  (With ordering points between
// ordinary instructions the compiler puts a wait state wherever a use directly follows such a
// point.)  A conversion must not directly follow the exponential it reads, nor a product by
// less than two instructions the conversion it reads; the windows keep them further apart.
__device__ __forceinline__ void exp2_to(float &p, float s) { asm volatile("v_exp_f32 %0, %1" : "=v"(p) : "v"(s)); }
__device__ __forceinline__ void pack_bf16(uint32_t &w, float lo, float hi) {
    asm volatile("v_cvt_pk_bf16_f32 %0, %1, %2" : "=v"(w) : "v"(lo), "v"(hi));
}

// Scores written by matrix instructions become readable by vector instructions: 16 wait
// states cover the passes of the last product plus its write-back.
template <int QB>
__device__ __forceinline__ void settle_scores(f32x4 (&s)[2][QB], bool wait) {
    if (wait) asm volatile("s_nop 15");
#pragma unroll
    for (int b = 0; b < 2; ++b)
#pragma unroll
        for (int qb = 0; qb < QB; ++qb) asm volatile("" : "+v"(s[b][qb]));
}

// The same for the accumulators in the AGPRs (before they are rescaled or stored), and, with
// after = true, between vector writes to them and the next matrix instruction.
template <int D, int QB>
__device__ __forceinline__ void settle_acc(f32x4 (&acc)[D / 16][QB], f32x4 (&l_acc)[QB], bool after) {
    if (after) asm volatile("s_nop 3");
    else asm volatile("s_nop 15\n\ts_nop 7");
#pragma unroll
    for (int qb = 0; qb < QB; ++qb) {
        asm volatile("" : "+a"(l_acc[qb]));
#pragma unroll
        for (int mb = 0; mb < D / 16; ++mb) asm volatile("" : "+a"(acc[mb][qb]));
    }
}

// Lazy running maximum.  Score accumulators start at neg_m = -m (m = running maximum, log2
// units), so s holds scores relative to m that will be exponentiated NEXT.  If any of them
// exceeds kRescaleThreshold, raise the maximum by delta and rescale what was accumulated
// under the old one: these scores, the output accumulators, the row sums, and the
// probabilities p_pending that have been computed but not yet multiplied into either.
// A query that has seen nothing but scores of -inf has no maximum yet, which neg_m = -0 says (no_maximum): the first
// score above -inf sets it, wherever that lies, and nothing has been accumulated that would have to be rescaled.
constexpr uint32_t kNoMaximum = 0x80000000u;                                   // -0; 0 - m and x - x are never that
__device__ __forceinline__ bool no_maximum(const f32x4 &neg_m) { return __float_as_uint(neg_m[0]) == kNoMaximum; }
template <int D, int QB>
__device__ __forceinline__ void raise_maximum(const float (&lane_max)[QB], f32x4 (&s)[2][QB], f32x4 (&neg_m)[QB],
                                              bf16x8 (&p_pending)[QB], f32x4 (&acc)[D / 16][QB], f32x4 (&l_acc)[QB]) {
    bool raise = false;
#pragma unroll
    for (int qb = 0; qb < QB; ++qb) raise = raise || (lane_max[qb] > (no_maximum(neg_m[qb]) ? -INFINITY : kRescaleThreshold));
    if (__builtin_expect(__any(raise) != 0, 0)) {     // the branch body is laid out away from the loop
        settle_acc<D, QB>(acc, l_acc, false);
#pragma unroll
        for (int qb = 0; qb < QB; ++qb) {
            const float top = quad_max(lane_max[qb]);
            const bool none = no_maximum(neg_m[qb]), sets = none && top != -INFINITY;
            const float delta = sets ? top : none ? 0.0f : fmaxf(top, 0.0f);   // a maximum never goes down
            const float alpha = none ? 0.0f : __builtin_amdgcn_exp2f(-delta);
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                s[0][qb][i] -= delta;
                s[1][qb][i] -= delta;
                neg_m[qb][i] = sets ? 0.0f - top : neg_m[qb][i] - delta;
                l_acc[qb][i] *= alpha;
            }
#pragma unroll
            for (int mb = 0; mb < D / 16; ++mb)
#pragma unroll
                for (int i = 0; i < 4; ++i) acc[mb][qb][i] *= alpha;
            Pack16 t;
            t.v = p_pending[qb];
            const uint32_t w[4] = {t.u.x, t.u.y, t.u.z, t.u.w};
#pragma unroll
            for (int e = 0; e < 4; ++e)
                t.p[e] = to_bf16x2(__uint_as_float(w[e] << 16) * alpha, __uint_as_float(w[e] & 0xffff0000u) * alpha);
            p_pending[qb] = t.v;
        }
        settle_acc<D, QB>(acc, l_acc, true);
    }
}

// One K operand (16 bytes of a K row) from LDS: operand g is block g % 2 of the d-step g / 2; SUB
// selects the first or second round of the tile OFF bytes after the one k_addr points into.
template <int D, int SUB, int OFF>
__device__ __forceinline__ bf16x8 load_k_operand(const uint32_t (&k_addr)[D / 32], int g) {
    return lds_load<bf16x8>(k_addr[g / 2] + OFF + (SUB * 32 + 4 * (g % 2)) * Tile<D>::kRowBytes);
}

// One V^T operand via two transposing reads.  Inside a group of 16 lanes, lane j supplies
// the 8-byte chunk (row j/4, columns 4*(j%4)..+3) and receives column j of that 4x16 block,
// i.e. 4 consecutive keys of one d.  Operand mb covers the round's 32 keys and rows 16 mb .. of
// O^T; HALF selects the first or second four of a lane's eight keys.
template <int D, int SUB, int HALF, int OFF>
__device__ __forceinline__ bf16x4 load_v_half(const uint32_t (&v_addr)[D / 16], int mb) {
    const uint32_t a0 = v_addr[mb] + OFF + (SUB * 32 + HALF * 4) * Tile<D>::kRowBytes;
    return __builtin_amdgcn_ds_read_tr16_b64_v4bf16(LP_LDS_PTR(bf16x4, uintptr_t(a0)));
}

// Everything one wavefront carries from step to step.
template <int D, int QB>
struct Pipe {
    bf16x8 qreg[QB][D / 32];      // Q^T operands (pre-scaled)
    bf16x8 opreg[D / 16];          // LDS operands: K rows before a score product, V^T blocks before a PV product
    bf16x8 ones;                   // 1.0 in every element: the A operand of the row sums
    f32x4 acc[D / 16][QB];        // O^T accumulators
    f32x4 l_acc[QB];              // row sums, each of the four elements (and every lane of a query) the same
    f32x4 neg_m[QB];              // -m in every element (m = running maximum, log2 units, common to
                                   // the four lanes of a query): the initial value of every score accumulator
    uint32_t k_addr[D / 32];       // LDS addresses of the K operands in the stage at k_off
    uint32_t v_addr[D / 16];       // LDS addresses of the V operands in the stage at v_off
    uint32_t k_off, v_off;         // stage offsets k_addr / v_addr currently point into
    uint32_t tile_off;             // stage offset of tile i/2
    uint32_t issue_off;            // stage offset the next issued tile goes to
    int issue_t;                   // index of the next tile to issue
};

// Writes 16 result rows of this wave (block qb of acc scaled by `inv`, rounded to bf16) to rows
// dst + r * row_stride, r < rows_valid.  A lane holds, for query `col`, rows
// d = 16 mb + 4 quad + i of O^T, i.e. 8-byte pieces of many rows; the pieces pass through the
// wave's own LDS (16-byte granules XORed with the row) and leave as whole 128-byte lines.
template <int D, int QB>
__device__ __forceinline__ void store_rows(uint32_t out_lds, const f32x4 (&acc)[D / 16][QB], int qb, float inv, __bf16 *dst,
                                           int64_t row_stride, int rows_valid, int lane) {
    constexpr int kGran = Tile<D>::kGran;
    const int col = lane % 16, quad = lane / 16;
#pragma unroll
    for (int mb = 0; mb < D / 16; ++mb) {
        const f32x4 &x = acc[mb][qb];
        union { u32x2 u; bf16x2 p[2]; } ow;
        ow.p[0] = to_bf16x2(x[0] * inv, x[1] * inv);
        ow.p[1] = to_bf16x2(x[2] * inv, x[3] * inv);
        *LP_LDS_PTR(u32x2, uintptr_t(out_lds + col * Tile<D>::kRowBytes + 16 * ((2 * mb + quad / 2) ^ (col % kGran)) + 8 * (quad % 2))) = ow.u;
    }
#pragma unroll
    for (int j = 0; j < 16 * kGran / 64; ++j) {
        const int r = (lane + 64 * j) / kGran, g = lane % kGran;
        const u32x4 u = lds_load<u32x4>(out_lds + r * Tile<D>::kRowBytes + 16 * (g ^ (r % kGran)));
        if (r < rows_valid) *reinterpret_cast<u32x4 *>(dst + r * row_stride + 8 * g) = u;
    }
}

// Rounds the pairs of probabilities [FROM, TO) to packed bf16 words and completes an operand with its fourth word.  Pair k
// holds scores 2 k, 2 k + 1 counted block by block: word k % 4 of the operand of query block k / 4.
template <int FROM, int TO, int QB>
__device__ __forceinline__ void convert_pairs(const float (&ex)[QB * 8], uint32_t (&pw)[QB][4], bf16x8 (&p_cur)[QB]) {
    static_for<FROM, TO>([&](auto kc) {
        constexpr int k = decltype(kc)::value, qb = k / 4, e = k % 4;
        pack_bf16(pw[qb][e], ex[2 * k], ex[2 * k + 1]);
        if constexpr (e == 3) {
            Pack16 t;
            t.u = make_uint4(pw[qb][0], pw[qb][1], pw[qb][2], pw[qb][3]);
            p_cur[qb] = t.v;
        }
    });
}

// Where in a step what stands.  A step is (2 G + 1) QB windows, one per product: G = D / 16 score groups, the group of
// the row sums, G PV groups (a group is the QB products that share an operand).  After an odd window there is room for
// two instructions, after an even one for the exponential that leads the next (see pipeline_step).
template <int D, int QB>
struct Windows {
    static constexpr int G = D / 16, M = (2 * G + 1) * QB;
    static constexpr int kPv = (G + 1) * QB;                             // first window of the PV phase
    static constexpr int E = QB * 8, kEvery = 2 * G * QB / E;           // exponentials, and windows per exponential
    static_assert(kEvery == 2 || kEvery == 1, "the exponentials fill the products' windows");
    static constexpr int odd(int m) { return m | 1; }
    // the V^T operand of PV group g is fetched into the registers that score group g has read, a half at a time
    static constexpr int fetch_v(int g, int half) { return odd(g * QB + QB - 1) + 2 * half; }
    // the K operand g of the next score phase into those that PV group g has read
    static constexpr int fetch_k(int g) { return g == G - 1 ? M - 1 : odd(kPv + g * QB + QB - 1); }
    // load g of the next tile (K block g / 2, then its V block), behind the write of M0 in the window of load g - 1
    static constexpr int load(int g) { return kPv + g * QB + QB - 3; }
    static constexpr int v_before(int m) {                                // V fetches (halves) issued before window m
        int c = 0;
        for (int g = 0; g < G; ++g)
            for (int h = 0; h < 2; ++h) c += fetch_v(g, h) < m;
        return c;
    }
    static constexpr int k_before(int m) {
        int c = 0;
        for (int g = 0; g < G; ++g) c += fetch_k(g) < m;
        return c;
    }
    static_assert(fetch_v(G - 1, 1) < kPv && fetch_k(G - 2) < M && load(0) >= G * QB && load(G - 1) < M, "a fetch stands in its own phase, a load behind its barrier");
};

template <int BYTES>
__device__ __forceinline__ uint32_t next_stage(uint32_t off) {
    off += BYTES;
    return off == kStages * BYTES ? 0u : off;
}

// Step i of the software pipeline (SUB = i % 2).  For ONE wavefront a step issues
//   MFMA:  S^T of round i+1, then O^T += V^T P^T of round i-1
//   VALU:  probabilities of round i (spread over the whole step), then the maximum check
//          for round i+1
//   LDS :  each score group is followed by the fetch of a V operand of round i-1 into the
//          registers it has just read, each PV group by the fetch of a K operand of round i+2
// so that an LDS operand is fetched half a step before its products, and K and V operands
// share one set of registers.
// Even steps open tile t+1 (t = i/2): at the end of their score phase they wait for its loads
// and pass the barrier (after which every wave has fetched its last operand from tile t-2), and
// over their PV phase they refill that stage with tile t+kStages-2.
// The same code runs at the ends of a segment: with MASK, keys past the segment's end get
// scores -inf (probabilities 0), and the round before the first has probabilities 0, so
// the products issued for rounds that do not exist add nothing; their operands are read
// from valid, if stale, LDS addresses.  MASK = false is for steps whose rounds i+1 lie
// wholly inside the segment and keeps the step free of conditionals.
//
// STAGE >= 0: tile i/2 lies in that LDS stage, known at compile time (the unrolled part of a segment,
// see run_segment): operand addresses then differ between stages by an instruction's offset, and
// by kReach stages where that does not reach.
template <int D, int QB, int SUB, bool MASK, bool CHECK, int STAGE = -1>
__device__ __forceinline__ void pipeline_step(uint32_t lds0, const Lane<D> &c, int i, bool first,
                                              Pipe<D, QB> &w, f32x4 (&s_cur)[2][QB], f32x4 (&s_nxt)[2][QB],
                                              bf16x8 (&p_prev)[QB], bf16x8 (&p_cur)[QB]) {
    using T = Tile<D>;
    // Per-tile bookkeeping is scalar and happens here; what it decides is carried out inside the
    // windows below, so that no stretch of the step is without a product to issue:
    //  * SUB == 0 opens tile t+1 (t = i/2).  Its K operands are first fetched in the PV phase, so
    //    the wait for its loads and the barrier (after which every wave has fetched its last
    //    operand from tile t-2) stand at the end of the score phase; each K operand address moves
    //    to the new stage right before its first fetch there; and the kLd load statements that
    //    refill tile t-2's stage with tile t+kStages-2 are spread over the PV phase.  Past the
    //    segment's end the loads are given an offset outside the buffer: they fetch nothing.
    //  * SUB == 1: round i-1 is the first of tile i/2, the V fetches move on to that tile --
    //    unless it lies past the segment and was never loaded (its probabilities are 0, and 0
    //    times whatever an unwritten stage holds need not be 0); each V operand address moves
    //    right before its first fetch of the step.
    constexpr bool kFixed = STAGE >= 0;
    constexpr int kKStage = (STAGE + 1) % kStages, kVStage = SUB == 0 ? (STAGE + kStages - 1) % kStages : STAGE;
    constexpr int kKOff = kFixed ? (kKStage % T::kReach) * T::kStageBytes : 0, kVOff = kFixed ? (kVStage % T::kReach) * T::kStageBytes : 0;
    // in the unrolled part: the step to the next kReach stages, taken by the fetch that enters them
    constexpr uint32_t kHop = T::kReach * T::kStageBytes;
    constexpr bool kKHop = kFixed && T::kReach < kStages && SUB == 0 && kKStage % T::kReach == 0;
    constexpr bool kVHop = kFixed && T::kReach < kStages && SUB == 1 && STAGE % T::kReach == 0;
    uint32_t k_delta = 0, v_delta = 0, issue_soff = 0, issue_stage = 0;
    if (kFixed) {
        k_delta = kKStage == 0 ? 0u - (kStages / T::kReach - 1) * kHop : kHop;
        v_delta = STAGE == 0 ? 0u - (kStages / T::kReach - 1) * kHop : kHop;
        if (SUB == 0) {
            issue_soff = w.issue_t < c.t_end ? uint32_t(w.issue_t) * c.tile_bytes : c.valid_bytes;
            ++w.issue_t;
        }
    } else if (SUB == 0) {
        if (!first) w.tile_off = next_stage<T::kStageBytes>(w.tile_off);
        const uint32_t nxt_off = next_stage<T::kStageBytes>(w.tile_off);
        k_delta = nxt_off - w.k_off;       // wraps; the sums do not
        w.k_off = nxt_off;
        issue_soff = w.issue_t < c.t_end ? uint32_t(w.issue_t) * c.tile_bytes : c.valid_bytes;
        issue_stage = w.issue_off;
        ++w.issue_t;
        w.issue_off = next_stage<T::kStageBytes>(w.issue_off);
    } else {
        if (i / 2 < c.t_end) {
            v_delta = w.tile_off - w.v_off;
            w.v_off = w.tile_off;
        }
    }

    // The step's products come in G score groups, the group of the row sums and G PV groups.  The wavefront is alone on
    // its SIMD, which takes an instruction of it every 4 cycles (an exponential 8) and gives a product 8 of the 16 it takes: the
    // matrix pipeline stays busy if no more than 8 cycles of other instructions stand between two products.  The
    // vector and LDS work of the step is therefore cut into one small window per product (struct Windows): at head_dim
    // 128 the exponentials of round i alternate with what is shorter, a conversion, the refill of the operand
    // registers that a group has read (half a V^T operand or a K operand), in even steps the next tile's loads.  At 64
    // there are twice as many exponentials to a product and the windows are longer than it.
    // Row sums are products too, with an operand of ones: four per step.  As v_dot2c_f32_bf16 of the packed pairs they
    // held the matrix pipeline as long as a product each, 16 of them a step.
    using W = Windows<D, QB>;
    constexpr int G = W::G, M = W::M, E = W::E, kEvery = W::kEvery;
    uint32_t pw[QB][4];
    float ex[E];
    Pack16 vop;
    static_for<0, M>([&](auto mc) {
        // every second group runs backwards: neighbours then share an operand throughout, and what does not change costs less
        // power (13230 tokens, 40 heads of 128: 2280 -> 2251 us)
        constexpr int m = decltype(mc)::value, g = m / QB, at = m % QB, qb = g % 2 ? QB - 1 - at : at;
        // pair k is rounded in the window behind its second exponential's
        if constexpr (m % (2 * kEvery) == 0 && m > 0 && m / kEvery <= E) convert_pairs<m / (2 * kEvery) - 1, m / (2 * kEvery)>(ex, pw, p_cur);
        if constexpr (m % kEvery == kEvery - 1 && m / kEvery < E) {
            constexpr int x = m / kEvery;
            exp2_to(ex[x], s_cur[(x / 4) % 2][x / 8][x % 4]);
        }
        // Operand arrivals are checked for half a phase at a time.  In issue order the LDS queue holds, at the start of the
        // score phase, the G K fetches of the previous PV phase: all but the newest G / 2 cover groups 0 .. G / 2 - 1;
        // by group G / 2 the newest are the V fetches so far.  The PV phase mirrors this with
        // 2 G V fetches followed by one K fetch per group.
        if constexpr (at == 0 && g == 0) lds_wait<G / 2>();
        if constexpr (at == 0 && g == G / 2) lds_wait<W::v_before(m)>();
        if constexpr (at == 0 && g == G + 1) lds_wait<G>();
        if constexpr (at == 0 && g == G + 1 + G / 2) lds_wait<W::k_before(m)>();
        if constexpr (g < 2) mfma_score_init(s_nxt[g % 2][qb], w.opreg[g], w.qreg[qb][0], w.neg_m[qb]);
        else if constexpr (g < G) mfma_score(s_nxt[g % 2][qb], w.opreg[g], w.qreg[qb][g / 2]);
        else if constexpr (g == G) mfma_pv(w.l_acc[qb], w.ones, p_prev[qb]);
        else mfma_pv(w.acc[g - G - 1][qb], w.opreg[g - G - 1], p_prev[qb]);
        static_for<0, G>([&](auto oc) {
            constexpr int o = decltype(oc)::value;
            if constexpr (m == W::fetch_v(o, 0)) {
                if constexpr (kFixed ? kVHop : SUB == 1) move_address(w.v_addr[o], v_delta);
                vop.h[0] = load_v_half<D, 1 - SUB, 0, kVOff>(w.v_addr, o);
            }
            if constexpr (m == W::fetch_v(o, 1)) {
                vop.h[1] = load_v_half<D, 1 - SUB, 1, kVOff>(w.v_addr, o);
                w.opreg[o] = vop.v;
            }
            if constexpr (m == W::fetch_k(o)) {
                if constexpr (o % 2 == 0 && (kFixed ? kKHop : SUB == 0)) move_address(w.k_addr[o / 2], k_delta);
                w.opreg[o] = load_k_operand<D, SUB, kKOff>(w.k_addr, o);
            }
            // the tile's load statements, one block to a PV group (both blocks to every second one outside the unrolled part)
            if constexpr (SUB == 0 && kFixed) {
                constexpr int kDst = ((STAGE + kStages - 2) % kStages) * T::kStageBytes;
                if constexpr (m == W::load(0) - 2 && o == 0) set_m0<kDst>(c.ld_base[0]);
                if constexpr (m == W::load(o)) {
                    if constexpr (o % 2 == 0) load_to_lds_16(c.k_rsrc, c.k_voff[o / 2], issue_soff);
                    else load_to_lds_16(c.v_rsrc, c.v_voff[o / 2], issue_soff);
                    if constexpr (o + 1 < G) set_m0<kDst + (o % 2 == 0 ? T::kTileBytes : 0)>(c.ld_base[(o + 1) / 2]);
                }
            }
            if constexpr (SUB == 0 && !kFixed && m == W::load(o) && o % 2 == 0) issue_tile_part<D, o / 2>(lds0, c, issue_soff, issue_stage);
        });
        if constexpr (SUB == 0 && m == G * QB - 1) {
            // tile t+1, issued one tile ago; what is still on its way from LDS is V of tile t-1
            asm volatile("s_waitcnt vmcnt(0)\n\ts_barrier" ::: "memory");
        }
        if constexpr (m == W::kPv + QB) {             // the last score product has left the pipeline
            settle_scores(s_nxt, false);
            if (MASK) mask_scores(i + 1, c.quad, c.key_end, s_nxt);
        }
    });
    if constexpr (CHECK) {                     // the repeated run only, see run_segment
        float lane_max[QB];
#pragma unroll
        for (int qb = 0; qb < QB; ++qb) {
            lane_max[qb] = s_nxt[0][qb][0];
#pragma unroll
            for (int e = 1; e < 8; ++e) lane_max[qb] = fmaxf(lane_max[qb], s_nxt[e / 4][qb][e % 4]);
        }
        raise_maximum<D, QB>(lane_max, s_nxt, w.neg_m, p_cur, w.acc, w.l_acc);
    }
}

// Element offset of the first token of head index bh = batch_item * heads + head.
__device__ __forceinline__ int64_t head_offset(const AttnParams &a, int bh) {
    const int b = bh / a.heads;
    return int64_t(b) * a.stride_batch + int64_t(bh - b * a.heads) * a.stride_head;
}

// First iteration of (logical) workgroup p when W iterations are dealt to P workgroups.
__device__ __forceinline__ uint32_t range_start(uint32_t p, uint32_t W, uint32_t P) {
    return uint32_t(uint64_t(p) * W / P);
}

// Position x in the space with imaginary tiles -> index of the first real tile at or after it.
__device__ __forceinline__ uint32_t real_tile(uint32_t x, uint32_t unit_cost, uint32_t tpu) {
    const uint32_t unit = x / unit_cost, r = x - unit * unit_cost, imaginary = unit_cost - tpu;
    return unit * tpu + (r > imaginary ? r - imaginary : 0u);
}

// A segment: the tiles [t_begin, t_stop) of the unit whose query rows start at row0 of a head.
struct Segment {
    int head, row0;
    int t_begin, t_stop;
    bool valid;
};

// Where a workgroup stands in its work: its range of the shared space first, then whole units.
struct Walk {
    uint32_t it, it_end;
    int whole_round;
};

template <int QB>
__device__ __forceinline__ Segment next_segment(Walk &k, const AttnParams &a, uint32_t tpu, uint32_t lp, uint32_t n_wg) {
    Segment s;
    s.valid = true;
    uint32_t unit = 0;
    if (k.it < k.it_end) {
        unit = k.it / tpu;
        s.t_begin = int(k.it - unit * tpu);
        s.t_stop = int(min(tpu, uint32_t(s.t_begin) + (k.it_end - k.it)));
        k.it += uint32_t(s.t_stop - s.t_begin);
    } else if (k.whole_round < a.whole_rounds) {
        unit = uint32_t(a.shared_units) + uint32_t(k.whole_round) * n_wg + lp;
        s.t_begin = 0;
        s.t_stop = int(tpu);
        ++k.whole_round;
    } else {
        s.t_begin = s.t_stop = 0;
        s.valid = false;
    }
    s.head = int(unit) / a.n_qtiles;
    s.row0 = (int(unit) - s.head * a.n_qtiles) * unit_rows(QB);
    return s;
}

// The smaller unit that (logical) workgroup lp takes in the last round, if any: they are spread evenly over the workgroups, those of
// the head that the large units end in first.
template <int QB>
__device__ __forceinline__ Segment tail_segment(const AttnParams &a, uint32_t tpu, uint32_t lp, uint32_t n_wg) {
    Segment s;
    const uint32_t t = range_start(lp, a.tail_units, n_wg);
    const int past = int(t) - a.tail_first;
    s.head = past < 0 ? a.tail_head : a.tail_head + 1 + past / a.tail_qtiles;
    s.row0 = past < 0 ? a.tail_row + int(t) * unit_rows(QB) : past % a.tail_qtiles * unit_rows(QB);
    s.t_begin = 0;
    s.t_stop = int(tpu);
    s.valid = range_start(lp + 1, a.tail_units, n_wg) > t;
    return s;
}

// Points the tile traffic at a segment and sends for its first kStages-2 tiles (the
// segment's tiles use the LDS stages in turn, from stage 0).  The caller has made sure
// that no wave still reads the stages.
template <int D>
__device__ __forceinline__ void start_tiles(uint32_t lds0, const AttnParams &a, const Segment &seg, Lane<D> &c, int n, int64_t stride_tok) {
    using T = Tile<D>;
    const int64_t head_off = head_offset(a, seg.head);
    c.key_end = min(n, seg.t_stop * kBN);
    c.t_end = seg.t_stop;
    {
        // raw buffers over this head's K and V, ending with the last element of token n-1
        // (flags: 32-bit data format, as every untyped buffer on this architecture)
        const int valid_bytes = int((int64_t(n - 1) * stride_tok + D) * 2);
        c.valid_bytes = uint32_t(valid_bytes);
        const __bf16 *kh = a.k + head_off, *vh = a.v + head_off;
        c.k_rsrc = __builtin_amdgcn_make_buffer_rsrc(const_cast<__bf16 *>(kh), 0, valid_bytes, 0x00020000);
        c.v_rsrc = __builtin_amdgcn_make_buffer_rsrc(const_cast<__bf16 *>(vh), 0, valid_bytes, 0x00020000);
    }
#pragma unroll
    for (int t = 0; t < kStages - 2; ++t)
        if (seg.t_begin + t < c.t_end) issue_tile<D>(lds0, c, seg.t_begin + t, t * T::kStageBytes);
}

// Loads a segment's raw Q rows: a lane holds, for query `col` of a block, d = 32 kk + 8 quad .. +7.
template <int D, int QB>
__device__ __forceinline__ void load_q(const AttnParams &a, const Segment &seg, Pipe<D, QB> &w, int n,
                                       int64_t stride_tok, int wave, int col, int quad) {
    const __bf16 *qh = a.q + head_offset(a, seg.head);
    const int q0 = seg.row0 + wave * (16 * QB);
#pragma unroll
    for (int qb = 0; qb < QB; ++qb) {
        const int qi = q0 + qb * 16 + col;
#pragma unroll
        for (int kk = 0; kk < D / 32; ++kk) {
            Pack16 t;
            t.u = make_uint4(0, 0, 0, 0);
            if (qi < n) t.u = *reinterpret_cast<const uint4 *>(qh + int64_t(qi) * stride_tok + kk * 32 + quad * 8);
            w.qreg[qb][kk] = t.v;
        }
    }
}

// One segment after the other: `seg`, whose first tiles have been sent for, then what `next` gives.  Behind the last of them the
// tiles of `after`, the first segment of units of another size, are sent for.
template <int D, int QB, typename Next>
__device__ __forceinline__ void run_units(uint32_t lds0, const AttnParams &a, Lane<D> &c, int wave, Segment seg, const Segment &after,
                                          uint32_t sharer, Next &&next) {
    using T = Tile<D>;
    constexpr int G = D / 16;         // LDS operands per phase: (block, d-step) of S^T, 16-row blocks of O^T
    const int lane_id = threadIdx.x % 64;
    const int quad = lane_id / 16;
    const int n = a.n;
    const int64_t stride_tok = a.stride_tok;
    const int n_rounds = (n + 31) / 32;
    const uint32_t tpu = uint32_t(a.tiles_per_unit);
    const uint32_t out_lds = lds0 + T::kRingBytes + wave * T::kOutBytes;
    bool first_segment = true;

    Pipe<D, QB> w;
    {
        Pack16 t;
        t.u = make_uint4(0x3f803f80, 0x3f803f80, 0x3f803f80, 0x3f803f80);
        w.ones = t.v;
        asm volatile("" : "+v"(w.ones));
    }
    load_q<D, QB>(a, seg, w, n, stride_tok, wave, lane_id % 16, quad);

    while (true) {
        const int64_t head_off = head_offset(a, seg.head);
        const int t_begin = seg.t_begin, t_stop = seg.t_stop;
        const int i_begin = 2 * t_begin;                 // rounds [i_begin, i_end) of 32 keys
        const int i_end = min(2 * t_stop, n_rounds);

        // ---- Q^T operands arrive raw; multiply by scale*log2(e) and round to bf16 again
#pragma unroll
        for (int qb = 0; qb < QB; ++qb)
#pragma unroll
            for (int kk = 0; kk < D / 32; ++kk) {
                Pack16 t;
                t.v = w.qreg[qb][kk];
                const uint32_t u[4] = {t.u.x, t.u.y, t.u.z, t.u.w};
#pragma unroll
                for (int e = 0; e < 4; ++e)   // a bf16 is the upper half of the binary32 with the same value
                    t.p[e] = to_bf16x2(__uint_as_float(u[e] << 16) * a.scale_log2e,
                                       __uint_as_float(u[e] & 0xffff0000u) * a.scale_log2e);
                w.qreg[qb][kk] = t.v;
            }
        // the Q^T operands now live in AGPRs for the whole segment (left to itself the register
        // allocator may keep them elsewhere and copy each into one shared AGPR quad right before
        // its product, overwriting the quad the product issued just before is still reading)
#pragma unroll
        for (int qb = 0; qb < QB; ++qb)
#pragma unroll
            for (int kk = 0; kk < D / 32; ++kk) asm volatile("" : "+a"(w.qreg[qb][kk]));

        // ---- the segment's rounds.  Run first without the running-maximum check (CHECK = false):
        // the maximum stays what the first round made it, a probability is exp2 of whatever the
        // score is above that, and as long as nothing overflows binary32 / bf16 (2^127) the result
        // is the same sum of the same terms, only scaled by another power of two on both sides of
        // the final division.  If a row sum or an accumulator does come out non-finite -- some
        // score exceeded the first round's maximum by about 2^7 in log2 units -- or a row sum as good as 0, the workgroup
        // runs the segment again with the check (CHECK = true), which raises the maximum as it goes.
        auto run_segment = [&](auto checked_c) {
        constexpr bool CHECK = decltype(checked_c)::value;
#pragma unroll
        for (int mb = 0; mb < G; ++mb)
#pragma unroll
            for (int qb = 0; qb < QB; ++qb) w.acc[mb][qb] = f32x4{0.0f, 0.0f, 0.0f, 0.0f};
#pragma unroll
        for (int qb = 0; qb < QB; ++qb) w.l_acc[qb] = f32x4{0.0f, 0.0f, 0.0f, 0.0f};
        settle_acc<D, QB>(w.acc, w.l_acc, true);

        // ---- LDS operand addresses in stage 0 (recomputed from an opaque copy of the lane
        // index: kept as loop invariants they would be held in registers through the pipeline)
        w.tile_off = 0;
        w.k_off = 0;
        w.v_off = 0;
        w.issue_off = (kStages - 2) * T::kStageBytes;    // as start_tiles left it
        w.issue_t = t_begin + kStages - 2;
        {
            const int lane = opaque(lane_id), col = lane % 16, quad = lane / 16;
            // K operand: the row of key 8 (col / 4) + col % 4 (block 1: 4 keys later), so that elements
            // 4 b + i of a lane are the keys 8 quad .. 8 quad + 7 of the round
            const int krow = 8 * (col / 4) + col % 4;
#pragma unroll
            for (int kk = 0; kk < D / 32; ++kk)
                w.k_addr[kk] = lds0 + krow * T::kRowBytes + 16 * ((4 * kk + quad) ^ T::swz_k(krow));
            const int vrow = 8 * quad + col / 4;
#pragma unroll
            for (int mb = 0; mb < G; ++mb)
                w.v_addr[mb] = lds0 + T::kTileBytes + vrow * T::kRowBytes + 8 * (col % 2) + 16 * ((2 * mb + (col % 4) / 2) ^ T::swz_v(vrow));
        }

        // ---- the segment's first round fixes the initial maximum
        wait_tile_loads<0>();
        __syncthreads();
        f32x4 s_a[2][QB], s_b[2][QB];
        bf16x8 p_a[QB], p_b[QB];
        {
            f32x4 zero4 = {0.0f, 0.0f, 0.0f, 0.0f};
            asm volatile("s_nop 1" : "+v"(zero4));       // two wait states before a product may read it
#pragma unroll
            for (int g = 0; g < G; ++g) w.opreg[g] = load_k_operand<D, 0, 0>(w.k_addr, g);
#pragma unroll
            for (int g = 0; g < G; ++g)
#pragma unroll
                for (int qb = 0; qb < QB; ++qb) {
                    if (g < 2) mfma_score_init(s_a[g % 2][qb], w.opreg[g], w.qreg[qb][0], zero4);
                    else mfma_score(s_a[g % 2][qb], w.opreg[g], w.qreg[qb][g / 2]);
                }
#pragma unroll
            for (int g = 0; g < G; ++g) w.opreg[g] = load_k_operand<D, 1, 0>(w.k_addr, g);
            settle_scores(s_a, true);
        }
        if ((i_begin + 1) * 32 > c.key_end) mask_scores(i_begin, quad, c.key_end, s_a);
#pragma unroll
        for (int qb = 0; qb < QB; ++qb) {
            float tmax = s_a[0][qb][0];
#pragma unroll
            for (int e = 1; e < 8; ++e) tmax = fmaxf(tmax, s_a[e / 4][qb][e % 4]);
            tmax = quad_max(tmax);
            // a round of nothing but -inf: scores are taken as they are, see no_maximum
            const float neg = tmax == -INFINITY ? __uint_as_float(kNoMaximum) : 0.0f - tmax;
#pragma unroll
            for (int e = 0; e < 4; ++e) {
                w.neg_m[qb][e] = neg;
                s_a[0][qb][e] += neg;
                s_a[1][qb][e] += neg;
            }
            s_b[0][qb] = s_a[0][qb];
            s_b[1][qb] = s_a[1][qb];
            Pack16 z;
            z.u = make_uint4(0, 0, 0, 0);
            p_b[qb] = z.v;                  // probabilities of the round before the first: none
            asm volatile("" : "+v"(p_b[qb]));            // in registers from here on, not formed in front of their product
        }

        // ---- the pipeline, two steps at a time; step i_end only flushes the PV product of the last round
        int i = i_begin;
        auto whole_tiles = [&](int end) {                // tiles while rounds i+1 and i+2 are whole
            for (; (i + 3) * 32 <= c.key_end && i < end; i += 2) {
                pipeline_step<D, QB, 0, false, CHECK>(lds0, c, i, i == i_begin, w, s_a, s_b, p_b, p_a);
                pipeline_step<D, QB, 1, false, CHECK>(lds0, c, i + 1, false, w, s_b, s_a, p_a, p_b);
            }
        };
        if (!CHECK && (i + 11) * 32 <= c.key_end) {
            // four tiles at a time, each with its stage known at compile time: 318, 260, 202 instructions a tile (QB = 4, 3, 2)
            // instead of 366, 309, 250 at head_dim 128, 221, 176, 134 instead of 258, 216, 174 at 64.  The first tile comes
            // before them (its V fetches stay in stage 0), so they start in stage 1.
            whole_tiles(i_begin + 2);
#pragma unroll
            for (int kk = 0; kk < D / 32; ++kk) w.k_addr[kk] -= T::kStageBytes;
            for (; (i + 9) * 32 <= c.key_end; i += 8) {
                static_for<1, kStages + 1>([&](auto tc) {
                    constexpr int STAGE = decltype(tc)::value % kStages, step = 2 * (decltype(tc)::value - 1);
                    pipeline_step<D, QB, 0, false, CHECK, STAGE>(lds0, c, i + step, false, w, s_a, s_b, p_b, p_a);
                    pipeline_step<D, QB, 1, false, CHECK, STAGE>(lds0, c, i + step + 1, false, w, s_b, s_a, p_a, p_b);
                });
            }
#pragma unroll
            for (int kk = 0; kk < D / 32; ++kk) w.k_addr[kk] += T::kStageBytes;
            w.issue_off = 3 * T::kStageBytes;            // as the first tile left it
        }
        whole_tiles(i_end);
        for (; i <= i_end; i += 2) {
            pipeline_step<D, QB, 0, true, CHECK>(lds0, c, i, i == i_begin, w, s_a, s_b, p_b, p_a);
            if (i < i_end) pipeline_step<D, QB, 1, true, CHECK>(lds0, c, i + 1, false, w, s_b, s_a, p_a, p_b);
        }
        };   // run_segment

        run_segment(std::false_type{});
        {
            // anything in this lane's row sums or accumulators that is not finite, or within 2^7 of
            // not being so (partial rows are stored as bf16)?  As integers, the largest positive and the largest negative
            // magnitude (an infinity and any NaN lie above every number): half an instruction each per register.
            // And a row sum far below 1, which the key of the maximum alone adds: no score of the first round was above -inf, and
            // those that followed lie too far below 0, what they were taken relative to.
            settle_acc<D, QB>(w.acc, w.l_acc, false);
            constexpr uint32_t kTooLarge = (127 + 121) << 23;          // 2^121
            int32_t pos = 0;
            uint32_t neg = 0;
            int32_t smallest = kTooLarge;
#pragma unroll
            for (int qb = 0; qb < QB; ++qb) smallest = min(smallest, int32_t(__float_as_uint(w.l_acc[qb][0])));
#pragma unroll
            for (int qb = 0; qb < QB; ++qb)
#pragma unroll
                for (int mb = 0; mb <= G; ++mb) {          // (of the row sums all four elements, which are the same)
                    const f32x4 &x = mb < G ? w.acc[mb][qb] : w.l_acc[qb];
#pragma unroll
                    for (int r = 0; r < 4; r += 2) {
                        const uint32_t y0 = __float_as_uint(x[r]), y1 = __float_as_uint(x[r + 1]);
                        pos = max(max(int32_t(y0), int32_t(y1)), pos);
                        neg = max(max(y0, y1), neg);
                    }
                }
            constexpr int32_t kTooSmall = (127 - 60) << 23;            // 2^-60
            const bool out_of_range = pos >= int32_t(kTooLarge) || neg >= (0x80000000u | kTooLarge) || smallest < kTooSmall;
            // the barrier also makes sure that every wave has left the segment's tiles
            if (__syncthreads_or(out_of_range)) {
                start_tiles<D>(lds0, a, seg, c, n, stride_tok);
                run_segment(std::true_type{});
            }
        }

        // ---- the next segment's first tiles set out before this segment's results are
        // stored, so that their latency hides behind the stores
        const Segment nxt = next();
        if (nxt.valid || after.valid) {
            __syncthreads();        // every wave has left this segment's tiles before their stages are refilled
            start_tiles<D>(lds0, a, nxt.valid ? nxt : after, c, n, stride_tok);
        }
        if (nxt.valid) {
            load_q<D, QB>(a, nxt, w, n, stride_tok, wave, opaque(lane_id) % 16, opaque(lane_id) / 16);
        }

        // ---- results of this segment: final rows, or (a unit shared with other workgroups)
        // running maximum, row sum and unnormalised rows into this workgroup's slot
        settle_acc<D, QB>(w.acc, w.l_acc, false);
        const int lane = opaque(lane_id), col = lane % 16, quad = lane / 16;
        const bool whole = QB < kMostQB || (t_begin == 0 && uint32_t(t_stop) == tpu);      // smaller units are not shared
#pragma unroll
        for (int qb = 0; qb < QB; ++qb) {
            const float l_tot = w.l_acc[qb][0];
            const int row0 = wave * (16 * QB) + qb * 16;
            if (whole) {
                const int q0 = seg.row0 + row0;
                store_rows<D, QB>(out_lds, w.acc, qb, 1.0f / l_tot, a.o + head_off + int64_t(q0) * stride_tok, stride_tok, n - q0, lane);
            } else {
                float *slot = a.ws + (size_t(2) * sharer + (first_segment ? 0 : 1)) * slot_floats<D>();
                if (quad == 0) {
                    slot[row0 + col] = l_tot == 0.0f ? -INFINITY : -w.neg_m[qb][0];        // 0: every key of this part at -inf
                    slot[kBM + row0 + col] = l_tot;
                }
                store_rows<D, QB>(out_lds, w.acc, qb, 1.0f, reinterpret_cast<__bf16 *>(slot + 2 * kBM) + row0 * D, D, 16, lane);
            }
        }
        first_segment = false;
        if (!nxt.valid) break;
        seg = nxt;
    }
}

template <int D, int QB, int TAIL>
__global__ __launch_bounds__(kWaves * 64) void attention_kernel(const AttnParams a) {
    using T = Tile<D>;
    using L = Lane<D>;
    extern __shared__ __attribute__((aligned(1024))) unsigned char smem[];
    const uint32_t lds0 = uint32_t(uintptr_t(LP_LDS_PTR(unsigned char, smem)));

    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x / 64);
    const int lane = threadIdx.x % 64;
    const int64_t stride_tok = a.stride_tok;

    // ---- lane constants of the tile traffic
    L c;
    c.quad = lane / 16;
    c.tile_bytes = uint32_t(kBN * stride_tok * 2);
#pragma unroll
    for (int i = 0; i < L::kLd; ++i) {
        const int instr = wave + i * kWaves;
        const int row = instr * T::kRowsPerInstr + lane / T::kGran;
        const int gran = lane % T::kGran;          // physical granule this lane fills
        c.ld_dst[i] = instr * 1024;
        c.ld_base[i] = __builtin_amdgcn_readfirstlane(lds0 + instr * 1024);
        c.k_voff[i] = uint32_t(row * stride_tok * 2) + 16 * (gran ^ T::swz_k(row));
        c.v_voff[i] = uint32_t(row * stride_tok * 2) + 16 * (gran ^ T::swz_v(row));
    }

    // ---- this workgroup's range of the shared (unit, tile) space, then its whole units, then its unit of the last round
    const uint32_t lp = logical_workgroup(blockIdx.x, gridDim.x);
    const uint32_t sharer = range_start(lp, a.shared_wgs, gridDim.x);
    const bool sharing = range_start(lp + 1, a.shared_wgs, gridDim.x) > sharer;
    const uint32_t tpu = uint32_t(a.tiles_per_unit);
    Walk walk;
    walk.it = sharing ? real_tile(range_start(sharer, a.shared_work, a.shared_wgs), a.unit_cost, tpu) : 0u;
    walk.it_end = sharing ? real_tile(range_start(sharer + 1, a.shared_work, a.shared_wgs), a.unit_cost, tpu) : 0u;
    walk.whole_round = 0;
    Segment last;
    last.valid = false;
    if constexpr (TAIL > 0) last = tail_segment<TAIL>(a, tpu, lp, gridDim.x);

    Segment seg = next_segment<QB>(walk, a, tpu, lp, gridDim.x);
    if (!seg.valid) return;
    start_tiles<D>(lds0, a, seg, c, a.n, stride_tok);
    run_units<D, QB>(lds0, a, c, wave, seg, last, sharer, [&] { return next_segment<QB>(walk, a, tpu, lp, gridDim.x); });
    if constexpr (TAIL > 0) {
        Segment none;
        none.valid = false;
        if (last.valid) run_units<D, TAIL>(lds0, a, c, wave, last, none, sharer, [&] { return none; });
    }
}

// Merges the partial results of every unit that more than one workgroup worked on:
//   m = max_s m_s,  l = sum_s l_s 2^(m_s - m),  O = sum_s O_s 2^(m_s - m) / l.
// grid = units * kBM / 32: a workgroup takes 32 query rows of one unit, a thread one row
// and 16 consecutive d.  The units are dealt to the XCDs as attention_kernel deals its ranges, so
// that most parts are read from the L2 they were written to; a unit has two parts more often than not, and
// both are fetched before either is used.
template <int D>
__global__ __launch_bounds__(32 * (D / 16)) void combine_kernel(const AttnParams a, uint32_t n_wg) {
    constexpr int kChunks = D / 16, kPieces = kBM / 32;
    const uint32_t piece = logical_workgroup(blockIdx.x, gridDim.x), unit = piece / kPieces;
    const uint32_t W = a.shared_work, tpu = uint32_t(a.tiles_per_unit);
    // the unit's real tiles sit at [x_lo, x_hi) of the shared space, after its imaginary ones
    const uint32_t x_hi = (unit + 1) * a.unit_cost, x_lo = x_hi - tpu;
    // workgroup holding position x: the largest p with range_start(p) <= x
    const uint32_t pf = uint32_t((uint64_t(x_lo + 1) * n_wg - 1) / W);
    const uint32_t pl = uint32_t((uint64_t(x_hi) * n_wg - 1) / W);
    if (pf == pl) return;                                      // computed whole by one workgroup
    const int head = int(unit) / a.n_qtiles, qtile = int(unit) % a.n_qtiles;
    const int row = int(piece % kPieces) * 32 + int(threadIdx.x) / kChunks, ch = int(threadIdx.x) % kChunks;
    const int qi = qtile * kBM + row;
    if (qi >= a.n) return;
    // a workgroup's first segment lies in slot 0, a later (its last) one in slot 1
    const bool pf_starts_here = range_start(pf, W, n_wg) >= unit * a.unit_cost;
    const float *slot0 = a.ws + (size_t(2) * pf + (pf_starts_here ? 0 : 1)) * slot_floats<D>();
    const size_t slot_step = size_t(2) * slot_floats<D>();    // every later workgroup starts inside the unit: slot 0
    const float *first_later = a.ws + size_t(2) * (pf + 1) * slot_floats<D>();
    struct Part {
        float m, l;
        uint4 x[2];
    };
    auto fetch = [&](const float *slot) {
        const uint4 *src = reinterpret_cast<const uint4 *>(reinterpret_cast<const __bf16 *>(slot + 2 * kBM) + row * D + ch * 16);
        return Part{slot[row], slot[kBM + row], {src[0], src[1]}};
    };
    const Part first = fetch(slot0), second = fetch(first_later);
    float m = fmaxf(first.m, second.m);
    for (uint32_t p = pf + 2; p <= pl; ++p) m = fmaxf(m, first_later[(p - pf - 1) * slot_step + row]);
    float l = 0.0f, acc[16];
#pragma unroll
    for (int e = 0; e < 16; ++e) acc[e] = 0.0f;
    auto add = [&](const Part &part) {
        const float f = __builtin_amdgcn_exp2f(part.m - m);
        l += part.l * f;
#pragma unroll
        for (int e = 0; e < 2; ++e) {
            const uint32_t wds[4] = {part.x[e].x, part.x[e].y, part.x[e].z, part.x[e].w};
#pragma unroll
            for (int j = 0; j < 4; ++j) {     // a bf16 is the upper half of the binary32 of the same value
                acc[8 * e + 2 * j + 0] += __uint_as_float(wds[j] << 16) * f;
                acc[8 * e + 2 * j + 1] += __uint_as_float(wds[j] & 0xffff0000u) * f;
            }
        }
    };
    add(first);
    add(second);
    for (uint32_t p = pf + 2; p <= pl; ++p) add(fetch(first_later + (p - pf - 1) * slot_step));
    const float inv = 1.0f / l;
    union { uint4 u[2]; bf16x2 p[8]; } ow;
#pragma unroll
    for (int e = 0; e < 8; ++e) ow.p[e] = to_bf16x2(acc[2 * e] * inv, acc[2 * e + 1] * inv);
    uint4 *dst = reinterpret_cast<uint4 *>(a.o + head_offset(a, head) + int64_t(qi) * a.stride_tok + ch * 16);
    dst[0] = ow.u[0];
    dst[1] = ow.u[1];
}

template <int D, int QB, int TAIL>
int launch_units(const AttnParams &a, uint32_t wgs, int dev, hipStream_t stream) {
    static std::atomic<uint64_t> attr_set{0};
    const void *kern = reinterpret_cast<const void *>(&attention_kernel<D, QB, TAIL>);
    const int rc = allow_lds(kern, Tile<D>::kBytes, dev, attr_set);
    if (rc != LP_OK) return rc;
    return lp::launch_kernel(kern, dim3(wgs), dim3(kWaves * 64), Tile<D>::kBytes, stream, a);
}

template <int D>
int launch_tiles(const AttnParams &a, int qb, int tail, uint32_t wgs, int dev, hipStream_t stream) {
    const int rc = tail != 0 ? launch_units<D, kMostQB, 3>(a, wgs, dev, stream)
                   : qb == 3 ? launch_units<D, 3, 0>(a, wgs, dev, stream)
                   : qb == 2 ? launch_units<D, 2, 0>(a, wgs, dev, stream)
                             : launch_units<D, kMostQB, 0>(a, wgs, dev, stream);
    if (rc != LP_OK || a.ws == nullptr) return rc;
    return lp::launch_kernel(reinterpret_cast<const void *>(&combine_kernel<D>), dim3(uint32_t(a.shared_units) * (kBM / 32)),
                             dim3(32 * (D / 16)), 0, stream, a, a.shared_wgs);
}

}  // namespace
