// lp_attention for short sequences and few heads.
//
// What bounds such a call is not the matrix pipeline but a chain: launch, first bytes of Q and K from
// memory, one round of products after the other, results.  attention_kernel (lp_attention_kernel.h) gives
// a workgroup 256 query rows, so 200 tokens of 4 heads are four workgroups that walk all keys one
// round after the other.  Here a workgroup takes 32 query rows of a head and its four wavefronts
// share the KEYS: wavefront w takes the rounds w, w + 4, ... of 32 keys, each with its own
// running maximum, row sum and output accumulators, and the four partial results are merged
// through LDS at the end (m = max m_w, l = sum l_w 2^(m_w - m), O = sum O_w 2^(m_w - m) / l).  The
// chain is a quarter as long and there are eight times as many workgroups; a wavefront's K and V
// pass through LDS of its own, so the loop has no barrier.  The price is that a K/V row is fetched for
// 32 query rows instead of 256, which is why long calls stay with attention_kernel: see
// attention_short_us for where the line lies.
//
// Products, operand layouts and the order of keys in a round are those of attention_kernel (16x16x32
// MFMA, S^T = K Q^T and O^T += V^T P^T, K rows permuted so that a lane's eight probabilities are eight
// consecutive keys, V read transposed); the products are builtins here: with 32 rows a wavefront
// needs 190 registers at head_dim 128 (126 at 64) and two (four) workgroups share a compute unit.
//
// Measured (us, attention_kernel in its best tiles / this): 200 tokens, 4 heads of 64: 7.8 / 4.8; 333, 3 of 128: 11.5 /
// 7.1; 1000, 12 of 128: 18.2 / 15.4; 2000, 12 of 128: 29 / 41; 3000, 12 of 128: 53 / 85.  One stage per
// wavefront, whose K half is refilled once the scores are formed and whose V half after the PV
// product, and two workgroups per compute unit are faster than two whole stages and one workgroup
// (1000 tokens, 12 heads of 128: 16.4 / 23.1); eight wavefronts per workgroup 20.9; 64 rows 22.8.
//
// A compute unit takes in about 100 GB/s through the global -> LDS path here (32 KB per 128 keys and workgroup in 0.33 us at
// head_dim 64), and its SIMDs issue for several wavefronts: what a round costs besides its products and exponentials counts.  The row
// sums as products, the score products started at -m without a look at it, and one write of M0 for four loads: 1000 tokens, 12
// heads of 64 10.0 -> 9.65 us, 600 x 24 of 64 8.05 -> 7.85, 333 x 3 of 128 7.15 -> 7.0, 200 x 4 of 64 4.7 as before.
// Not kept: a merge of one barrier in which each wavefront finishes a quarter of the columns (200 x 4 of 64 4.95), 64 rows at
// head_dim 64 and 48 at 128 with two workgroups to a compute unit (1628 x 25 of 64 28.7 / 30.9; 3000 x 12 of 128 84.8 / 68,
// 59 in 256-row tiles).
#include <hip/hip_runtime.h>

#include <atomic>

#include "lp_device.h"

namespace {

using namespace lp;

constexpr int kWaves = 4;                     // wavefronts of a workgroup; they share the keys
constexpr int kQB = 2;                        // 16-row query blocks of a workgroup
constexpr int kRows = 16 * kQB;
constexpr float kRescaleThreshold = 8.0f;     // log2 units the running maximum may lag behind

struct ShortParams {
    const __bf16 *q, *k, *v;
    __bf16 *o;
    int64_t stride_tok, stride_head, stride_batch;
    int heads;                 // heads per batch item
    int n, n_blocks;           // tokens, and blocks of kRows of them
    float scale_log2e;
};

template <int D>
struct Round : TileSwizzle<D> {
    static constexpr int kRowBytes = D * 2, kGran = kRowBytes / 16;    // a K or V row and its 16-byte granules
    static constexpr int kTileBytes = 32 * kRowBytes;                  // K or V of a round
    static constexpr int kRingBytes = kWaves * 2 * kTileBytes;         // K then V, for every wavefront
    static constexpr int kPartBytes = kRows * D * 4;                   // partial rows of a wavefront in the merge
    static constexpr int kMergeBytes = kWaves * (kPartBytes + kRows * 8);
    static constexpr int kLds = kRingBytes > kMergeBytes ? kRingBytes : kMergeBytes;
    static constexpr int kRowsPerLoad = 1024 / kRowBytes, kLoads = 32 / kRowsPerLoad;   // wave-wide loads of a tile
};

// At most PENDING of this wavefront's loads are still in flight.
template <int PENDING>
__device__ __forceinline__ void wait_loads() {
    asm volatile("s_waitcnt vmcnt(%0)" ::"n"(PENDING) : "memory");
}

// Four wave-wide global -> LDS loads to consecutive KB of LDS behind one write of M0: an instruction's offset counts on both
// sides, so lane offset i has to lie 1024 i below the bytes it fetches.
__device__ __forceinline__ void load_to_lds_4x16(__amdgpu_buffer_rsrc_t rsrc, uint32_t lds_addr, uint32_t v0, uint32_t v1, uint32_t v2, uint32_t v3, uint32_t soff) {
    asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tbuffer_load_dwordx4 %1, %5, %6 offen lds\n\tbuffer_load_dwordx4 %2, %5, %6 offen offset:1024 lds\n\t"
                 "buffer_load_dwordx4 %3, %5, %6 offen offset:2048 lds\n\tbuffer_load_dwordx4 %4, %5, %6 offen offset:3072 lds"
                 :
                 : "s"(lds_addr), "v"(v0), "v"(v1), "v"(v2), "v"(v3), "s"(rsrc), "s"(soff)
                 : "memory", "m0");
}

// FAR: tokens so far apart that the 32 rows of a round reach past 2^32 bytes, so that a 32-bit offset would place some of the
// rows past the last inside the buffer (which has less than 2^31 bytes).  They all go where the first of them lies, behind it.  A kernel of its own: the clamp in every call cost one of 1248 tokens x 4 heads of 128 4 %.
template <int D, bool FAR>
__global__ __launch_bounds__(kWaves * 64, 2) void attention_short_kernel(const ShortParams a) {
    using T = Round<D>;
    constexpr int KS = D / 32, MB = D / 16;
    extern __shared__ __attribute__((aligned(1024))) unsigned char smem[];
    const uint32_t lds0 = uint32_t(uintptr_t(LP_LDS_PTR(unsigned char, smem)));
    const int tid = threadIdx.x;
    const int wave = __builtin_amdgcn_readfirstlane(tid / 64);
    const int lane = tid % 64, col = lane % 16, quad = lane / 16;
    const int n = a.n;

    const uint32_t unit = logical_workgroup(blockIdx.x, gridDim.x);        // the blocks of a head go to one XCD
    const int bh = int(unit) / a.n_blocks, q0 = (int(unit) - bh * a.n_blocks) * kRows;
    const int item = bh / a.heads;
    const int64_t head_off = int64_t(item) * a.stride_batch + int64_t(bh - item * a.heads) * a.stride_head;

    // K and V of this head as raw buffers ending with token n-1
    const int valid_bytes = int((int64_t(n - 1) * a.stride_tok + D) * 2);
    const __amdgpu_buffer_rsrc_t k_rsrc = __builtin_amdgcn_make_buffer_rsrc(const_cast<__bf16 *>(a.k + head_off), 0, valid_bytes, 0x00020000);
    const __amdgpu_buffer_rsrc_t v_rsrc = __builtin_amdgcn_make_buffer_rsrc(const_cast<__bf16 *>(a.v + head_off), 0, valid_bytes, 0x00020000);
    const uint32_t tok_bytes = uint32_t(a.stride_tok * 2);
    const uint32_t k_lds = lds0 + wave * 2 * T::kTileBytes, v_lds = k_lds + T::kTileBytes;
    uint32_t k_voff[T::kLoads], v_voff[T::kLoads];
#pragma unroll
    for (int i = 0; i < T::kLoads; ++i) {
        const int row = i * T::kRowsPerLoad + lane / T::kGran, g = lane % T::kGran;
        const uint32_t row_off = uint32_t(FAR ? min(row, n) : row) * tok_bytes - 1024 * (i % 4);     // not below 0: rows do not overlap
        k_voff[i] = row_off + 16 * (g ^ T::swz_k(row));
        v_voff[i] = row_off + 16 * (g ^ T::swz_v(row));
    }
    auto issue = [&](const __amdgpu_buffer_rsrc_t &rsrc, uint32_t lds, const uint32_t (&voff)[T::kLoads], int round) {
#pragma unroll
        for (int i = 0; i < T::kLoads; i += 4)
            load_to_lds_4x16(rsrc, __builtin_amdgcn_readfirstlane(lds + i * 1024), voff[i], voff[i + 1], voff[i + 2], voff[i + 3],
                             uint32_t(round) * 32 * tok_bytes);
    };
    const int n_rounds = (n + 31) / 32;
    int round = wave;
    if (round < n_rounds) {
        issue(k_rsrc, k_lds, k_voff, round);
        issue(v_rsrc, v_lds, v_voff, round);
    }

    // Q^T operands, multiplied by scale * log2(e) and rounded to bf16 again; rows past the end repeat
    // the last one and are not stored
    bf16x8 q[kQB][KS];
#pragma unroll
    for (int qb = 0; qb < kQB; ++qb) {
        const __bf16 *row = a.q + head_off + int64_t(min(q0 + qb * 16 + col, n - 1)) * a.stride_tok;
#pragma unroll
        for (int kk = 0; kk < KS; ++kk) {
            Pack16 t;
            t.u = *reinterpret_cast<const uint4 *>(row + kk * 32 + quad * 8);
            const uint32_t u[4] = {t.u.x, t.u.y, t.u.z, t.u.w};
#pragma unroll
            for (int e = 0; e < 4; ++e)       // a bf16 is the upper half of the binary32 with the same value
                t.p[e] = to_bf16x2(__uint_as_float(u[e] << 16) * a.scale_log2e, __uint_as_float(u[e] & 0xffff0000u) * a.scale_log2e);
            q[qb][kk] = t.v;
        }
    }

    // LDS addresses of the K operands (rows 8 (r / 4) + r % 4, block 1 four rows later) and V^T operands
    const int krow = 8 * (col / 4) + col % 4, vrow = 8 * quad + col / 4;
    uint32_t k_addr[KS], v_addr[MB];
#pragma unroll
    for (int kk = 0; kk < KS; ++kk) k_addr[kk] = k_lds + krow * T::kRowBytes + 16 * ((4 * kk + quad) ^ T::swz_k(krow));
#pragma unroll
    for (int mb = 0; mb < MB; ++mb)
        v_addr[mb] = v_lds + vrow * T::kRowBytes + 8 * (col % 2) + 16 * ((2 * mb + (col % 4) / 2) ^ T::swz_v(vrow));

    // neg_m = -m in every element (m: running maximum, log2 units, common to the four lanes of a query), what the score products
    // start at; 0 as long as no score was above -inf, which limit = -inf says.  l: row sums, the same in every element.
    f32x4 acc[MB][kQB], l[kQB], neg_m[kQB];
    float limit[kQB];                           // a score relative to m above this raises m
    Pack16 ones;
    ones.u = make_uint4(0x3f803f80, 0x3f803f80, 0x3f803f80, 0x3f803f80);
#pragma unroll
    for (int qb = 0; qb < kQB; ++qb) {
        limit[qb] = -INFINITY;
        l[qb] = neg_m[qb] = f32x4{0.0f, 0.0f, 0.0f, 0.0f};
#pragma unroll
        for (int mb = 0; mb < MB; ++mb) acc[mb][qb] = f32x4{0.0f, 0.0f, 0.0f, 0.0f};
    }

    for (; round < n_rounds; round += kWaves) {
        const bool more = round + kWaves < n_rounds;
        wait_loads<T::kLoads>();                // K of this round; behind it only V
        f32x4 s[2][kQB];
#pragma unroll
        for (int kk = 0; kk < KS; ++kk)
#pragma unroll
            for (int b = 0; b < 2; ++b) {
                const bf16x8 ka = lds_load<bf16x8>(k_addr[kk] + 4 * b * T::kRowBytes);
#pragma unroll
                for (int qb = 0; qb < kQB; ++qb)
                    s[b][qb] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(ka, q[qb][kk], kk == 0 ? neg_m[qb] : s[b][qb], 0, 0, 0);
            }
        if (more) {
            asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");     // every K operand has left LDS
            issue(k_rsrc, k_lds, k_voff, round + kWaves);
        }
        if (__builtin_expect((round + 1) * 32 > n, 0)) {           // keys past the end: score -inf
            const int kbase = round * 32 + 8 * quad;
#pragma unroll
            for (int e = 0; e < 8; ++e) {
                const bool past = kbase + e >= n;
#pragma unroll
                for (int qb = 0; qb < kQB; ++qb) s[e / 4][qb][e % 4] = past ? -INFINITY : s[e / 4][qb][e % 4];
            }
        }
        // the maximum is set by the first round with a score above -inf, and raised when a score exceeds it
        // by more than the threshold
        float mx[kQB];
        bool raise = false;
#pragma unroll
        for (int qb = 0; qb < kQB; ++qb) {
            mx[qb] = s[0][qb][0];
#pragma unroll
            for (int e = 1; e < 8; ++e) mx[qb] = fmaxf(mx[qb], s[e / 4][qb][e % 4]);
            raise = raise | (mx[qb] > limit[qb]);
        }
        if (__builtin_expect(__builtin_amdgcn_ballot_w64(raise) != 0, 0)) {
#pragma unroll
            for (int qb = 0; qb < kQB; ++qb) {
                const bool fresh = limit[qb] == -INFINITY;
                const float top = quad_max(mx[qb]);
                const float d = fresh ? (top == -INFINITY ? 0.0f : top) : fmaxf(top, 0.0f);
                const float f = fresh ? 0.0f : __builtin_amdgcn_exp2f(-d);
                limit[qb] = fresh && top == -INFINITY ? -INFINITY : kRescaleThreshold;
                neg_m[qb] -= d;
                l[qb] *= f;
                s[0][qb] -= d;
                s[1][qb] -= d;
#pragma unroll
                for (int mb = 0; mb < MB; ++mb) acc[mb][qb] *= f;
            }
        }
        bf16x8 p[kQB];
#pragma unroll
        for (int qb = 0; qb < kQB; ++qb) {
            Pack16 t;
#pragma unroll
            for (int e = 0; e < 4; ++e)
                t.p[e] = to_bf16x2(__builtin_amdgcn_exp2f(s[e / 2][qb][(2 * e) % 4]), __builtin_amdgcn_exp2f(s[e / 2][qb][(2 * e) % 4 + 1]));
            p[qb] = t.v;
            // the row sum adds the rounded probabilities, as one product (a v_dot2 per pair holds the matrix pipeline as long each)
            l[qb] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(ones.v, p[qb], l[qb], 0, 0, 0);
        }
        if (more) wait_loads<T::kLoads>();      // V of this round; behind it only the next round's K
        else wait_loads<0>();
#pragma unroll
        for (int mb = 0; mb < MB; ++mb) {
            Pack16 t;
#pragma unroll
            for (int hf = 0; hf < 2; ++hf)
                t.h[hf] = __builtin_amdgcn_ds_read_tr16_b64_v4bf16(LP_LDS_PTR(bf16x4, uintptr_t(v_addr[mb] + 4 * hf * T::kRowBytes)));
#pragma unroll
            for (int qb = 0; qb < kQB; ++qb) acc[mb][qb] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(t.v, p[qb], acc[mb][qb], 0, 0, 0);
        }
        if (more) {
            asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");     // every V operand has left LDS
            issue(v_rsrc, v_lds, v_voff, round + kWaves);
        }
    }

    // ---- merge: maxima and row sums through LDS, then the rows, scaled to the common maximum
    __syncthreads();                            // every wavefront has left its ring (its loads have all landed)
    const uint32_t ml_lds = lds0 + kWaves * T::kPartBytes;
    float m[kQB];
#pragma unroll
    for (int qb = 0; qb < kQB; ++qb) {
        m[qb] = limit[qb] == -INFINITY ? -INFINITY : -neg_m[qb][0];
        if (quad == 0) lds_store(ml_lds + 8 * (wave * kRows + qb * 16 + col), f32x2{m[qb], l[qb][0]});
    }
    __syncthreads();
#pragma unroll
    for (int qb = 0; qb < kQB; ++qb) {
        const int row = qb * 16 + col;
        f32x2 part[kWaves];
        float top = -INFINITY, sum = 0.0f;      // wavefront 0 always has a round, so top is finite
#pragma unroll
        for (int w = 0; w < kWaves; ++w) {
            part[w] = lds_load<f32x2>(ml_lds + 8 * (w * kRows + row));
            top = fmaxf(top, part[w].x);
        }
#pragma unroll
        for (int w = 0; w < kWaves; ++w) sum += part[w].y * __builtin_amdgcn_exp2f(part[w].x - top);
        const float f = __builtin_amdgcn_exp2f(m[qb] - top) / sum;
#pragma unroll
        for (int mb = 0; mb < MB; ++mb)
            lds_store(lds0 + wave * T::kPartBytes + row * D * 4 + 16 * ((4 * mb + quad) ^ col), acc[mb][qb] * f);
    }
    __syncthreads();
#pragma unroll
    for (int j = 0; j < kRows * D / 8 / (64 * kWaves); ++j) {       // eight consecutive d of a row per thread
        const int c = tid + 64 * kWaves * j, row = c / (D / 8), ch = c % (D / 8);
        f32x4 lo = {0.0f, 0.0f, 0.0f, 0.0f}, hi = {0.0f, 0.0f, 0.0f, 0.0f};
#pragma unroll
        for (int w = 0; w < kWaves; ++w) {
            const uint32_t part = lds0 + w * T::kPartBytes + row * D * 4;
            lo += lds_load<f32x4>(part + 16 * ((2 * ch) ^ (row % 16)));
            hi += lds_load<f32x4>(part + 16 * ((2 * ch + 1) ^ (row % 16)));
        }
        Pack16 t;
        t.p[0] = to_bf16x2(lo[0], lo[1]);
        t.p[1] = to_bf16x2(lo[2], lo[3]);
        t.p[2] = to_bf16x2(hi[0], hi[1]);
        t.p[3] = to_bf16x2(hi[2], hi[3]);
        if (q0 + row < n) *reinterpret_cast<uint4 *>(a.o + head_off + int64_t(q0 + row) * a.stride_tok + 8 * ch) = t.u;
    }
}

template <int D, bool FAR>
int launch_short(ShortParams a, int64_t groups, hipStream_t stream) {
    static std::atomic<uint64_t> attr_set{0};
    const void *kern = reinterpret_cast<const void *>(&attention_short_kernel<D, FAR>);
    int dev = 0;
    device_compute_units(&dev);
    const int rc = allow_lds(kern, Round<D>::kLds, dev, attr_set);
    if (rc != LP_OK) return rc;
    return lp::launch_kernel(kern, dim3(uint32_t(groups)), dim3(kWaves * 64), Round<D>::kLds, stream, a);
}

int64_t short_groups(int64_t n, int64_t all_heads) { return all_heads * ((n + kRows - 1) / kRows); }

}  // namespace

namespace lp {

bool attention_short_launchable(int64_t n, int64_t all_heads) { return short_groups(n, all_heads) * (64 * kWaves) <= kMaxLaunchThreads; }

// us: launch and first fetch, then the workgroups of a compute unit, each a quarter of the rounds long.
// A compute unit holds several: two of them take 1.5 times as long as one.  Many heads bring q, k, v and o
// from and to memory faster than their few tokens need products: part of those transfers comes on top (192
// tokens x 2000 heads of 128: 176 us, 83 without it).  Off by 7 % (rms) at 1 .. 5000 tokens x 1 .. 5000 heads.
// Rows that lie split over one line more than they fill, with other heads' rows in between (padded or side by side at odd
// offsets), take a round of a full chip a third longer, as every K / V row is fetched once per 32 query rows: 1628 tokens x
// 25 heads of 64 45.2 us, 27.6 in whole lines; the 256-row tiles lose nothing (26.6 / 25.8).  A head of few rounds stays in the
// caches close by and loses little at head_dim 64: 153 x 411 14.6, 14.4 in whole lines.
float attention_short_us(int64_t n, int64_t all_heads, int head_dim, int cus, bool split) {
    const int64_t groups = short_groups(n, all_heads), rounds = (n + 127) / 128;
    const int64_t per_cu = (groups + cus - 1) / cus;
    if (per_cu <= 1) return head_dim == 128 ? 4.73f + 0.75f * float(rounds) : 4.274f + 0.437f * float(rounds);
    const float bytes_us = attention_bytes_us(n, all_heads, head_dim);
    if (head_dim == 64) {
        const float more = split && rounds > 2 ? 0.147f * (float(rounds) - 2.5f) : 0.0f;
        return 4.026f + float(per_cu) * (0.26f + 0.328f * float(rounds) + more) + 0.404f * bytes_us;
    }
    return 3.76f + 0.516f * float(per_cu) + float((per_cu + 1) / 2) * (split ? 1.386f : 1.066f) * float(rounds) + 0.782f * bytes_us;
}

int attention_short(const AttentionCall &c, hipStream_t stream) {
    ShortParams a;
    a.q = static_cast<const __bf16 *>(c.q);
    a.k = static_cast<const __bf16 *>(c.k);
    a.v = static_cast<const __bf16 *>(c.v);
    a.o = static_cast<__bf16 *>(c.o);
    a.stride_tok = c.stride_tok;
    a.stride_head = c.stride_head;
    a.stride_batch = c.stride_batch;
    a.heads = c.heads;
    a.n = c.n;
    a.n_blocks = (c.n + kRows - 1) / kRows;
    a.scale_log2e = c.scale_log2e;
    const int64_t groups = short_groups(c.n, c.all_heads);
    const bool far = c.stride_tok * 2 * 32 >= int64_t(1) << 32;
    if (c.head_dim == 128) return far ? launch_short<128, true>(a, groups, stream) : launch_short<128, false>(a, groups, stream);
    return far ? launch_short<64, true>(a, groups, stream) : launch_short<64, false>(a, groups, stream);
}

}  // namespace lp
