// lp_attention: which kernel a call runs and how its work is dealt out, the argument checks and the entry points.  The
// kernels: lp_attention_kernel.h, and lp_attention_short.hip for short calls.
#include <hip/hip_runtime.h>

#include <atomic>

#include "lp_attention.h"

namespace {

using namespace lp;

template <int D>
int64_t workspace_bytes_for(int cus) { return int64_t(2) * cus * slot_floats<D>() * int64_t(sizeof(float)); }

// ---- which way a call goes.  Times in us on 256 compute units, fitted to 4262 calls (1 .. 16000 tokens x 1 .. 5000
// heads, both head dims, rows in whole lines, split over lines and head-major), each timed on every way it can go: the short
// kernel; units of 256 rows whole or cut; units of 192 and of 128 rows; rounds of 256 with a last one of 192.  The choice is off
// the best way by 0.11 % on average (calls of 96 and more tokens and up to 80 heads), by more than 10 % in 9 calls, by 18 % at
// worst.  29 % of the calls take units of 192 or 128 rows, 15 % less time on average than the best of the other ways.

// What attention_kernel's units of 16 kWaves qb rows cost: launch, first tiles and Q, the first round, stores; from one unit to the
// next, in tile times; a tile while a part kBusy of the compute units works: one workgroup's own pace, slower
// as the power limit lowers the clock of a full chip.  A tile's time falls less than its rows: every operand fetched from LDS feeds
// one product per 16 rows of a wavefront, and at head_dim 128 and 32 rows the fetches take as long as the products.
// `split` comes on top of a tile where rows lie split over lines (rows_split): the fewer rows a unit has, the more often K and V are
// fetched, over more lines each time.  From 700 and 500 calls on every way in three layouts; the choice is off the best
// way by 0.18 % of their time (0.39 % without it and with a constant surcharge in the short kernel).
struct UnitCost {
    float once, change, split, tile[4];
};
constexpr float kBusy[4] = {0.5f, 0.8f, 0.94f, 1.0f};
constexpr UnitCost kUnit128[3] = {{8.017f, 4.443f, 0.03f, {0.571f, 0.645f, 0.707f, 0.759f}},      // qb 2, 3, 4
                                  {9.034f, 4.944f, 0.012f, {0.794f, 0.903f, 0.931f, 1.045f}},
                                  {11.446f, 3.748f, 0.0f, {1.088f, 1.117f, 1.293f, 1.330f}}};
constexpr UnitCost kUnit64[3] = {{6.289f, 5.242f, 0.01f, {0.380f, 0.414f, 0.419f, 0.475f}},
                                 {7.139f, 5.685f, 0.035f, {0.476f, 0.533f, 0.587f, 0.622f}},
                                 {8.726f, 4.981f, 0.0f, {0.729f, 0.749f, 0.776f, 0.796f}}};
const UnitCost &unit_cost(int head_dim, int qb) { return (head_dim == 128 ? kUnit128 : kUnit64)[qb - 2]; }

float tile_us(const UnitCost &c, float busy) {
    if (busy <= kBusy[0]) return c.tile[0];
    int i = 1;
    while (i < 3 && busy > kBusy[i]) ++i;
    return c.tile[i - 1] + (c.tile[i] - c.tile[i - 1]) * (busy - kBusy[i - 1]) / (kBusy[i] - kBusy[i - 1]);
}

// How attention_kernel's workgroups deal the units out.
struct Deal {
    int qb;              // 16-query blocks of a wavefront,
    int tail;            // and of those of the last round, if it is in smaller units (else 0)
    uint32_t wgs, rounds, shared, sharers;
    float us;
};

// Whole units to everybody for as many rounds as they fill, and one each of those left over.
Deal deal_whole(int head_dim, int qb, int64_t n, int all_heads, uint32_t cus, bool split) {
    const UnitCost &c = unit_cost(head_dim, qb);
    const uint32_t units = uint32_t((n + unit_rows(qb) - 1) / unit_rows(qb)) * uint32_t(all_heads), tpu = uint32_t((n + kBN - 1) / kBN);
    Deal d;
    d.qb = qb;
    d.tail = 0;
    d.wgs = units < cus ? units : cus;
    d.rounds = units / cus;
    d.shared = units - d.rounds * cus;
    d.sharers = d.shared;
    const float changes = float(d.rounds) - (d.rounds > 0 && d.shared == 0 ? 1.0f : 0.0f);
    // what of the transfers the products do not cover
    const float transfers = (head_dim == 128 ? 0.318f : 0.306f) * lp::attention_bytes_us(n, all_heads, head_dim);
    d.us = c.once + transfers + (float(d.rounds) * float(tpu) + changes * c.change) * tile_us(c, 1.0f);
    if (d.shared > 0) d.us += float(tpu) * tile_us(c, float(d.shared) / float(cus));
    if (split) d.us += float(d.rounds + (d.shared > 0 ? 1 : 0)) * float(tpu) * c.split;
    return d;
}

// Units of 256 rows: those left over after whole rounds taken whole by as many workgroups (no scratch memory, no merge) or cut into
// even ranges for as many as get kMinTiles tiles each.  Measured, whole / cut: 3780 tokens x 12 heads of 128 (180 units on 256) 76 / 83,
// 4680 x 12 102 / 116, 13230 x 40 (8 rounds and 32 units) 2460 / 2250; of 64: 2999 x 16 40 / 44, 4639 x 7 60 / 51.
Deal deal_large(int head_dim, int64_t n, int all_heads, uint32_t cus, bool may_cut) {
    constexpr uint32_t kMinTiles = 8;
    static_assert(kBoundaryTiles < kMinTiles, "a range of kMinTiles positions must hold a real tile");
    const float merge = head_dim == 128 ? 6.023f : 5.574f;                // combine_kernel and the parts it reads
    const UnitCost &c = unit_cost(head_dim, kMostQB);
    const uint32_t tpu = uint32_t((n + kBN - 1) / kBN);
    Deal d = deal_whole(head_dim, kMostQB, n, all_heads, cus, false);    // 256-row units lose nothing by split rows
    if (!may_cut || d.shared == 0) return d;
    uint32_t sharers = uint32_t(uint64_t(d.shared) * tpu / kMinTiles);
    if (sharers > cus) sharers = cus;
    if (sharers <= d.shared) return d;                                    // cutting adds no parallelism
    const float share = float(d.shared) * float(tpu) / float(sharers);
    const float cut_us = d.us - float(tpu) * tile_us(c, float(d.shared) / float(cus)) + merge +
                         (share + float(kBoundaryTiles)) * tile_us(c, float(sharers) / float(cus));
    if (cut_us < d.us) {
        if (d.rounds == 0) d.wgs = sharers;
        d.sharers = sharers;
        d.us = cut_us;
    }
    return d;
}

// Smaller units where they fill the chip better than `large` does: 192 or 128 rows throughout (they also leave fewer rows past the
// end of a head), or 192 in a last round that takes one to a workgroup.  Measured, 256 rows (whole or cut) / 192 / 128: 3780 x 12 of
// 128 76 / 70 / 91, 1625 x 38 70 / 63 / 53, 2304 x 40 of 64 63 / 57 / 68, 861 x 201 69 / 55 / 62; 2 x 7410 x 12 of 128
// 466, 452 with a last round of 192.
Deal deal_finer(int head_dim, int64_t n, int all_heads, uint32_t cus, bool split, const Deal &large) {
    Deal best = large;
    for (int qb = kMostQB - 1; qb >= 2; --qb) {
        const Deal d = deal_whole(head_dim, qb, n, all_heads, cus, split);
        if (d.us < best.us) best = d;
    }
    Deal d = deal_whole(head_dim, kMostQB, n, all_heads, cus, false);
    if (d.rounds > 0 && d.shared > 0) {
        constexpr int64_t kRows = unit_rows(kMostQB), kTail = unit_rows(3);
        const int64_t tiles = (n + kRows - 1) / kRows, whole = int64_t(d.rounds) * cus, row = whole % tiles * kRows;
        const int64_t units = (n - row + kTail - 1) / kTail + (all_heads - whole / tiles - 1) * ((n + kTail - 1) / kTail);
        const float tpu = float((n + kBN - 1) / kBN);
        if (units <= int64_t(cus)) {
            const UnitCost &c = unit_cost(head_dim, 3);
            d.us += tpu * (tile_us(c, float(units) / float(cus)) - tile_us(unit_cost(head_dim, kMostQB), float(d.shared) / float(cus)));
            if (split) d.us += tpu * c.split;
            d.tail = 3;
            d.shared = d.sharers = uint32_t(units);
            if (d.us < best.us) best = d;
        }
    }
    return best;
}

// What runs: the short kernel, or units as `deal` says.
struct Route {
    bool short_kernel;
    bool cut;            // units of the last round are shared and merged
    Deal deal;
};

// The cheapest of the short kernel, where its grid is one that can be launched, and units of 256 rows, whole or cut, and of fewer.
Route pick_route(int head_dim, int64_t n, int all_heads, int cus, bool scratch, bool split) {
    Route r;
    r.deal = deal_finer(head_dim, n, all_heads, uint32_t(cus), split, deal_large(head_dim, n, all_heads, uint32_t(cus), scratch));
    // up to 32 tokens are the short kernel's whatever the prices say: they may lie so far apart that the 64 rows of a tile, most of
    // them past the end, reach past 2^32 bytes, which attention_kernel's offsets do not hold
    r.short_kernel = lp::attention_short_launchable(n, all_heads) && (n <= 32 || lp::attention_short_us(n, all_heads, head_dim, cus, split) < r.deal.us);
    r.cut = !r.short_kernel && r.deal.sharers != r.deal.shared;
    return r;
}

// Whether the rows of a head's K or V are split over 128-byte lines that they do not fill: neither whole lines of
// their own nor one directly behind the other.
bool rows_split(uint64_t k, uint64_t v, int64_t stride_tok, int64_t stride_head, int64_t stride_batch, int heads, int batch, int head_dim) {
    const uint64_t offsets = k | v | uint64_t(stride_tok) * 2 | (heads > 1 ? uint64_t(stride_head) * 2 : 0) | (batch > 1 ? uint64_t(stride_batch) * 2 : 0);
    return offsets % 128 != 0 && (stride_tok - head_dim) * 2 >= 128;
}

template <int D>
int launch(AttnParams a, int heads, void *workspace, int64_t workspace_bytes, hipStream_t stream) {
    int dev = 0;
    const int cus = lp::device_compute_units(&dev);
    if (cus <= 0) return LP_ERR_HIP;
    a.tiles_per_unit = (a.n + kBN - 1) / kBN;
    const uint32_t tpu = uint32_t(a.tiles_per_unit);
    const bool scratch = workspace != nullptr && workspace_bytes >= workspace_bytes_for<D>(cus);
    const bool split = rows_split(uint64_t(uintptr_t(a.k)), uint64_t(uintptr_t(a.v)), a.stride_tok, a.stride_head, a.stride_batch, a.heads,
                                  heads / a.heads, D);
    const Route r = pick_route(D, a.n, heads, cus, scratch, split);
    const Deal &d = r.deal;
    // short calls go to attention_short_kernel, which needs no scratch memory
    if (r.short_kernel)
        return lp::attention_short({a.q, a.k, a.v, a.o, a.stride_tok, a.stride_head, a.stride_batch, a.heads, heads, D, a.n, a.scale_log2e}, stream);
    a.ws = r.cut ? static_cast<float *>(workspace) : nullptr;
    a.n_qtiles = (a.n + unit_rows(d.qb) - 1) / unit_rows(d.qb);
    if (d.tail != 0) {                      // d.shared of these, behind the rounds
        const int large = int(d.rounds * d.wgs);
        a.tail_units = d.shared;
        a.tail_head = large / a.n_qtiles;
        a.tail_row = large % a.n_qtiles * unit_rows(d.qb);
        a.tail_qtiles = (a.n + unit_rows(d.tail) - 1) / unit_rows(d.tail);
        a.tail_first = (a.n - a.tail_row + unit_rows(d.tail) - 1) / unit_rows(d.tail);
    }
    a.shared_units = d.tail != 0 ? 0 : int(d.shared);
    a.whole_rounds = int(d.rounds);
    a.unit_cost = tpu + (r.cut ? kBoundaryTiles : 0);
    a.shared_work = uint32_t(a.shared_units) * a.unit_cost;
    a.shared_wgs = d.tail != 0 ? 0 : d.sharers;
    return (D == 128 ? lp::attention_tiles_128 : lp::attention_tiles_64)(a, d.qb, d.tail, d.wgs, dev, stream);
}

}  // namespace

extern "C" int lp_internal_attention_tiles(int64_t n, int32_t all_heads, int32_t head_dim, int32_t cus, int32_t scratch, int32_t split, int32_t tiles[3]) {
    const Route r = pick_route(head_dim, n, all_heads, cus, scratch != 0, split != 0);
    tiles[0] = r.short_kernel ? 0 : unit_rows(r.deal.qb);
    tiles[1] = r.short_kernel ? 0 : unit_rows(r.deal.tail);
    tiles[2] = r.cut;
    return LP_OK;
}

extern "C" int lp_internal_attention_rows_split(uint64_t k, uint64_t v, int64_t stride_tok, int64_t stride_head, int64_t stride_batch, int32_t heads,
                                                int32_t batch, int32_t head_dim) {
    return rows_split(k, v, stride_tok, stride_head, stride_batch, heads, batch, head_dim);
}

extern "C" int64_t lp_attention_workspace_size(int32_t head_dim) {
    if (head_dim != 64 && head_dim != 128) return LP_ERR_UNSUPPORTED;
    const int cus = lp::device_compute_units();
    if (cus <= 0) return LP_ERR_HIP;
    return head_dim == 128 ? workspace_bytes_for<128>(cus) : workspace_bytes_for<64>(cus);
}

namespace {

// Argument checks shared by the entry points; no HIP call.  LP_OK: launch; kNothingToDo: succeed
// without a launch; negative: the error to return.
constexpr int kNothingToDo = 1;

int attention_check(const void *q, const void *k, const void *v, void *o, int32_t batch, int64_t n_tokens, int32_t heads,
                    int32_t head_dim, int64_t stride_batch, int64_t stride_tok, int64_t stride_head,
                    void *workspace, int64_t workspace_bytes) {
    if (n_tokens < 0 || heads < 1 || batch < 1) return LP_ERR_INVALID_ARG;
    if (head_dim != 64 && head_dim != 128) return LP_ERR_UNSUPPORTED;
    if (n_tokens == 0) return kNothingToDo;
    if (q == nullptr || k == nullptr || v == nullptr || o == nullptr) return LP_ERR_INVALID_ARG;
    if (!aligned16(q) || !aligned16(k) || !aligned16(v) || !aligned16(o)) return LP_ERR_INVALID_ARG;
    if (o == q || o == k || o == v) return LP_ERR_INVALID_ARG;   // the output is written while inputs are still read
    if (workspace != nullptr && (!aligned16(workspace) || workspace_bytes < 0)) return LP_ERR_INVALID_ARG;
    if (stride_head < head_dim || stride_head % 8 != 0 || stride_tok % 8 != 0) return LP_ERR_INVALID_ARG;
    // rows of different (token, head) pairs must not overlap: either token-major or head-major
    const bool token_major = stride_tok >= int64_t(heads) * stride_head;
    const bool head_major = stride_head >= n_tokens * stride_tok && stride_tok >= head_dim;
    if (!token_major && !head_major) return LP_ERR_INVALID_ARG;
    if (batch > 1) {
        // items one after the other, or (token-major) the items of a token side by side
        if (stride_batch < 0 || stride_batch % 8 != 0) return LP_ERR_INVALID_ARG;
        const int64_t item = token_major ? n_tokens * stride_tok : int64_t(heads) * stride_head;
        const bool outer = stride_batch >= item;
        const bool inner = stride_tok >= int64_t(batch) * stride_batch && stride_batch >= int64_t(heads) * stride_head;
        if (!outer && !inner) return LP_ERR_INVALID_ARG;
    }
    // 32-bit addressing inside one head: byte offsets below 2^31, work items below 2^31
    if (n_tokens > (int64_t(1) << 24) || (n_tokens * stride_tok + head_dim) * 2 >= (int64_t(1) << 31)) return LP_ERR_UNSUPPORTED;
    const int64_t all_heads = int64_t(batch) * heads;
    if (all_heads >= (int64_t(1) << 24)) return LP_ERR_UNSUPPORTED;
    const int64_t units = all_heads * ((n_tokens + kBM - 1) / kBM);
    if (units * ((n_tokens + kBN - 1) / kBN + kBoundaryTiles) >= (int64_t(1) << 31)) return LP_ERR_UNSUPPORTED;
    return LP_OK;
}

int attention_call(const void *q, const void *k, const void *v, void *o, int32_t batch, int64_t n_tokens, int32_t heads,
                   int32_t head_dim, int64_t stride_batch, int64_t stride_tok, int64_t stride_head, float scale,
                   void *workspace, int64_t workspace_bytes, void *stream) {
    const int chk = attention_check(q, k, v, o, batch, n_tokens, heads, head_dim, stride_batch, stride_tok, stride_head,
                                    workspace, workspace_bytes);
    if (chk != LP_OK) return chk == kNothingToDo ? LP_OK : chk;
    const int64_t all_heads = int64_t(batch) * heads;
    if (!(scale > 0.0f)) scale = 1.0f / sqrtf(float(head_dim));
    AttnParams a{};
    a.q = static_cast<const __bf16 *>(q);
    a.k = static_cast<const __bf16 *>(k);
    a.v = static_cast<const __bf16 *>(v);
    a.o = static_cast<__bf16 *>(o);
    a.stride_tok = stride_tok;
    a.stride_head = stride_head;
    a.stride_batch = batch > 1 ? stride_batch : 0;
    a.heads = heads;
    a.scale_log2e = scale * 1.4426950408889634f;
    a.n = int(n_tokens);
    hipStream_t st = static_cast<hipStream_t>(stream);
    if (head_dim == 128) return launch<128>(a, int(all_heads), workspace, workspace_bytes, st);
    return launch<64>(a, int(all_heads), workspace, workspace_bytes, st);
}

}  // namespace

// ---- scratch for callers that cannot allocate (lp_attention_static)
// Sized for the partial-result slots of head_dim 128 on kStaticMaxCUs compute units (the
// largest case; head_dim 64 needs less).  Every device the library runs on holds its own copy
// of this array, at its own address, until the process ends.  In host code the array's name
// is only a handle for hipGetSymbolAddress: kernels are given the address that call returns.
constexpr int kStaticMaxCUs = 256;
constexpr size_t kStaticScratchFloats = size_t(2) * kStaticMaxCUs * slot_floats<128>();
static __device__ __align__(256) float scratch[kStaticScratchFloats];

namespace {

constexpr int kMaxDevices = 64;
std::atomic<float *> g_scratch_ptr[kMaxDevices];

// Device address of `scratch` on the current device; looked up once per device, with that
// device current.  Returns nullptr (and records the HIP error) on failure.
float *static_scratch(int *status) {
    int dev = 0;
    hipError_t e = hipGetDevice(&dev);
    if (e != hipSuccess) {
        lp::set_last_hip_error(int(e));
        *status = LP_ERR_HIP;
        return nullptr;
    }
    if (dev < 0 || dev >= kMaxDevices) {
        *status = LP_ERR_LIMIT;
        return nullptr;
    }
    float *p = g_scratch_ptr[dev].load(std::memory_order_acquire);
    if (p == nullptr) {
        void *sym = nullptr;
        e = hipGetSymbolAddress(&sym, HIP_SYMBOL(scratch));
        if (e != hipSuccess || sym == nullptr) {
            lp::set_last_hip_error(int(e));
            *status = LP_ERR_HIP;
            return nullptr;
        }
        p = static_cast<float *>(sym);
        g_scratch_ptr[dev].store(p, std::memory_order_release);   // a racing thread stores the same address
    }
    *status = LP_OK;
    return p;
}

}  // namespace

extern "C" int64_t lp_attention_static_scratch_bytes(void) { return int64_t(kStaticScratchFloats * sizeof(float)); }

extern "C" int lp_attention_static(const void *q, const void *k, const void *v, void *o, int64_t n_tokens,
                                   int32_t heads, int32_t head_dim, int64_t stride_tok, int64_t stride_head,
                                   float scale, void *stream) {
    const int chk = attention_check(q, k, v, o, 1, n_tokens, heads, head_dim, 0, stride_tok, stride_head, nullptr, 0);
    if (chk != LP_OK) return chk == kNothingToDo ? LP_OK : chk;
    const int cus = lp::device_compute_units();
    if (cus <= 0) return LP_ERR_HIP;
    // the slots of every compute unit must fit the fixed array
    const int64_t need = head_dim == 128 ? workspace_bytes_for<128>(cus) : workspace_bytes_for<64>(cus);
    if (need > int64_t(kStaticScratchFloats * sizeof(float))) return LP_ERR_LIMIT;
    int status = LP_OK;
    float *ws = static_scratch(&status);
    if (ws == nullptr) return status;
    return attention_call(q, k, v, o, 1, n_tokens, heads, head_dim, 0, stride_tok, stride_head, scale, ws, need, stream);
}

extern "C" int lp_attention(const void *q, const void *k, const void *v, void *o, int64_t n_tokens,
                            int32_t heads, int32_t head_dim, int64_t stride_tok, int64_t stride_head,
                            float scale, void *workspace, int64_t workspace_bytes, void *stream) {
    return attention_call(q, k, v, o, 1, n_tokens, heads, head_dim, 0, stride_tok, stride_head, scale, workspace,
                          workspace_bytes, stream);
}

extern "C" int lp_attention_batch(const void *q, const void *k, const void *v, void *o, int32_t batch, int64_t n_tokens,
                                  int32_t heads, int32_t head_dim, int64_t stride_batch, int64_t stride_tok,
                                  int64_t stride_head, float scale, void *workspace, int64_t workspace_bytes,
                                  void *stream) {
    return attention_call(q, k, v, o, batch, n_tokens, heads, head_dim, stride_batch, stride_tok, stride_head, scale,
                          workspace, workspace_bytes, stream);
}
