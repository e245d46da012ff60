// What the dispatch of lp_attention (lp_attention.hip) and its kernels (lp_attention_kernel.h) share (not installed).
#pragma once
#include <hip/hip_runtime.h>

#include "lp_device.h"

namespace lp {

constexpr int kWaves = 4;                     // wavefronts per workgroup, one per SIMD
constexpr int kMostQB = 4;                    // 16-query blocks of a wavefront: 4, 64 rows, wherever that fills the chip
constexpr int unit_rows(int qb) { return 16 * kWaves * qb; }              // query rows per workgroup
constexpr int kBM = unit_rows(kMostQB);
constexpr int kBN = 64;                       // keys per LDS tile (two rounds of 32)
constexpr uint32_t kBoundaryTiles = 4;        // what changing units costs a workgroup, in tile times

// Launch parameters.  A unit is one query tile of one head, 256 rows unless said otherwise; every unit walks
// tiles_per_unit tiles of 64 keys.  With P workgroups, the units are served in two parts:
//  * the first shared_units units form a (unit, key tile) iteration space that is cut into
//    shared_wgs <= P contiguous ranges (never empty), so a workgroup may start and end in
//    the middle of a unit; such partial results go to `ws` and are merged by combine_kernel.
//    The workgroups that take one are spread evenly over the P.  With shared_wgs = shared_units
//    every range is a whole unit and nothing is left to merge.
//    The cut is even in COST, not in tiles: every unit is preceded by kBoundaryTiles
//    imaginary tiles that stand for what a workgroup pays to change units (drain and
//    refill of the pipeline, stores, a new Q), the space of shared_units * unit_cost
//    real and imaginary tiles is cut into equal ranges, and a range's imaginary tiles are
//    dropped.  A workgroup that changes units thus gets fewer tiles than one that does not.
//  * the remaining whole_rounds * P units are taken whole, unit shared_units + r*P + p by
//    workgroup p in round r: the workgroups of an XCD then walk the keys of one head in
//    step and share its K/V stream through the L2.
// A call whose last round is in smaller units has no shared ones, and whole_rounds * P units before them.
struct AttnParams {
    const __bf16 *q, *k, *v;
    __bf16 *o;
    float *ws;                 // slots for partial results: 2 per workgroup
    int64_t stride_tok, stride_head, stride_batch;
    int heads;                 // heads per batch item; a unit's head index counts batch * heads + head
    float scale_log2e;
    int n, n_qtiles, tiles_per_unit;
    int shared_units, whole_rounds;
    uint32_t shared_work;      // shared_units * unit_cost
    uint32_t unit_cost;        // tiles_per_unit + kBoundaryTiles
    uint32_t tail_units;       // smaller units of the last round, one to a workgroup; the rows before (tail_head, tail_row) are in large ones
    int tail_head, tail_row;
    int tail_first, tail_qtiles;   // smaller units of tail_head, and of a whole head
    uint32_t shared_wgs;       // ranges of the shared space; workgroup p (logical order) takes range r if r is the only
                               // number in [p shared_wgs / P, (p + 1) shared_wgs / P), both rounded down
};

// A slot holds, for the 256 query rows of a unit: m[256] and l[256] in binary32, then the
// unnormalised O rows [256][D] rounded to bf16 (the merged row is rounded to bf16 on store
// anyway; halving the rows halves the traffic of the merge).
template <int D>
constexpr int slot_floats() { return kBM * (D / 2 + 2); }

// The tiles a call is dealt in: units of 16 kWaves qb query rows, and of 16 kWaves tail rows in the last round if tail is
// not 0.  Compiled: qb 2 .. kMostQB alone, kMostQB with a tail of 3.  Launches attention_kernel on `wgs` workgroups and, where
// a.ws is given, combine_kernel behind it.
int attention_tiles_64(const AttnParams &a, int qb, int tail, uint32_t wgs, int dev, hipStream_t stream);
int attention_tiles_128(const AttnParams &a, int qb, int tail, uint32_t wgs, int dev, hipStream_t stream);

}  // namespace lp
