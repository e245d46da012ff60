// Internal declarations shared by the library's translation units (not installed).
#pragma once
#include <stdint.h>

#include "lp.h"

// Host-side plan: the integers of Sec. 3.3 (Eq. 7-9) and Sec. 3.4 (Eq. 11) for
// every partition, plus what the copy kernels need to address the packed buffer.
struct lp_plan {
    lp_config cfg;
    int32_t dim;          // 0 = T, 1 = H, 2 = W
    int32_t K;
    int32_t N;            // patches along dim
    int32_t L;            // core patches per partition, ceil(N / K)
    int32_t O;            // overlap patches
    int32_t extent;       // latent extent along dim
    int64_t inner;        // product of the extents after dim (elements per unit step along dim)
    int64_t outer;        // product of the extents before dim, channels included
    int64_t latent_elems; // C*T*H*W
    int64_t total_elems;  // sum of the sub-latent sizes
    lp_part_info part[LP_MAX_PARTS];
};

namespace lp {
void set_last_hip_error(int err);

// A launch has at most this many threads (a dispatch states its grid as 32-bit thread counts).
constexpr int64_t kMaxLaunchThreads = (int64_t(1) << 32) - 1;
}

// Which way a call of these sizes goes on a device of `cus` compute units.  Host arithmetic for the tests (a
// test of one kernel states that its sizes run that kernel); not part of the library's interface.
extern "C" {
// tiles: query rows of attention_kernel's tiles (0: the short kernel, whose wavefronts share the keys), those of its last round (0: the
// same), 1 if the tiles of the last round are cut into ranges and merged
int lp_internal_attention_tiles(int64_t n, int32_t all_heads, int32_t head_dim, int32_t cus, int32_t scratch, int32_t split, int32_t tiles[3]);
// 1 if the rows of K or V lie split over cache lines (`split` above; addresses in bytes, strides in elements)
int lp_internal_attention_rows_split(uint64_t k, uint64_t v, int64_t stride_tok, int64_t stride_head, int64_t stride_batch, int32_t heads,
                                     int32_t batch, int32_t head_dim);
// head_dim 0: lp_linear.  way: features and tokens of a tile, those of the tiles that cut the last round (0: none),
// the workgroups, and the threads of each.
int lp_internal_gemm_way(int64_t n, int32_t d_in, int32_t d_out, int32_t head_dim, int32_t cus, int64_t way[6]);
}

#ifdef __HIPCC__
#include <hip/hip_runtime.h>
namespace lp {
// Launch through hipLaunchKernel so that the status is this launch's own return
// value (hipGetLastError would also report errors other code left behind).
template <typename... Args>
inline int launch_kernel(const void *fn, dim3 grid, dim3 block, size_t lds_bytes, hipStream_t stream, Args... args) {
    void *argv[] = {static_cast<void *>(&args)...};
    const hipError_t e = hipLaunchKernel(fn, grid, block, argv, lds_bytes, stream);
    if (e != hipSuccess) {
        set_last_hip_error(int(e));
        return LP_ERR_HIP;
    }
    return LP_OK;
}

// lp_attention's arguments after the checks.
struct AttentionCall {
    const void *q, *k, *v;
    void *o;
    int64_t stride_tok, stride_head, stride_batch;
    int32_t heads, all_heads, head_dim;   // heads of one batch item, of all items
    int32_t n;
    float scale_log2e;
};
// The kernel for short sequences (lp_attention_short.hip), whether its grid fits a launch, and what it is expected to take.
int attention_short(const AttentionCall &c, hipStream_t stream);
bool attention_short_launchable(int64_t n, int64_t all_heads);
float attention_short_us(int64_t n, int64_t all_heads, int head_dim, int cus, bool split);
// us that q, k, v and o take at the rate of a large copy, 4.7 TB/s
inline float attention_bytes_us(int64_t n, int64_t all_heads, int head_dim) {
    return 8.0f * float(n) * float(all_heads) * float(head_dim) / 4.7e6f;
}

// Compute units of the current device (each host thread remembers the last device it asked about); 0,
// with the HIP error recorded, if there is none.
inline int device_compute_units(int *device = nullptr) {
    static thread_local int cached_dev = -1, cached_cus = 0;
    int dev = 0;
    hipError_t e = hipGetDevice(&dev);
    if (e == hipSuccess && dev != cached_dev) {
        int cus = 0;
        e = hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, dev);
        if (e == hipSuccess) {
            cached_cus = cus;
            cached_dev = dev;
        }
    }
    if (e != hipSuccess) {
        set_last_hip_error(int(e));
        return 0;
    }
    if (device != nullptr) *device = dev;
    return cached_cus;
}
}  // namespace lp
#endif
