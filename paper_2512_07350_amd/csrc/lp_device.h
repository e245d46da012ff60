// Device helpers that more than one translation unit uses (not installed).
#pragma once
#include <hip/hip_runtime.h>

#include <atomic>
#include <type_traits>

#include "lp_internal.h"

#define LP_LDS_PTR(T, p) ((__attribute__((address_space(3))) T *)(p))

namespace lp {

typedef __attribute__((ext_vector_type(8))) __bf16 bf16x8;
typedef __attribute__((ext_vector_type(4))) __bf16 bf16x4;
typedef __attribute__((ext_vector_type(2))) __bf16 bf16x2;
typedef __attribute__((ext_vector_type(4))) float f32x4;
typedef __attribute__((ext_vector_type(2))) float f32x2;
typedef __attribute__((ext_vector_type(2))) uint32_t u32x2;
typedef __attribute__((ext_vector_type(4))) uint32_t u32x4;

union Pack16 {
    uint4 u;
    bf16x8 v;
    bf16x4 h[2];
    bf16x2 p[4];
};

// floor(n / d) for 0 <= n < 2^31 as (n * magic) >> shift with a 64-bit product.
// With l = ceil(log2 d), magic = floor(2^(31+l) / d) + 1 < 2^32 and shift = 31 + l,
// magic*d = 2^shift + e with 0 < e <= 2^l, so the error term n*e/(d*2^shift) < 1/d.
struct FastDiv {
    uint32_t magic;
    uint32_t shift;
    uint32_t d;
};

inline FastDiv make_fastdiv(uint32_t d) {
    FastDiv f;
    f.d = d;
    uint32_t l = 0;
    while ((uint64_t(1) << l) < d) ++l;
    f.shift = 31 + l;
    f.magic = uint32_t(((unsigned __int128)1 << f.shift) / d + 1);
    return f;
}

__device__ __forceinline__ uint32_t fastdiv(uint32_t n, const FastDiv &f) {
    return uint32_t((uint64_t(n) * f.magic) >> f.shift);
}

// f(integral_constant<int, I>) for I = FROM .. TO-1: a loop whose index is a constant
// expression inside the body.
template <int FROM, int TO, typename F>
__device__ __forceinline__ void static_for(F &&f) {
    if constexpr (FROM < TO) {
        f(std::integral_constant<int, FROM>{});
        static_for<FROM + 1, TO>(f);
    }
}

__device__ __forceinline__ bf16x2 to_bf16x2(float lo, float hi) {
    f32x2 f = {lo, hi};
    return __builtin_convertvector(f, bf16x2);
}

// LDS accesses use 32-bit LDS byte addresses held in registers.
template <typename V>
__device__ __forceinline__ V lds_load(uint32_t addr) {
    return *LP_LDS_PTR(const V, uintptr_t(addr));
}
template <typename V>
__device__ __forceinline__ void lds_store(uint32_t addr, const V &x) {
    *LP_LDS_PTR(V, uintptr_t(addr)) = x;
}

// One wave-wide global -> LDS load of 1024 bytes: lane L fetches the 16 bytes at byte offset voff + soff of the
// buffer and they land at LDS address lds_addr + 16 L (lds_addr is wave-uniform and goes through M0; bytes outside
// the buffer arrive as zeros).  Written as an assembly statement so that the compiler keeps no record of it: told about
// such a load, it waits for ALL of them (vmcnt(0)) before the next LDS read of any address, which would put the whole
// memory latency of the tile just sent for in front of the operand reads of the tiles in use.  The users order these
// loads against the reads of their own stage with vmcnt waits and barriers, and use M0 for nothing else.
__device__ __forceinline__ void load_to_lds_16(__amdgpu_buffer_rsrc_t rsrc, uint32_t lds_addr, uint32_t voff, uint32_t soff) {
    asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tbuffer_load_dwordx4 %1, %2, %3 offen lds"
                 :
                 : "s"(lds_addr), "v"(voff), "s"(rsrc), "s"(soff)
                 : "memory", "m0");
}

// Granule XOR masks of the attention kernels' K and V tiles in LDS (rows of D bf16 in 16-byte granules); reader and writer
// use the same functions.  A K read takes, per 16 lanes, one granule of the rows 8 (r / 4) + r % 4 (+ 4): their 16 places
// must differ modulo the 256 bytes of the banks.  A V read takes, per 32 lanes, two granules of the rows 0-3 and
// 8-11 (+ 4, + 16).
template <int D>
struct TileSwizzle {
    __device__ static int swz_k(int row) { return D == 128 ? (row & 3) | ((row >> 1) & 12) : ((row >> 1) & 1) | ((row >> 2) & 6); }
    __device__ static int swz_v(int row) { return D == 128 ? 2 * ((row & 3) | ((row >> 1) & 4)) : (row & 2) | ((row >> 1) & 4); }
};

// Workgroup ids are dealt round robin to the 8 XCDs; remap so that each XCD owns a contiguous stretch of the logical
// order and what neighbours in it share stays in one XCD's L2.
__device__ __forceinline__ uint32_t logical_workgroup(uint32_t b, uint32_t n_wg) {
    const uint32_t xcd = b % 8, slot = b / 8;
    const uint32_t base = n_wg / 8, rem = n_wg % 8;
    return xcd * base + (xcd < rem ? xcd : rem) + slot;
}

// op over the four lanes of equal lane % 16 (the four quads of a matrix instruction's column), in every
// one of them.  The swaps exchange rows of 16 (32) lanes between two copies of x, after which one copy
// holds the first and the other the second of each pair of rows.
template <typename Op>
__device__ __forceinline__ float over_quads(float x, Op &&op) {
    const auto a = __builtin_amdgcn_permlane16_swap(__float_as_uint(x), __float_as_uint(x), false, false);
    x = op(__uint_as_float(a[0]), __uint_as_float(a[1]));
    const auto b = __builtin_amdgcn_permlane32_swap(__float_as_uint(x), __float_as_uint(x), false, false);
    return op(__uint_as_float(b[0]), __uint_as_float(b[1]));
}
__device__ __forceinline__ float quad_max(float x) { return over_quads(x, [](float a, float b) { return fmaxf(a, b); }); }

// Lets kernel `fn` have `bytes` of dynamic LDS on device `dev`.  The limit is an attribute of the function on a device: set
// once per device, `done` holding a bit for each (a repeated set by a racing host thread is harmless).
inline int allow_lds(const void *fn, int bytes, int dev, std::atomic<uint64_t> &done) {
    const uint64_t dev_bit = dev < 64 ? (uint64_t(1) << dev) : 0;
    if ((done.load(std::memory_order_relaxed) & dev_bit) == 0) {
        const hipError_t e = hipFuncSetAttribute(fn, hipFuncAttributeMaxDynamicSharedMemorySize, bytes);
        if (e != hipSuccess) {
            set_last_hip_error(int(e));
            return LP_ERR_HIP;
        }
        done.fetch_or(dev_bit, std::memory_order_relaxed);
    }
    return LP_OK;
}

inline bool aligned16(const void *p) { return (reinterpret_cast<uintptr_t>(p) & 15) == 0; }

}  // namespace lp
