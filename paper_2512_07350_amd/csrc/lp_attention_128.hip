// attention_kernel at head_dim 128 (a file of its own, so that the head dims compile side by side).
#include "lp_attention_kernel.h"

int lp::attention_tiles_128(const AttnParams &a, int qb, int tail, uint32_t wgs, int dev, hipStream_t stream) {
    return launch_tiles<128>(a, qb, tail, wgs, dev, stream);
}
