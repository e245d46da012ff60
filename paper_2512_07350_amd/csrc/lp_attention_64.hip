// attention_kernel at head_dim 64 (a file of its own, so that the head dims compile side by side).
#include "lp_attention_kernel.h"

int lp::attention_tiles_64(const AttnParams &a, int qb, int tail, uint32_t wgs, int dev, hipStream_t stream) {
    return launch_tiles<64>(a, qb, tail, wgs, dev, stream);
}
