// Instances of the streaming kernel: FP8 LayerNorm forward.
#include "stream_fp8.h"

namespace credit {

const void *stream_kernel_ln_fp8(bool split, bool full) {
    if (split) return full ? (const void *)&k_stream_ln_fp8<true, true> : (const void *)&k_stream_ln_fp8<true, false>;
    return full ? (const void *)&k_stream_ln_fp8<false, true> : (const void *)&k_stream_ln_fp8<false, false>;
}

}  // namespace credit
