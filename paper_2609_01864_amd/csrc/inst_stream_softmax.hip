// Instances of the streaming kernel: softmax forward.
#include "stream_softmax.h"

namespace credit {

#define CREDIT_K(DT, V, R, SPLIT) \
    (full ? (const void *)&k_stream_softmax<OP_SOFTMAX_FWD, DT, V, R, SPLIT, true> : (const void *)&k_stream_softmax<OP_SOFTMAX_FWD, DT, V, R, SPLIT, false>)
#define CREDIT_S(DT, V, R) \
    if (dt == DT && v == V && r == R) return split ? CREDIT_K(DT, V, R, true) : CREDIT_K(DT, V, R, false);

const void *stream_kernel_softmax(int dt, int v, int r, bool split, bool full) {
    CREDIT_S(DT_F32, 1, 2) CREDIT_S(DT_F32, 2, 2) CREDIT_S(DT_F32, 4, 1) CREDIT_S(DT_F32, 8, 1)
    CREDIT_S(DT_BF16, 1, 2) CREDIT_S(DT_BF16, 2, 2) CREDIT_S(DT_BF16, 4, 1) CREDIT_S(DT_BF16, 8, 1)
    if (dt == DT_FP8 && v == 4 && r == 1) {  // split: whole slices only
        if (full) return split ? (const void *)&k_stream_softmax<OP_SOFTMAX_FWD, DT_FP8, 4, 1, true, true>
                               : (const void *)&k_stream_softmax<OP_SOFTMAX_FWD, DT_FP8, 4, 1, false, true>;
        if (!split) return (const void *)&k_stream_softmax<OP_SOFTMAX_FWD, DT_FP8, 4, 1, false, false>;
    }
    return nullptr;
}

}  // namespace credit
