// Instances of the streaming kernel: RMSNorm forward
// (those that the rules of host.cpp choose).
#include "stream.h"

namespace credit {

#define CREDIT_1(DT, V, R, SPLIT, FULL) \
    if (dt == DT && v == V && r == R && split == SPLIT && full == FULL) \
        return (const void *)&k_stream<OP_RMS_FWD, DT, V, R, SPLIT, FULL>;
#define CREDIT_S(DT, V, R, SPLIT) CREDIT_1(DT, V, R, SPLIT, true) CREDIT_1(DT, V, R, SPLIT, false)

const void *stream_kernel_rms_fwd(int dt, int v, int r, bool split, bool full) {
    CREDIT_S(DT_F32, 2, 2, false) CREDIT_S(DT_F32, 4, 1, false) CREDIT_S(DT_F32, 8, 1, false)
    CREDIT_S(DT_F32, 1, 4, true) CREDIT_1(DT_F32, 2, 2, true, true) CREDIT_S(DT_F32, 2, 4, true)
    CREDIT_S(DT_F32, 4, 1, true) CREDIT_S(DT_F32, 8, 1, true)
    CREDIT_S(DT_BF16, 2, 2, false) CREDIT_S(DT_BF16, 2, 4, false) CREDIT_S(DT_BF16, 4, 1, false)
    CREDIT_S(DT_BF16, 8, 1, false)
    CREDIT_S(DT_BF16, 1, 4, true) CREDIT_S(DT_BF16, 2, 2, true) CREDIT_1(DT_BF16, 2, 4, true, true)
    CREDIT_1(DT_BF16, 4, 1, true, true) CREDIT_1(DT_BF16, 8, 1, true, false)
    return nullptr;
}

}  // namespace credit
