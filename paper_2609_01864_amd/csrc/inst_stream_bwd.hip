// Instances of the streaming kernel: the LayerNorm / RMSNorm backward
// (those that the rules of host.cpp choose).
#include "stream.h"

namespace credit {

#define CREDIT_1(OP, DT, V, R, SPLIT, FULL) \
    if (op == OP && dt == DT && v == V && r == R && split == SPLIT && full == FULL) \
        return (const void *)&k_stream<OP, DT, V, R, SPLIT, FULL>;
#define CREDIT_S(OP, DT, V, R, SPLIT) CREDIT_1(OP, DT, V, R, SPLIT, true) CREDIT_1(OP, DT, V, R, SPLIT, false)

const void *stream_kernel_bwd(int op, int dt, int v, int r, bool split, bool full) {
    CREDIT_S(OP_LN_BWD, DT_F32, 1, 4, false) CREDIT_S(OP_LN_BWD, DT_F32, 2, 2, false)
    CREDIT_S(OP_LN_BWD, DT_F32, 4, 1, false)
    CREDIT_S(OP_LN_BWD, DT_F32, 1, 2, true) CREDIT_S(OP_LN_BWD, DT_F32, 1, 4, true)
    CREDIT_S(OP_LN_BWD, DT_F32, 2, 2, true)
    CREDIT_S(OP_LN_BWD, DT_BF16, 1, 4, false) CREDIT_S(OP_LN_BWD, DT_BF16, 2, 2, false)
    CREDIT_S(OP_LN_BWD, DT_BF16, 1, 4, true) CREDIT_S(OP_LN_BWD, DT_BF16, 2, 2, true)
    CREDIT_S(OP_LN_BWD, DT_BF16, 2, 4, true)
    CREDIT_S(OP_RMS_BWD, DT_F32, 1, 4, false) CREDIT_S(OP_RMS_BWD, DT_F32, 2, 2, false)
    CREDIT_S(OP_RMS_BWD, DT_F32, 4, 1, false)
    CREDIT_S(OP_RMS_BWD, DT_F32, 1, 2, true) CREDIT_S(OP_RMS_BWD, DT_F32, 1, 4, true)
    CREDIT_S(OP_RMS_BWD, DT_F32, 2, 2, true) CREDIT_S(OP_RMS_BWD, DT_F32, 4, 1, true)
    CREDIT_S(OP_RMS_BWD, DT_BF16, 1, 4, false) CREDIT_S(OP_RMS_BWD, DT_BF16, 2, 2, false)
    CREDIT_S(OP_RMS_BWD, DT_BF16, 4, 1, false)
    CREDIT_S(OP_RMS_BWD, DT_BF16, 1, 2, true) CREDIT_S(OP_RMS_BWD, DT_BF16, 1, 4, true)
    CREDIT_S(OP_RMS_BWD, DT_BF16, 2, 2, true)
    return nullptr;
}

}  // namespace credit
