// Instances of the streaming kernel: the LayerNorm / RMSNorm backward.
#include "stream.h"

namespace credit {

#define CREDIT_K(OP, DT, V, R, SPLIT) \
    (full ? (const void *)&k_stream<OP, DT, V, R, SPLIT, true> : (const void *)&k_stream<OP, DT, V, R, SPLIT, false>)
#define CREDIT_S(OP, DT, V, R) \
    if (op == OP && dt == DT && v == V && r == R) \
        return split ? CREDIT_K(OP, DT, V, R, true) : CREDIT_K(OP, DT, V, R, false);
#define CREDIT_SV(OP, DT) \
    CREDIT_S(OP, DT, 1, 4) CREDIT_S(OP, DT, 1, 2) CREDIT_S(OP, DT, 2, 2) CREDIT_S(OP, DT, 2, 4) CREDIT_S(OP, DT, 4, 1)

const void *stream_kernel_bwd(int op, int dt, int v, int r, bool split, bool full) {
    CREDIT_SV(OP_LN_BWD, DT_F32)
    CREDIT_SV(OP_LN_BWD, DT_BF16)
    CREDIT_SV(OP_RMS_BWD, DT_F32)
    CREDIT_SV(OP_RMS_BWD, DT_BF16)
    return nullptr;
}

}  // namespace credit
