// Instances of the streaming kernel: row-wise int8 quantisation.
#include "stream_quant.h"

namespace credit {

#define CREDIT_K(DT, V, R, SPLIT) \
    (full ? (const void *)&k_stream_quant<DT, V, R, SPLIT, true> : (const void *)&k_stream_quant<DT, V, R, SPLIT, false>)
#define CREDIT_S(DT, V, R) \
    if (dt == DT && v == V && r == R) return split ? CREDIT_K(DT, V, R, true) : CREDIT_K(DT, V, R, false);
#define CREDIT_W(DT) \
    if (dt == DT && v == 8 && r == 1 && !split) return CREDIT_K(DT, 8, 1, false);  // the widest: resident rows only

const void *stream_kernel_quant(int dt, int v, int r, bool split, bool full) {
    CREDIT_S(DT_F32, 1, 2) CREDIT_S(DT_F32, 2, 2) CREDIT_S(DT_F32, 4, 1) CREDIT_W(DT_F32)
    CREDIT_S(DT_BF16, 1, 2) CREDIT_S(DT_BF16, 2, 2) CREDIT_S(DT_BF16, 4, 1) CREDIT_W(DT_BF16)
    return nullptr;
}

}  // namespace credit
