// k_fused for fp16 rows of more than 4 KB, up to 16 KB.
#include "fused_instances.h"

const void* coral_fused_long_f16(bool dense, int gate, bool routed, bool logprob, int segs) {
    return fused_long_rows<kF16>(dense, gate, routed, logprob, segs);
}
