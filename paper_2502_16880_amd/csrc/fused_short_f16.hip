// k_fused for fp16 rows of up to 4 KB.
#include "fused_instances.h"

const void* coral_fused_short_f16(bool dense, int gate, bool routed, bool logprob, int segs) {
    return fused_short_rows<kF16>(dense, gate, routed, logprob, segs);
}
