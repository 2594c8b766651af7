// k_fused for bf16 rows of more than 4 KB, up to 16 KB.
#include "fused_instances.h"

const void* coral_fused_long_bf16(bool dense, int gate, bool routed, bool logprob, int segs) {
    return fused_long_rows<kBF16>(dense, gate, routed, logprob, segs);
}
