// Addresses of the single-launch kernel's instantiations (k_fused, fused_path.h), which are
// compiled in translation units of their own: rows of up to 4 KB (segs 2, 4) and longer ones
// (segs 8, 16) per storage type.
#pragma once

#define CORAL_FUSED_GETTER(name) \
    __attribute__((visibility("hidden"))) const void* name(bool dense, int gate, bool routed, bool logprob, int segs)

CORAL_FUSED_GETTER(coral_fused_short_f32);
CORAL_FUSED_GETTER(coral_fused_long_f32);
CORAL_FUSED_GETTER(coral_fused_short_bf16);
CORAL_FUSED_GETTER(coral_fused_long_bf16);
CORAL_FUSED_GETTER(coral_fused_short_f16);
CORAL_FUSED_GETTER(coral_fused_long_f16);
