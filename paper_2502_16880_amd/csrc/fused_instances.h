// The instantiations of k_fused for one storage type and row lengths; the translation units
// fused_*.hip hold one set each so that they compile side by side.
#pragma once
#include "fused_kernels.h"
#include "fused_path.h"

namespace {

template <int DT, int SEGS>
const void* fused_instance(bool dense, int gate, bool routed, bool logprob) {
#define CORAL_FUSED(...) reinterpret_cast<const void*>(&k_fused<DT, __VA_ARGS__, SEGS>)
    if (dense) return CORAL_FUSED(true, kGateVector, false, false);
    if (gate == kGateShared)
        return logprob ? (routed ? CORAL_FUSED(false, kGateShared, true, true) : CORAL_FUSED(false, kGateShared, false, true))
                       : (routed ? CORAL_FUSED(false, kGateShared, true, false) : CORAL_FUSED(false, kGateShared, false, false));
    if constexpr (DT != kF32) {
        if (gate == kGateMfma && !logprob)
            return routed ? CORAL_FUSED(false, kGateMfma, true, false) : CORAL_FUSED(false, kGateMfma, false, false);
        if constexpr (SEGS <= 8) {     // (rows beyond 8 KB with log-probabilities: always shared, or another path)
            if (gate == kGateMfma)
                return routed ? CORAL_FUSED(false, kGateMfma, true, true) : CORAL_FUSED(false, kGateMfma, false, true);
        } else {
            if (gate == kGateMfma) return nullptr;
        }
    }
    return logprob ? (routed ? CORAL_FUSED(false, kGateVector, true, true) : CORAL_FUSED(false, kGateVector, false, true))
                   : (routed ? CORAL_FUSED(false, kGateVector, true, false) : CORAL_FUSED(false, kGateVector, false, false));
#undef CORAL_FUSED
}

template <int DT>
const void* fused_short_rows(bool dense, int gate, bool routed, bool logprob, int segs) {
    return segs <= 2 ? fused_instance<DT, 2>(dense, gate, routed, logprob)
                     : fused_instance<DT, 4>(dense, gate, routed, logprob);
}
template <int DT>
const void* fused_long_rows(bool dense, int gate, bool routed, bool logprob, int segs) {
    return segs <= 8 ? fused_instance<DT, 8>(dense, gate, routed, logprob)
                     : fused_instance<DT, 16>(dense, gate, routed, logprob);
}

}  // namespace
