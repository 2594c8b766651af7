// Map of the control words at the start of the workspace (32-bit words, all but kGatePolls and
// kGateGaveUp zero between calls; coral_lmhead_workspace_init prepares them once, every kernel that
// uses one leaves it as it was).  Plain constants so that a host compiler can include this file too:
// a test builds the table below and checks that no two entries overlap and all lie inside the
// control area.
#pragma once

namespace coral_ctrl {

struct Entry {
    const char* name;
    int first_word;
    int n_words;
};

constexpr int kWords = 128;                 // size of the control area in words (512 bytes)
constexpr int kFusedArrival = 0;            // single-launch path: workgroups that have published
constexpr int kGateSelectArrival = 8;       // tile path: per token tile, k_gate_select workgroups that
constexpr int kGateSelectArrivalWords = 4;  //   have stored their scores (at most 4 token tiles)
constexpr int kTileQueue = 4;               // tile path: next block of k_tiles
constexpr int kLpGroupArrival = 64;         // log-probability mode: one counter per activated
constexpr int kLpGroupArrivalWords = 64;    //   group (at most 64 in the single-launch kernel)
constexpr int kGateDone = 1;                // single-launch path, shared gate: workgroups that have read the scores,
constexpr int kGateGaveUp = 2;              //   how many had to compute the gate alone so far,
constexpr int kGatePolls = 32;              //   and how often a workgroup asks for the scores at most (0: nobody
                                            //   has cleared the score words yet; the next such call does);
                                            //   in a 128-byte line without counters, as it is read through the caches

// Behind the control area: the shared gate's scores, group by group (bit patterns; 0: not there yet, and
// so between calls).
constexpr int kGateScores = kWords;
constexpr int kGateScoreWords = 4096;
constexpr int kPreparedWords = kWords + kGateScoreWords;

constexpr Entry kMap[] = {
    {"fused_arrival", kFusedArrival, 1},
    {"gate_select_arrival", kGateSelectArrival, kGateSelectArrivalWords},
    {"tile_queue", kTileQueue, 1},
    {"logprob_group_arrival", kLpGroupArrival, kLpGroupArrivalWords},
    {"gate_done", kGateDone, 1},
    {"gate_polls", kGatePolls, 1},
    {"gate_gave_up", kGateGaveUp, 1},
};
constexpr int kMapEntries = sizeof(kMap) / sizeof(kMap[0]);

}  // namespace coral_ctrl
