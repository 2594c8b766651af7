// Single-launch path of the grouped / dense LM head.
//
// One persistent workgroup of 16 waves per compute unit.  Every workgroup
//   1. stages the M hidden vectors in LDS,
//   2. gets the gate s[M,G] (Eq. 7's W2 projection): computes all of it from the L2-resident
//      gate matrix, or, where that takes longer than a hand-over between the workgroups, its
//      share of the groups, and reads the others' scores (kGateShared); selects the g best
//      groups per token and builds the list of activated groups with their token masks,
//   3. streams its share of the activated rows: a wave takes a batch of consecutive rows of
//      one group at a time, sixteen 1 KB non-temporal loads whatever the rows' length (SEGS
//      loads per row, 16 / SEGS rows: one row of 16 KB up to eight rows of 2 KB), and dots
//      them with the hidden vectors of the tokens that selected the group
//      (v_dot2c_f32_bf16, fp32 accumulation); the sums across lanes of all the batch's
//      (row, token) pairs are taken together, one result per group of lanes,
//   4. collects the logits per token in LDS where a workgroup meets few rows per token;
//      otherwise keeps per (wave, token) a sorted list of the k best, touched only when a
//      logit beats the wave's current k-th,
//   5. publishes its k best per token; the workgroup that arrives last merges all
//      workgroups' lists and writes the result.
// The logits row never exists in memory.  No workgroup depends on another's progress: the only wait,
// for the shared gate's scores, is bounded, and who gives up computes them.
//
// Log-probability mode (LP, Eq. 8: log p(x) = log p_router(n) + z[x] - lse_n, the softmax
// taken inside each selected group): a workgroup streams rows of one group only, the
// workgroups shared out among the activated groups by cost; beside the candidates
// every wave notes the (max, sum of exp) of every batch of rows for token t, and the workgroup
// sums these pieces in batch order (the result then does not depend on which wave drew
// which batch); the last workgroup of each group finishes the group (lse_n, offset, the
// group's k best per token) and the last group merges every token's g lists.  A draft-level
// call also expands the tree level in that last workgroup (tree_expand.h).
#pragma once
#include "control_words.h"
#include "device_utils.h"
#include "tree_expand.h"
#include "wave_topk.h"

namespace {

constexpr int kFusedWaves = 16;
constexpr int kFusedBlock = kFusedWaves * kWave;
// A wave holds a batch of fused_rows(SEGS) rows of up to SEGS 1 KB segments in registers, 16
// loads in all.  SEGS = 2, 4, 8, 16: with a fixed two rows of eight segments, rows of 1 KB left
// seven loads in eight unused and paid a cross-lane sum and a list step per row.
constexpr int kFusedLoads = 16;
constexpr int kFusedMaxSegs = 16;
__host__ __device__ constexpr int fused_rows(int segs) { return kFusedLoads / segs; }
inline int fused_segs(int jp) { return jp <= 2 ? 2 : jp <= 4 ? 4 : jp <= 8 ? 8 : 16; }
__host__ __device__ constexpr int log2_small(int n) { return n <= 1 ? 0 : 1 + log2_small(n / 2); }
constexpr int kLdsLimit = 160 * 1024;
// Log-probability mode: a batch's cost in a workgroup's time by the tokens that selected its group: its load,
// and their dot products (10 + tokens).  16-bit rows beyond 4 KB, groups with two to three and a half tokens on
// average: little more than the load while the tokens are few, more than that beyond four.  10 + tokens against
// this over 1722 random heads: there 1.01 times as fast on average, 0.98 to 1.05 (us: bf16 H = 3584, 152064
// rows, 16 tokens 164.6, 162.1); fewer tokens a group 0.998, 0.97 to 1.03; more 1.007, 0.93 to 1.06; shorter
// rows and fp32 the same on average.
template <int DT, int SEGS>
__device__ __forceinline__ int lp_batch_cost(int tokens, int pairs, int groups) {
    if (DT == kF32 || SEGS < 8 || pairs < 2 * groups || 2 * pairs > 7 * groups) return 10 + tokens;   // wave-uniform
    return 2 * (20 + tokens) + (tokens > 4 ? 4 * (tokens - 4) : 0);
}
// Batches of a workgroup where there are few: fewer workgroups then leave fewer lists to merge (three
// groups of 101 rows, one token: 24.8 us with all 256, 22.0 with four batches each, 22.4 with 16; six
// tokens over 9500 rows 29.1, 29.0, 39.4; over small heads 4 % with 5 to 7 tokens, 1 % with 10 to 17).
constexpr int kLpFewBatches = 4;
constexpr int kLpPiecesMax = 16 * 1024;    // LDS for a workgroup's log-sum-exp pieces, at most
// Collected candidates: where a workgroup meets few rows per token (the configured shapes:
// g * v / 256, about 63), the waves append every logit to one buffer per token instead of
// keeping sorted lists, and one wave per token ranks the buffer at the end.
constexpr int kCollectMax = kTopkLdsMax;       // entries per token, at most
// Batches dealt out: a workgroup takes this many consecutive ones while there are few rounds
// (see step 3), half as many with less than a round, else single ones; the host's bound on
// collected rows is that for D = 8, which the others do not exceed.
constexpr int kDealFew = 8;
constexpr int kLpGroupCounters = coral_ctrl::kLpGroupArrival - coral_ctrl::kFusedArrival;   // from p.counter
// How the gate (step 2a) is computed: by every workgroup for itself, on the vector units or on the matrix
// cores (16-bit storage, four tokens or more), or shared between the workgroups (see fused_gate_shared in
// coral_lmhead.hip).  The LDS plan goes by the first two whichever runs.
enum GateMode { kGateVector = 0, kGateMfma = 1, kGateShared = 2 };
// Shared gate: its words behind FusedParams::counter, and how often a score is asked for (about 1 us each)
// before the workgroup stops waiting (the control word holds this number, or less: 0 where the score words
// are not cleared).  Undisturbed, nobody gives up with 16 requests over eight heads, with 12 up to a sixth
// do; other kernels in the way, the number hardly matters from 12 to 48.  What the waiting then costs, own
// gate against shared, us a step: Llama3 shape, 8 tokens, beside large matrix products 247, 260, beside
// the same step on another stream 201, 209, H = 8192, one token 199, 205 and 67.5, 74.9; with a large
// gate it is ahead there too (120 groups, H = 8192, 8 tokens 212, 189 and 99, 39).
constexpr int kGateScoresAt = coral_ctrl::kGateScores - coral_ctrl::kFusedArrival;
constexpr int kGateDoneAt = coral_ctrl::kGateDone - coral_ctrl::kFusedArrival;
constexpr int kGatePollsAt = coral_ctrl::kGatePolls - coral_ctrl::kFusedArrival;
constexpr int kGateGaveUpAt = coral_ctrl::kGateGaveUp - coral_ctrl::kFusedArrival;
constexpr int kGatePollsMax = 24;
// Groups left that a workgroup which gave up computes without publishing them or looking again: two rounds
// of its waves, where 256 workgroups' stores to the same few lines take longer (fp32 Llama2, 16 groups, all
// giving up: 45 us a step, 270 with them).  With many left it is the other way round (every workgroup alone
// and a pair at a time: 120 groups, H = 8192, 8 tokens 150 us, 52; 1000 groups, 4 tokens 340, 74).
constexpr int kGateAloneGroups = 2 * kFusedWaves;
static_assert(coral_ctrl::kGateScoreWords <= kFusedBlock * 4, "a thread reads four scores");
constexpr int kGateTileFloats = 256;          // a wave's partial 16 x 16 tile

struct FusedParams {
    const uint4* hidden;        // [M, n_vec]   what the LM head sees
    const uint4* gate_hidden;   // [M, n_vec]   what the router sees (grouped; may equal hidden)
    const uint4* gate_W;        // [G, n_vec]   (grouped)
    const float* bias;          // [G] or null  (grouped)
    const uint4* lm_W;          // [V, n_vec]
    const int32_t* offsets;     // [G+1]        (grouped)
    const int32_t* rows;        // [V]          (grouped)
    int32_t* sel_out;           // [M, g] or null
    Cand* part;                 // [M, k, gridDim.x] per-workgroup lists, entry-major
    unsigned long long* lse_part;   // [M, gridDim.x] (max, sum of exp) pairs (log-probability mode)
    Cand* glist;                // [M, g, k] a token's list per selected group (log-probability mode)
    unsigned long long* pair_lse;   // (max, sum of exp) of every (batch of rows, token) (same mode)
    // Draft-level call (log-probability mode): the tokens are the nodes of a tree level and
    // the workgroup that writes the result also expands the level (tree_expand.h).
    const float* parent_score;  // [M] cumulative log-probabilities of the nodes, or null (zero)
    int32_t* next_parent;       // [n_next], or null: no expansion
    int32_t* next_token;        // [n_next]
    float* next_score;          // [n_next]
    int n_next;
    unsigned int* counter;      // arrival counter, zero between calls; the log-probability
                                // mode also uses words kLpGroupCounters .. + 63, the shared gate
                                // kGateDoneAt and kGateScoresAt .. + M G - 1, zero as well, and
                                // kGatePollsAt, kGateGaveUpAt (control_words.h)
    int32_t* topk_ids;          // [M, k]
    float* topk_logits;         // [M, k]
    int M, V, G, g, k;
    int n_vec, jp;
    int cap;                    // entries per token of the LDS buffer of collected candidates; 0: lists per
                                // wave.  Log-probability mode: every workgroup decides by its rows
    int deal_single;            // batches are dealt singly in any case (cap holds only then)
    int stream_waves;           // waves of a workgroup that stream weight rows (1..16)
};

struct FusedLds {
    int o_hidden, o_lists, o_s, o_mask, o_ugroup, o_ustart, o_uend, o_uprefix, o_umask, o_flags, o_count;
    int o_keys, o_offsets, o_bias;
    int o_sel, o_wgstart;       // log-probability mode only
    int o_pieces, pieces_bytes; // same mode: the log-sum-exp pieces of a workgroup's batches, if they fit
    int o_tree, tree_bytes;     // same mode: a draft level's tables, at the end of the lists' region
    int total;
};

// 16-byte vectors between consecutive hidden vectors in LDS: the row length plus one, so
// that the matrix-core gate, which reads a column of 16 rows at a time, meets no bank conflicts.
__host__ __device__ inline int hidden_lds_stride(int jp) { return jp * kWave + 1; }

// Byte offsets of the kernel's regions in dynamic LDS (the host sizes the launch with the
// same function the kernel lays its pointers out with).
__host__ __device__ inline FusedLds fused_lds_layout(int M, int G, int g, int k, int jp, bool dense,
                                                     int gate_mode, bool logprob = false,
                                                     int cap = 0) {
    FusedLds L;
    int off = 0;
    auto take = [&](size_t bytes) {
        int at = off;
        off = (int)((off + bytes + 15) / 16 * 16);
        return at;
    };
    long long um = (long long)M * g < G ? (long long)M * g : G;   // activated groups at most
    if (dense || um < 1) um = 1;
    size_t hidden_bytes = (size_t)M * hidden_lds_stride(jp) * sizeof(uint4);
    // reused when a workgroup ranks its own candidates: 64 keys per wave
    const size_t own_bytes = (size_t)kFusedWaves * kWave * sizeof(unsigned long long);
    if (hidden_bytes < own_bytes) hidden_bytes = own_bytes;
    size_t lists_bytes = cap && !logprob ? 0 : (size_t)kFusedWaves * M * k * sizeof(Cand);
    if (lists_bytes < (size_t)M * cap * sizeof(unsigned long long)) lists_bytes = (size_t)M * cap * sizeof(unsigned long long);
    // the MFMA gate parks its per-wave partial tiles here before the lists are initialised
    const size_t gate_part_bytes =
        (!dense && gate_mode != kGateVector)
            ? (size_t)kFusedWaves * ((M + 15) / 16) * kGateTileFloats * sizeof(float)
            : 0;
    if (lists_bytes < gate_part_bytes) lists_bytes = gate_part_bytes;
    // Both regions are free when the published lists are merged: the scratch of that lies over
    // them, and in the log-probability mode a draft level's tables behind it.
    L.tree_bytes = logprob ? M * k * (int)(sizeof(unsigned long long) + sizeof(int) + sizeof(float)) : 0;   // (a multiple of 16)
    const size_t merge_bytes = (size_t)kFusedWaves * sizeof(MergeScratch) + L.tree_bytes;
    if (hidden_bytes + lists_bytes < merge_bytes) hidden_bytes = merge_bytes - lists_bytes;
    L.o_hidden = take(hidden_bytes);
    L.o_lists = take(lists_bytes);
    L.o_tree = off - L.tree_bytes;
    L.o_s = take(dense ? 16 : (size_t)M * G * sizeof(float));
    L.o_mask = take(dense ? 16 : (size_t)G * sizeof(unsigned long long));
    L.o_ugroup = take((size_t)um * sizeof(int));
    L.o_ustart = take((size_t)um * sizeof(int));
    L.o_uend = take((size_t)um * sizeof(int));
    L.o_uprefix = take((size_t)(um + 1) * sizeof(int));
    L.o_umask = take((size_t)um * sizeof(unsigned long long));
    L.o_flags = take(16);
    L.o_count = take(cap || logprob ? (size_t)M * sizeof(int) : 0);   // collected candidates per token
    L.o_keys = take(dense ? 16 : (size_t)kFusedWaves * kWave * sizeof(unsigned long long));
    L.o_offsets = take(dense ? 16 : (size_t)(G + 1) * sizeof(int));
    L.o_bias = take(dense ? 16 : (size_t)G * sizeof(float));
    L.o_sel = take(logprob ? (size_t)M * g * sizeof(int) : 0);
    L.o_wgstart = take(logprob ? (size_t)(um + 1) * sizeof(int) : 0);
    L.o_pieces = off;
    L.pieces_bytes = 0;
    if (logprob) {                                     // what is left, up to kLpPiecesMax
        const int left = (kLdsLimit - off) / 16 * 16;
        L.pieces_bytes = left < 0 ? 0 : left < kLpPiecesMax ? left : kLpPiecesMax;
        off += L.pieces_bytes;
    }
    L.total = off;
    return L;
}

__device__ __forceinline__ int uni(int x) { return __builtin_amdgcn_readfirstlane(x); }
__device__ __forceinline__ unsigned long long uni64(unsigned long long x) {
    const unsigned lo = (unsigned)__builtin_amdgcn_readfirstlane((int)(unsigned)x);
    const unsigned hi = (unsigned)__builtin_amdgcn_readfirstlane((int)(unsigned)(x >> 32));
    return ((unsigned long long)hi << 32) | lo;
}

// Insert the wave-uniform candidate (z, id) of token t into that token's LDS list if it
// beats the list's k-th entry.  thr_v / thr_i cache the k-th entry of every token's list
// of this wave, token t in lane t.
__device__ __forceinline__ void lds_list_insert(Cand* list, int k, int lane, float z, int id,
                                                float& thr_v, int& thr_i, int t) {
    const float tv = __int_as_float(__builtin_amdgcn_readlane(__float_as_int(thr_v), t));
    const int ti = __builtin_amdgcn_readlane(thr_i, t);
    if (!better(z, id, tv, ti)) return;                // wave-uniform
    Cand c = sentinel();
    if (lane < k) c = list[lane];
    const unsigned long long b = __ballot(better(z, id, c.v, c.id));
    const int pos = __ffsll(b) - 1;                    // <= k-1: the k-th entry is beaten
    const float sv = lane_below(c.v);
    const int si = lane_below(c.id);
    if (lane == pos) {
        c.v = z;
        c.id = id;
    } else if (lane > pos) {
        c.v = sv;
        c.id = si;
    }
    if (lane < k) list[lane] = c;
    const float nv = __int_as_float(__builtin_amdgcn_readlane(__float_as_int(c.v), k - 1));
    const int ni = __builtin_amdgcn_readlane(c.id, k - 1);
    if (lane == t) {
        thr_v = nv;
        thr_i = ni;
    }
}

__device__ __forceinline__ unsigned long long pack_lse(float m, float s) {
    return ((unsigned long long)__float_as_uint(s) << 32) | __float_as_uint(m);
}
// Takes a packed (max, sum) piece into the running state (m, s).
__device__ __forceinline__ void lse_take(float& m, float& s, unsigned long long piece) {
    const float pm = __uint_as_float((unsigned)(piece & 0xffffffffull));
    const float ps = __uint_as_float((unsigned)(piece >> 32));
    const float nm = fmaxf(m, pm);
    if (nm > -INFINITY) s = s * expf(m - nm) + ps * expf(pm - nm);
    m = nm;
}

// Combines the (max, sum) states of all lanes (absent: (-inf, 0)) into log(sum of exp); -inf
// if there is nothing to sum.
__device__ __forceinline__ float lse_finish(float m, float s) {
    const float wm = wave_max(m);
    const float ws = wave_sum(wm > -INFINITY ? s * expf(m - wm) : 0.f);
    return wm + logf(ws);
}

// One lane's place in a batch: bit 5 of the lane is the row's lowest bit, and so on downwards; the
// bits below number the tokens of a pass (see wave_sum_spread).
template <int ROWS>
__device__ __forceinline__ int batch_row(int lane) {
    int r = 0;
#pragma unroll
    for (int i = 0; i < log2_small(ROWS); ++i) r |= ((lane >> (5 - i)) & 1) << i;
    return r;
}
__host__ __device__ constexpr int batch_lane(int row) {        // the first lane of a row
    return ((row & 1) << 5) | ((row & 2) << 3) | ((row & 4) << 1) | ((row & 8) >> 1);
}

struct BatchSink {                      // where a batch's logits go (wave-uniform but for thr_*)
    Cand* lists;                        // [M, k] this wave's lists
    unsigned long long* keys;           // [M, cap] collected candidates of the workgroup
    int* count;                         // [M]
    int cap;                            // 0: lists
    unsigned long long* lds_pieces;     // log-probability mode: piece of (token slot j, batch) at
    unsigned long long* mem_pieces;     // pieces[j * stride + at], in LDS or in memory
    int pieces_stride, pieces_at;
    bool pieces_in_lds;
    float thr_v;                        // lane t: the k-th entry of token t's list of this wave
    int thr_i;
};

// The next NT tokens of `rem` against the batch in w: dot products, sums across lanes, and the
// logits on their way (to the buffers or lists; in the log-probability mode their (max, sum of
// exp) over the batch's rows too).  rid: this lane's row id; n_rows: rows that exist.
template <int DT, int NT, bool LP, int SEGS>
__device__ __forceinline__ void fused_tokens(const FusedParams& p, const uint4* hs,
                                             const uint4 (&w)[fused_rows(SEGS)][SEGS],
                                             unsigned long long& rem, int& slot, int rid, int n_rows, BatchSink& out) {
    constexpr int ROWS = fused_rows(SEGS);
    constexpr int N = ROWS * NT;
    constexpr int LR = log2_small(ROWS);
    const int lane = threadIdx.x & (kWave - 1);
    const int hs_stride = hidden_lds_stride(p.jp);
    int tok[NT];
#pragma unroll
    for (int i = 0; i < NT; ++i) {
        tok[i] = __ffsll(rem) - 1;
        rem &= rem - 1ull;
    }
    float acc[N];
#pragma unroll
    for (int i = 0; i < N; ++i) acc[i] = 0.f;
#pragma unroll
    for (int j = 0; j < SEGS; ++j) {
        if (j < p.jp) {                                // uniform
#pragma unroll
            for (int i = 0; i < NT; ++i) {
                const uint4 h = hs[tok[i] * hs_stride + j * kWave + lane];
#pragma unroll
                for (int r = 0; r < ROWS; ++r) acc[i * ROWS + r] = dot_vec<DT>(w[r][j], h, acc[i * ROWS + r]);
            }
        }
    }
    const float z = wave_sum_spread<N>(acc, lane);
    int i = 0;                                         // this lane's token of the pass
    int t = tok[0];
    if (NT >= 2) {
        const bool b0 = (lane >> (5 - LR)) & 1;
        t = b0 ? tok[1] : tok[0];
        i = b0 ? 1 : 0;
        if (NT >= 4) {
            const bool b1 = (lane >> (4 - LR)) & 1;
            const int t2 = b0 ? tok[NT >= 4 ? 3 : 0] : tok[NT >= 4 ? 2 : 0];
            t = b1 ? t2 : t;
            i += b1 ? 2 : 0;
        }
    }
    const int row = batch_row<ROWS>(lane);
    const bool first = (lane & (kWave / N - 1)) == 0;  // (a result is in kWave / N neighbouring lanes)
    const bool mine = first && row < n_rows;
    if (out.cap) {                                     // uniform: the token's buffer takes every logit
        if (mine) {
            const int at = atomicAdd(&out.count[t], 1);
            if (at < out.cap) out.keys[(size_t)t * out.cap + at] = cand_key(z, rid);   // (the host's bound holds)
        }
    } else {
        // the token's k-th entry: uniform reads and a select (a lane permute would go through LDS)
        auto thr_of = [&](int i, float& v, int& id) {
            v = __int_as_float(__builtin_amdgcn_readlane(__float_as_int(out.thr_v), tok[i]));
            id = __builtin_amdgcn_readlane(out.thr_i, tok[i]);
        };
        float tv;
        int ti;
        thr_of(0, tv, ti);
#pragma unroll
        for (int q = 1; q < NT; ++q) {
            float v;
            int id;
            thr_of(q, v, id);
            tv = i == q ? v : tv;
            ti = i == q ? id : ti;
        }
        unsigned long long pass = __ballot(mine && better(z, rid, tv, ti));
        while (pass) {                                 // wave-uniform
            const int src = __ffsll(pass) - 1;
            pass &= pass - 1ull;
            const int ts = __builtin_amdgcn_readlane(t, src);
            lds_list_insert(out.lists + ts * p.k, p.k, lane,
                            __int_as_float(__builtin_amdgcn_readlane(__float_as_int(z), src)),
                            __builtin_amdgcn_readlane(rid, src), out.thr_v, out.thr_i, ts);
        }
    }
    if (LP) {                                          // the pass's pieces, one per token
        const float zv = row < n_rows ? z : -INFINITY;
        float m = zv;
        if (ROWS >= 2) m = lane_xor_max<32>(m);
        if (ROWS >= 4) m = lane_xor_max<16>(m);
        if (ROWS >= 8) m = lane_xor_max<8>(m);
        float s = m > -INFINITY ? expf(zv - m) : 0.f;
        if (ROWS >= 2) s = lane_xor_sum<32>(s);
        if (ROWS >= 4) s = lane_xor_sum<16>(s);
        if (ROWS >= 8) s = lane_xor_sum<8>(s);
        if (first && row == 0) {
            const int at = (slot + i) * out.pieces_stride + out.pieces_at;
            if (out.pieces_in_lds)                     // uniform
                out.lds_pieces[at] = pack_lse(m, s);
            else
                __hip_atomic_store(out.mem_pieces + at, pack_lse(m, s), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
        }
    }
    slot += NT;
}

template <int DT, bool DENSE, int GATE, bool ROUTED, bool LP, int SEGS>
__global__ __launch_bounds__(kFusedBlock) void k_fused(FusedParams p) {
    static_assert(!(LP && DENSE), "the log-probability mode belongs to the grouped head");
    constexpr int ROWS = fused_rows(SEGS);
    extern __shared__ uint4 smem[];
    char* lds = reinterpret_cast<char*>(smem);
    const int lds_gate = GATE != kGateShared ? GATE : DT == kF32 || p.M <= 3 ? kGateVector : kGateMfma;
    const FusedLds lay = fused_lds_layout(p.M, p.G, p.g, p.k, p.jp, DENSE, lds_gate, LP, p.cap);
    uint4* hs = reinterpret_cast<uint4*>(lds + lay.o_hidden);
    Cand* lists = reinterpret_cast<Cand*>(lds + lay.o_lists);
    float* s_lds = reinterpret_cast<float*>(lds + lay.o_s);
    unsigned long long* mask_lds = reinterpret_cast<unsigned long long*>(lds + lay.o_mask);
    int* ugroup = reinterpret_cast<int*>(lds + lay.o_ugroup);
    int* ustart = reinterpret_cast<int*>(lds + lay.o_ustart);
    int* uend = reinterpret_cast<int*>(lds + lay.o_uend);
    int* uprefix = reinterpret_cast<int*>(lds + lay.o_uprefix);
    unsigned long long* umask = reinterpret_cast<unsigned long long*>(lds + lay.o_umask);
    int* flags = reinterpret_cast<int*>(lds + lay.o_flags);
    int* collect_count = reinterpret_cast<int*>(lds + lay.o_count);                  // [M], collected candidates only
    unsigned long long* collect_keys = reinterpret_cast<unsigned long long*>(lds + lay.o_lists);   // [M][cap]
    int* off_lds = reinterpret_cast<int*>(lds + lay.o_offsets);
    float* bias_lds = reinterpret_cast<float*>(lds + lay.o_bias);
    int* sel_lds = reinterpret_cast<int*>(lds + lay.o_sel);          // LP: [M, g] selections
    int* wgstart = reinterpret_cast<int*>(lds + lay.o_wgstart);      // LP: first workgroup of a group

    const int lane = threadIdx.x & (kWave - 1);
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x / kWave);
    const int hs_stride = hidden_lds_stride(p.jp);
    const int M = p.M, k = p.k;

    // batch counter, see step 3: a wave's first batch is fixed (i = wave), the others are drawn
    if (threadIdx.x == 0) {
        flags[2] = LP ? 0 : p.stream_waves;
        flags[3] = 0;                                  // shared gate: whether a score did not come in time
    }
    if ((LP || p.cap) && (int)threadIdx.x < p.M) collect_count[threadIdx.x] = 0;     // (seen by all after the gate's barriers)
    // ---- 1. hidden vectors: requested first, written to LDS only after the grouped
    // variants have requested their first gate rows as well (loads return in order, so the
    // wait for the hidden vectors does not wait for the gate rows behind them)
    constexpr int kHU = 4;
    const int row_vecs = p.jp * kWave;                     // <= 1024: at least one row a pass
    int h_mm = threadIdx.x / row_vecs;
    int h_vec = threadIdx.x - h_mm * row_vecs;
    const int rows_per_pass = kFusedBlock / row_vecs;
    uint4 htmp[kHU];
    // The router may see another vector than the LM head (Eq. 7: W2 is applied to
    // act(W1 h) + h): then the gate's vectors are staged first and the LM head's replace
    // them after the gate, their loads in flight during the selection (ROUTED, compiled
    // apart: the kernel has no registers to spare).
    const uint4* h_src = ROUTED ? p.gate_hidden : p.hidden;
    auto hidden_request = [&](int m0) {
#pragma unroll
        for (int u = 0; u < kHU; ++u) {
            const int m = m0 + u * rows_per_pass + h_mm;
            htmp[u] = make_uint4(0, 0, 0, 0);
            if (h_mm < rows_per_pass && m < M && h_vec < p.n_vec)
                htmp[u] = h_src[(size_t)m * p.n_vec + h_vec];
        }
    };
    auto hidden_commit = [&](int m0) {                     // then the passes that remain
#pragma unroll
        for (int u = 0; u < kHU; ++u) {
            const int m = m0 + u * rows_per_pass + h_mm;
            if (h_mm < rows_per_pass && m < M) hs[m * hs_stride + h_vec] = htmp[u];
        }
    };
    auto hidden_rest = [&]() {
        for (int m0 = rows_per_pass * kHU; m0 < M; m0 += rows_per_pass * kHU) {
            hidden_request(m0);
            hidden_commit(m0);
        }
    };
    hidden_request(0);
    // group offsets and bias travel with them (G <= 1024 = the workgroup's size), so that
    // no later step waits for memory
    int off_r0 = 0, off_r1 = 0;
    float bias_r = 0.f;
    if (!DENSE) {
        if ((int)threadIdx.x <= p.G) off_r0 = p.offsets[threadIdx.x];
        if ((int)threadIdx.x + kFusedBlock <= p.G) off_r1 = p.offsets[threadIdx.x + kFusedBlock];
        if ((int)threadIdx.x < p.G && p.bias) bias_r = p.bias[threadIdx.x];
    }
    auto small_commit = [&]() {
        if ((int)threadIdx.x <= p.G) off_lds[threadIdx.x] = off_r0;
        if ((int)threadIdx.x + kFusedBlock <= p.G) off_lds[threadIdx.x + kFusedBlock] = off_r1;
        if ((int)threadIdx.x < p.G) bias_lds[threadIdx.x] = bias_r;
    };
    Cand* my_lists = lists + (size_t)wave * M * k;

    int total_batches;
    if (DENSE) {
        hidden_commit(0);
        hidden_rest();
        total_batches = (p.V + ROWS - 1) / ROWS;
        __syncthreads();
    } else {
        for (int n = threadIdx.x; n < p.G; n += kFusedBlock) mask_lds[n] = 0ull;
        if (GATE == kGateShared) {
            // ---- 2a. every workgroup computes the scores of its share of the groups (blockIdx, blockIdx +
            // #workgroups, ...; one wave a (group, token) pair at a time, the row's first request in flight
            // with the hidden vectors), publishes them and reads everyone's.  A word is its own flag: it is
            // zero between calls, and a score of +0 is published as -0.  They are read with
            // 16-byte loads past the caches, a wave's 256 words in one request; four scores of one group
            // are neighbours, so that a workgroup's stores touch one line: with a word per
            // load and stores scattered over the lines of all groups the hand-over took 4 us longer
            // than with these (256 workgroups ask for the same lines while the stores are on their way).
            // Bounded: the workgroups before this one may not be running yet where other kernels
            // hold the compute units.  After as many requests as the control word says, the workgroups that
            // run compute what is still missing between them: a wave a group with all its tokens at a time,
            // each workgroup's from another place on, published like a share, and what others have
            // published read in between.  Any workgroup gets to the end of that by itself.  A score has the
            // same bits wherever it is computed.
            uint4 ga[SEGS];
            auto load_gate_row = [&](int n) {
                int left = p.n_vec - lane;
                asm volatile("" : "+v"(left));
#pragma unroll
                for (int j = 0; j < SEGS; ++j) {
                    ga[j] = make_uint4(0, 0, 0, 0);
                    if (j * kWave < left) ga[j] = p.gate_W[(size_t)n * p.n_vec + j * kWave + lane];
                }
            };
            auto score = [&](int n, int m) {
                float s = 0.f;
#pragma unroll
                for (int j = 0; j < SEGS; ++j)
                    if (j < p.jp) s = dot_vec<DT>(ga[j], hs[m * hs_stride + j * kWave + lane], s);
                s = wave_sum(s) + bias_lds[n];
                if (lane == 0) s_lds[m * p.G + n] = s == 0.f ? -0.f : s;
            };
            int polls_at = kGatePollsAt;
            asm volatile("" : "+v"(polls_at));         // (a vector load: a scalar one holds up the gate rows' addresses)
            const unsigned polls_r = p.counter[polls_at];
            const int first_n = blockIdx.x, step_n = gridDim.x;
            const int pairs = first_n < p.G ? ((p.G - 1 - first_n) / step_n + 1) * M : 0;
            if (wave < pairs) load_gate_row(first_n + wave / M * step_n);
            const int n_words = M * p.G;
            for (int e = threadIdx.x; e < n_words; e += kFusedBlock) s_lds[e] = 0.f;       // (+0: missing)
            hidden_commit(0);
            small_commit();
            hidden_rest();
            __syncthreads();
            const int polls = (int)min((unsigned)uni((int)polls_r), (unsigned)kGatePollsMax);
            unsigned* words = p.counter + kGateScoresAt;       // [G][M]
            auto publish = [&](int n, int m, float s) {
                __hip_atomic_store(words + n * M + m, __float_as_uint(s), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            };
            // this wave's words, asked for up to `times` times; whether all are there
            auto read_scores = [&](int times) {
                const auto rsrc = __builtin_amdgcn_make_buffer_rsrc(words, 0, n_words * (int)sizeof(unsigned), 0x00027000);
                int ln = lane;
                asm volatile("" : "+v"(ln));
                const int e0 = (wave * kWave + ln) * 4;
                u32x4_t v = {0u, 0u, 0u, 0u};
                bool all = false;
                for (int i = 0; i < times; ++i) {
                    v = __builtin_amdgcn_raw_buffer_load_b128(rsrc, e0 * (int)sizeof(unsigned), 0, 16 /* sc1: from memory */);
                    asm volatile("" ::: "memory");     // (the request is made again)
                    all = true;
#pragma unroll
                    for (int c = 0; c < 4; ++c) all = all && (e0 + c >= n_words || v[c] != 0u);
                    if (__ballot(!all) == 0ull) break;
                    __builtin_amdgcn_s_sleep(2);
                }
#pragma unroll
                for (int c = 0; c < 4; ++c) {
                    const int e = e0 + c, n = e / M;
                    if (e < n_words && v[c] != 0u) s_lds[(e - n * M) * p.G + n] = __uint_as_float(v[c]);
                }
                return all;
            };
            const bool reads = polls > 0 && wave * 4 * kWave < n_words;        // wave-uniform
            for (int q = wave; q < pairs; q += kFusedWaves) {  // wave-uniform
                const int i = q / M, n = first_n + i * step_n;
                if (q != wave) load_gate_row(n);
                score(n, q - i * M);
            }
            __syncthreads();
            if (wave == 0)                             // (one wave: gate_through waits for its stores)
                for (int q = lane; q < pairs; q += kWave) {
                    const int i = q / M, m = q - i * M, n = first_n + i * step_n;
                    publish(n, m, s_lds[m * p.G + n]);
                }
            if (polls == 0 || (reads && !read_scores(polls))) flags[3] = 1;
            __syncthreads();
            if (uni(flags[3])) {                       // block-uniform
                if (threadIdx.x == 0)
                    __hip_atomic_fetch_add(p.counter + kGateGaveUpAt, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
                auto missing = [&](int base) {         // of the 64 groups from base on
                    const int n = base + lane;
                    bool out = false;
                    if (n < p.G)
                        for (int m = 0; m < M; ++m) out = out || __float_as_uint(s_lds[m * p.G + n]) == 0u;
                    return __ballot(out);
                };
                for (;;) {
                    int total = 0;
                    for (int base = 0; base < p.G; base += kWave) total += __popcll(missing(base));
                    int rank = (int)(blockIdx.x * kFusedWaves + wave) % max(total, 1), mine = -1;
                    if (wave < total)
                        for (int base = 0; mine < 0; base += kWave) {
                            const unsigned long long b = missing(base);
                            const unsigned long long before = b & ((1ull << lane) - 1ull);
                            const unsigned long long at = __ballot((b >> lane & 1ull) && __popcll(before) == rank);
                            if (at) mine = base + __ffsll(at) - 1;
                            rank -= __popcll(b);
                        }
                    __syncthreads();                   // (nobody writes a score before all have looked)
                    if (total == 0) break;             // block-uniform
                    const bool shares = polls > 0 && total > kGateAloneGroups;
                    if (mine >= 0) {
                        load_gate_row(mine);
#pragma unroll 1
                        for (int m = 0; m < M; ++m) score(mine, m);
                        if (shares) {                  // (the wave's own LDS words: in order)
                            if (lane < M) publish(mine, lane, s_lds[lane * p.G + mine]);
                            __builtin_amdgcn_s_waitcnt(0x0F70);    // vmcnt(0), for gate_through
                        }
                    }
                    if (shares && reads) read_scores(1);
                    __syncthreads();
                }
            }
        } else if (GATE == kGateMfma) {
            // ---- 2a. gate on the matrix cores: s[16 groups x 16 tokens] tiles, the H
            // columns split over the 16 waves in steps of 32 (v_mfma_f32_16x16x32_bf16:
            // lane l feeds row l%16, columns 8*(l/16)..+8 of both operands and receives
            // rows 4*(l/16)..+4, column l%16 of the tile); the waves' partial tiles are
            // summed in wave order.
            const int r16 = lane & 15, q4 = lane >> 4;
            const int n_gt = (p.G + 15) / 16, n_tt = (M + 15) / 16;
            constexpr int kSlice = kGateTileFloats;
            float* gpart = reinterpret_cast<float*>(lds + lay.o_lists);   // [wave][n_tt][kSlice]
            // waves 0-7 work on the even tile of a pair of group tiles, waves 8-15 on the odd
            // one; wave kw of either half takes the 256-byte blocks kw, kw + 8, kw + 16, ... of
            // the gate rows, at most four of them in one pass (rows of more than 8 KB take four
            // passes of two; they come with 16 tokens at most).  A block is four wave loads of
            // four rows x 256 contiguous bytes, transposed in registers to the operands of four
            // 32-column steps (mfma_operands_from_quad_rows in device_utils.h): register
            // 4 B + c then feeds rows 0..15, 16-byte chunks {c, 4 + c, 8 + c, 12 + c} of block
            // 8 B + kw, and the hidden vectors are read from LDS with the same choice.
            const int half = wave >> 3, kw = wave & 7;
            constexpr int kPasses = SEGS > 8 ? SEGS / 4 : 1;   // (two passes of four blocks run out of registers)
            constexpr int kSteps = 2 * SEGS / kPasses;
            uint4 ga[kSteps];
            // (every workgroup sums the columns in the same order: the scores, and with them
            // the selection, must come out bit-identical in all of them)
            auto load_gate_tile = [&](int gt, int pass) {
                int n_vec = p.n_vec;                           // (opaque: the lane masks are not kept for later)
                asm volatile("" : "+s"(n_vec));
#pragma unroll
                for (int i = 0; i < kSteps; ++i) {
                    const int n = gt * 16 + ((lane >> 2) & 3) * 4 + (i & 3);
                    const int vec = ((pass * (kSteps / 4) + (i >> 2)) * 8 + kw) * 16 + q4 * 4 + (lane & 3);
                    ga[i] = make_uint4(0, 0, 0, 0);
                    if (vec < n_vec && n < p.G) ga[i] = p.gate_W[(size_t)n * p.n_vec + vec];
                }
            };
            auto to_operand_layout = [&]() {
#pragma unroll
                for (int i = 0; i < kSteps; i += 4)
                    mfma_operands_from_quad_rows(ga[i], ga[i + 1], ga[i + 2], ga[i + 3], lane);
            };
            load_gate_tile(half, 0);
            hidden_commit(0);
            small_commit();
            hidden_rest();
            // The first tile's rows are transposed before the barrier, while the workgroup
            // waits for its last wave's hidden vectors (1.6 us at 8 tokens).
            to_operand_layout();
            __syncthreads();
            for (int pair = 0; pair * 2 < n_gt; ++pair) {
                if (pair) {
                    load_gate_tile(pair * 2 + half, 0);
                    to_operand_layout();
                }
                auto multiply = [&](f32x4_t acc, int tt, int pass) {
                    const int m = tt * 16 + r16;
                    const int mc = m < M ? m : M - 1;          // clamped: the load is unconditional
                    int n_vec = p.n_vec;
                    asm volatile("" : "+s"(n_vec));
#pragma unroll
                    for (int i0 = 0; i0 < kSteps; i0 += 2) {
                        uint4 hb[2];
#pragma unroll
                        for (int u = 0; u < 2; ++u) {
                            const int vec = ((pass * (kSteps / 4) + ((i0 + u) >> 2)) * 8 + kw) * 16 + q4 * 4 + ((i0 + u) & 3);
                            const bool in = vec < n_vec;
                            hb[u] = hs[mc * hs_stride + (in ? vec : 0)];
                            if (m >= M || !in) hb[u] = make_uint4(0, 0, 0, 0);
                        }
#pragma unroll
                        for (int u = 0; u < 2; ++u)
                            acc = mfma_tile<DT>(ga[i0 + u], hb[u], acc);
                    }
                    return acc;
                };
                if (kPasses == 1) {
                    for (int tt = 0; tt < n_tt; ++tt)          // uniform
                        *reinterpret_cast<f32x4_t*>(gpart + ((size_t)wave * n_tt + tt) * kSlice + lane * 4) =
                            multiply(f32x4_t{0.f, 0.f, 0.f, 0.f}, tt, 0);
                } else {                                       // one token tile
                    f32x4_t acc = multiply(f32x4_t{0.f, 0.f, 0.f, 0.f}, 0, 0);
#pragma unroll 1
                    for (int pass = 1; pass < kPasses; ++pass) {
                        load_gate_tile(pair * 2 + half, pass);
                        to_operand_layout();
                        acc = multiply(acc, 0, pass);
                    }
                    *reinterpret_cast<f32x4_t*>(gpart + (size_t)wave * kSlice + lane * 4) = acc;
                }
                __syncthreads();
                for (int idx = threadIdx.x; idx < 2 * n_tt * 256; idx += kFusedBlock) {
                    const int hh = idx / (n_tt * 256);
                    const int rest = idx - hh * n_tt * 256;
                    const int tt = rest >> 8, e = rest & 255;
                    const int l = e >> 2, i = e & 3;
                    const int n = (pair * 2 + hh) * 16 + (l >> 4) * 4 + i;
                    const int m = tt * 16 + (l & 15);
                    float sum = 0.f;
                    for (int w = hh * 8; w < hh * 8 + 8; ++w)
                        sum += gpart[((size_t)w * n_tt + tt) * kSlice + e];
                    if (n < p.G && m < M) s_lds[m * p.G + n] = sum + bias_lds[n];
                }
                __syncthreads();
            }
        } else {
            // ---- 2a. gate on the vector units (fp32 storage, or few tokens): each wave takes
            // rows n0 and n0 + 16 per pass (one row where it fills the registers)
            constexpr bool kTwo = SEGS <= 8;
            constexpr int kGateStep = (kTwo ? 2 : 1) * kFusedWaves;
            uint4 ga[SEGS], gb[kTwo ? SEGS : 1];
            auto load_gate_rows = [&](int n0) {
                const int n1 = n0 + kFusedWaves;
                int left = p.n_vec - lane;
                asm volatile("" : "+v"(left));
#pragma unroll
                for (int j = 0; j < SEGS; ++j) {
                    const int vec = j * kWave + lane;
                    ga[j] = make_uint4(0, 0, 0, 0);
                    if (kTwo) gb[kTwo ? j : 0] = make_uint4(0, 0, 0, 0);
                    if (j * kWave < left) {
                        if (n0 < p.G) ga[j] = p.gate_W[(size_t)n0 * p.n_vec + vec];
                        if (kTwo && n1 < p.G) gb[kTwo ? j : 0] = p.gate_W[(size_t)n1 * p.n_vec + vec];
                    }
                }
            };
            load_gate_rows(wave);
            hidden_commit(0);
            small_commit();
            hidden_rest();
            __syncthreads();
            for (int n0 = wave; n0 < p.G; n0 += kGateStep) {
                if (n0 != wave) load_gate_rows(n0);
                const int n1 = kTwo ? n0 + kFusedWaves : p.G;      // (p.G: none)
#pragma unroll 1
                for (int m = 0; m + 1 < M; m += 2) {           // two tokens per pass
                    const int m1 = m + 1;
                    float a0 = 0.f, b0 = 0.f, a1 = 0.f, b1 = 0.f;
#pragma unroll
                    for (int j = 0; j < SEGS; ++j)
                        if (j < p.jp) {
                            const uint4 h0 = hs[m * hs_stride + j * kWave + lane];
                            const uint4 h1 = hs[m1 * hs_stride + j * kWave + lane];
                            a0 = dot_vec<DT>(ga[j], h0, a0);
                            if (kTwo) b0 = dot_vec<DT>(gb[kTwo ? j : 0], h0, b0);
                            a1 = dot_vec<DT>(ga[j], h1, a1);
                            if (kTwo) b1 = dot_vec<DT>(gb[kTwo ? j : 0], h1, b1);
                        }
                    a0 = wave_sum(a0);
                    if (kTwo) b0 = wave_sum(b0);
                    a1 = wave_sum(a1);
                    if (kTwo) b1 = wave_sum(b1);
                    if (lane == 0) {
                        const float bias0 = bias_lds[n0];
                        const float bias1 = n1 < p.G ? bias_lds[n1] : 0.f;
                        s_lds[m * p.G + n0] = a0 + bias0;
                        s_lds[m1 * p.G + n0] = a1 + bias0;
                        if (n1 < p.G) {
                            s_lds[m * p.G + n1] = b0 + bias1;
                            s_lds[m1 * p.G + n1] = b1 + bias1;
                        }
                    }
                }
                if (M & 1) {                                   // the last of an odd number of tokens
                    const int m = M - 1;                       // (the dot instructions bound this step)
                    float a0 = 0.f, b0 = 0.f;
#pragma unroll
                    for (int j = 0; j < SEGS; ++j)
                        if (j < p.jp) {
                            const uint4 h0 = hs[m * hs_stride + j * kWave + lane];
                            a0 = dot_vec<DT>(ga[j], h0, a0);
                            if (kTwo) b0 = dot_vec<DT>(gb[kTwo ? j : 0], h0, b0);
                        }
                    a0 = wave_sum(a0);
                    if (kTwo) b0 = wave_sum(b0);
                    if (lane == 0) {
                        s_lds[m * p.G + n0] = a0 + bias_lds[n0];
                        if (n1 < p.G) s_lds[m * p.G + n1] = b0 + bias_lds[n1];
                    }
                }
            }
            __syncthreads();
        }
        if (ROUTED) {                                  // the gate's last read of hs is behind a barrier
            h_src = p.hidden;
            // (recomputed behind a compiler barrier: the first staging's addresses would
            // otherwise be kept through the gate, where there are no registers to spare)
            int tid = threadIdx.x;
            asm volatile("" : "+v"(tid));
            h_mm = tid / row_vecs;
            h_vec = tid - h_mm * row_vecs;
            hidden_request(0);
        }
        // Log-probability mode: every workgroup streams rows of one group only (it keeps one
        // list and one log-sum-exp state per token, Eq. 8 normalises per group), so the
        // workgroups are shared out among the count <= 64 activated groups in proportion to
        // their cost, batches x lp_batch_cost(tokens that selected the group): one each,
        // the rest by the groups' shares rounded down, what is then left one more each to the
        // groups with the highest cost per workgroup.  The numbers add up to n_share: gridDim.x, or
        // fewer where there are few batches (the workgroups behind leave before the stream: P_act).
        // One wave's work (activated group u in lane u), after it has written the tables of 2c.
        auto share_out_workgroups = [&](int count, int all_pairs) {
            const int n_share = min((int)gridDim.x, max(count, (all_pairs + kLpFewBatches - 1) / kLpFewBatches));
            const int nb_u = lane < count ? uprefix[lane + 1] - uprefix[lane] : 0;
            // (batches scaled to 16 bits so that the products below stay in 31)
            const int shift = max(0, 16 - __clz(all_pairs));
            const unsigned cost =
                lane < count ? (unsigned)(nb_u >> shift) *
                                   (unsigned)lp_batch_cost<DT, SEGS>(__popcll(umask[lane]), M * p.g, count) : 0u;
            const unsigned total = (unsigned)__builtin_amdgcn_readlane(wave_scan_inclusive((int)cost), 63);
            // (the reciprocal rounded down, so that the shares never add up to more than there are)
            const float scale = (float)(n_share - count) * __builtin_amdgcn_rcpf((float)(total ? total : 1u)) * (1.f - 0x1p-20f);
            int n_wg = lane < count ? 1 + (int)((float)cost * scale) : 0;
            const int left = n_share - __builtin_amdgcn_readlane(wave_scan_inclusive(n_wg), 63);
            if (left > 0) {                            // wave-uniform
                unsigned long long* rank_keys =
                    reinterpret_cast<unsigned long long*>(lds + lay.o_keys) + (size_t)wave * kWave;
                const int rank = wave_rank(rank_keys, (float)cost * __builtin_amdgcn_rcpf((float)n_wg), lane, count, lane);
                if (lane < count && rank < left) ++n_wg;
            }
            const int incl_wg = wave_scan_inclusive(n_wg);
            if (lane < count) wgstart[lane] = incl_wg - n_wg;
            if (lane == 0) wgstart[count] = n_share;
        };
        // ---- 2b. per-token top-g by rank counting: group n of token m is selected iff
        // fewer than g groups beat it (larger score first, then lower group id); its rank
        // is its position in the selection
        if (p.G <= kWave) {
            // group n in lane n.  gm: the tokens that selected this lane's group.
            unsigned long long gm = 0ull;
            unsigned long long* sel_keys =
                reinterpret_cast<unsigned long long*>(lds + lay.o_keys) + (size_t)wave * kWave;
            for (int m = wave; m < M; m += kFusedWaves) {  // one wave per token
                float v = lane < p.G ? s_lds[m * p.G + lane] : -INFINITY;
                if (!(v == v)) v = -INFINITY;              // NaN: unspecified, but keep a total order
                const int rank = wave_rank(sel_keys, v, lane, p.G, lane);
                if (lane < p.G && rank < p.g) {
                    atomicOr(&mask_lds[lane], 1ull << m);
                    if (p.sel_out && blockIdx.x == 0) p.sel_out[m * p.g + rank] = lane;
                    if (LP) sel_lds[m * p.g + rank] = lane;
                }
            }
            __syncthreads();
            if (lane < p.G) gm = mask_lds[lane];
            // ---- 2c. activated groups in ascending id order, their row ranges and the row
            // pairs before each.  Every wave builds the same tables and writes them to the
            // same LDS words (equal values), then reads back only what it wrote itself: no
            // barrier, no wave waits for another.
            const unsigned long long act = __ballot(gm != 0ull);
            const int count = __popcll(act);
            const int at = __popcll(act & ((1ull << lane) - 1ull));
            int lo = 0, hi = 0;
            if (gm != 0ull) {
                lo = off_lds[lane];
                hi = off_lds[lane + 1];
            }
            const int nb = (hi - lo + ROWS - 1) / ROWS;       // 0 for the others
            const int incl = wave_scan_inclusive(nb);
            if (gm != 0ull) {
                ugroup[at] = lane;
                umask[at] = gm;
                ustart[at] = lo;
                uend[at] = hi;
                uprefix[at] = incl - nb;
            }
            const int all_pairs = __builtin_amdgcn_readlane(incl, 63);
            if (lane == 0) {
                uprefix[count] = all_pairs;
                flags[0] = count;
            }
            if (LP) share_out_workgroups(count, all_pairs);
            if (ROUTED) {
                hidden_commit(0);
                hidden_rest();
                __syncthreads();
            }
            total_batches = all_pairs;
        } else {
            // more groups than lanes: one wave per token, up to 16 scores per lane; the g best
            // are cut out by bisection (wave_bound) and ranked among themselves.  (A count over
            // all pairs of groups by the whole workgroup took 23 us at 9 tokens and 100 groups.)
            auto select_token = [&](auto regs, int m) {
                constexpr int N = decltype(regs)::value;
                unsigned long long key[N];
#pragma unroll
                for (int i = 0; i < N; ++i) {
                    const int n = i * kWave + lane;
                    float v = n < p.G ? s_lds[m * p.G + n] : -INFINITY;
                    if (!(v == v)) v = -INFINITY;
                    key[i] = n < p.G ? cand_key(v, n) : 0ull;
                }
                auto chosen = [&](int rank, int n) {
                    atomicOr(&mask_lds[n], 1ull << m);
                    if (p.sel_out && blockIdx.x == 0) p.sel_out[m * p.g + rank] = n;
                    if (LP) sel_lds[m * p.g + rank] = n;
                };
                if (p.g <= kWave) {                        // uniform
                    wave_topk<N>(key, p.g, lane, reinterpret_cast<unsigned long long*>(lds + lay.o_keys) + (size_t)wave * kWave,
                                 [&](int rank, unsigned long long kk) { chosen(rank, key_id(kk)); });
                } else {
#pragma unroll
                    for (int i = 0; i < N; ++i) {
                        int rank = 0;
                        for (int o = 0; o < p.G; ++o) {
                            float ov = s_lds[m * p.G + o];
                            if (!(ov == ov)) ov = -INFINITY;
                            rank += cand_key(ov, o) > key[i] ? 1 : 0;
                        }
                        if (key[i] != 0ull && rank < p.g) chosen(rank, i * kWave + lane);
                    }
                }
            };
            for (int m = wave; m < M; m += kFusedWaves) {
                if (p.G <= 2 * kWave) select_token(std::integral_constant<int, 2>(), m);       // uniform
                else if (p.G <= 4 * kWave) select_token(std::integral_constant<int, 4>(), m);
                else select_token(std::integral_constant<int, 16>(), m);
            }
            __syncthreads();
            if (wave == 0) {
                int count = 0;
                for (int base = 0; base < p.G; base += kWave) {
                    const int n = base + lane;
                    const unsigned long long gm = n < p.G ? mask_lds[n] : 0ull;
                    const unsigned long long b = __ballot(gm != 0ull);
                    if (gm != 0ull) {
                        const int u = count + __popcll(b & ((1ull << lane) - 1ull));
                        ugroup[u] = n;
                        umask[u] = gm;
                        ustart[u] = off_lds[n];
                        uend[u] = off_lds[n + 1];
                    }
                    count += __popcll(b);
                }
                int carry = 0;                             // batches before each activated group
                for (int base = 0; base < count; base += kWave) {
                    const int u = base + lane;
                    const int nb = u < count ? (uend[u] - ustart[u] + ROWS - 1) / ROWS : 0;
                    const int incl = wave_scan_inclusive(nb);
                    if (u < count) uprefix[u] = carry + incl - nb;
                    carry += __builtin_amdgcn_readlane(incl, 63);
                }
                if (lane == 0) {
                    uprefix[count] = carry;
                    flags[0] = count;
                }
                if (LP) share_out_workgroups(count, carry);
            }
            if (ROUTED) {
                hidden_commit(0);
                hidden_rest();
            }
            __syncthreads();
            total_batches = uni(uprefix[uni(flags[0])]);
        }
    }

    // ---- 3./4. stream batches of ROWS rows (the lists share LDS with the gate's partial tiles,
    // so they are emptied only now; each wave touches its own lists only)
    BatchSink out;
    out.lists = my_lists;
    out.keys = collect_keys;
    out.count = collect_count;
    out.cap = p.cap;
    out.lds_pieces = reinterpret_cast<unsigned long long*>(lds + lay.o_pieces);
    out.mem_pieces = p.pair_lse;
    out.pieces_stride = out.pieces_at = 0;
    out.pieces_in_lds = false;
    out.thr_v = -INFINITY;
    out.thr_i = INT_MAX;
    // The workgroup's batches are b(i) = (i / D) * D * #workgroups + D * blockIdx + i % D for
    // i = 0, 1, ...; its waves draw i from an LDS counter, so a wave that the memory system
    // serves faster takes more of them and all waves finish together.  D = 1 shares the
    // batches out evenly, D = 8 keeps neighbouring rows in one workgroup.  Measured (us):
    // two rounds (Llama3 shape, M = 1) D = 8 33.0, D = 1 33.5; ten (M = 10) 131.0, 130.1; 15
    // (dense) 159.0, 156.4; a fifth of a round (1024-wide head, 8 tokens) D = 4 20.9, D = 8 22.4; a
    // tenth, one token 11.7, 11.3.  Few enough batches for all lists to be fetched in one trip with
    // D = 8 (256-wide head, 4 tokens): 14.3, 13.6; not quite (2 tokens, k = 20): 14.4, 14.7.  (Up to four
    // tokens: with more the fewer workgroups have too many products each.  Time with D = 8 over D = 4, 14 to 17
    // small heads each: 5 tokens 1.015, 6 1.03, 7 1.035, 8 1.015.)
    // (Log-probability mode: the workgroup's share is a contiguous range of one group's
    // batches instead, the j-th of the equal parts its group's workgroups cut the group into.)
    const int round = gridDim.x * kFusedWaves;
    const bool one_trip = M <= 4 && total_batches * k <= kDealFew * 8 * kWave;   // (see wave_merge_lists)
    const int deal = total_batches >= 4 * round || p.deal_single ? 0
                     : total_batches >= round || one_trip ? log2_small(kDealFew) : log2_small(kDealFew / 2);
    auto dealt = [&](int i) {
        return (int)(((i >> deal) * gridDim.x + blockIdx.x) << deal) + (i & ((1 << deal) - 1));
    };
    // Workgroups without a batch leave here; the last merge goes by the others' lists.
    const int P_act = LP ? uni(wgstart[uni(flags[0])]) : min((int)gridDim.x, (total_batches + (1 << deal) - 1) >> deal);
    // Shared gate: the workgroup has read the scores and its own are in memory; the last of all
    // workgroups that gets here, those without a batch among them, leaves the words at zero for the next call
    // (all that any call may use, where nobody has cleared them before).
    auto gate_through = [&]() {
        if (GATE != kGateShared || wave != 0) return;
        __builtin_amdgcn_s_waitcnt(0x0F70);            // vmcnt(0): this wave's stores are out
        int through = 0;
        if (lane == 0)
            through = (int)__hip_atomic_fetch_add(p.counter + kGateDoneAt, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        if (uni(through) != (int)gridDim.x - 1) return;
        int ln = lane;
        asm volatile("" : "+v"(ln));                   // (see wave_merge_lists)
        const bool first =
            uni((int)__hip_atomic_load(p.counter + kGatePollsAt, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT)) == 0;
        const int n_words = first ? coral_ctrl::kGateScoreWords : M * p.G;
        for (int e = ln; e < n_words; e += kWave)
            __hip_atomic_store(p.counter + kGateScoresAt + e, 0u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        if (lane == 0) {
            __hip_atomic_store(p.counter + kGateDoneAt, 0u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            if (first)
                __hip_atomic_store(p.counter + kGatePollsAt, (unsigned)kGatePollsMax, __ATOMIC_RELAXED,
                                   __HIP_MEMORY_SCOPE_AGENT);
        }
    };
    if ((int)blockIdx.x >= P_act) {                    // block-uniform
        gate_through();
        return;
    }
    int u = 0;
    int lp_lo = 0, lp_nwg = 0;
    // The (max, sum of exp) pieces are kept per batch and summed in batch order at the end: a
    // running state per wave would make the sum depend on which wave drew which batch, and the
    // result would not repeat bit for bit.
    int lp_stride = 0, lp_origin = 0;                  // piece of (token slot j, batch b): j * lp_stride + b - lp_origin
    if (LP) {
        const int count = uni(flags[0]);
        const int nxt = lane < count ? wgstart[lane + 1] : INT_MAX;
        u = __popcll(__ballot(nxt <= (int)blockIdx.x));    // wgstart[u] <= blockIdx.x < wgstart[u + 1]
        const int j = blockIdx.x - uni(wgstart[u]);
        lp_nwg = uni(wgstart[u + 1]) - uni(wgstart[u]);
        const int nb = uni(uprefix[u + 1]) - uni(uprefix[u]);
        const int per = (nb + lp_nwg - 1) / lp_nwg;
        lp_lo = uni(uprefix[u]) + min(j * per, nb);
        total_batches = uni(uprefix[u]) + min((j + 1) * per, nb);  // the end of this workgroup's range
        const int n_mine = total_batches - lp_lo;
        if (n_mine * ROWS > p.cap) out.cap = 0;        // too many rows to collect: lists, in the same place
        // The pieces stay in LDS if this workgroup's fit there; else they go through memory,
        // this group's behind those of the activated groups before it.
        if ((size_t)n_mine * __popcll(uni64(umask[u])) * sizeof(unsigned long long) <= (size_t)lay.pieces_bytes) {
            out.pieces_in_lds = true;
            lp_stride = n_mine;
            lp_origin = lp_lo;
        } else {
            const int before = lane < u ? (uprefix[lane + 1] - uprefix[lane]) * __popcll(umask[lane]) : 0;
            out.mem_pieces = p.pair_lse + (size_t)__builtin_amdgcn_readlane(wave_scan_inclusive(before), 63);
            lp_stride = nb;
            lp_origin = uni(uprefix[u]);
        }
        out.pieces_stride = lp_stride;
    }
    if (!out.cap)
        for (int i = lane; i < M * k; i += kWave) my_lists[i] = sentinel();
    auto draw_batch = [&]() {
        int i = 0;
        if (lane == 0) i = atomicAdd(&flags[2], 1);
        i = uni(i);
        return LP ? lp_lo + i : dealt(i);
    };
    const unsigned long long all_tokens = M >= 64 ? ~0ull : ((1ull << M) - 1ull);
    // The batch's row ids, each in its row's lanes (rows past the group's end repeat the last).
    const int my_row = batch_row<ROWS>(lane);
    auto describe = [&](int b, int& rid, int& n_rows, unsigned long long& bm) {
        if (DENSE) {
            n_rows = min(ROWS, p.V - b * ROWS);
            rid = b * ROWS + min(my_row, n_rows - 1);
            bm = all_tokens;
        } else {
            while (b >= uni(uprefix[u + 1])) ++u;      // b < total_batches = uprefix[count]
            const int r0 = uni(ustart[u]) + (b - uni(uprefix[u])) * ROWS;
            n_rows = min(ROWS, uni(uend[u]) - r0);
            rid = p.rows[r0 + min(my_row, n_rows - 1)];
            bm = uni64(umask[u]);
        }
    };
    // the first batch is fixed (i = wave), the others are drawn from the LDS counter
    // (With few tokens the dense head's consecutive rows stream fastest with 64 to 160 KB in
    // flight per compute unit rather than 256 KB: its waves beyond p.stream_waves sit out.)
    int b = LP ? draw_batch() : wave < p.stream_waves ? dealt(wave) : total_batches;
    int rid = 0, n_rows = 0;
    unsigned long long bm = 0ull;
    if (b < total_batches) describe(b, rid, n_rows, bm);
    while (b < total_batches) {                        // wave-uniform
        uint4 w[ROWS][SEGS];
        const uint4* row_ptr[ROWS];
        int left = p.n_vec - lane;                     // vectors of a row from this lane's first one on
        asm volatile("" : "+v"(left));                 // (else the segments' lane masks are kept across the whole kernel)
#pragma unroll
        for (int r = 0; r < ROWS; ++r)
            row_ptr[r] = p.lm_W + (size_t)__builtin_amdgcn_readlane(rid, batch_lane(r)) * p.n_vec;
#pragma unroll
        for (int j = 0; j < SEGS; ++j) {
            const int vec = j * kWave + lane;
#pragma unroll
            for (int r = 0; r < ROWS; ++r) w[r][j] = make_uint4(0, 0, 0, 0);
            if (j * kWave < left) {
#pragma unroll
                for (int r = 0; r < ROWS; ++r) w[r][j] = load_stream(row_ptr[r] + vec);
            }
        }
        const int nb = draw_batch();
        int nrid = 0, nn_rows = 0;
        unsigned long long nbm = 0ull;
        if (nb < total_batches) describe(nb, nrid, nn_rows, nbm);

        if (LP) out.pieces_at = b - lp_origin;
        unsigned long long rem = bm;
        int slot = 0;
        while (rem) {                                  // wave-uniform
            const int cnt = __popcll(rem);
            if (ROWS <= 4 && cnt >= 4)
                fused_tokens<DT, ROWS <= 4 ? 4 : 2, LP, SEGS>(p, hs, w, rem, slot, rid, n_rows, out);
            else if (cnt >= 2)
                fused_tokens<DT, 2, LP, SEGS>(p, hs, w, rem, slot, rid, n_rows, out);
            else
                fused_tokens<DT, 1, LP, SEGS>(p, hs, w, rem, slot, rid, n_rows, out);
        }
        b = nb;
        rid = nrid;
        n_rows = nn_rows;
        bm = nbm;
    }

    gate_through();
    // ---- 5. rank the workgroup's candidates, publish, last workgroup merges all
    // the hidden vectors are no longer needed: their LDS is the ranking scratch
    unsigned long long* rank_buf = reinterpret_cast<unsigned long long*>(lds + lay.o_hidden) + (size_t)wave * kWave;
    const int P = gridDim.x;
    // published lists are entry-major, part[(t*k + i)*P + workgroup]: the first entries of
    // all workgroups, which bound the result, are contiguous
    auto publish_token = [&](int t) {
        Cand* dst = p.part + (size_t)t * k * P + blockIdx.x;
        auto put = [&](int r, unsigned long long key) {
            const Cand c = key_cand(key);
            publish_cand(dst + (size_t)r * P, c.v, c.id);
        };
        if (out.cap) {                                 // uniform
            wave_topk_lds(collect_keys + (size_t)t * out.cap, min(uni(collect_count[t]), out.cap), k, lane, rank_buf, put);
        } else {                                       // the 16 waves' lists: at most 1024 entries
            auto rank_lists = [&](auto regs) {
                constexpr int N = decltype(regs)::value;
                const int inv_k = inv_small(k);
                int ln = lane;
                asm volatile("" : "+v"(ln));           // (see wave_merge_lists)
                unsigned long long key[N];
#pragma unroll
                for (int i = 0; i < N; ++i) {
                    const int e = i * kWave + ln;
                    const int l = div_small(e, inv_k);
                    key[i] = e < kFusedWaves * k ? real_key(lists[((size_t)l * M + t) * k + e - l * k]) : 0ull;
                }
                wave_topk<N>(key, k, ln, rank_buf, put);
            };
            if (k <= 16) rank_lists(std::integral_constant<int, 4>());
            else rank_lists(std::integral_constant<int, 16>());
        }
    };
    // Where two waves share a task (log-probability mode): wave i < 8 and this one.  The four SIMDs
    // have every fourth wave each, so the first waves spread over them, and so do the second ones.
    auto second_wave = [](int i) { return kFusedWaves / 2 + ((i + 2) & (kFusedWaves / 2 - 1)); };
    auto shared_task = [](int w) { return w < kFusedWaves / 2 ? w : (w - 2) & (kFusedWaves / 2 - 1); };
    auto publish_all = [&]() {                         // logit mode, every wave of the workgroup
        if (out.cap && out.cap <= 2 * kWave && M <= kFusedWaves / 2) {
            // Fewer tokens than waves and at most two candidates per lane: S waves share a token,
            // each counts over a slice of the keys how many are above its lanes' (the keys are
            // distinct) and the token's first wave adds the counts up.
            const int S = M <= 1 ? 16 : M <= 2 ? 8 : M <= 4 ? 4 : 2;
            unsigned short* partial = reinterpret_cast<unsigned short*>(lds + lay.o_hidden);   // [wave][2][64]
            const int t = wave / S, slice = wave % S;
            const unsigned long long* keys = collect_keys + (size_t)(t < M ? t : 0) * out.cap;
            const int n = t < M ? min(uni(collect_count[t]), out.cap) : 0;
            const unsigned long long c0 = lane < n ? keys[lane] : 0ull;
            const unsigned long long c1 = lane + kWave < n ? keys[lane + kWave] : 0ull;
            const int per = (n + S - 1) / S;
            const int j1 = min(n, (slice + 1) * per);
            int r0 = 0, r1 = 0;
            if (n <= kWave) {                              // wave-uniform
#pragma unroll 8
                for (int j = slice * per; j < j1; ++j) r0 += keys[j] > c0 ? 1 : 0;
            } else {
#pragma unroll 8
                for (int j = slice * per; j < j1; ++j) {
                    const unsigned long long o = keys[j];
                    r0 += o > c0 ? 1 : 0;
                    r1 += o > c1 ? 1 : 0;
                }
            }
            partial[wave * 2 * kWave + lane] = (unsigned short)r0;
            partial[wave * 2 * kWave + kWave + lane] = (unsigned short)r1;
            __syncthreads();
            if (t < M && slice == 0) {
                for (int q = 1; q < S; ++q) {
                    r0 += partial[(wave + q) * 2 * kWave + lane];
                    r1 += partial[(wave + q) * 2 * kWave + kWave + lane];
                }
                Cand* dst = p.part + (size_t)t * k * P + blockIdx.x;
                if (c0 != 0ull && r0 < k) publish_cand(dst + (size_t)r0 * P, key_value(c0), key_id(c0));
                if (c1 != 0ull && r1 < k) publish_cand(dst + (size_t)r1 * P, key_value(c1), key_id(c1));
                if (lane >= n && lane < k) publish_cand(dst + (size_t)lane * P, -INFINITY, INT_MAX);
            }
        } else {
            for (int t = wave; t < M; t += kFusedWaves) publish_token(t);
        }
    };
    if (LP) {
        __syncthreads();
        // the tokens of this workgroup's group only: their lists, ranked by logit (inside
        // a group that is the order of log p as well), and their log-sum-exp pieces.  Up to eight
        // tokens: two waves each, one for the list and one for the pieces (a wave alone on its SIMD
        // issues a dependent instruction every eight to ten cycles: one after the other 3.7 us
        // from the last row to the list in memory at the Llama3 shape).
        unsigned long long rem = uni64(umask[u]);
        const bool split = 2 * __popcll(rem) <= kFusedWaves;
        for (int idx = 0; rem; ++idx, rem &= rem - 1ull) {     // block-uniform
            const bool lists = (idx & (kFusedWaves - 1)) == wave;
            const bool pieces = split ? second_wave(idx) == wave : lists;
            if (!lists && !pieces) continue;           // wave-uniform
            const int t = __ffsll(rem) - 1;
            // the pieces of this workgroup's batches for token slot idx, summed in batch order;
            // the first 256 are requested before the ranking, which hides their latency
            const int q0 = idx * lp_stride + lp_lo - lp_origin + lane;
            const int q_end = idx * lp_stride + total_batches - lp_origin;
            auto piece_at = [&](int q) {
                return out.pieces_in_lds ? out.lds_pieces[q]
                                         : __hip_atomic_load(out.mem_pieces + q, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
            };
            unsigned long long early[4];
#pragma unroll
            for (int c = 0; c < 4; ++c) {
                early[c] = 0xff800000ull;              // (-inf, 0)
                if (pieces && q0 + c * kWave < q_end) early[c] = piece_at(q0 + c * kWave);
            }
            if (lists) publish_token(t);
            if (!pieces) continue;
            // (the maximum first, then every piece scaled to it: independent exponentials)
            float late_m = -INFINITY, late_s = 0.f;    // batches beyond the first 256, if any
            for (int q = q0 + 4 * kWave; q < q_end; q += kWave) lse_take(late_m, late_s, piece_at(q));
            float wm = late_m;
#pragma unroll
            for (int c = 0; c < 4; ++c) wm = fmaxf(wm, __uint_as_float((unsigned)(early[c] & 0xffffffffull)));
            wm = wave_max(wm);
            float mine_s = 0.f;
            if (wm > -INFINITY) {
#pragma unroll
                for (int c = 0; c < 4; ++c)            // ascending batch order
                    mine_s += __uint_as_float((unsigned)(early[c] >> 32)) *
                              expf(__uint_as_float((unsigned)(early[c] & 0xffffffffull)) - wm);
                mine_s += late_s * expf(late_m - wm);
            }
            const float tot = wave_sum(mine_s);
            if (lane == 0)
                __hip_atomic_store(p.lse_part + (size_t)t * P + blockIdx.x,
                                   pack_lse(wm, tot), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        }
    }
    // (what the merges overwrite, candidates and ranking scratch, is used up when they run)
    MergeScratch* ms = reinterpret_cast<MergeScratch*>(lds + lay.o_hidden) + wave;
    if (LP) {
        __builtin_amdgcn_s_waitcnt(0x0F70);            // vmcnt(0): the published lists are out
        __syncthreads();
        // Eq. 8: log p(x) = log p_router(n) + z[x] - lse_n.  finish(t, gu) is the work for token t and
        // its selected group ugroup[gu], of one wave or shared by two (lists: this
        // wave's part is to merge the group's published lists by logit; shifts: to combine the
        // log-sum-exp pieces of the group's workgroups and take the router's log-softmax over all
        // G scores).  Leaves the k best, offset added, in the lanes (lane r = rank r) of the wave
        // that merges.  With `split` it is called by every wave, `on` or not, up to the barrier.
        auto finish = [&](bool on, bool lists, bool shifts, bool split, int t, int gu) {
            const int n = uni(ugroup[gu]);
            const int w0 = uni(wgstart[gu]);
            const int n_wg = uni(wgstart[gu + 1]) - w0;
            float shift = 0.f;
            // the pieces are requested first and used after the merge, whose own loads
            // then share their trip to memory
            unsigned long long piece[4];
            if (on && shifts) {
#pragma unroll
                for (int c = 0; c < 4; ++c) {
                    const int l = c * kWave + lane;
                    piece[c] = 0xff800000ull;          // (-inf, 0)
                    if (l < n_wg)
                        piece[c] = __hip_atomic_load(p.lse_part + (size_t)t * P + w0 + l, __ATOMIC_RELAXED,
                                                     __HIP_MEMORY_SCOPE_AGENT);
                }
            }
            if (on && lists) {
                const Cand* src = p.part + (size_t)t * k * P + w0;
                wave_merge_lists(
                    n_wg, k, lane, ms, [&](int l, int e) { return fetch_cand(src + (size_t)e * P + l); },
                    [&](int r, unsigned long long key) { ms->out[r] = key_cand(key); });
            }
            if (on && shifts) {
                float rm = -INFINITY, rs = 0.f, s_n = 0.f;
                for (int o = lane; o < p.G; o += kWave) {
                    float v = s_lds[t * p.G + o];
                    if (!(v == v)) v = -INFINITY;
                    if (o == n) s_n = v;
                    const float nm = fmaxf(rm, v);
                    if (nm > -INFINITY) rs = rs * expf(rm - nm) + expf(v - nm);
                    rm = nm;
                }
                s_n = wave_sum(s_n);                   // one lane holds it, the others zero
                const float logp = s_n - lse_finish(rm, rs);
                float bm = -INFINITY, bs = 0.f;
#pragma unroll
                for (int c = 0; c < 4; ++c)            // ascending workgroup order
                    if (c * kWave < n_wg) lse_take(bm, bs, piece[c]);   // uniform
                shift = logp - lse_finish(bm, bs);
            }
            if (split) {                               // block-uniform
                if (on && shifts && lane == 0) ms->out[0].v = shift;
                __syncthreads();
                if (on && lists) shift = (ms - wave + second_wave(wave))->out[0].v;
            }
            Cand c = sentinel();
            if (on && lists && lane < k) c = ms->out[lane];
            if (is_real(c)) c.v += shift;
            return c;
        };
        // Draft-level call: the results also go to a table of tree keys in LDS (behind the merge
        // scratch), from which the level is expanded below.
        const bool expand = p.next_parent != nullptr;  // uniform
        unsigned long long* tree_keys = reinterpret_cast<unsigned long long*>(lds + lay.o_tree);   // [M * k]
        int* tree_ids = reinterpret_cast<int*>(tree_keys + M * k);
        float* tree_scores = reinterpret_cast<float*>(tree_ids + M * k);
        auto write_result = [&](int t, int r, Cand c) {
            p.topk_ids[(size_t)t * k + r] = c.id;
            p.topk_logits[(size_t)t * k + r] = c.v;
            if (expand) {
                const int e = t * k + r;
                const float parent = p.parent_score ? p.parent_score[t] : 0.f;
                tree_keys[e] = tree_key(parent, c.v, is_real(c) ? c.id : -1, e);
                tree_ids[e] = c.id;
                tree_scores[e] = parent + c.v;
            }
        };
        auto expand_level = [&]() {                    // called by every thread of the workgroup
            if (!expand) return;
            __syncthreads();
            if (p.n_next <= kWave && M * k <= 4 * kWave) {     // uniform
                if (wave != 0) return;
                int ln = lane;
                asm volatile("" : "+v"(ln));           // (see wave_merge_lists)
                tree_topk<4>(
                    M * k, p.n_next, ln, ms->keys, [&](int e) { return tree_keys[e]; },
                    [&](unsigned long long key, int) { return key; },
                    [&](int r, unsigned long long key) {
                        const int e = key != 0ull ? key_id(key) : 0;
                        p.next_parent[r] = key != 0ull ? div_small(e, inv_small(k)) : -1;
                        p.next_token[r] = key != 0ull ? tree_ids[e] : -1;
                        p.next_score[r] = key != 0ull ? tree_scores[e] : -INFINITY;
                    });
                return;
            }
            for (int m = wave; m < M; m += kFusedWaves) {
                int e;
                bool keep;
                const int rank = tree_rank_node(tree_keys, M, k, p.n_next, m, lane, e, keep);
                if (keep) {
                    p.next_parent[rank] = m;
                    p.next_token[rank] = tree_ids[e];
                    p.next_score[rank] = tree_scores[e];
                }
            }
            if (wave == 0) {
                int n_real = 0;
                for (int e = lane; e < M * k; e += kWave) n_real += tree_keys[e] != 0ull ? 1 : 0;
                n_real = wave_scan_inclusive(n_real);
                n_real = __builtin_amdgcn_readlane(n_real, 63);
                tree_pad(n_real, p.n_next, lane, p.next_parent, p.next_token, p.next_score);
            }
        };
        if (2 * M * p.g <= kFusedWaves) {
            // Few (token, group) pairs: the workgroup that arrives last takes them all, two
            // waves each, and merges every token's g lists through LDS (two hand-overs through
            // memory fewer than below; from about 16 pairs on the scheme below is faster).
            if (threadIdx.x == 0) {
                const unsigned int old = __hip_atomic_fetch_add(p.counter, 1u, __ATOMIC_RELAXED,
                                                                __HIP_MEMORY_SCOPE_AGENT);
                flags[1] = old == (unsigned)P_act - 1u ? 1 : 0;
            }
            __syncthreads();
            if (!uni(flags[1])) return;                // block-uniform
            const int count = uni(flags[0]);
            Cand* glists = reinterpret_cast<Cand*>(lds + lay.o_keys);   // [M * g, k], <= 16 x 64 entries
            {
                const int pair = shared_task(wave);    // two waves each
                const bool on = pair < M * p.g, lists = wave < kFusedWaves / 2;
                const int n = uni(sel_lds[on ? pair : 0]);
                const int gu = __ffsll(__ballot(lane < count && ugroup[lane] == n)) - 1;
                const Cand c = finish(on, lists, !lists, true, on ? pair / p.g : 0, gu);
                if (on && lists && lane < k) glists[pair * k + lane] = c;
            }
            __syncthreads();
            if (wave < M) {
                const Cand* src = glists + (size_t)wave * p.g * k;
                wave_merge_lists(
                    p.g, k, lane, ms, [&](int l, int e) { return src[l * k + e]; },
                    [&](int r, unsigned long long key) { write_result(wave, r, key_cand(key)); });
            }
            expand_level();
            if (threadIdx.x == 0)                      // ready for the next call
                __hip_atomic_store(p.counter, 0u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            return;
        }
        // More pairs than half of the waves: the workgroup of a group that arrives last (a counter per
        // activated group) finishes the group, two waves per token that selected it up to eight tokens,
        // one beyond, and
        // publishes the lists; the group that finishes last (one more counter) merges every
        // token's g lists.  The groups' last workgroups work side by side, most of them
        // while other groups still stream.
        unsigned int* group_counter = p.counter + kLpGroupCounters + u;
        if (threadIdx.x == 0) {
            const unsigned int old = __hip_atomic_fetch_add(group_counter, 1u, __ATOMIC_RELAXED,
                                                            __HIP_MEMORY_SCOPE_AGENT);
            flags[1] = old == (unsigned)lp_nwg - 1u ? 1 : 0;
        }
        __syncthreads();
        if (!uni(flags[1])) return;                    // block-uniform
        if (threadIdx.x == 0)                          // ready for the next call
            __hip_atomic_store(group_counter, 0u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        const int n = uni(ugroup[u]);
        unsigned long long rem = uni64(umask[u]);
        while (rem) {                                  // block-uniform: 8 tokens or up to 16 at a time
            const int todo = __popcll(rem);
            const bool split = 2 * todo <= kFusedWaves;
            const int mine = split ? shared_task(wave) : wave;
            const bool on = mine < todo;
            unsigned long long at = rem;               // this wave's token: the mine-th of those left
            for (int i = 0; i < kFusedWaves && i < todo; ++i) {
                if (on && i < mine) at &= at - 1ull;
                if (!split) rem &= rem - 1ull;
            }
            if (split) rem = 0ull;
            const int t = __ffsll(at) - 1;
            const bool lists = !split || wave < kFusedWaves / 2, shifts = !split || wave >= kFusedWaves / 2;
            const int i = __ffsll(__ballot(lane < p.g && sel_lds[t * p.g + lane] == n)) - 1;
            const Cand c = finish(on, lists, shifts, split, t, u);
            if (on && lists && lane < k) publish_cand(p.glist + ((size_t)t * p.g + i) * k + lane, c.v, c.id);
        }
        __builtin_amdgcn_s_waitcnt(0x0F70);            // vmcnt(0): the group's lists are out
        __syncthreads();
        if (threadIdx.x == 0) {
            const unsigned int old = __hip_atomic_fetch_add(p.counter, 1u, __ATOMIC_RELAXED,
                                                            __HIP_MEMORY_SCOPE_AGENT);
            flags[1] = old == (unsigned)uni(flags[0]) - 1u ? 1 : 0;
        }
        __syncthreads();
        if (!uni(flags[1])) return;                    // block-uniform
        for (int t = wave; t < M; t += kFusedWaves) {
            const Cand* src = p.glist + (size_t)t * p.g * k;
            wave_merge_lists(
                p.g, k, lane, ms, [&](int l, int e) { return fetch_cand(src + l * k + e); },
                [&](int r, unsigned long long key) { write_result(t, r, key_cand(key)); });
        }
        expand_level();
        if (threadIdx.x == 0)
            __hip_atomic_store(p.counter, 0u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        return;
    }
    __syncthreads();
    publish_all();
    __builtin_amdgcn_s_waitcnt(0x0F70);                // vmcnt(0): the published lists are out
    __syncthreads();
    if (threadIdx.x == 0) {
        const unsigned int old = __hip_atomic_fetch_add(p.counter, 1u, __ATOMIC_RELAXED,
                                                        __HIP_MEMORY_SCOPE_AGENT);
        flags[1] = old == (unsigned)P_act - 1u ? 1 : 0;
    }
    __syncthreads();
    if (!uni(flags[1])) return;                        // block-uniform

    // Last workgroup: one wave per token merges the published lists, one per workgroup with batches.
    for (int t = wave; t < M; t += kFusedWaves) {
        const Cand* src = p.part + (size_t)t * k * P;
        wave_merge_lists(
            P_act, k, lane, ms,
            [&](int l, int i) { return fetch_cand(src + (size_t)i * P + l); },
            [&](int r, unsigned long long key) {
                const Cand c = key_cand(key);
                p.topk_ids[(size_t)t * k + r] = c.id;
                p.topk_logits[(size_t)t * k + r] = c.v;
            });
    }
    if (threadIdx.x == 0)                              // ready for the next call
        __hip_atomic_store(p.counter, 0u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

}  // namespace
