// Weight-grouped LM head of a speculative-decoding draft model, gfx950 (MI355X).
//
// Paper section 3.3 ("LM Head Router"): the router's W2 projection scores G
// vocabulary groups per draft token, the g best groups are activated, logits are
// computed over the rows of those groups only and the k best candidates per token
// go to tree expansion (appendix "Discussion on LM Head Router").  The paper gives
// no kernel; this design is for CDNA4: the path is bound by streaming the active
// weight rows from HBM once, so
//   - one wavefront reads one weight row as consecutive 1 KB segments (64 lanes x
//     16 B), several rows in flight, non-temporal so the stream does not evict the
//     small reused operands from L2;
//   - the hidden vectors of the tokens that selected the group sit in LDS and are
//     re-used for every row of the chunk; bf16 pairs go through v_dot2c_f32_bf16
//     with fp32 accumulation;
//   - where the hidden vectors fit on chip the logits row never leaves it: a workgroup collects
//     its logits per token in LDS, publishes its k best, and the last workgroup merges all.
//     With many tokens the matrix cores take over and the activated rows' logits go through
//     memory to a ranking kernel.
// A group selected by several tokens is read once for all of them (the union of the
// tokens' groups that the appendix's tree-decoding paragraph activates).
#include <hip/hip_runtime.h>
#include <hip/hip_ext.h>
#include <limits.h>
#include <stdint.h>
#include <stdlib.h>

#include <mutex>

#include "coral_lmhead.h"
#include "control_words.h"
#include "device_utils.h"
#include "fused_kernels.h"
#include "fused_path.h"
#include "router_premix.h"
#include "staged_path.h"
#include "tile_path.h"
#include "tree_expand.h"

// Scratch memory of coral_lmhead_grouped_noalloc: what the other entry points take as their
// caller-provided workspace.  One copy per GPU the library runs on, held until the process
// ends; in host code the name is only a handle for hipGetSymbolAddress, never an address.
constexpr size_t kStaticScratchBytes = (size_t)CORAL_NOALLOC_SCRATCH_BYTES;
// The array is larger than what calls are counted by (static_counted_bytes): the statistics of blocks
// processed in halves, of which half of the workgroups have one at most, and the gate's scores behind the
// 512 bytes of control words.
constexpr int kMaxWorkgroups = 256;    // upper bound of the persistent kernels' grids
constexpr size_t upper_stat_bytes(int M) { return (size_t)(kMaxWorkgroups / 2) * M * sizeof(float2); }
constexpr size_t kCtrlBytes = coral_ctrl::kWords * sizeof(unsigned int);   // control words at the start of the workspace
constexpr size_t kGateScoreBytes = coral_ctrl::kGateScoreWords * sizeof(unsigned int);   // and the scores behind them
static_assert(kCtrlBytes % 256 == 0 && kGateScoreBytes % 256 == 0, "");
constexpr size_t kStaticArrayBytes = kStaticScratchBytes + upper_stat_bytes(kMaxM) + kGateScoreBytes;
static __device__ __align__(256) unsigned char scratch[kStaticArrayBytes];

namespace {

// The first n words of a workspace: control words, and the gate's scores as far as n goes.  Only where
// it holds all of these may the workgroups wait for each other's scores.
__global__ void k_prepare_words(unsigned int* p, int n) {
    const int i = blockIdx.x * blockDim.x + threadIdx.x;
    if (i < n) p[i] = i == coral_ctrl::kGatePolls && n >= coral_ctrl::kPreparedWords ? (unsigned)kGatePollsMax : 0u;
}

coral_status prepare_words(void* workspace, size_t bytes, hipStream_t stream) {
    const size_t most = coral_ctrl::kPreparedWords * sizeof(unsigned int);
    const int n = (int)((bytes < most ? bytes : most) / sizeof(unsigned int));
    hipLaunchKernelGGL(k_prepare_words, dim3((n + 255) / 256), dim3(256), 0, stream, static_cast<unsigned int*>(workspace), n);
    return hipGetLastError() == hipSuccess ? CORAL_OK : CORAL_ERR_HIP;
}

// ---------------------------------------------------------------- host side
inline size_t align_up(size_t x, size_t a) { return (x + a - 1) / a * a; }

inline bool dtype_ok(coral_dtype dt) { return dt == CORAL_F32 || dt == CORAL_BF16 || dt == CORAL_F16; }
inline bool is_16bit(coral_dtype dt) { return dt != CORAL_F32; }
// One of three instantiations by storage type (kernels without an fp32 form pass nullptr).
#define CORAL_PICK_DT(dt, f32, bf16, f16) ((dt) == CORAL_F32 ? (f32) : (dt) == CORAL_BF16 ? (bf16) : (f16))

static_assert(coral_ctrl::kLpGroupArrivalWords >= kWave, "one arrival counter per activated group");
static_assert(coral_ctrl::kGateSelectArrivalWords * 16 >= kMaxM, "one arrival counter per token tile");

struct Layout {
    size_t ctrl, fused_part, fused_lse, fused_glist, fused_pairs, s, sel, mask, union_list, n_union, chunk_base, slot_count, part, lse_part, logp_sel, tile_mask, tile_first_block, tile_z, tile_stat, tile_upper, total;
    int part_stride;
};

bool sizes_ok(int M, int H, int V, int G, int g, int k) {
    if (M < 1 || H < 1 || V < 1 || k < 1) return false;
    if (G < 0 || g < 0 || (G == 0) != (g == 0) || g > G) return false;
    return true;
}

// Which paths' arrays a layout holds: all that calls with these sizes can take (a workspace), or
// those of one path only (the static scratch array; kCounted: what its calls are counted by).
enum class LayoutFor { kWorkspace, kSingleLaunch, kTiles, kCounted };

// pieces: the log-probability mode's table of per-batch pieces (layout_pieces).  tiles: whether the
// shape can take the tile kernels (their logits buffer and statistics are left out otherwise), as
// the matrix-core path proper or on the general path, and whether with blocks of 32 rows.
enum class Tiles { kNone, kGeneral, kOwn };
struct TileArrays {
    Tiles kind;
    bool small;
};
struct Pieces {
    size_t entries;             // 0 if the single-launch kernel cannot run the mode
    bool shared;                // in the memory of the multi-kernel paths' arrays
};
Layout make_layout(int M, int V, int G, int g, int k, Pieces pieces, TileArrays tile_arrays,
                   LayoutFor what = LayoutFor::kWorkspace) {
    Layout L;
    const Tiles tiles = tile_arrays.kind;
    size_t off = 0;
    auto take = [&](size_t bytes) {
        size_t at = off;
        off = align_up(off + bytes, 256);
        return at;
    };
    L.ctrl = take(kCtrlBytes + kGateScoreBytes);
    const size_t single = what != LayoutFor::kTiles && what != LayoutFor::kCounted ? 1 : 0;
    const size_t logprob = what == LayoutFor::kWorkspace ? 1 : 0;
    const size_t staged = what == LayoutFor::kWorkspace ? 1 : 0;
    L.fused_part = take(single * kMaxWorkgroups * M * k * sizeof(Cand));
    L.fused_lse = take(logprob * kMaxWorkgroups * M * sizeof(unsigned long long));   // log-probability mode
    L.fused_glist = take(logprob * M * (g ? g : 1) * k * sizeof(Cand));
    L.fused_pairs = off;
    const size_t pieces_end = align_up(off + pieces.entries * sizeof(unsigned long long), 256);
    if (!pieces.shared) off = pieces_end;
    L.s = take((size_t)kGateParts * M * (G ? G : 1) * sizeof(float));
    L.sel = take((size_t)M * (g ? g : 1) * sizeof(int32_t));
    L.mask = take((size_t)(G ? G : 1) * sizeof(unsigned long long));
    L.union_list = take((size_t)(G ? G : 1) * sizeof(int32_t));
    L.n_union = take(sizeof(int32_t));
    L.chunk_base = take((size_t)M * (g ? g : 1) * sizeof(int32_t));
    L.slot_count = take((size_t)M * (g ? g : 1) * sizeof(int32_t));
    L.logp_sel = take((size_t)M * (g ? g : 1) * sizeof(float));
    L.tile_mask = take((size_t)((kMaxM + 15) / 16) * (G ? G : 1) * sizeof(unsigned long long));
    L.tile_first_block = take((size_t)(G ? G : 1) * sizeof(int32_t));
    L.part_stride = (V + kChunkRows - 1) / kChunkRows + g;
    const size_t lists = off;
    L.part = take(staged * M * L.part_stride * k * sizeof(Cand));
    L.lse_part = take(staged * M * L.part_stride * 2 * sizeof(float));     // log-probability mode
    // A group's blocks round up: V / 128 + G blocks at most (dense: V itself rounds up).  On the
    // general path the logits take the place of the staged kernels' lists, which no call uses
    // with them.
    const size_t after = off;
    if (tiles == Tiles::kGeneral) off = lists;
    const size_t tile_blocks = (size_t)V / kTileRows + G + (tiles == Tiles::kOwn || G == 0 ? 1 : 0);
    L.tile_z = take(tiles != Tiles::kNone ? tile_blocks * M * kTileRows * sizeof(float) : 0);
    // (with blocks of 32 rows the logits take no more, their statistics V / 32 + G entries)
    const size_t stat_blocks = (size_t)V / (tile_arrays.small ? kTileRowsSmall : kTileRows) + G + 1;
    L.tile_stat = take(tiles != Tiles::kNone ? stat_blocks * M * sizeof(float2) : 0);
    L.tile_upper = take(tiles == Tiles::kOwn && what != LayoutFor::kCounted ? upper_stat_bytes(M) : 0);   // of blocks in halves
    if (off < after) off = after;
    L.total = off > pieces_end ? off : pieces_end;
    return L;
}

coral_status check_common(const void* hidden, const void* lm_W, int M, int H, int V, int k,
                          coral_dtype dt, const int32_t* topk_ids, const float* topk_logits) {
    if (!hidden || !lm_W || !topk_ids || !topk_logits) return CORAL_ERR_NULL;
    if (!dtype_ok(dt)) return CORAL_ERR_SHAPE;
    if (M < 1 || H < 1 || V < 1 || k < 1) return CORAL_ERR_SHAPE;
    if (M > kMaxM || k > kMaxK) return CORAL_ERR_UNSUPPORTED;
    if (H % (is_16bit(dt) ? 8 : 4) != 0) return CORAL_ERR_UNSUPPORTED;
    if (((uintptr_t)hidden | (uintptr_t)lm_W) & 15u) return CORAL_ERR_UNSUPPORTED;
    return CORAL_OK;
}

coral_status check_workspace(const void* ws, size_t have, size_t need) {
    if (!ws) return CORAL_ERR_WORKSPACE;
    if ((uintptr_t)ws & 255u) return CORAL_ERR_WORKSPACE;
    if (have < need) return CORAL_ERR_WORKSPACE;
    return CORAL_OK;
}

size_t logits_lds_bytes(int tb_max, int jp, int k) {
    return (size_t)tb_max * jp * kWave * sizeof(uint4) + (size_t)kWavesPerBlock * k * sizeof(Cand);
}

inline coral_status launch_status() {
    return hipGetLastError() == hipSuccess ? CORAL_OK : CORAL_ERR_HIP;
}

// Launch of the kernel that streams the weight rows.  The measurement entry points pass two
// events: they are bound to this launch and take the kernel's own start and stop times (what
// a kernel trace reports as its duration), not the times at which event records before and
// after it would be reached, which include the dispatch latency.
coral_status launch_timed(const void* fn, dim3 grid, dim3 block, size_t lds, hipStream_t stream, void* ev_before,
                          void* ev_after, void** args) {
    const hipError_t e =
        ev_before && ev_after
            ? hipExtLaunchKernel(fn, grid, block, args, lds, stream, static_cast<hipEvent_t>(ev_before),
                                 static_cast<hipEvent_t>(ev_after), 0)
            : hipLaunchKernel(fn, grid, block, args, lds, stream);
    return e == hipSuccess ? launch_status() : CORAL_ERR_HIP;
}
template <class F, class... Args>
coral_status launch_timed(F fn, dim3 grid, dim3 block, size_t lds, hipStream_t stream, void* ev_before,
                          void* ev_after, Args... args) {
    if (ev_before && ev_after)
        hipExtLaunchKernelGGL(fn, grid, block, (uint32_t)lds, stream, static_cast<hipEvent_t>(ev_before),
                              static_cast<hipEvent_t>(ev_after), 0, args...);
    else
        hipLaunchKernelGGL(fn, grid, block, lds, stream, args...);
    return launch_status();
}

// The only state the library keeps between calls: per device, the number of compute units
// (the single-launch path runs one workgroup on each) and the largest dynamic LDS size each
// kernel has been allowed so far.  Both are properties of the device and of the loaded code
// object, looked up once instead of on every call; a mutex guards them.
constexpr int kMaxDevices = 64;
constexpr int kMaxKernels = 192;
struct DeviceCache {
    int compute_units;
    void* scratch_ptr;          // this device's copy of `scratch`, looked up on first use
    int n_kernels;
    const void* kernel[kMaxKernels];
    int lds_bytes[kMaxKernels];
};
DeviceCache g_cache[kMaxDevices];
std::mutex g_cache_mutex;

int compute_units() {
    int dev = 0;
    if (hipGetDevice(&dev) != hipSuccess || dev < 0 || dev >= kMaxDevices) return 0;
    std::lock_guard<std::mutex> lock(g_cache_mutex);
    if (g_cache[dev].compute_units == 0) {
        int n = 0;
        if (hipDeviceGetAttribute(&n, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess)
            return 0;
        g_cache[dev].compute_units = n;
    }
    return g_cache[dev].compute_units;
}

// Device address of this device's copy of the static scratch array.
coral_status static_scratch(void** out) {
    int dev = 0;
    if (hipGetDevice(&dev) != hipSuccess || dev < 0 || dev >= kMaxDevices) return CORAL_ERR_HIP;
    std::lock_guard<std::mutex> lock(g_cache_mutex);
    if (!g_cache[dev].scratch_ptr) {
        void* ptr = nullptr;
        if (hipGetSymbolAddress(&ptr, HIP_SYMBOL(scratch)) != hipSuccess || !ptr) return CORAL_ERR_HIP;
        g_cache[dev].scratch_ptr = ptr;
    }
    *out = g_cache[dev].scratch_ptr;
    return CORAL_OK;
}

// Lets kernel `fn` use `bytes` of dynamic LDS on the current device (needed above 64 KB).
bool allow_lds(const void* fn, int bytes) {
    if (bytes <= 64 * 1024) return true;
    int dev = 0;
    if (hipGetDevice(&dev) != hipSuccess) return false;
    DeviceCache* c = dev >= 0 && dev < kMaxDevices ? &g_cache[dev] : nullptr;
    std::lock_guard<std::mutex> lock(g_cache_mutex);
    int slot = -1;
    if (c) {
        for (int i = 0; i < c->n_kernels; ++i)
            if (c->kernel[i] == fn) slot = i;
        if (slot >= 0 && c->lds_bytes[slot] >= bytes) return true;
    }
    if (hipFuncSetAttribute(fn, hipFuncAttributeMaxDynamicSharedMemorySize, bytes) != hipSuccess)
        return false;
    if (c) {
        if (slot < 0 && c->n_kernels < kMaxKernels) {
            slot = c->n_kernels++;
            c->kernel[slot] = fn;
        }
        if (slot >= 0) c->lds_bytes[slot] = bytes;
    }
    return true;
}

// Gate of the single-launch path where every workgroup computes it, and what the LDS plan goes by:
// from four tokens on it goes through the matrix cores (16-bit storage only; measured at the Llama3
// shape: two tokens 52.1 against 50.8 us on the vector units, three equal, four 81.0 against 81.5).
int fused_gate_mode(bool dense, int M, int G, int g, int k, int jp, coral_dtype dt, bool logprob = false) {
    (void)G; (void)g; (void)k; (void)jp; (void)logprob;
    return dense || !is_16bit(dt) || M <= 3 ? kGateVector : kGateMfma;
}

// Whether the single launch's gate is shared between the workgroups (kGateShared): where it would take
// every workgroup by itself longer than the hand-over, about 4 us.  Estimates in us of the former: on the
// matrix cores by passes of 32 groups, on the vector units of 16 groups and two tokens, each with the bytes
// of its rows.  Fitted to 2 x 343 heads (512 to 8192 columns, 8 to 120 groups, 1 to 32 tokens, bf16 and fp32,
// 24000 rows): 1.08 times as fast on average (log-probabilities 1.05).  us, own gate against shared: bf16, 8
// tokens, H = 8192, 8 groups 59, 55, 120 groups 74, 43; H = 4096, 16 groups 27.8, 26.5, 64 groups 36, 28; H =
// 2048, 32 groups 22.0, 22.2; H = 512, 120 groups 22.8, 20.6, 32 groups 16.4, 18.5; fp32, 16 tokens, H = 1024,
// 16 groups 33, 29, 4 tokens, H = 4096, 16 groups 30.4, 29.1, 64 groups 43, 30.
// With up to three tokens the own gate starts early and goes by the bytes of the whole gate.  Over 1291 heads
// (8192 rows and more, 8 to 256 groups) with those below kFewTokensKb the worst are 0.907 (one token), 0.927
// (two) and 0.951 (three) times as fast as with the own gate, without them 0.963, 0.976 and 1.008; the heads
// left out are 0.98, 1.00 and 1.03 on average (one token, H = 2776, 66 groups 16.7, 18.4; H = 8192, 32 groups 56.1, 54.5).
bool fused_gate_shared(int M, int G, int n_vec, coral_dtype dt) {
    constexpr double kFewTokensKb[3] = {500, 300, 200};
    if (M * G > coral_ctrl::kGateScoreWords) return false;
    const double kb = n_vec / 64.0;                        // of a gate row
    if (M <= 3 && G * kb < kFewTokensKb[M - 1]) return false;
    const double own = is_16bit(dt) && M >= 4 ? (G + 31) / 32 * (0.4 + 0.68 * kb)
                                              : (G + 15) / 16 * 0.5 * (0.3 + 0.05 * M + (0.1 + 0.11 * M) * kb);
    return own > 3.5;
}

// Rows the single-launch kernel takes (by their 16-byte vectors): up to 8 KB, and from 8.25 to 16 KB.  (Rows of
// nine segments leave seven of a batch's sixteen loads empty: nine_segs_take_fused.  Below a quarter of the
// ninth segment two heads measured 1.5 and 2.5 times as fast on the single launch: not a loss, but these
// widths are where the general path's form of long rows is pinned, and they stay there.)
bool fused_rows_fit(int n_vec) {
    return n_vec <= 8 * kWave || (n_vec >= 8 * kWave + kWave / 4 && n_vec <= kFusedMaxSegs * kWave);
}

// Log-probability mode: beyond 32 tokens the single-launch kernel's per-wave lists (one per token,
// hardly ever filled) and per-token pieces cost more than the tile kernels' three launches
// (264-wide head, 59 tokens, 3 of 29 groups: 82 us against 34).
constexpr int kLogprobFusedMaxTokens = 32;

// Activated groups at most.
inline long long max_union(int M, int G, int g) { return (long long)M * g < G ? (long long)M * g : G; }

// The single-launch kernel's log-probability mode gives every activated group workgroups of
// its own and ranks the groups in one wave: at most 64 activated groups, fewer than half the
// workgroups; a token's g lists share the LDS of one wave's lists.
bool fused_logprob_fits(int M, int G, int g, int k, int jp, coral_dtype dt, int workgroups) {
    if (g > kFusedWaves) return false;
    const long long um = max_union(M, G, g);
    if (um > kWave || 2 * um > workgroups) return false;
    return fused_lds_layout(M, G, g, k, jp, false, fused_gate_mode(false, M, G, g, k, jp, dt, true), true)
               .total <= kLdsLimit;
}

// Tile kernels: weights below 4 GiB, LDS plan within the limit.
bool tile_kernels_fit(int M, int H, int V, int G, int g, int k, coral_dtype dt, int* u_max_out, int* lds_out) {
    if (k > kMaxK || M > 64) return false;
    if ((unsigned long long)V * H * (is_16bit(dt) ? 2ull : 4ull) >= (1ull << 32)) return false;   // 32-bit weight offsets
    long long um = (long long)M * g < G ? (long long)M * g : G;
    if (um < 1) um = 1;
    const TileLds T = tile_lds_layout((int)um);
    if (T.total > kLdsLimit) return false;
    // the ranking kernel keeps a few words per block of a token's groups in LDS
    if ((long long)V / kTileRows + g + 1 > (1 << 16)) return false;
    if (tile_select_lds_layout(g > 0 ? g : 1, V / kTileRows + g + 1).total > kLdsLimit) return false;
    *u_max_out = (int)um;
    *lds_out = T.total;
    return true;
}

// Matrix-core path proper: 16-bit storage and whole 512-column chunks as well.
bool tiles_fit(int M, int H, int V, int G, int g, int k, coral_dtype dt, int* u_max_out, int* lds_out) {
    return is_16bit(dt) && H % (kChunkVecs * 8) == 0 && tile_kernels_fit(M, H, V, G, g, k, dt, u_max_out, lds_out);
}

// Groups that M tokens activate if each draws its g of G by lot, and their 128-row blocks.
double expected_groups(int M, int G, int g) {
    double out = 1.0;                          // chance that a group stays out: (1 - g / G) ^ M
    double power = 1.0 - (double)g / G;
    for (int m = M; m; m >>= 1, power *= power)
        if (m & 1) out *= power;
    return G * (1.0 - out);
}
double expected_blocks(int M, int V, int G, int g) {
    return expected_groups(M, G, g) * ((V / G + kTileRows - 1) / kTileRows);
}

// Rows of nine segments (4224 to 4608 columns, fp32 half of that): whether the single launch takes them.  us,
// multi-kernel paths against single launch, over 8000 random heads (8 to 4000 groups, 1 to 17 tokens, any k) that
// had all taken it:
//   - grouped: 1.9 times as fast off the matrix-core path, 1.2 times beside it, while a group has few tokens.
//     With many, a row's products on the vector units take longer than its load: k <= 16, beside the matrix-core
//     path from six tokens a group on 0.84 on average (f16 H = 4608, 106958 rows, 5 of 8 groups, 14 tokens 175,
//     261); off it, where the other path's blocks fill rounds over the compute units, 16 bits from 7.5 on 0.97, 0.57
//     to 1.2 (H = 4224, 16 of 26 groups, 14 tokens 150, 225), fp32 from 8.5 on 0.98, 0.68 to 1.3 (H = 2144, 25 of 27
//     groups, 15 tokens 138, 202).  Where they fill half of a round, or little of the second, the single launch
//     stays ahead (1.2 and 1.25, but six of 130 heads 0.80 to 0.97).  Beyond k = 16 (the other paths' merges go by
//     whole lists) it is up to ten tokens a group, 1.05 and more on average, above 0.98;
//   - more scores than the workgroups can share, where the other choice is the matrix-core path: every workgroup
//     computed them all, 54 heads 0.13 to 0.57 (bf16 H = 4608, 1021 groups, 6 tokens 40, 294);
//   - log-probabilities: up to eight tokens 1.6 times as fast off the matrix-core path (16 bits, k <= 16, from six
//     tokens a group on and several rounds of blocks 0.88 to 1.1), 1.17 beside it, but from 3.5 tokens a group on
//     0.92 to 1.26, and where a token's groups have more than 520 candidates between them 0.75 to 1.05 (bf16, 10 of
//     47 groups, 3 tokens, k = 64 51, 64; up to 520 1.05 and more); with more tokens 0.75 to 2.3 (bf16 H = 4328, 6 of 8 groups, 12 tokens 176, 234);
//   - dense: up to seven tokens 2.9 times as fast off the matrix-core path, 1.3 beside it, but there seven tokens
//     0.92 to 0.99 from 22000 rows on (f16 H = 4608, 83005 rows 133, 144; 9057 rows 1.35); more tokens f16 H = 4480,
//     94129 rows, 9 tokens 146, 166, bf16 H = 4352, 24624 rows, 15 tokens 49, 70.
constexpr int kNineSegsDenseTokens = 7, kNineSegsLogprobTokens = 8;
bool nine_segs_take_fused(int M, int H, int V, int G, int g, int k, coral_dtype dt, bool logprob) {
    int um, lds;
    const bool tiles = tiles_fit(M, H, V, G, g, k, dt, &um, &lds) && (!logprob || G <= kWave);
    const double group_tokens = M * g / expected_groups(M, G, g);
    if (logprob) {
        if (M > kNineSegsLogprobTokens) return false;
        if (tiles) return group_tokens <= 3.5 && g * k <= 520;
        return group_tokens <= 6.0 || k > 16 || !is_16bit(dt) || expected_blocks(M, V, G, g) <= kMaxWorkgroups;
    }
    if (tiles && M * G > coral_ctrl::kGateScoreWords) return false;
    if (group_tokens <= (k > 16 ? 10.0 : tiles ? 6.0 : is_16bit(dt) ? 7.5 : 8.5)) return true;
    const double rounds = expected_blocks(M, V, G, g) / kMaxWorkgroups;
    return !tiles && (rounds <= 0.75 || (rounds > 1.0 && rounds <= 1.5));
}
bool nine_segs_take_fused_dense(int M, int H, int V, int k, coral_dtype dt) {
    int um, lds;
    if (M != kNineSegsDenseTokens) return M < kNineSegsDenseTokens;
    return V < 16384 || !tiles_fit(M, H, V, 0, 0, k, dt, &um, &lds);
}

// Rows beyond 8 KB: the single launch takes them where the workgroups can share the gate's scores.  us, the
// general path against it, over the heads off the matrix-core path among 380 random ones (8 to 1000 groups, 1 to
// 14 tokens) that the own gate had kept there: 1.5 to 1.9 times as fast on average, none slower by more than 2 %;
// bf16 H = 7296, 117 groups, 6 tokens 76, 36; fp32 H = 3072, 109 groups, 5 tokens 56, 28; log-probabilities, f16
// H = 6144, 128 groups, 8 tokens 74, 29; bf16 H = 5632, 83 groups, 9 tokens 131, 134.  Not where a group has
// more than ten tokens (fp32 H = 2816, 109 of 126 groups, 12 tokens 246, 278).
// The lines from before that stay where
//   - the matrix-core path is the other choice: taken while tokens are few or where its blocks do not fill a
//     good part of one round over the compute units (H = 5120, 6 tokens, 32 groups 97, 83; with the shared gate
//     the single launch would be ahead beyond them too, by 4 to 27 %: 7 tokens, 126 groups 79, 68);
//   - the last of a row's segments is filled to less than a quarter, or there are more scores than words for
//     them: few groups and tokens, or many candidates (the staged merges go by whole lists; own gate, H = 4616,
//     128100 rows, one token, 128 groups 40, 30, 300 groups 38, 46; 6 tokens, 80 groups 72, 62, 300 groups
//     46, 103; log-probabilities, 6 tokens, 64 groups 79, 80).  Both are pinned by the routes' tests.
bool long_rows_take_fused(int M, int H, int V, int G, int g, int k, coral_dtype dt, bool logprob) {
    int um, lds;
    const int n_vec = H / (is_16bit(dt) ? 8 : 4), last = n_vec % kWave;
    if (n_vec <= 9 * kWave && !nine_segs_take_fused(M, H, V, G, g, k, dt, logprob)) return false;
    if (tiles_fit(M, H, V, G, g, k, dt, &um, &lds) && (!logprob || G <= kWave)) {
        const double blocks = expected_blocks(M, V, G, g);
        return M < 4 || k > 10 || blocks <= (logprob ? 110 : 145) || blocks > kMaxWorkgroups + 6;
    }
    if (M * G <= coral_ctrl::kGateScoreWords && (last == 0 || last >= kWave / 4) &&
        (n_vec <= 9 * kWave || M * g <= 10 * expected_groups(M, G, g)))
        return true;
    return G <= (!logprob ? 64 : M >= 7 ? 60 : 40) || G + 6 * M <= (logprob ? 80 : 135) + (k > 10 ? 8 * (k - 10) : 0);
}

// Log-probability mode: whether the single-launch kernel runs a call.  (Beyond 32 tokens only where
// the tile kernels cannot: 256-wide head, V = 900000, 36 tokens, 2 of 32 groups 180 us here, 707 us
// with the staged kernels, which are left then.)
bool logprob_takes_fused(int M, int H, int V, int G, int g, int k, int jp, coral_dtype dt) {
    int um, lds;
    return fused_rows_fit(H / (is_16bit(dt) ? 8 : 4)) && fused_logprob_fits(M, G, g, k, jp, dt, kMaxWorkgroups) &&
           (jp <= 8 || long_rows_take_fused(M, H, V, G, g, k, dt, true)) &&
           (M <= kLogprobFusedMaxTokens || !tile_kernels_fit(M, H, V, G, g, k, dt, &um, &lds));
}

// What a draft-level call adds to the log-probability head: the expansion of the tree level
// whose nodes are the call's tokens.
struct LevelExpand {
    const float* parent_score;
    int n_next;
    int32_t* next_parent;
    int32_t* next_token;
    float* next_score;
};

// Enqueues the expansion of a level from the candidate lists in memory.
coral_status launch_tree_expand(const LevelExpand& level, const int32_t* cand_ids, const float* cand_logp, int M, int k,
                                hipStream_t stream) {
    if (level.n_next <= kWave && M * k <= kTreeTopkMax)
        hipLaunchKernelGGL(level.parent_score ? k_tree_topk<true> : k_tree_topk<false>, dim3(1), dim3(kWave), 0, stream,
                           level.parent_score, cand_ids, cand_logp, M, k, level.n_next, level.next_parent,
                           level.next_token, level.next_score);
    else
        hipLaunchKernelGGL(k_tree_expand, dim3(M), dim3(kWave), (size_t)M * k * sizeof(unsigned long long), stream,
                           level.parent_score, cand_ids, cand_logp, M, k, level.n_next, level.next_parent,
                           level.next_token, level.next_score);
    return launch_status();
}

// The single-launch log-probability mode's table of pieces: one (max, sum) per (batch of rows of
// a selected group, token that selected it); a token's g groups are distinct, so their batches
// number V / rows + g at most.  Rows beyond 8 KB (one to a batch): the table shares the memory of
// the multi-kernel paths' arrays, which no call uses with it.
Pieces layout_pieces(int M, int H, int V, int G, int g, int k, coral_dtype dt) {
    if (G < 1 || !dtype_ok(dt)) return {0, false};
    const int n_vec = H / (is_16bit(dt) ? 8 : 4);
    const int jp = (n_vec + kWave - 1) / kWave;
    if (jp < 1 || !logprob_takes_fused(M, H, V, G, g, k, jp, dt)) return {0, false};
    return {(size_t)M * ((size_t)V / fused_rows(fused_segs(jp)) + g), jp > 8};
}

// Collected candidates instead of per-wave lists, where a workgroup is sure to meet at
// most kCollectMax rows per token: it takes D consecutive batches out of every D P of the
// concatenated activated groups, so of any group (a run of at most n batches) it meets no
// more than D * (n / D P) + min(D, n % D P), and a token has g groups.  D = kDealFew (the
// bound for the smaller D that the kernel uses as well is never larger), or, where buffers
// that size do not fit, D = 1 throughout (512-wide head, 55 tokens, 7 of 61 groups: 64
// entries per token instead of 448, 148 us with lists, 57 with buffers).  Returns the entries
// per token, 0 for lists.
int collect_cap(bool dense, int M, int G, int g, int k, int jp, int gate, int group_rows, int P, bool* deal_single) {
    const int rows = fused_rows(fused_segs(jp));
    for (int deal = kDealFew; deal >= 1; deal -= kDealFew - 1) {
        const long long period = (long long)deal * P;
        const long long n = ((long long)group_rows + rows - 1) / rows;
        const long long rest = n % period;
        const long long per_group = deal * (n / period) + (rest < deal ? rest : deal);
        const long long bound = (rows * per_group * (dense ? 1 : g) + kWave - 1) / kWave * kWave;
        *deal_single = deal == 1;
        if (bound > 0 && bound <= kCollectMax &&
            fused_lds_layout(M, G, g, k, jp, dense, gate, false, (int)bound).total <= kLdsLimit)
            return (int)bound;
    }
    *deal_single = false;
    return 0;
}

// Enqueues the single-launch path (the caller has checked with plan_path that it fits).
coral_status launch_fused(bool dense, const void* hidden, const void* gate_hidden, const void* gate_W,
               const float* gate_bias,
               const void* lm_W, const coral_group_index* gi, int M, int H, int V, int G, int g,
               int k, coral_dtype dt, int32_t* topk_ids, float* topk_logits, int32_t* sel_groups,
               char* ws, const Layout& L, hipStream_t stream, void* ev_before, void* ev_after,
               bool logprob = false, const LevelExpand* level = nullptr, int max_group_rows = 0) {
    const int n_vec = H / (is_16bit(dt) ? 8 : 4);
    const int jp = (n_vec + kWave - 1) / kWave;
    const int gate = fused_gate_mode(dense, M, G, g, k, jp, dt, logprob);
    int P = compute_units();
    if (P < 1) return CORAL_ERR_HIP;
    if (P > kMaxWorkgroups) P = kMaxWorkgroups;
    const int segs = fused_segs(jp);
    int cap = 0;
    bool deal_single = false;
    if (!logprob) {
        cap = collect_cap(dense, M, G, g, k, jp, gate, dense ? V : max_group_rows, P, &deal_single);
    } else {
        // a workgroup's rows depend on the selection: buffers as large as fit beside the pieces,
        // used by the workgroups whose rows they hold
        for (int c = kCollectMax; !cap && c > kFusedWaves * k; c -= kWave) {
            const FusedLds L2 = fused_lds_layout(M, G, g, k, jp, false, gate, true, c);
            if (L2.total <= kLdsLimit && L2.pieces_bytes >= kLpPiecesMax) cap = c;
        }
        if (!cap) cap = kFusedWaves * k;               // the lists' own size
    }
    const FusedLds F = fused_lds_layout(M, G, g, k, jp, dense, gate, logprob, cap);
    if (!fused_rows_fit(n_vec) || F.total > kLdsLimit) return CORAL_ERR_UNSUPPORTED;   // not reached
    if (jp > 8 && gate == kGateMfma && M > 16) return CORAL_ERR_UNSUPPORTED;        // not reached: LDS
    FusedParams p = {};
    p.cap = cap;
    p.deal_single = deal_single ? 1 : 0;
    // Measured with rows of 8 KB (Llama shapes): dense head, one or two tokens: 6 waves 158 us
    // against 165 us with all 16 (Llama2: 46.5 against 48.5 us); four tokens: 10 waves 162 us
    // against 168 us.  Rows of 7 KB (Qwen shape) and the grouped head's gathered rows are
    // fastest with all 16 (Qwen dense: 163 us against 170 us with 6).
    const bool rows_of_8k = ((size_t)n_vec * 16) % 8192 == 0;
    p.stream_waves = !dense || !rows_of_8k ? kFusedWaves : M <= 2 ? 6 : M <= 4 ? 10 : kFusedWaves;
    p.hidden = static_cast<const uint4*>(hidden);
    p.gate_hidden = static_cast<const uint4*>(gate_hidden);
    p.gate_W = static_cast<const uint4*>(gate_W);
    p.bias = gate_bias;
    p.lm_W = static_cast<const uint4*>(lm_W);
    p.offsets = gi ? gi->group_offsets : nullptr;
    p.rows = gi ? gi->group_rows : nullptr;
    p.sel_out = sel_groups;
    p.part = reinterpret_cast<Cand*>(ws + L.fused_part);
    p.lse_part = reinterpret_cast<unsigned long long*>(ws + L.fused_lse);
    p.glist = reinterpret_cast<Cand*>(ws + L.fused_glist);
    p.pair_lse = reinterpret_cast<unsigned long long*>(ws + L.fused_pairs);
    if (level) {
        p.parent_score = level->parent_score;
        p.n_next = level->n_next;
        p.next_parent = level->next_parent;
        p.next_token = level->next_token;
        p.next_score = level->next_score;
    }
    p.counter = reinterpret_cast<unsigned int*>(ws + L.ctrl) + coral_ctrl::kFusedArrival;
    p.topk_ids = topk_ids;
    p.topk_logits = topk_logits;
    p.M = M; p.V = V; p.G = G; p.g = g; p.k = k;
    p.n_vec = n_vec; p.jp = jp;
    const bool routed = !dense && gate_hidden != hidden;
    if (logprob && (dense || 2 * max_union(M, G, g) > P)) return CORAL_ERR_UNSUPPORTED;   // not reached
    const bool short_rows = segs <= 4;
    const auto getter = CORAL_PICK_DT(dt, short_rows ? coral_fused_short_f32 : coral_fused_long_f32,
                                      short_rows ? coral_fused_short_bf16 : coral_fused_long_bf16,
                                      short_rows ? coral_fused_short_f16 : coral_fused_long_f16);
    const bool shared = !dense && fused_gate_shared(M, G, n_vec, dt);
    const void* fn = getter(dense, shared ? (int)kGateShared : gate, routed, logprob, segs);
    if (!fn) return CORAL_ERR_UNSUPPORTED;             // not reached
    if (!allow_lds(fn, F.total)) return CORAL_ERR_HIP;
    void* args[] = {&p};
    return launch_timed(fn, dim3(P), dim3(kFusedBlock), F.total, stream, ev_before, ev_after, args);
}

// The dense head goes to the matrix-core path from 8 tokens on, if the vocabulary gives every
// workgroup at least two 128-row blocks (below that its per-block set-up and epilogue
// dominate and the vector path is faster).
bool dense_prefers_tiles(int M, int V) { return M >= 8 && V >= 2 * kMaxWorkgroups * kTileRows; }

// Which path a call takes, decided in one place for the entry points and the path query.
struct PathPlan {
    int path;            // 0 general, 1 single launch, 2 tiles, -1 none (the staged kernels'
                         // token batch and lists do not fit LDS: rows beyond about 10 K values)
    int tile_umax, tile_lds;
    bool tile_kernels;   // paths 0 and 2: the tile kernels run (path 0: else the staged ones)
    bool tile_small;     // ... with blocks of 32 rows
};

bool staged_fits(int M, int jp, int k) {
    return logits_lds_bytes(M < kTokBatch ? M : kTokBatch, jp, k) <= (size_t)kLdsLimit;
}

// Dense heads that fit the single launch: whether the tile kernels' general form takes less time, by
// estimates in us fitted to 1200 heads of 8 to 152 K rows and 64 to 4096 columns, 16 to 31 tokens (fp32: 24
// to 32), new weights in every call (root mean square error 4 to 5 %).  The single launch dots every row
// with every token on the vector units (rows padded to its segments of 64 vectors); the tile kernels take
// whole rounds of 128-row blocks, chunk by chunk, whatever the tokens, less with one token tile, and their
// weights' stream is slower where rows are no whole 128-byte lines.  (fp32: few blocks take less than
// estimated, hence the form of the line.)  Over these heads times are 0.75 of the single launch's (fp32 0.88),
// 5 and 9 of them more than 2 % above it, the worst 1.09 and 1.11; with all of them on the tile kernels 37 and
// 68 were, the worst 1.28 and 1.50.  bf16 H = 1024, V = 38654, 26 tokens 54 on the single launch, 28 on the
// tiles; H = 1736, V = 11449, 18 tokens, k = 33 29, 37 (90 blocks); H = 2320, V = 33780, 19 tokens 61, 67 (264
// blocks, a second round for eight); fp32 H = 944, V = 33304, 26 tokens 54, 70.  The general form's sums
// are as exact as the vector units': 3.4e-8 against 4.4e-8 off.
// Fewer than 8192 rows or 16 tokens (fp32 24) stay on the single launch: up to there such calls have been
// moved, which is not where the two cross.  Measured on the other side, all on the tile kernels: 16 bits, 12
// tokens 0.97 of the single launch's time on average, 0.75 to 1.32, 14 tokens 0.88, 0.66 to 1.35; below 8192
// rows 16 tokens 1.07, 24 tokens 0.88; fp32 16 tokens 1.10, 23 tokens 0.96; below 8192 rows 24 tokens 1.34.
bool general_tiles_faster(int M, int V, int n_vec, int k, coral_dtype dt) {
    const int blocks = (V + kTileRows - 1) / kTileRows;
    const double chunks = (n_vec + kChunkVecs - 1) / kChunkVecs;
    const double steps = (blocks + kMaxWorkgroups - 1) / kMaxWorkgroups * chunks;      // chunks of a workgroup
    const double mb = (double)V * n_vec * 16e-6, odd_mb = n_vec % 8 != 0 ? mb : 0.0;
    const double rows = (double)M * V * 1e-6, dots = rows * 1e-3 * chunks * kWave;
    if (is_16bit(dt))
        return 10.4 + (M <= 16 ? 2.05 : 3.0) * steps + 3.3 * blocks / kMaxWorkgroups + 0.074 * mb + 0.043 * odd_mb + 0.164 * k <
               0.97 * (8.0 + 0.39 * M + 133.0 * dots + 10.4 * rows + 0.051 * mb + 0.097 * k);
    return 11.0 + 5.4 * steps + 4.1 * blocks / kMaxWorkgroups + 0.066 * mb + 0.03 * odd_mb + 0.15 * k <
           4.0 + 0.9 * (7.7 + 0.42 * M + 98.0 * dots + 7.3 * rows + 0.041 * mb + 0.097 * k);
}

// The static scratch array (logit ranking only, no table of pieces).  Which shapes it takes is a
// matter of sizes that callers rely on, and does not move with the kernels that run them: the
// published and the staged lists must fit; or, for 16-bit heads of whole 512-column chunks whose rows
// are beyond 8 KB or whose tokens and lists do not share the LDS of a workgroup with 24 KB for
// merges, the tile path's arrays with 128-row blocks.
size_t static_counted_bytes(int M, int H, int V, int G, int g, int k, coral_dtype dt) {
    int um, lds;
    bool tiles = tiles_fit(M, H, V, G, g, k, dt, &um, &lds);
    const int jp = (H / (is_16bit(dt) ? 8 : 4) + kWave - 1) / kWave;
    if (tiles && jp <= 8) {
        const FusedLds F = fused_lds_layout(M, G, g, k, jp, false, fused_gate_mode(false, M, G, g, k, jp, dt));
        const int hidden = M * hidden_lds_stride(jp) * (int)sizeof(uint4), merges = 24 * 1024;
        tiles = F.total - F.o_lists + (hidden > merges ? hidden : merges) > kLdsLimit;
    }
    return make_layout(M, V, G, g, k, Pieces{}, {tiles ? Tiles::kOwn : Tiles::kNone, false},
                       tiles ? LayoutFor::kCounted : LayoutFor::kWorkspace).total - kGateScoreBytes;
}

// Grouped heads that fit the single launch, with many tokens: whether the tile kernels take less time.  16 bits,
// from 37 tokens on (the single launch dots every row with each of its group's tokens on the vector units and
// ranks every token's candidates in every workgroup).  Up to 49 tokens, and nine to a group, not where
//   - one or two candidates are wanted (the single launch's ranking goes by k) and a row is more than one chunk,
//     or part of one and the blocks more than one round over the compute units, or
//   - the last chunk is partly filled (it costs as much as a whole one), there are about two rounds of chunks over
//     the compute units or more, and two tokens or more to a group.
// Single launch against tiles over 5500 random heads of 8 to 152 K rows, 8 to 1024 groups and 256 to 1096 columns:
// 1.47 times as fast on average, the worst 0.97, over 1000 more the worst 0.93 (us: bf16 H = 256, 48720 rows, 53
// tokens 41, 28; H = 512, 150991 rows, one of 28 groups, 37 tokens 40, 43); in the two exceptions, 7 in a hundred
// heads, 1.19, but down to 0.86 (f16 H = 776, 38275 rows, 41 tokens, k = 1 35, 41; bf16 H = 488, 125086 rows, 37
// tokens 44, 50).  33 to 36 tokens 1.18, 0.87 to 1.4 (H = 816, 146627 rows, 35 tokens 71, 82); 25 to 32 tokens
// 1.07, 0.85 to 1.40; up to 16 tokens 0.80; fp32 0.87.  Not where the entry point without a workspace
// would have to go through the tokens in batches, reading the weights again for each.
bool grouped_tiles_faster(int M, int H, int V, int G, int g, int k, coral_dtype dt) {
    if (!is_16bit(dt) || V < 8192 || H < 256 || M < 37) return false;
    const int chunk = kChunkVecs * 8, chunks = (H + chunk - 1) / chunk;
    const double group_tokens = M * g / expected_groups(M, G, g);
    if (M < 50 && group_tokens <= 9.0) {
        const bool part = H % chunk != 0;
        if (k <= 2 && (chunks > 1 || (part && V > kMaxWorkgroups * kTileRows))) return false;
        if (part && group_tokens >= 1.8 && (long long)V * chunks > 62000) return false;
    }
    const Tiles kind = H % (kChunkVecs * 8) == 0 ? Tiles::kOwn : Tiles::kGeneral;
    return make_layout(M, V, G, g, k, Pieces{}, {kind, false}, LayoutFor::kTiles).total <= kStaticArrayBytes ||
           static_counted_bytes(M, H, V, G, g, k, dt) > kStaticScratchBytes;
}

// The general path takes what the other two do not: fp32 rows beyond the single-launch kernel,
// widths that are no multiple of 512, more than 64 groups with log-probabilities.  It runs the
// tile kernels too, whose column tail is then guarded and whose fp32 form multiplies in full fp32
// (v_mfma_f32_16x16x4_f32), wherever these fit; the staged kernels stay for what is left (weights
// of 4 GiB and more, hundreds of activated groups).  The staged kernels stage eight tokens at a
// time and read a group's rows again for every eight, and their last merge is one workgroup per
// token over every chunk's list: fp32 H = 768, 58 tokens 319 us against 61 us here; 16-bit
// H = 5432, 43 tokens, log-probabilities 529 against 160; 16-bit H = 1664, 40 tokens 97 against 35.
PathPlan plan_path_kind(bool dense, int M, int H, int V, int G, int g, int k, coral_dtype dt, bool logprob) {
    PathPlan pl = {};
    const int n_vec = H / (is_16bit(dt) ? 8 : 4);
    const int jp = (n_vec + kWave - 1) / kWave;
    if (logprob) {     // the single-launch kernel, else the tile path, else the general path
        pl.path = staged_fits(M, jp, k) ? 0 : -1;
        if (dense) return pl;
        if (logprob_takes_fused(M, H, V, G, g, k, jp, dt)) {
            pl.path = 1;
        } else if (tiles_fit(M, H, V, G, g, k, dt, &pl.tile_umax, &pl.tile_lds) && G <= kWave) {
            pl.path = 2;                    // (more than 64 groups: the general path, whose form of the
                                            // same kernels serves any number; not measured in this one)
        }
        return pl;
    }
    const bool fused_ok =
        fused_rows_fit(n_vec) &&
        (dense ? jp != 9 || nine_segs_take_fused_dense(M, H, V, k, dt)
               : jp <= 8 || long_rows_take_fused(M, H, V, G, g, k, dt, false)) &&
        fused_lds_layout(M, dense ? 0 : G, dense ? 0 : g, k, jp, dense,
                         fused_gate_mode(dense, M, dense ? 0 : G, dense ? 0 : g, k, jp, dt)).total <= kLdsLimit;
    const bool tiles_ok =
        tiles_fit(M, H, V, dense ? 0 : G, dense ? 0 : g, k, dt, &pl.tile_umax, &pl.tile_lds);
    // (Many tokens: also where the single launch could not collect its candidates and would keep
    // sorted lists, every logit of every token against them: dense bf16 H = 1024, V = 58000, 40
    // tokens 323 us, tile kernels 37; H = 4096, 16 tokens 164, 91; grouped bf16 H = 512, V = 128256,
    // 64 tokens, 2 of 4 groups 435, 52.  Equal groups: what is decided here depends on sizes only.)
    bool single;
    const bool lists = M >= (dense ? 16 : 32) && fused_ok &&
                       !collect_cap(dense, M, dense ? 0 : G, dense ? 0 : g, k, jp,
                                    fused_gate_mode(dense, M, G, g, k, jp, dt), dense ? V : (V + G - 1) / G,
                                    kMaxWorkgroups, &single);
    const bool many = fused_ok && (dense ? V >= 8192 && M >= (is_16bit(dt) ? 16 : 24) && general_tiles_faster(M, V, n_vec, k, dt)
                                         : grouped_tiles_faster(M, H, V, G, g, k, dt));
    if (((dense ? dense_prefers_tiles(M, V) : many) || lists) && tiles_ok)
        pl.path = 2;
    else if ((lists || many) && tile_kernels_fit(M, H, V, dense ? 0 : G, dense ? 0 : g, k, dt, &pl.tile_umax, &pl.tile_lds))
        pl.path = 0;
    else if (fused_ok)
        pl.path = 1;
    else if (tiles_ok)
        pl.path = 2;
    else
        pl.path = staged_fits(M, jp, k) ? 0 : -1;
    return pl;
}

// Blocks of 32 rows instead of 128, where the rows of the groups that the tokens activate fill fewer
// 128-row blocks than half of the compute units, a group's tokens fit one token tile on average
// (every block stages them again, against a quarter of the weight bytes) and a row is long (a block's
// start and end, about 4 us, against its chunks).  Measured, 128 rows against 32: bf16 H = 4608, 16
// tokens, dense 4000 rows 35 against 23 us, 16000 rows 44 against 42, 18000 rows 43 against 52; over
// 730 heads with 8 to 18 chunks the mean ratio is 0.7 up to 80 blocks, 0.9 from there on and 1.1
// beyond 138.  Groups far from a multiple of 128 rows leave larger blocks empty: fp32 H = 2432, 76
// groups of 133 rows, 48 tokens 121 against 61.  The other way round bf16 H = 1664, 13 groups of 2005
// rows, 40 tokens 35 against 48; dense f16 H = 5632, 62 tokens 64 against 173.
bool tile_small_blocks(int V, int g, double rows, long long group_tokens, int n_chunks) {
    return rows < kMaxWorkgroups / 2 * kTileRows && group_tokens <= 16 && n_chunks >= 8 &&
           V / kTileRowsSmall + g + 1 <= (1 << 16) &&
           tile_select_lds_layout(g > 0 ? g : 1, V / kTileRowsSmall + g + 1).total <= kLdsLimit;
}

// The general path's steps that the staged kernels run faster than the tile kernels (`rows`: rows of
// the activated groups at most):
//   - one batch of tokens and fewer 128-row blocks than compute units, as their 32-row chunks spread
//     over more of these: fp32 H = 2304, one token, one group of 710 rows 32 us staged, 54 tiles;
//   - k <= 16 (their merges go by whole lists: dense bf16 H = 4136, one token, k = 64 720, 370) and a
//     few (token, group) pairs, hardly any of them in the same group: fp32 H = 2304, 9 tokens, one
//     of 300 groups each 28, 37; but one of 32 groups of 187 rows each 41, 32;
//   - rows beyond 8 KB that leave a chunk partly filled (whole ones: fp32 H = 4352, 12 groups of 7223
//     rows, 12 tokens 242, 170), up to two tokens per group, more than one round of blocks, k <= 10
//     (k = 16: H = 4352, 7 groups, 3 tokens 144, 101).  The tile kernels' time goes by whole rounds of
//     blocks, whatever the tokens; the staged kernels stream rows as they come, at a cost per token,
//     and their gate and selection grow with tokens x groups (fp32 most: H = 2304, 128 groups, 8
//     tokens 141, 108; 300 groups, 48 tokens 193, 110).  us, staged against tiles, bf16: H = 4104,
//     128256 rows, 32 groups, 4 tokens 103, 125, 8 tokens 156, 183, 14 tokens 225, 210, 33 tokens 383,
//     275; H = 4360, 16 groups, 14 tokens 236, 260; H = 8200, 3 tokens 152, 228; 128 groups, 10 tokens
//     177, 224, but with 50176 rows in all (one round), 14 tokens 130, 118; fp32 H = 3332, V = 99984,
//     2 of 48 groups, 9 tokens 134, 188; dense H = 8200, 50257 rows, one token 178, 226, 3 tokens
//     197, 226, 4 tokens 230, 226; dense H = 4104, 2 tokens 121, 120, 4 tokens 143, 118.
bool staged_preferred(bool dense, int M, int H, int V, int G, int g, int k, coral_dtype dt, long long rows) {
    const int jp = (H / (is_16bit(dt) ? 8 : 4) + kWave - 1) / kWave;
    if (!staged_fits(M, jp, k)) return false;
    if (M <= kTokBatch && rows < (long long)kMaxWorkgroups * kTileRows) return true;
    if (k > 16) return false;
    if (!dense && M * g <= 12 && M * g <= 1.1 * expected_groups(M, G, g)) return true;
    if (jp <= 8 || H % (kChunkVecs * (is_16bit(dt) ? 8 : 4)) == 0) return false;
    if (dense) return M <= (jp > 16 ? 3 : 2);
    return k <= 10 && M <= 24 && M * g <= 2.1 * expected_groups(M, G, g) && M * G <= (is_16bit(dt) ? 3072 : 800) &&
           expected_blocks(M, V, G, g) > kMaxWorkgroups - 6;
}

PathPlan plan_path(bool dense, int M, int H, int V, int G, int g, int k, coral_dtype dt, bool logprob = false) {
    PathPlan pl = plan_path_kind(dense, M, H, V, G, g, k, dt, logprob);
    const long long rows = dense ? V : max_union(M, G, g) * V / (G > 0 ? G : 1);
    pl.tile_kernels = pl.path == 2 || (pl.path == 0 && !staged_preferred(dense, M, H, V, G, g, k, dt, rows) &&
                                       tile_kernels_fit(M, H, V, dense ? 0 : G, dense ? 0 : g, k, dt, &pl.tile_umax, &pl.tile_lds));
    const long long groups = dense ? 1 : max_union(M, G, g);
    const int n_chunks = (H / (is_16bit(dt) ? 8 : 4) + kChunkVecs - 1) / kChunkVecs;
    pl.tile_small = pl.tile_kernels && groups > 0 &&
                    tile_small_blocks(V, dense ? 0 : g, dense ? V : expected_groups(M, G, g) * V / G,
                                      dense ? M : ((long long)M * g + groups - 1) / groups, n_chunks);
    return pl;
}

// Whether a call with these sizes (grouped in either output mode, or dense when G = 0) can run
// the tile kernels: the workspace then holds their logits buffer.
TileArrays layout_tiles(int M, int H, int V, int G, int g, int k, coral_dtype dt) {
    if (!dtype_ok(dt) || H % (is_16bit(dt) ? 8 : 4) != 0) return {Tiles::kNone, false};
    const PathPlan plans[3] = {plan_path(true, M, H, V, 0, 0, k, dt),
                               G < 1 ? PathPlan{-1} : plan_path(false, M, H, V, G, g, k, dt),
                               G < 1 ? PathPlan{-1} : plan_path(false, M, H, V, G, g, k, dt, true)};
    TileArrays t = {Tiles::kNone, false};
    for (const PathPlan& p : plans) {
        if (p.path == 2) t.kind = Tiles::kOwn;
        else if (p.path == 0 && p.tile_kernels && t.kind == Tiles::kNone) t.kind = Tiles::kGeneral;
        t.small = t.small || p.tile_small;
    }
    return t;
}

// From how many activated rows on k_tiles reads the weights past the caches (non-temporal): 0 always,
// INT_MAX never.  Few rows are read through them, as a draft loop's next step may find them in the
// last-level cache; that costs where it does not, from 128 MB on more than it gives where it does.  us,
// through the caches against past them, new weights in every step and the same: two of 32 groups, H = 5120, 95
// MB 46.1, 43.8 and 35.4, 41.1, 177 MB 60.1, 55.9 and 54.7, 58.1; three of 48, H = 2560, 80 MB 41.0, 39.6
// and 38.5, 40.7, 165 MB 57.6, 52.9 and 51.0, 53.3, 238 MB 70.7, 64.2 and 59.6, 63.6; H = 8192, 410 MB
// 111.7, 100.1 and 106.2, 93.1.  The kernel counts the rows (what tokens activate goes by the scores: with
// a router's bias of N(0, 2^2) 80 MB of the 197 that they would draw by lot).  In any case through the
// caches: rows that are no whole 128-byte lines (a line is then wanted by two loads of a wave, the second of
// which should find it: dense H = 5680, 22 tokens 165 us past the caches, 146 through them, H = 2280, 13
// tokens 32.0, 22.5), and blocks that come round again for the next 32 tokens (fp32 H = 1536, 43 tokens,
// 484 MB 245, 228).  In any case past them: blocks of 32 rows, whose waves read longer runs of a row (H =
// 5120, 35 tokens 53.5, 56.2), and the dense head's consecutive rows of whole chunks (new weights in every
// step, 24 tokens, H = 1536, 201 MB 51.6, 47.0, H = 512, 67 MB 30.6, 29.1).
int tile_stream_rows(bool dense, bool general, bool small, int M, int G, int g, int n_vec) {
    if (n_vec % 8 != 0) return INT_MAX;
    if (small || (dense && !general)) return 0;
    if (general && (dense ? M : M * g / expected_groups(M, G, g)) > 32.0) return INT_MAX;
    return (int)(128000000 / (n_vec * 16)) + 1;
}

// Enqueues k_tiles and the ranking of the logits it leaves.  For the grouped head the gate
// and selection kernel must already be enqueued (selection, the token tiles' masks; in the
// log-probability mode log p_router of the selection too).
coral_status launch_tiles(bool dense, const PathPlan& plan, const void* hidden, const void* lm_W,
                          const coral_group_index* gi, int M, int H, int V,
                          int G, int k, coral_dtype dt, int32_t* topk_ids,
                          float* topk_out, char* ws, const Layout& L, hipStream_t stream,
                          void* ev_before, void* ev_after, const int32_t* sel = nullptr, int g = 0,
                          bool logprob = false, bool halves = true) {
    int P = compute_units();
    if (P < 1) return CORAL_ERR_HIP;
    if (P > kMaxWorkgroups) P = kMaxWorkgroups;
    TileParams p = {};
    p.hidden = static_cast<const uint4*>(hidden);
    p.lm_W = static_cast<const uint4*>(lm_W);
    p.rows = gi ? gi->group_rows : nullptr;
    p.offsets = gi ? gi->group_offsets : nullptr;
    p.tile_mask = reinterpret_cast<const unsigned long long*>(ws + L.tile_mask);
    p.group_mask = reinterpret_cast<unsigned long long*>(ws + L.mask);
    p.group_first_block = reinterpret_cast<int32_t*>(ws + L.tile_first_block);
    p.z = reinterpret_cast<float*>(ws + L.tile_z);
    p.stat = reinterpret_cast<float2*>(ws + L.tile_stat);
    p.stat_upper = reinterpret_cast<float2*>(ws + L.tile_upper);
    p.split_from = reinterpret_cast<int32_t*>(ws + L.n_union);
    p.halves = halves ? 1 : 0;
    p.want_lse = logprob ? 1 : 0;
    p.next_block = reinterpret_cast<unsigned int*>(ws + L.ctrl) + coral_ctrl::kTileQueue;
    p.M = M; p.V = V; p.G = G;
    p.n_vec = H / (is_16bit(dt) ? 8 : 4);
    p.n_chunks = (p.n_vec + kChunkVecs - 1) / kChunkVecs;
    p.u_max = plan.tile_umax;
    typedef void (*tiles_fn)(TileParams, int);
    const bool small = plan.tile_small, general = plan.path == 0;
    const int lds = plan.tile_lds;
    const int rows_per_block = small ? kTileRowsSmall : kTileRows;
    p.stream_rows = tile_stream_rows(dense, general, small, M, G, g, p.n_vec);
    const tiles_fn fn =
        small     ? CORAL_PICK_DT(dt, (k_tiles<kF32, true, kTileSplitSmall>), (k_tiles<kBF16, true, kTileSplitSmall>), (k_tiles<kF16, true, kTileSplitSmall>))
        : general ? CORAL_PICK_DT(dt, (k_tiles<kF32, true, kTileSplit>), (k_tiles<kBF16, true, kTileSplit>), (k_tiles<kF16, true, kTileSplit>))
        : dt == CORAL_F16 ? k_tiles<kF16, false, kTileSplit> : k_tiles<kBF16, false, kTileSplit>;
    if (!allow_lds(reinterpret_cast<const void*>(fn), lds)) return CORAL_ERR_HIP;
    coral_status st;
    if ((st = launch_timed(fn, dim3(P), dim3(kTileBlock), lds, stream, ev_before, ev_after, p, dense ? 1 : 0)) !=
        CORAL_OK)
        return st;

    TileSelectParams q = {};
    q.z = p.z;
    q.stat = p.stat;
    q.stat_upper = p.stat_upper;
    q.split_from = p.split_from;
    q.sel = sel;
    q.offsets = p.offsets;
    q.rows = p.rows;
    q.group_first_block = p.group_first_block;
    q.group_mask = p.group_mask;
    q.logp_sel = reinterpret_cast<const float*>(ws + L.logp_sel);
    q.next_block = p.next_block;
    q.topk_ids = topk_ids;
    q.topk_out = topk_out;
    q.M = M; q.V = V; q.g = g; q.k = k;
    q.max_blocks = V / rows_per_block + g + 1;
    static_assert(kTileRowsSmall == 1 << 5 && kTileRows == 1 << 7, "");
    const int select_lds = tile_select_lds_layout(dense ? 1 : g, q.max_blocks).total;
    typedef void (*select_fn)(TileSelectParams);
    const select_fn sf =
        dense     ? (small ? k_tile_select<true, false, 5> : k_tile_select<true, false, 7>)
        : logprob ? (small ? k_tile_select<false, true, 5> : k_tile_select<false, true, 7>)
                  : (small ? k_tile_select<false, false, 5> : k_tile_select<false, false, 7>);
    if (!allow_lds(reinterpret_cast<const void*>(sf), select_lds)) return CORAL_ERR_HIP;
    hipLaunchKernelGGL(sf, dim3(M), dim3(kSelectThreads), select_lds, stream, q);
    return launch_status();
}

}  // namespace

// Yardstick for the bench line: a kernel that only reads, in the single-launch path's shape.
// One workgroup per compute unit, `waves` waves each; a wave takes consecutive 16 KB pieces
// dealt round robin over waves and workgroups, 16 non-temporal 1 KB loads in flight per piece.
namespace {
__global__ __launch_bounds__(kFusedBlock) void k_probe_read(const uint4* __restrict__ src, unsigned long long pieces) {
    const int lane = threadIdx.x & (kWave - 1);
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x / kWave);
    const unsigned long long stride = (unsigned long long)gridDim.x * (blockDim.x / kWave);
    unsigned x = 0u;
    for (unsigned long long q = (unsigned long long)blockIdx.x * (blockDim.x / kWave) + wave; q < pieces; q += stride) {
        const uint4* p = src + q * 1024 + lane;
        uint4 v[16];
#pragma unroll
        for (int i = 0; i < 16; ++i) v[i] = load_stream(p + i * kWave);
#pragma unroll
        for (int i = 0; i < 16; ++i) x ^= v[i].x ^ v[i].y ^ v[i].z ^ v[i].w;
    }
    asm volatile("" ::"v"(x));                          // (keeps the loads: nothing is written)
}
}  // namespace

extern "C" coral_status coral_probe_read(const void* src, size_t bytes, int waves, void* hip_stream,
                                         void* ev_before, void* ev_after) {
    if (!src || !ev_before || !ev_after) return CORAL_ERR_NULL;
    if (bytes < 16384 || bytes % 16384 != 0 || waves < 1 || waves > kFusedWaves) return CORAL_ERR_SHAPE;
    if ((uintptr_t)src & 15u) return CORAL_ERR_UNSUPPORTED;
    int P = compute_units();
    if (P < 1) return CORAL_ERR_HIP;
    if (P > kMaxWorkgroups) P = kMaxWorkgroups;
    return launch_timed(k_probe_read, dim3(P), dim3(waves * kWave), 0, static_cast<hipStream_t>(hip_stream),
                        ev_before, ev_after, static_cast<const uint4*>(src), (unsigned long long)(bytes / 16384));
}

extern "C" const char* coral_status_string(coral_status st) {
    switch (st) {
        case CORAL_OK: return "ok";
        case CORAL_ERR_NULL: return "a required pointer is NULL";
        case CORAL_ERR_SHAPE: return "a size is out of range or inconsistent";
        case CORAL_ERR_GROUP_INDEX: return "the group index is not a partition of the vocabulary";
        case CORAL_ERR_UNSUPPORTED: return "request outside the kernels' stated limits";
        case CORAL_ERR_WORKSPACE: return "workspace missing, misaligned or too small";
        case CORAL_ERR_HIP: return "the HIP runtime refused a launch";
    }
    return "unknown status";
}

extern "C" coral_status coral_group_index_validate(const int32_t* host_offsets,
                                                   const int32_t* host_rows, int G, int V) {
    if (!host_offsets || !host_rows) return CORAL_ERR_NULL;
    if (G < 1 || V < 1) return CORAL_ERR_SHAPE;
    if (host_offsets[0] != 0 || host_offsets[G] != V) return CORAL_ERR_GROUP_INDEX;
    for (int n = 0; n < G; ++n)
        if (host_offsets[n + 1] < host_offsets[n]) return CORAL_ERR_GROUP_INDEX;
    unsigned char* seen = static_cast<unsigned char*>(calloc((size_t)V, 1));
    if (!seen) return CORAL_ERR_SHAPE;
    coral_status st = CORAL_OK;
    for (int i = 0; i < V; ++i) {
        const int32_t r = host_rows[i];
        if (r < 0 || r >= V || seen[r]) {
            st = CORAL_ERR_GROUP_INDEX;
            break;
        }
        seen[r] = 1;
    }
    free(seen);
    return st;
}

extern "C" size_t coral_lmhead_workspace_bytes(int M, int H, int V, int G, int g, int k,
                                               coral_dtype dt) {
    if (!sizes_ok(M, H, V, G, g, k)) return 0;
    // (fewer tokens can need more, where they take a route with larger arrays)
    size_t most = 0;
    for (int m = M; m >= 1; m = m > kMaxM ? kMaxM : m - 1) {
        const size_t need = make_layout(m, V, G, g, k, layout_pieces(m, H, V, G, g, k, dt),
                                        layout_tiles(m, H, V, G, g, k, dt)).total;
        if (need > most) most = need;
    }
    return most;
}

extern "C" int coral_lmhead_path(int dense, int M, int H, int V, int G, int g, int k,
                                 coral_dtype dt) {
    if (!dtype_ok(dt)) return -1;
    if (M < 1 || H < 1 || V < 1 || k < 1 || M > kMaxM || k > kMaxK) return -1;
    if (H % (is_16bit(dt) ? 8 : 4) != 0) return -1;
    if (!dense && (G < 1 || g < 1 || g > G || G > kMaxG)) return -1;
    return plan_path(dense != 0, M, H, V, G, g, k, dt).path;
}

extern "C" int coral_lmhead_logprob_path(int M, int H, int V, int G, int g, int k, coral_dtype dt) {
    if (coral_lmhead_path(0, M, H, V, G, g, k, dt) < 0) return -1;
    return plan_path(false, M, H, V, G, g, k, dt, true).path;
}

extern "C" coral_status coral_lmhead_workspace_init(void* workspace, size_t workspace_bytes,
                                                    void* hip_stream) {
    coral_status st = check_workspace(workspace, workspace_bytes, kCtrlBytes);
    if (st != CORAL_OK) return st;
    return prepare_words(workspace, workspace_bytes, static_cast<hipStream_t>(hip_stream));
}

namespace {

// The tile kernels' arrays for M tokens in the static scratch.
Layout static_tiles_layout(const PathPlan& plan, int M, int V, int G, int g, int k) {
    return make_layout(M, V, G, g, k, Pieces{}, {plan.path == 2 ? Tiles::kOwn : Tiles::kGeneral, plan.tile_small},
                       LayoutFor::kTiles);
}

// The arrays of the kernels that run a call, in the static scratch.  The tile kernels' may be more
// than the call is counted by: then they run for the tokens in equal batches, which leaves every bit
// of a token's result as it is where no block is processed in halves (one token's arrays fit: 4 V bytes
// of logits, with V limited by the ranking kernel's LDS).
Layout static_layout(const PathPlan& plan, int M, int V, int G, int g, int k, int* batch) {
    *batch = M;
    if (plan.path == 1) return make_layout(M, V, G, g, k, Pieces{}, TileArrays{}, LayoutFor::kSingleLaunch);
    if (!plan.tile_kernels) return make_layout(M, V, G, g, k, Pieces{}, TileArrays{});
    Layout L = {};
    for (int n = 1; n <= M; ++n) {
        *batch = (M + n - 1) / n;
        L = static_tiles_layout(plan, *batch, V, G, g, k);
        if (L.total <= kStaticArrayBytes) break;
    }
    return L;
}

// Whether the grouped head's blocks may be processed in halves.  A half's columns are summed in four
// parts instead of two, so its logits round differently, and which blocks are halved goes by the groups
// of all tokens of a launch.  Shapes whose tokens go in batches in the static scratch are therefore never
// halved, there and with a workspace, and give the same bits either way.  (bf16 H = 1024, V = 100000, two
// of eight groups, 64 tokens in four batches; the log-probability mode has no static form.)
bool tiles_take_halves(const PathPlan& plan, int M, int H, int V, int G, int g, int k, coral_dtype dt) {
    return plan.path != 2 || static_tiles_layout(plan, M, V, G, g, k).total <= kStaticArrayBytes ||
           static_counted_bytes(M, H, V, G, g, k, dt) > kStaticScratchBytes;
}

coral_status grouped_impl(const void* hidden, const void* gate_hidden, const void* gate_W,
                          const float* gate_bias, const void* lm_W, const coral_group_index* gi, int M, int H, int V,
                          int g, int k, coral_dtype dt, int32_t* topk_ids, float* topk_logits,
                          int32_t* sel_groups, void* workspace, size_t workspace_bytes,
                          void* hip_stream, void* ev_before, void* ev_after, bool logprob,
                          const LevelExpand* level = nullptr, bool static_workspace = false) {
    if (!gate_W || !gi) return CORAL_ERR_NULL;
    coral_status st = check_common(hidden, lm_W, M, H, V, k, dt, topk_ids, topk_logits);
    if (st != CORAL_OK) return st;
    if (!gi->group_offsets_host || !gi->group_offsets || !gi->group_rows) return CORAL_ERR_NULL;
    const int G = gi->G;
    if (G < 1 || g < 1 || g > G) return CORAL_ERR_SHAPE;
    if (G > kMaxG) return CORAL_ERR_UNSUPPORTED;
    if (!gate_hidden) gate_hidden = hidden;      // the router sees what the LM head sees
    if (((uintptr_t)gate_W | (uintptr_t)gate_hidden) & 15u) return CORAL_ERR_UNSUPPORTED;
    const int32_t* off = gi->group_offsets_host;
    if (off[0] != 0 || off[G] != V) return CORAL_ERR_GROUP_INDEX;
    int max_rows = 0;
    // the g smallest groups bound the number of candidates a token can have
    int smallest[kMaxG];
    for (int n = 0; n < G; ++n) {
        const int len = off[n + 1] - off[n];
        if (len < 0) return CORAL_ERR_GROUP_INDEX;
        if (len > max_rows) max_rows = len;
        smallest[n] = len;
    }
    long long min_cand = 0;
    for (int i = 0; i < g; ++i) {           // partial selection sort, g <= G <= 1024
        int best = i;
        for (int n = i + 1; n < G; ++n)
            if (smallest[n] < smallest[best]) best = n;
        const int tmp = smallest[i];
        smallest[i] = smallest[best];
        smallest[best] = tmp;
        min_cand += smallest[i];
    }
    if ((long long)k > min_cand) return CORAL_ERR_SHAPE;
    PathPlan plan = plan_path(false, M, H, V, G, g, k, dt, logprob);
    Layout L;
    int tile_tokens = M;                       // tokens that the tile kernels take at a time
    if (static_workspace) {
        if (logprob || static_counted_bytes(M, H, V, G, g, k, dt) > kStaticScratchBytes) return CORAL_ERR_WORKSPACE;
        L = static_layout(plan, M, V, G, g, k, &tile_tokens);
        if (L.total > kStaticArrayBytes) return CORAL_ERR_WORKSPACE;               // not reached
    } else {
        L = make_layout(M, V, G, g, k, layout_pieces(M, H, V, G, g, k, dt), layout_tiles(M, H, V, G, g, k, dt));
        st = check_workspace(workspace, workspace_bytes, L.total);
        if (st != CORAL_OK) return st;
    }

    hipStream_t stream = static_cast<hipStream_t>(hip_stream);
    if (logprob && plan.path == 1) {   // a device with few compute units: see fused_logprob_fits
        const int cu = compute_units();
        if (2 * max_union(M, G, g) > (cu < kMaxWorkgroups ? cu : kMaxWorkgroups))
            plan.path = staged_fits(M, ((H / (is_16bit(dt) ? 8 : 4)) + kWave - 1) / kWave, k) ? 0 : -1;
    }
    if (plan.path < 0) return CORAL_ERR_UNSUPPORTED;       // before anything is enqueued
    if (static_workspace) {
        // this device's copy of the array; its control words are prepared by a fill kernel on
        // the call's stream (the array keeps whatever the last call on this GPU left there); the
        // scores' words only where they are used (small heads 0.1 us)
        if ((st = static_scratch(&workspace)) != CORAL_OK) return st;
        const bool shared = plan.path == 1 && fused_gate_shared(M, G, H / (is_16bit(dt) ? 8 : 4), dt);
        if ((st = prepare_words(workspace, shared ? kStaticArrayBytes : kCtrlBytes, stream)) != CORAL_OK) return st;
    }
    char* ws = static_cast<char*>(workspace);
    if (plan.path == 1)
        return launch_fused(false, hidden, gate_hidden, gate_W, gate_bias, lm_W, gi, M, H, V, G, g, k, dt, topk_ids,
                            topk_logits, sel_groups, ws, L, stream, ev_before, ev_after, logprob, level, max_rows);
    float* s = reinterpret_cast<float*>(ws + L.s);
    int32_t* sel = sel_groups ? sel_groups : reinterpret_cast<int32_t*>(ws + L.sel);
    unsigned long long* mask = reinterpret_cast<unsigned long long*>(ws + L.mask);
    int32_t* union_list = reinterpret_cast<int32_t*>(ws + L.union_list);
    int32_t* n_union = reinterpret_cast<int32_t*>(ws + L.n_union);
    int32_t* chunk_base = reinterpret_cast<int32_t*>(ws + L.chunk_base);
    Cand* part = reinterpret_cast<Cand*>(ws + L.part);

    const int n_vec = H / (is_16bit(dt) ? 8 : 4);
    const uint4* hid = static_cast<const uint4*>(hidden);
    const uint4* ghid = static_cast<const uint4*>(gate_hidden);
    const uint4* gw = static_cast<const uint4*>(gate_W);
    if (plan.tile_kernels) {
        const int tiles_g = (G + 15) / 16;
        typedef void (*gate_select_fn)(GateSelParams);
        const gate_select_fn gs = CORAL_PICK_DT(dt, k_gate_select<kF32>, k_gate_select<kBF16>, k_gate_select<kF16>);
        const bool halves = logprob || tiles_take_halves(plan, M, H, V, G, g, k, dt);
        for (int m0 = 0; m0 < M; m0 += tile_tokens) {          // (one turn but for the static scratch)
            const int m = M - m0 < tile_tokens ? M - m0 : tile_tokens;
            int32_t* sel_m = sel_groups ? sel + (size_t)m0 * g : sel;
            GateSelParams q = {};
            q.hidden = ghid + (size_t)m0 * n_vec;
            q.gate_W = gw; q.bias = gate_bias; q.s = s; q.sel = sel_m;
            q.tile_mask = reinterpret_cast<unsigned long long*>(ws + L.tile_mask);
            q.counters = reinterpret_cast<unsigned int*>(ws + L.ctrl) + coral_ctrl::kGateSelectArrival;
            q.M = m; q.G = G; q.g = g; q.n_vec = n_vec;
            if (logprob) q.logp_sel = reinterpret_cast<float*>(ws + L.logp_sel);
            hipLaunchKernelGGL(gs, dim3(tiles_g * ((m + 15) / 16), kGateParts), dim3(kFusedBlock), 0, stream, q);
            if ((st = launch_status()) != CORAL_OK) return st;
            st = launch_tiles(false, plan, hid + (size_t)m0 * n_vec, lm_W, gi, m, H, V, G, k, dt,
                              topk_ids + (size_t)m0 * k, topk_logits + (size_t)m0 * k, ws, L, stream, ev_before,
                              ev_after, sel_m, g, logprob, halves);
            if (st != CORAL_OK) return st;
        }
        if (!level) return CORAL_OK;
        return launch_tree_expand(*level, topk_ids, topk_logits, M, k, stream);
    }
    typedef void (*gate_fn)(const uint4*, const uint4*, const float*, int, int, int, float*);
    const gate_fn gate_kernel = CORAL_PICK_DT(dt, k_gate<kF32>, k_gate<kBF16>, k_gate<kF16>);
    hipLaunchKernelGGL(gate_kernel, dim3(G), dim3(kBlock), 0, stream, ghid, gw, gate_bias, M, G, n_vec, s);
    if ((st = launch_status()) != CORAL_OK) return st;
    float* logp_sel = logprob ? reinterpret_cast<float*>(ws + L.logp_sel) : nullptr;
    hipLaunchKernelGGL(k_select, dim3(1), dim3(kBlock), 0, stream, s, gi->group_offsets, M, G, g, sel,
                       mask, union_list, n_union, chunk_base, logp_sel,
                       logprob ? reinterpret_cast<int32_t*>(ws + L.slot_count) : nullptr);
    if ((st = launch_status()) != CORAL_OK) return st;

    LogitsParams p;
    p.hidden = hid;
    p.lm_W = static_cast<const uint4*>(lm_W);
    p.offsets = gi->group_offsets;
    p.rows = gi->group_rows;
    p.sel = sel;
    p.group_mask = mask;
    p.union_list = union_list;
    p.n_union = n_union;
    p.chunk_base = chunk_base;
    p.part = part;
    p.lse_part = logprob ? reinterpret_cast<float*>(ws + L.lse_part) : nullptr;
    p.M = M; p.V = V; p.G = G; p.g = g; p.k = k;
    p.n_vec = n_vec;
    p.jp = (n_vec + kWave - 1) / kWave;
    p.tb_max = M < kTokBatch ? M : kTokBatch;
    p.part_stride = L.part_stride;
    const size_t lds = logits_lds_bytes(p.tb_max, p.jp, k);       // fits: plan_path checked it
    const int chunks = (max_rows + kChunkRows - 1) / kChunkRows;
    const long long union_max = max_union(M, G, g);
    if (chunks < 1) return CORAL_ERR_SHAPE;
    dim3 grid(chunks, (unsigned)union_max);
    typedef void (*logits_fn)(LogitsParams);
    const logits_fn fn =
        logprob ? CORAL_PICK_DT(dt, (k_logits<kF32, false, true>), (k_logits<kBF16, false, true>),
                                (k_logits<kF16, false, true>))
                : CORAL_PICK_DT(dt, (k_logits<kF32, false, false>), (k_logits<kBF16, false, false>),
                                (k_logits<kF16, false, false>));
    if (!allow_lds(reinterpret_cast<const void*>(fn), (int)lds)) return CORAL_ERR_HIP;
    if ((st = launch_timed(fn, grid, dim3(kBlock), lds, stream, ev_before, ev_after, p)) != CORAL_OK) return st;
    if (logprob)
        hipLaunchKernelGGL(k_merge_logprob<4>, dim3(M), dim3(kBlock), 0, stream, part, p.lse_part,
                           L.part_stride, reinterpret_cast<const int32_t*>(ws + L.slot_count), chunk_base,
                           logp_sel, g, k, topk_ids, topk_logits);
    else
        hipLaunchKernelGGL(k_merge, dim3(M), dim3(kBlock), 0, stream, part, L.part_stride, sel,
                           gi->group_offsets, g, 0, k, topk_ids, topk_logits);
    if ((st = launch_status()) != CORAL_OK || !level) return st;
    // draft-level call on the multi-kernel path: the expansion is one more launch
    return launch_tree_expand(*level, topk_ids, topk_logits, M, k, stream);
}

coral_status dense_impl(const void* hidden, const void* lm_W, int M, int H, int V, int k,
                        coral_dtype dt, int32_t* topk_ids, float* topk_logits, void* workspace,
                        size_t workspace_bytes, void* hip_stream, void* ev_before,
                        void* ev_after) {
    coral_status st = check_common(hidden, lm_W, M, H, V, k, dt, topk_ids, topk_logits);
    if (st != CORAL_OK) return st;
    if (k > V) return CORAL_ERR_SHAPE;
    const Layout L = make_layout(M, V, 0, 0, k, Pieces{}, layout_tiles(M, H, V, 0, 0, k, dt));
    st = check_workspace(workspace, workspace_bytes, L.total);
    if (st != CORAL_OK) return st;

    hipStream_t stream = static_cast<hipStream_t>(hip_stream);
    char* ws = static_cast<char*>(workspace);
    const PathPlan plan = plan_path(true, M, H, V, 0, 0, k, dt);
    if (plan.path < 0) return CORAL_ERR_UNSUPPORTED;
    // many tokens per row: the contraction is no longer cheap on the vector units
    if (plan.tile_kernels)
        return launch_tiles(true, plan, hidden, lm_W, nullptr, M, H, V, 0, k, dt, topk_ids, topk_logits, ws, L,
                            stream, ev_before, ev_after);
    if (plan.path == 1)
        return launch_fused(true, hidden, nullptr, nullptr, nullptr, lm_W, nullptr, M, H, V, 0, 0, k, dt, topk_ids,
                            topk_logits, nullptr, ws, L, stream, ev_before, ev_after);
    LogitsParams p = {};
    p.hidden = static_cast<const uint4*>(hidden);
    p.lm_W = static_cast<const uint4*>(lm_W);
    p.part = reinterpret_cast<Cand*>(ws + L.part);
    p.M = M; p.V = V; p.G = 0; p.g = 0; p.k = k;
    p.n_vec = H / (is_16bit(dt) ? 8 : 4);
    p.jp = (p.n_vec + kWave - 1) / kWave;
    p.tb_max = M < kTokBatch ? M : kTokBatch;
    p.part_stride = L.part_stride;
    const size_t lds = logits_lds_bytes(p.tb_max, p.jp, k);
    const int chunks = (V + kChunkRows - 1) / kChunkRows;
    typedef void (*logits_fn)(LogitsParams);
    const logits_fn fn = CORAL_PICK_DT(dt, (k_logits<kF32, true>), (k_logits<kBF16, true>), (k_logits<kF16, true>));
    if (!allow_lds(reinterpret_cast<const void*>(fn), (int)lds)) return CORAL_ERR_HIP;
    if ((st = launch_timed(fn, dim3(chunks), dim3(kBlock), lds, stream, ev_before, ev_after, p)) != CORAL_OK) return st;
    hipLaunchKernelGGL(k_merge, dim3(M), dim3(kBlock), 0, stream, p.part, L.part_stride,
                       (const int32_t*)nullptr, (const int32_t*)nullptr, 0, chunks, k, topk_ids,
                       topk_logits);
    return launch_status();
}

}  // namespace

extern "C" coral_status coral_lmhead_grouped(const void* hidden, const void* gate_W,
                                             const float* gate_bias, const void* lm_W,
                                             const coral_group_index* gi, int M, int H, int V,
                                             int g, int k, coral_dtype dt, int32_t* topk_ids,
                                             float* topk_logits, int32_t* sel_groups,
                                             void* workspace, size_t workspace_bytes,
                                             void* hip_stream) {
    return grouped_impl(hidden, nullptr, gate_W, gate_bias, lm_W, gi, M, H, V, g, k, dt, topk_ids,
                        topk_logits, sel_groups, workspace, workspace_bytes, hip_stream, nullptr,
                        nullptr, false);
}

extern "C" coral_status coral_lmhead_grouped_noalloc(const void* hidden, const void* gate_W,
                                                     const float* gate_bias, const void* lm_W,
                                                     const coral_group_index* gi, int M, int H, int V,
                                                     int g, int k, coral_dtype dt, int32_t* topk_ids,
                                                     float* topk_logits, int32_t* sel_groups,
                                                     void* hip_stream) {
    return grouped_impl(hidden, nullptr, gate_W, gate_bias, lm_W, gi, M, H, V, g, k, dt, topk_ids,
                        topk_logits, sel_groups, nullptr, 0, hip_stream, nullptr, nullptr, false,
                        nullptr, true);
}

extern "C" coral_status coral_lmhead_grouped_routed(
    const void* hidden, const void* gate_hidden, const void* gate_W, const float* gate_bias,
    const void* lm_W, const coral_group_index* gi, int M, int H, int V, int g, int k,
    coral_dtype dt, int logprob, int32_t* topk_ids, float* topk_out, int32_t* sel_groups,
    void* workspace, size_t workspace_bytes, void* hip_stream) {
    return grouped_impl(hidden, gate_hidden, gate_W, gate_bias, lm_W, gi, M, H, V, g, k, dt, topk_ids,
                        topk_out, sel_groups, workspace, workspace_bytes, hip_stream, nullptr,
                        nullptr, logprob != 0);
}

extern "C" coral_status coral_lmhead_draft_level(
    const void* hidden, const void* gate_hidden, const void* gate_W, const float* gate_bias,
    const void* lm_W, const coral_group_index* gi, int M, int H, int V, int g, int k,
    coral_dtype dt, const float* parent_score, int n_next, int32_t* topk_ids, float* topk_logprob,
    int32_t* sel_groups, int32_t* next_parent, int32_t* next_token, float* next_score,
    void* workspace, size_t workspace_bytes, void* hip_stream) {
    if (!next_parent || !next_token || !next_score) return CORAL_ERR_NULL;
    if (M < 1 || k < 1 || n_next < 1) return CORAL_ERR_SHAPE;
    if (M > kMaxM || k > kMaxK) return CORAL_ERR_UNSUPPORTED;
    if (n_next > M * k) return CORAL_ERR_SHAPE;
    const LevelExpand level = {parent_score, n_next, next_parent, next_token, next_score};
    return grouped_impl(hidden, gate_hidden, gate_W, gate_bias, lm_W, gi, M, H, V, g, k, dt, topk_ids,
                        topk_logprob, sel_groups, workspace, workspace_bytes, hip_stream, nullptr,
                        nullptr, true, &level);
}

extern "C" coral_status coral_tree_expand(const float* parent_score, const int32_t* cand_ids,
                                          const float* cand_logp, int M, int k, int n_next,
                                          int32_t* next_parent, int32_t* next_token,
                                          float* next_score, void* hip_stream) {
    if (!cand_ids || !cand_logp || !next_parent || !next_token || !next_score) return CORAL_ERR_NULL;
    if (M < 1 || k < 1 || n_next < 1) return CORAL_ERR_SHAPE;
    if (M > kMaxM || k > kMaxK) return CORAL_ERR_UNSUPPORTED;
    if (n_next > M * k) return CORAL_ERR_SHAPE;
    const LevelExpand level = {parent_score, n_next, next_parent, next_token, next_score};
    return launch_tree_expand(level, cand_ids, cand_logp, M, k, static_cast<hipStream_t>(hip_stream));
}

extern "C" coral_status coral_router_premix(const void* hidden, const void* W1, int M, int H,
                                            coral_dtype dt, coral_activation act, void* u_out,
                                            void* hip_stream) {
    if (!hidden || !W1 || !u_out) return CORAL_ERR_NULL;
    if (!dtype_ok(dt)) return CORAL_ERR_SHAPE;
    if (act != CORAL_ACT_SILU && act != CORAL_ACT_RELU && act != CORAL_ACT_IDENTITY) return CORAL_ERR_SHAPE;
    if (M < 1 || H < 1) return CORAL_ERR_SHAPE;
    const bool w16 = is_16bit(dt);
    if (H % (w16 ? 8 : 4) != 0) return CORAL_ERR_UNSUPPORTED;
    if (((uintptr_t)hidden | (uintptr_t)W1 | (uintptr_t)u_out) & 15u) return CORAL_ERR_UNSUPPORTED;
    const size_t row_bytes = (size_t)H * (w16 ? 2 : 4);
    if (row_bytes > (size_t)kLdsLimit) return CORAL_ERR_UNSUPPORTED;
    {   // u_out must not overlap hidden: workgroups read hidden rows that others write
        const uintptr_t a = (uintptr_t)hidden, b = (uintptr_t)u_out;
        const size_t bytes = (size_t)M * row_bytes;
        if (a < b + bytes && b < a + bytes) return CORAL_ERR_UNSUPPORTED;
    }
    PremixParams p = {};
    p.hidden = static_cast<const uint4*>(hidden);
    p.W1 = static_cast<const uint4*>(W1);
    p.out = u_out;
    p.M = M; p.H = H; p.act = (int)act;
    p.n_vec = H / (w16 ? 8 : 4);
    hipStream_t stream = static_cast<hipStream_t>(hip_stream);
    typedef void (*premix_fn)(PremixParams);
    // Which kernel, us (k_premix_wide, k_premix_blocks): H = 2560, 8 tokens 6.3, 6.6, 15 6.3, 7.0; H =
    // 3584, 8 tokens 8.3, 8.3; H = 4096, 1 to 8 tokens 9.4, 9.0, 15 9.8, 10.0, 40 12.6, 13.8.
    if (w16 && M >= 4 && M <= 64 && H % (kPremixChunkVecs * 8) == 0 &&
        H / (kPremixChunkVecs * 8) <= kPremixMaxChunks && (M > 8 || H <= 3072)) {     // matrix cores, tokens staged in chunks
        typedef void (*wide_fn)(PremixParams);
        const int n_ct = (M + 15) / 16;
        const bool f16 = dt == CORAL_F16;
        // (three or four token tiles at the full width of 8 chunks: both streams issued a few
        // chunks ahead, see k_premix_wide)
        const bool ring = n_ct >= 3 && p.n_vec / kPremixChunkVecs == kPremixMaxChunks;
        const wide_fn wf =
            n_ct == 1   ? (f16 ? k_premix_wide<kF16, 1> : k_premix_wide<kBF16, 1>)
            : n_ct == 2 ? (f16 ? k_premix_wide<kF16, 2> : k_premix_wide<kBF16, 2>)
            : n_ct == 3 ? (ring ? (f16 ? k_premix_wide<kF16, 3, true> : k_premix_wide<kBF16, 3, true>)
                                : (f16 ? k_premix_wide<kF16, 3> : k_premix_wide<kBF16, 3>))
                        : (ring ? (f16 ? k_premix_wide<kF16, 4, true> : k_premix_wide<kBF16, 4, true>)
                                : (f16 ? k_premix_wide<kF16, 4> : k_premix_wide<kBF16, 4>));
        const int lds = (int)premix_wide_lds_bytes();
        if (!allow_lds(reinterpret_cast<const void*>(wf), lds)) return CORAL_ERR_HIP;
        hipLaunchKernelGGL(wf, dim3(H / 16), dim3(kPremixWideBlock), lds, stream, p);
        return launch_status();
    }
    // ... (k_premix, k_premix_blocks): 16 bits, H = 512, one token 4.6, 3.6, H = 5120 14.1, 13.3, H =
    // 6016 15.3, 16.2, 2 tokens 17.1, 16.1; H = 8192, 1 to 4 tokens 24.9, 27.9, 25.8, 27.7, 27.1, 27.5,
    // 34.0, 27.4; fp32, H = 1536, 4 tokens 7.4, 7.5, 8 tokens 10.0, 7.5; H = 4096, one token 15.2, 19.0, 4
    // tokens 16.9, 19.1, 8 tokens 31.4, 19.0.  (fp32 rows of less than 6 KB: the vector units' sums are the
    // more exact ones, 3.45e-8 against 3.6e-8 at H = 512; 5.7e-8 against 5.3e-8 at 1536.)
    if (w16 ? M >= 4 || H <= 5632 || (M >= 2 && H <= 7680) : M >= 5 && H >= 1536) {
        const int n_ct = M <= 16 ? 1 : M <= 32 ? 2 : M <= 48 ? 3 : 4;
        // (as many blocks ahead as the registers hold)
        const premix_fn fn =
            n_ct == 1   ? CORAL_PICK_DT(dt, (k_premix_blocks<kF32, 1, 2>), (k_premix_blocks<kBF16, 1, 2>), (k_premix_blocks<kF16, 1, 2>))
            : n_ct == 2 ? CORAL_PICK_DT(dt, (k_premix_blocks<kF32, 2, 3>), (k_premix_blocks<kBF16, 2, 2>), (k_premix_blocks<kF16, 2, 2>))
            : n_ct == 3 ? CORAL_PICK_DT(dt, (k_premix_blocks<kF32, 3, 2>), (k_premix_blocks<kBF16, 3, 1>), (k_premix_blocks<kF16, 3, 1>))
                        : CORAL_PICK_DT(dt, (k_premix_blocks<kF32, 4, 1>), (k_premix_blocks<kBF16, 4, 1>), (k_premix_blocks<kF16, 4, 1>));
        hipLaunchKernelGGL(fn, dim3((H + 15) / 16, (M + n_ct * 16 - 1) / (n_ct * 16)), dim3(kPremixBlockThreads), 0, stream, p);
        return launch_status();
    }
    int tok = (int)((size_t)kLdsLimit / 2 / row_bytes);       // two workgroups per compute unit
    if (tok < 1) tok = 1;
    if (tok > kPremixTok) tok = kPremixTok;
    if (tok > M) tok = M;
    p.tok_per_wg = tok;
    const int lds = (int)((size_t)tok * row_bytes);
    const int pairs = (H + 1) / 2;
    int gx = (pairs + kWavesPerBlock - 1) / kWavesPerBlock;
    if (gx > 2 * kMaxWorkgroups) gx = 2 * kMaxWorkgroups;
    const dim3 grid(gx, (M + tok - 1) / tok);
    const premix_fn fn = CORAL_PICK_DT(dt, k_premix<kF32>, k_premix<kBF16>, k_premix<kF16>);
    if (!allow_lds(reinterpret_cast<const void*>(fn), lds)) return CORAL_ERR_HIP;
    hipLaunchKernelGGL(fn, grid, dim3(kBlock), lds, stream, p);
    return launch_status();
}

extern "C" coral_status coral_lmhead_grouped_logprob(
    const void* hidden, const void* gate_W, const float* gate_bias, const void* lm_W,
    const coral_group_index* gi, int M, int H, int V, int g, int k, coral_dtype dt,
    int32_t* topk_ids, float* topk_logprob, int32_t* sel_groups, void* workspace,
    size_t workspace_bytes, void* hip_stream) {
    return grouped_impl(hidden, nullptr, gate_W, gate_bias, lm_W, gi, M, H, V, g, k, dt, topk_ids,
                        topk_logprob, sel_groups, workspace, workspace_bytes, hip_stream, nullptr,
                        nullptr, true);
}

extern "C" coral_status coral_lmhead_grouped_logprob_profiled(
    const void* hidden, const void* gate_W, const float* gate_bias, const void* lm_W,
    const coral_group_index* gi, int M, int H, int V, int g, int k, coral_dtype dt,
    int32_t* topk_ids, float* topk_logprob, int32_t* sel_groups, void* workspace,
    size_t workspace_bytes, void* hip_stream, void* ev_before, void* ev_after) {
    if (!ev_before || !ev_after) return CORAL_ERR_NULL;
    return grouped_impl(hidden, nullptr, gate_W, gate_bias, lm_W, gi, M, H, V, g, k, dt, topk_ids,
                        topk_logprob, sel_groups, workspace, workspace_bytes, hip_stream, ev_before,
                        ev_after, true);
}

extern "C" coral_status coral_lmhead_grouped_profiled(
    const void* hidden, const void* gate_W, const float* gate_bias, const void* lm_W,
    const coral_group_index* gi, int M, int H, int V, int g, int k, coral_dtype dt,
    int32_t* topk_ids, float* topk_logits, int32_t* sel_groups, void* workspace,
    size_t workspace_bytes, void* hip_stream, void* ev_before, void* ev_after) {
    if (!ev_before || !ev_after) return CORAL_ERR_NULL;
    return grouped_impl(hidden, nullptr, gate_W, gate_bias, lm_W, gi, M, H, V, g, k, dt, topk_ids,
                        topk_logits, sel_groups, workspace, workspace_bytes, hip_stream, ev_before,
                        ev_after, false);
}

extern "C" coral_status coral_lmhead_dense(const void* hidden, const void* lm_W, int M, int H,
                                           int V, int k, coral_dtype dt, int32_t* topk_ids,
                                           float* topk_logits, void* workspace,
                                           size_t workspace_bytes, void* hip_stream) {
    return dense_impl(hidden, lm_W, M, H, V, k, dt, topk_ids, topk_logits, workspace,
                      workspace_bytes, hip_stream, nullptr, nullptr);
}

extern "C" coral_status coral_lmhead_dense_profiled(const void* hidden, const void* lm_W, int M,
                                                    int H, int V, int k, coral_dtype dt,
                                                    int32_t* topk_ids, float* topk_logits,
                                                    void* workspace, size_t workspace_bytes,
                                                    void* hip_stream, void* ev_before,
                                                    void* ev_after) {
    if (!ev_before || !ev_after) return CORAL_ERR_NULL;
    return dense_impl(hidden, lm_W, M, H, V, k, dt, topk_ids, topk_logits, workspace,
                      workspace_bytes, hip_stream, ev_before, ev_after);
}
