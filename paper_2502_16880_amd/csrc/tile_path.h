// Matrix-core path for groups that many tokens selected (wide draft-tree steps) and for
// the dense head with many tokens: the logits of a block of 128 weight rows for up to 64
// tokens are 16x16 tiles of v_mfma_f32_16x16x32_bf16.
//
// k_tiles: one persistent workgroup of 8 waves per compute unit; wave = (row group rg =
// wave/2: 32 rows = two row tiles, half kq = wave%2 of every 512-column chunk).  Per block of
// 128 rows of one group:
//   - the weight rows go from HBM into registers in whole 128-byte lines (a wave load
//     covers 8 rows x 128 B), and pairs of such registers go through a wave-private LDS
//     slice into the MFMA A operands of two 32-column steps; 16 KB per wave in flight,
//     the next block's first 16 loads issued before this block's epilogue;
//   - the hidden vectors of the tokens that selected the group are staged chunk by chunk
//     (512 columns, double buffered) in LDS and read as B operands, each fragment used for
//     both row tiles of the wave;
//   - the two half sums of each tile are added in a fixed order through LDS, which
//     leaves, per token, the block's 128 logits two per lane of a wave; they go to memory as
//     they are, 512 bytes per (block, token), with the largest of them (and the sum of exp in
//     the log-probability mode): a few MB per step against the hundreds of MB of weight rows,
//     and the workgroup is back in its next block's K loop within a few microseconds.
// k_gate_select in front of it: gate and selection per tile of 16 tokens.  k_tile_select behind
// it: one workgroup per token bounds the token's k-th logit by the k-th largest block maximum,
// reads the logits of the blocks that reach the bound and ranks them (Eq. 8's offsets added
// per group in the log-probability mode).
#pragma once
#include "device_utils.h"
#include "fused_path.h"
#include <type_traits>

namespace {

constexpr int kTileWaves = 8;
// Waves that share a row group of 32 rows (split of a chunk's columns): two, a block then being
// 128 rows, or all eight with blocks of 32 rows, for steps whose 128-row blocks would leave
// compute units without work (see tile_small_blocks in coral_lmhead.hip).
constexpr int kTileSplit = 2, kTileSplitHalf = 4, kTileSplitSmall = 8;
__host__ __device__ constexpr int tile_rows(int split) { return 32 * kTileWaves / split; }
constexpr int kTileHalfTokens = 32;              // tokens of a group whose blocks can be processed in halves
constexpr int kTileBlock = kTileWaves * kWave;
constexpr int kTileRows = tile_rows(kTileSplit);          // weight rows per block (4 row groups of 32)
constexpr int kTileRowsSmall = tile_rows(kTileSplitSmall);
static_assert(tile_rows(kTileSplitHalf) * 2 == kTileRows && tile_rows(kTileSplitHalf) == kWave, "");
constexpr int kChunkVecs = 64;                   // 16-byte vectors per 512-column chunk
constexpr int kHbStride = kChunkVecs + 1;        // LDS row stride in vectors (pad: no bank conflicts)
constexpr int kHbBufVecs = 64 * kHbStride;       // one staging buffer: 64 token slots
constexpr int kRing = 16;                        // weight loads of a wave in flight
constexpr int kGateParts = 2;                    // workgroups that share the columns of a gate tile
// Strides (floats) of the accumulator tiles parked in LDS for the epilogue: token tile,
// row tile of a wave, wave.  Modulo the 64 banks they are 16, 16 and 48.
constexpr int kRedCt = 272, kRedTile = 4 * kRedCt + 16, kRedWave = 2 * kRedTile + 16;
static_assert(kTileWaves * kRedWave * 4 <= 2 * kHbBufVecs * 16, "the parked tiles fit the staging buffers");
// Compiler-only barrier: no memory access is moved across it.  Keeps global loads at the
// place in the instruction stream where the source puts them (the compiler would otherwise
// sink them to their first use, which defeats prefetching).
__device__ __forceinline__ void keep_memory_order() { asm volatile("" ::: "memory"); }

struct TileParams {
    const uint4* hidden;                    // [M, n_vec]
    const uint4* lm_W;                      // [V, n_vec]
    const int32_t* rows;                    // [V]     (grouped)
    const int32_t* offsets;                 // [G+1]   (grouped)
    const unsigned long long* tile_mask;    // [token tiles, G] (grouped) what k_gate_select left
    unsigned long long* group_mask;         // [G] out (grouped): tokens that selected the group
    int32_t* group_first_block;             // [G] out (grouped): first block of an activated group
    float* z;                               // [blocks, M, rows of a block] out: logits of (block, token slot)
    float2* stat;                           // [blocks, M] out: the slot's largest logit, and in the
                                            // log-probability mode the sum of exp(z - largest)
    float2* stat_upper;                     // [blocks from split_from on, M] out: the same of rows 64 to 127
    int32_t* split_from;                    // out: the first block processed in halves
    int halves;                             // whether blocks may be (see tiles_take_halves in coral_lmhead.hip)
    int stream_rows;                        // weights past the caches from so many activated rows on (tile_stream_rows)
    int want_lse;
    unsigned int* next_block;               // block queue: zero before the launch
    int M, V, G;
    int n_vec, n_chunks;
    int u_max;                              // capacity of the activated-group arrays
};

struct TileLds {
    int o_hbuf, o_scratch, o_ustart, o_uend, o_uprefix, o_umask, o_flags, total;
};

__host__ __device__ inline TileLds tile_lds_layout(int u_max) {
    TileLds L;
    int off = 0;
    auto take = [&](size_t bytes) {
        int at = off;
        off = (int)((off + bytes + 15) / 16 * 16);
        return at;
    };
    L.o_hbuf = take((size_t)2 * kHbBufVecs * sizeof(uint4));
    L.o_scratch = take((size_t)kTileWaves * kLinePairSlots * sizeof(uint4));
    L.o_ustart = take((size_t)u_max * sizeof(int));
    L.o_uend = take((size_t)u_max * sizeof(int));
    L.o_uprefix = take((size_t)(u_max + 1) * sizeof(int));
    L.o_umask = take((size_t)u_max * sizeof(unsigned long long));
    L.o_flags = take(16);
    // (256 bytes more than are used: which shapes fit, and with them the route and the size checks of
    // calls, stays as it was when the kernel kept its tokens here)
    L.total = off + 256;
    return L;
}

// One 512-column chunk of a block's K loop for NCT token tiles (a compile-time count: no
// branch inside a chunk, so that LDS reads, matrix instructions and loads of neighbouring
// steps interleave).  REFILL: a next chunk exists; its weight lines refill the ring slots as
// they are consumed.  Its hidden vectors are requested at the top of the chunk, before those
// refills, and written to the other staging buffer only in the chunk's last step pair: loads
// complete in order, and the requests are younger than all 16 weight lines of this chunk, so
// an earlier write would wait for lines that are not needed yet (and were requested least
// long ago), while by the last step pair all of them have been consumed anyway.
struct TileStage {                                     // staging registers, 2 NCT in use
    uint4 r0, r1, r2, r3, r4, r5, r6, r7;
};

// The tokens of a wave's staging slots wave, wave + 8, ... (wave-uniform), slots past the unit's tokens
// repeating its last one.
struct TileTokens {
    int t0, t1, t2, t3, t4, t5, t6, t7;
};
// ... of a unit of n_t tokens, those of the mask from the first-th on.
__device__ __forceinline__ TileTokens tile_tokens(unsigned long long mask, int first, int n_t, int lane, int wave) {
    const int below = __builtin_amdgcn_mbcnt_hi((unsigned)(mask >> 32), __builtin_amdgcn_mbcnt_lo((unsigned)mask, 0u)) - first;
    const int mine = (mask >> lane) & 1ull ? below : -1;   // this lane's token's slot
    auto tok = [&](int i) {
        const int s = wave + i * kTileWaves;
        return __ffsll(__ballot(mine == (s < n_t ? s : n_t - 1))) - 1;
    };
    return {tok(0), tok(1), tok(2), tok(3), tok(4), tok(5), tok(6), tok(7)};
}

template <int NCT, bool GENERAL>
__device__ __forceinline__ void tile_fetch_hidden(const TileParams& p, const TileTokens& tok, TileStage& hst, int c, int lane) {
    constexpr int kN = 2 * NCT;
    // (past the row's end, in the last chunk: the row's last vector, stored as zero)
    const int last = p.n_vec - 1 - c * kChunkVecs;
    const uint4* src = p.hidden + c * kChunkVecs;
    const unsigned at = (unsigned)(GENERAL && lane > last ? last : lane) * 16u;
    int n_vec = p.n_vec;
    asm volatile("" : "+s"(n_vec));                    // (the rows' offsets are not kept from chunk to chunk)
    auto load = [&](int t) {
        return load_vec(reinterpret_cast<const uint4*>(reinterpret_cast<const char*>(src + (unsigned)t * (unsigned)n_vec) + at));
    };
    if (kN > 0) hst.r0 = load(tok.t0);
    if (kN > 1) hst.r1 = load(tok.t1);
    if (kN > 2) hst.r2 = load(tok.t2);
    if (kN > 3) hst.r3 = load(tok.t3);
    if (kN > 4) hst.r4 = load(tok.t4);
    if (kN > 5) hst.r5 = load(tok.t5);
    if (kN > 6) hst.r6 = load(tok.t6);
    if (kN > 7) hst.r7 = load(tok.t7);
}
// The first chunk's hidden vectors of a unit with up to two token tiles (with more there are no registers
// for them beside the parked tiles), n2 = 2 or 4 staging slots per wave, in r0 ... r3; of a half with one
// tile the second chunk's behind them.
template <bool GENERAL>
__device__ __forceinline__ void tile_fetch_first(const TileParams& p, const TileTokens& tok, TileStage& hst, int n2, bool half, int lane) {
    if (n2 > 4) return;                                // (all conditions are uniform)
    const uint4* src = p.hidden + (GENERAL && lane > p.n_vec - 1 ? p.n_vec - 1 : lane);
    auto load = [&](int t, int c) { return load_vec(src + c * kChunkVecs + (size_t)t * p.n_vec); };
    hst.r0 = load(tok.t0, 0);
    hst.r1 = load(tok.t1, 0);
    if (n2 == 4 || half) {
        hst.r2 = load(n2 == 4 ? tok.t2 : tok.t0, n2 == 4 ? 0 : 1);
        hst.r3 = load(n2 == 4 ? tok.t3 : tok.t1, n2 == 4 ? 0 : 1);
    }
    keep_memory_order();
}
template <int NCT, bool GENERAL>
__device__ __forceinline__ void tile_store_hidden(int n_vec, const TileStage& hst, uint4* hbuf, int c, int lane,
                                                  int wave) {
    constexpr int kN = 2 * NCT;
    uint4* dst = hbuf + (size_t)(c & 1) * kHbBufVecs + (size_t)wave * kHbStride + lane;
    if (GENERAL && c * kChunkVecs + lane >= n_vec) {    // past the row's end
#pragma unroll
        for (int i = 0; i < kN; ++i) store_vec(dst + i * kTileWaves * kHbStride, make_uint4(0, 0, 0, 0));
    } else {
        if (kN > 0) store_vec(dst + 0 * kTileWaves * kHbStride, hst.r0);
        if (kN > 1) store_vec(dst + 1 * kTileWaves * kHbStride, hst.r1);
        if (kN > 2) store_vec(dst + 2 * kTileWaves * kHbStride, hst.r2);
        if (kN > 3) store_vec(dst + 3 * kTileWaves * kHbStride, hst.r3);
        if (kN > 4) store_vec(dst + 4 * kTileWaves * kHbStride, hst.r4);
        if (kN > 5) store_vec(dst + 5 * kTileWaves * kHbStride, hst.r5);
        if (kN > 6) store_vec(dst + 6 * kTileWaves * kHbStride, hst.r6);
        if (kN > 7) store_vec(dst + 7 * kTileWaves * kHbStride, hst.r7);
    }
}

// This lane's vector of step pair sp of chunk c, counted from the row's start.
template <int SPLIT>
__device__ __forceinline__ int tile_lane_vec(int c, int sp) {
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x / kWave);
    return c * kChunkVecs + sp * 8 + (wave % SPLIT) * (kChunkVecs / SPLIT) +
           line_load_chunk(threadIdx.x & (kWave - 1));
}

// The 128-byte line of step pair sp of chunk c in the lane's row at byte offset `row` of
// the weight matrix (offsets are 32-bit: the path takes matrices below 4 GiB).  GENERAL: `row` is
// the row's start, and lanes past its end read its last vector (dropped in tile_step_pair);
// otherwise the lane's place in a chunk is part of `row`.  STREAM: non-temporal (see tile_stream_rows).
template <bool STREAM, bool GENERAL, int SPLIT>
__device__ __forceinline__ uint4 tile_load_w(const TileParams& p, unsigned row, int c, int sp) {
    unsigned off;
    if (GENERAL) {
        const int vec = tile_lane_vec<SPLIT>(c, sp);
        off = row + (unsigned)(vec < p.n_vec ? vec : p.n_vec - 1) * 16u;
    } else {
        off = row + (unsigned)(c * kChunkVecs + sp * 8) * 16u;
    }
    const uint4* src = reinterpret_cast<const uint4*>(reinterpret_cast<const char*>(p.lm_W) + off);
    return STREAM ? load_stream(src) : load_vec(src);
}

// Step pair SP of a chunk: the two 32-column steps whose weight lines sit in ring slots
// 4 SLOT .. 4 SLOT + 3.  A wave has 8 / SPLIT step pairs of a chunk, so the ring's four cover
// SPLIT / 2 chunks and are refilled that far ahead.
template <bool STREAM, int DT, int NCT, bool REFILL, bool STORE, int SP, bool GENERAL, int SPLIT, int SLOT, int AHEAD>
__device__ __forceinline__ void tile_step_pair(const TileParams& p, int c, uint4 (&a)[kRing],
                                               f32x4_t (&acc)[2][4], f32x4_t (&low)[2][4],
                                               const unsigned (&wrow)[4],
                                               uint4* hbuf, TileStage& hst, uint4* my_slice, int lane) {
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x / kWave);
    const int r16 = lane & 15, q4 = lane >> 4;
    const int kq = wave % SPLIT;
    constexpr int kSteps = 16 / SPLIT;
    const uint4* hb = hbuf + (size_t)(c & 1) * kHbBufVecs;
    if (GENERAL && (!REFILL || SPLIT == kTileSplitSmall)) {    // the last chunk: nothing past the row's end
        const unsigned in = tile_lane_vec<SPLIT>(c, SP) < p.n_vec ? 0xffffffffu : 0u;
#pragma unroll
        for (int o = 0; o < 4; ++o)
            a[SLOT * 4 + o] = make_uint4(a[SLOT * 4 + o].x & in, a[SLOT * 4 + o].y & in, a[SLOT * 4 + o].z & in, a[SLOT * 4 + o].w & in);
    }
    uint4 op[2][2];                                    // [row tile][step of the pair]
#pragma unroll
    for (int t = 0; t < 2; ++t) {
        mfma_operands_from_lines(a[SLOT * 4 + 2 * t], a[SLOT * 4 + 2 * t + 1], lane, my_slice, op[t][0],
                                 op[t][1]);
        if (REFILL) {                                  // refill the two slots just consumed
            a[SLOT * 4 + 2 * t] = tile_load_w<STREAM, GENERAL, SPLIT>(p, wrow[2 * t], c + AHEAD, SP);
            a[SLOT * 4 + 2 * t + 1] = tile_load_w<STREAM, GENERAL, SPLIT>(p, wrow[2 * t + 1], c + AHEAD, SP);
        }
    }
    if (REFILL) keep_memory_order();
    if (STORE) {                                       // the other buffer is free since the last barrier
        tile_store_hidden<NCT, GENERAL>(p.n_vec, hst, hbuf, c + 1, lane, wave);
        keep_memory_order();
    }
    if (GENERAL) {
        // One running fp32 sum over a row's hundreds of products would be less exact than the
        // staged kernels' lane-split sums (fp32, 2048 columns: 4e-7 against 7e-8).  So the step
        // pair's products start from zero and are added to the running sum with their rounding
        // error kept (two-sum).  (The barrier: reading several operands ahead, as the compiler
        // would, costs more registers than there are.)
#pragma unroll
        for (int ct = 0; ct < NCT; ++ct) {
            f32x4_t x[2] = {f32x4_t{0.f, 0.f, 0.f, 0.f}, f32x4_t{0.f, 0.f, 0.f, 0.f}};
#pragma unroll
            for (int s2 = 0; s2 < 2; ++s2) {
                const uint4 hv = hb[(ct * 16 + r16) * kHbStride + (kq * kSteps + 2 * SP + s2) * 4 + q4];
#pragma unroll
                for (int t = 0; t < 2; ++t) x[t] = mfma_tile<DT>(op[t][s2], hv, x[t]);
            }
            __builtin_amdgcn_sched_barrier(0);
#pragma unroll
            for (int t = 0; t < 2; ++t)
#pragma unroll
                for (int i = 0; i < 4; ++i) {
                    const float hi = acc[t][ct][i], sum = hi + x[t][i], back = sum - hi;
                    low[t][ct][i] += (hi - (sum - back)) + (x[t][i] - back);
                    acc[t][ct][i] = sum;
                }
        }
        return;
    }
#pragma unroll
    for (int s2 = 0; s2 < 2; ++s2) {
        const int off = (kq * kSteps + 2 * SP + s2) * 4 + q4;
#pragma unroll
        for (int ct = 0; ct < NCT; ++ct) {
            const uint4 hv = hb[(ct * 16 + r16) * kHbStride + off];
#pragma unroll
            for (int t = 0; t < 2; ++t)
                acc[t][ct] = mfma_tile<DT>(op[t][s2], hv, acc[t][ct]);
        }
    }
}

template <bool STREAM, int DT, int NCT, bool REFILL, bool GENERAL>
__device__ __forceinline__ void tile_chunk(const TileParams& p, int c, uint4 (&a)[kRing],
                                           f32x4_t (&acc)[2][4], f32x4_t (&low)[2][4],
                                           const unsigned (&wrow)[4],
                                           uint4* hbuf, const TileTokens& tok, uint4* my_slice) {
    TileStage hst;
    int lane = threadIdx.x & (kWave - 1);
    asm volatile("" : "+v"(lane));                     // (what is derived from it is not kept from chunk to chunk)
    // (the scheduling barriers keep the compiler from sinking the loads to where their
    // registers are first needed, which would undo the ordering)
    // (general form with two token tiles: after the first step pair, fp32 after the second, there
    // are no registers for them before)
    constexpr int kFetchAt = !GENERAL || NCT == 1 ? 0 : DT == kF32 ? 2 : 1;
    auto fetch = [&]() {
        tile_fetch_hidden<NCT, GENERAL>(p, tok, hst, c + 1, lane);
        keep_memory_order();
    };
    if (REFILL && kFetchAt == 0) fetch();
    tile_step_pair<STREAM, DT, NCT, REFILL, false, 0, GENERAL, kTileSplit, 0, 1>(p, c, a, acc, low, wrow, hbuf, hst, my_slice, lane);
    if (REFILL && kFetchAt == 1) fetch();
    tile_step_pair<STREAM, DT, NCT, REFILL, false, 1, GENERAL, kTileSplit, 1, 1>(p, c, a, acc, low, wrow, hbuf, hst, my_slice, lane);
    if (REFILL && kFetchAt == 2) fetch();
    tile_step_pair<STREAM, DT, NCT, REFILL, false, 2, GENERAL, kTileSplit, 2, 1>(p, c, a, acc, low, wrow, hbuf, hst, my_slice, lane);
    tile_step_pair<STREAM, DT, NCT, REFILL, REFILL, 3, GENERAL, kTileSplit, 3, 1>(p, c, a, acc, low, wrow, hbuf, hst, my_slice, lane);
    __syncthreads();
}

// The same with four waves on a row group (halves of 64 rows): two step pairs of a chunk per wave, so
// that the ring holds two chunks.  Hidden vectors are requested two chunks ahead as well: a chunk ahead
// they would be younger than all of the next chunk's weight lines, and waiting for them would drain
// the ring.  PH = c % 2.  `fetched` takes those of chunk c + 2 (REFILL: there is one), `held` are those
// of chunk c + 1 (STORE).
template <bool STREAM, int DT, int NCT, bool REFILL, bool STORE, int PH>
__device__ __forceinline__ void tile_chunk_half(const TileParams& p, int c, uint4 (&a)[kRing],
                                                f32x4_t (&acc)[2][4], f32x4_t (&low)[2][4],
                                                const unsigned (&wrow)[4], uint4* hbuf, const TileTokens& tok,
                                                uint4* my_slice, TileStage& fetched, TileStage& held) {
    int lane = threadIdx.x & (kWave - 1);
    asm volatile("" : "+v"(lane));
    if (REFILL) {
        tile_fetch_hidden<NCT, false>(p, tok, fetched, c + 2, lane);
        keep_memory_order();
    }
    tile_step_pair<STREAM, DT, NCT, REFILL, false, 0, false, kTileSplitHalf, PH * 2, 2>(p, c, a, acc, low, wrow, hbuf, held, my_slice, lane);
    tile_step_pair<STREAM, DT, NCT, REFILL, STORE, 1, false, kTileSplitHalf, PH * 2 + 1, 2>(p, c, a, acc, low, wrow, hbuf, held, my_slice, lane);
    __syncthreads();
}

// The same with all eight waves on one row group (general form): one step pair of the chunk per
// wave, from ring slot PH = c % 4.
template <bool STREAM, int DT, int NCT, int PH>
__device__ __forceinline__ void tile_chunk_small(const TileParams& p, int c, uint4 (&a)[kRing],
                                                 f32x4_t (&acc)[2][4], f32x4_t (&low)[2][4],
                                                 const unsigned (&wrow)[4],
                                                 uint4* hbuf, const TileTokens& tok, uint4* my_slice) {
    const int lane = threadIdx.x & (kWave - 1);
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x / kWave);
    const bool more = c + 1 < p.n_chunks;              // uniform
    TileStage hst;
    if (more) {
        tile_fetch_hidden<NCT, true>(p, tok, hst, c + 1, lane);
        keep_memory_order();
    }
    // (past the last chunk the refills read the row's last vector, which nothing uses: a form
    // without them beside this one costs more registers than there are)
    tile_step_pair<STREAM, DT, NCT, true, false, 0, true, kTileSplitSmall, PH, 4>(p, c, a, acc, low, wrow, hbuf, hst, my_slice, threadIdx.x & (kWave - 1));
    if (more) tile_store_hidden<NCT, true>(p.n_vec, hst, hbuf, c + 1, lane, wave);
    __syncthreads();
}

// The K loop of one block.  Hidden chunk staging: slots wave, wave + 8, ... below 16 NCT;
// lane = vector inside the chunk; slots past the group's tokens repeat its last token
// (their columns of the tiles are never read back).
template <bool STREAM, int DT, int NCT, bool GENERAL, int SPLIT>
__device__ __forceinline__ void tile_k_loop(const TileParams& p, uint4 (&a)[kRing], f32x4_t (&acc)[2][4],
                                            const unsigned (&wrow)[4], uint4* hbuf,
                                            const TileTokens& tok, const TileStage& first, uint4* my_slice) {
    int lane = threadIdx.x & (kWave - 1);
    asm volatile("" : "+v"(lane));
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x / kWave);
    TileStage even, odd;                               // (halves) hidden vectors of the next even and odd chunk
    if (SPLIT == kTileSplitHalf && NCT == 1) {         // (see tile_fetch_first)
        odd.r0 = first.r2;
        odd.r1 = first.r3;
    }
    if (SPLIT == kTileSplitHalf && NCT == 2) {
        tile_fetch_hidden<NCT, GENERAL>(p, tok, odd, 1, lane);
        keep_memory_order();
    }
    if (NCT > 2) tile_fetch_hidden<NCT, GENERAL>(p, tok, even, 0, lane);
    tile_store_hidden<NCT, GENERAL>(p.n_vec, NCT > 2 ? even : first, hbuf, 0, lane, wave);
    __syncthreads();
    f32x4_t low[2][4];                                 // (general form) what the running sums have rounded off
#pragma unroll
    for (int t = 0; t < 2; ++t)
#pragma unroll
        for (int ct = 0; ct < 4; ++ct) low[t][ct] = f32x4_t{0.f, 0.f, 0.f, 0.f};
    if constexpr (SPLIT == kTileSplitHalf) {
        const int n = p.n_chunks;                      // at least two
        int c = 0;
        for (; c + 3 < n; c += 2) {                    // uniform
            tile_chunk_half<STREAM, DT, NCT, true, true, 0>(p, c, a, acc, low, wrow, hbuf, tok, my_slice, even, odd);
            tile_chunk_half<STREAM, DT, NCT, true, true, 1>(p, c + 1, a, acc, low, wrow, hbuf, tok, my_slice, odd, even);
        }
        if (c + 2 < n) {                               // three left
            tile_chunk_half<STREAM, DT, NCT, true, true, 0>(p, c, a, acc, low, wrow, hbuf, tok, my_slice, even, odd);
            tile_chunk_half<STREAM, DT, NCT, false, true, 1>(p, c + 1, a, acc, low, wrow, hbuf, tok, my_slice, odd, even);
            tile_chunk_half<STREAM, DT, NCT, false, false, 0>(p, c + 2, a, acc, low, wrow, hbuf, tok, my_slice, even, odd);
        } else {
            tile_chunk_half<STREAM, DT, NCT, false, true, 0>(p, c, a, acc, low, wrow, hbuf, tok, my_slice, even, odd);
            tile_chunk_half<STREAM, DT, NCT, false, false, 1>(p, c + 1, a, acc, low, wrow, hbuf, tok, my_slice, odd, even);
        }
    } else if constexpr (SPLIT == kTileSplit) {
        for (int c = 0; c + 1 < p.n_chunks; ++c)
            tile_chunk<STREAM, DT, NCT, true, GENERAL>(p, c, a, acc, low, wrow, hbuf, tok, my_slice);
        tile_chunk<STREAM, DT, NCT, false, GENERAL>(p, p.n_chunks - 1, a, acc, low, wrow, hbuf, tok, my_slice);
    } else {
        for (int c = 0; c < p.n_chunks; c += 4) {      // uniform
            tile_chunk_small<STREAM, DT, NCT, 0>(p, c, a, acc, low, wrow, hbuf, tok, my_slice);
            if (c + 1 < p.n_chunks) tile_chunk_small<STREAM, DT, NCT, 1>(p, c + 1, a, acc, low, wrow, hbuf, tok, my_slice);
            if (c + 2 < p.n_chunks) tile_chunk_small<STREAM, DT, NCT, 2>(p, c + 2, a, acc, low, wrow, hbuf, tok, my_slice);
            if (c + 3 < p.n_chunks) tile_chunk_small<STREAM, DT, NCT, 3>(p, c + 3, a, acc, low, wrow, hbuf, tok, my_slice);
        }
    }
    if (GENERAL) {
        // (an infinite sum has no rounding error: the two-sum's is inf - inf, NaN)
#pragma unroll
        for (int t = 0; t < 2; ++t)
#pragma unroll
            for (int ct = 0; ct < NCT; ++ct)
#pragma unroll
                for (int i = 0; i < 4; ++i) {
                    const float sum = acc[t][ct][i] + low[t][ct][i];
                    acc[t][ct][i] = __builtin_isfinite(sum) ? sum : acc[t][ct][i];
                }
    }
}

// The workgroup's blocks, drawn from the queue one by one (`at`: its first draw), once the table of the
// activated groups is in LDS.
template <bool STREAM, int DT, bool GENERAL, int SPLIT>
__device__ __forceinline__ void tile_units(const TileParams& p, bool dense, int at, int total_blocks, const TileLds& lay, char* lds) {
    constexpr int ROWS = tile_rows(SPLIT);
    constexpr bool HALVES = !GENERAL;                  // blocks can be processed in halves (see split_from)
    uint4* hbuf = reinterpret_cast<uint4*>(lds + lay.o_hbuf);
    int* ustart = reinterpret_cast<int*>(lds + lay.o_ustart);
    int* uend = reinterpret_cast<int*>(lds + lay.o_uend);
    int* uprefix = reinterpret_cast<int*>(lds + lay.o_uprefix);
    unsigned long long* umask = reinterpret_cast<unsigned long long*>(lds + lay.o_umask);
    int* flags = reinterpret_cast<int*>(lds + lay.o_flags);
    const int lane = threadIdx.x & (kWave - 1);
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x / kWave);
    const int M = p.M;
    uint4* my_slice = reinterpret_cast<uint4*>(lds + lay.o_scratch) + (size_t)wave * kLinePairSlots;
    unsigned int drawn = 0u;
    const unsigned long long all_tokens = M >= 64 ? ~0ull : ((1ull << M) - 1ull);
    // Where the last round of blocks would occupy no more than half of the workgroups, its blocks are
    // handed out in halves of 64 rows (four waves on a row group): one workgroup alone reads a block
    // at 50 GB/s, and 32 blocks in a third round held up the wide tree's step by 20 us (136.6 us a
    // call, 126.5 with halves; 2.5 % on average over inputs); heads with fewer blocks than that in all
    // likewise (ragged head, 24 tokens 42.2, 37.5).  Not those of groups with more than 32 tokens
    // (behind flags[2] there is none): the hidden vectors of the next two chunks do not fit the
    // registers beside three or four token tiles, and a form that waits for them a chunk ahead made
    // the whole kernel slower (wide tree 126 -> 134 us, by the registers it takes).
    const int P = gridDim.x;
    const int over = total_blocks % P;
    const int split_from = HALVES && p.halves && p.n_chunks > 1 && 2 * over <= P ? max(total_blocks - over, uni(flags[2])) : total_blocks;
    const int total_units = 2 * total_blocks - split_from;
    if (blockIdx.x == 0 && threadIdx.x == 0) *p.split_from = split_from;
    int u = 0;
    // A unit of the queue: block b, of it all rows or those of one half; its first row and the end of
    // its group (row indices into p.rows, or vocabulary ids).
    struct Unit {
        int b, half;                                   // half: -1 all rows, 0 the first 64, 1 the others
        int first, end;
        unsigned long long bm;
    };
    auto locate = [&](int at) {
        Unit x;
        x.b = at;
        x.half = -1;
        if (HALVES && at >= split_from) {
            x.b = split_from + ((at - split_from) >> 1);
            x.half = (at - split_from) & 1;
        }
        if (dense) {
            x.first = x.b * ROWS;
            x.end = p.V;
            x.bm = all_tokens;
        } else {
            while (x.b >= uni(uprefix[u + 1])) ++u;    // blocks come in increasing order
            x.first = uni(ustart[u]) + (x.b - uni(uprefix[u])) * ROWS;
            x.end = uni(uend[u]);
            x.bm = uni64(umask[u]);
        }
        if (HALVES && x.half == 1) x.first += ROWS / 2;
        return x;
    };
    // This lane's four weight rows: row (lane / 8) of each 8-row octet o of the wave's 32
    // rows (clamped inside the group; the logits of the duplicates are never read), as byte offsets
    // of its place in a chunk; and the ring's first slots.  Slot sp * 4 + o holds octet o's 128-byte
    // line of step pair sp of the first chunk, or (halves) of pair sp % 2 of chunk sp / 2, or (all
    // waves on one row group) of the one step pair of chunk sp (past the last chunk: clamped to the
    // row's end, not used).
    // The hidden vectors of the first chunk (halves: two) are requested before them: behind them they
    // would arrive after the last line, and the K loop's first refills with them.
    uint4 a[kRing];
    unsigned wrow[4];
    TileTokens tok;
    TileStage first;
    // General form: the running sums' rounding errors take the registers of two token tiles, so a
    // block serves 32 tokens at a time and comes round again for the next 32.
    constexpr bool kPasses = GENERAL;
    constexpr int kPassTokens = kPasses ? 32 : kMaxM;
    // tokens of a unit's pass from slot s0 on
    auto pass_tokens = [&](unsigned long long bm, int s0) {
        const int left = __popcll(bm) - (kPasses ? s0 : 0);
        return kPasses && left > kPassTokens ? kPassTokens : left;
    };
    auto start_unit = [&](const Unit& x, int s0, int lane) {
        const bool half = HALVES && x.half >= 0;       // uniform
        const int split = half ? kTileSplitHalf : SPLIT;
        const int rg = wave / split, kq = wave % split;
        int rid[4];
#pragma unroll
        for (int o = 0; o < 4; ++o) {
            int idx = x.first + rg * 32 + o * 8 + line_load_row(lane);
            if (idx >= x.end) idx = x.end - 1;
            rid[o] = dense ? idx : p.rows[idx];
        }
        const int n_t = pass_tokens(x.bm, s0);
        tok = tile_tokens(x.bm, s0, n_t, lane, wave);
        tile_fetch_first<GENERAL>(p, tok, first, 2 * ((n_t + 15) >> 4), half, lane);
#pragma unroll
        for (int o = 0; o < 4; ++o)
            wrow[o] = ((unsigned)rid[o] * (unsigned)p.n_vec + (GENERAL ? 0 : kq * (kChunkVecs / split) + line_load_chunk(lane))) * 16u;
#pragma unroll
        for (int sp = 0; sp < 4; ++sp) {
            int c = SPLIT == kTileSplit ? 0 : sp, pair = SPLIT == kTileSplit ? sp : 0;
            if (HALVES && x.half >= 0) {               // uniform
                c = sp >> 1;
                pair = sp & 1;
            }
#pragma unroll
            for (int o = 0; o < 4; ++o) a[sp * 4 + o] = tile_load_w<STREAM, GENERAL, SPLIT>(p, wrow[o], c, pair);
        }
    };

    Unit now = {0, -1, 0, 0, 0ull};
    if (at < total_units) {
        now = locate(at);
        start_unit(now, 0, lane);
    }
    int s0 = 0;                                        // first token slot of this pass
    while (at < total_units) {                         // block-uniform
        int ln = lane;                                 // (what is derived from it is not kept from block to block:
        asm volatile("" : "+v"(ln));                   // there are no registers for that)
        const unsigned long long bm = now.bm;
        const bool last_pass = !kPasses || s0 + kPassTokens >= __popcll(bm);
        if (threadIdx.x == 0 && last_pass)             // the draw returns long before the K loop ends
            drawn = __hip_atomic_fetch_add(p.next_block, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        const int n_t = pass_tokens(bm, s0);
        const int n_ct = (n_t + 15) >> 4;

        f32x4_t acc[2][4];
#pragma unroll
        for (int t = 0; t < 2; ++t)
#pragma unroll
            for (int ct = 0; ct < 4; ++ct) acc[t][ct] = f32x4_t{0.f, 0.f, 0.f, 0.f};

        if constexpr (GENERAL) {
            if (n_ct == 1) tile_k_loop<STREAM, DT, 1, GENERAL, SPLIT>(p, a, acc, wrow, hbuf, tok, first, my_slice);   // block-uniform
            else tile_k_loop<STREAM, DT, 2, GENERAL, SPLIT>(p, a, acc, wrow, hbuf, tok, first, my_slice);
        } else {
            auto run = [&](auto tiles) {
                constexpr int NCT = decltype(tiles)::value;
                if constexpr (NCT <= 2)
                    if (now.half >= 0) return tile_k_loop<STREAM, DT, NCT, GENERAL, kTileSplitHalf>(p, a, acc, wrow, hbuf, tok, first, my_slice);
                tile_k_loop<STREAM, DT, NCT, GENERAL, SPLIT>(p, a, acc, wrow, hbuf, tok, first, my_slice);
            };
            switch (n_ct) {                                // block-uniform
                case 1: run(std::integral_constant<int, 1>()); break;
                case 2: run(std::integral_constant<int, 2>()); break;
                case 3: run(std::integral_constant<int, 3>()); break;
                default: run(std::integral_constant<int, 4>()); break;
            }
        }

        // next block: locate it and start its first 16 weight loads before the epilogue
        // (flags[1] was last read before this block's barriers)
        if (threadIdx.x == 0 && last_pass) flags[1] = (int)drawn;
        __syncthreads();
        const int next_at = last_pass ? uni(flags[1]) : at;
        Unit next = now;
        if (next_at < total_units) {
            if (last_pass) next = locate(next_at);
            start_unit(next, last_pass ? 0 : s0 + kPassTokens, ln);
        }

        // half sums -> LDS (over the staging buffers, free after the last barrier).  A
        // tile's accumulators sit at ln * 4 plus 4 floats of padding per 16 lanes, and the
        // strides between tiles are chosen so that the reads below, whose 64 lanes want one
        // column of four different tiles, fall on 64 different banks.
        float* red = reinterpret_cast<float*>(hbuf);
        const int red_lane = ln * 4 + (ln >> 4) * 4;
#pragma unroll
        for (int t = 0; t < 2; ++t)
#pragma unroll
            for (int ct = 0; ct < 4; ++ct)
                if (ct < n_ct)
                    *reinterpret_cast<f32x4_t*>(red + wave * kRedWave + t * kRedTile + ct * kRedCt + red_lane) =
                        acc[t][ct];
        __syncthreads();
        // one wave per token slot, the block's rows in two halves of 64: ln = (row tile,
        // row) -> 64 logits of the slot, 256 consecutive bytes of the block's logits
        // and the slot's largest logit (rows past the group's end do not count): the ranking
        // kernel reads the logits only of blocks whose largest can matter.  Log-probability
        // mode: the sum of exp(z - largest) as well, the block's piece of the group's lse.
        // (A form each for whole blocks and halves: with the split a run-time value whole blocks took
        // 0.3 us longer, dense H = 512, 65536 rows, 64 tokens 34.8 us a call against 34.2, H = 3584, 32000
        // rows 69.8, 66.2.)
        auto finish = [&](auto halved) {
            constexpr bool HALF = decltype(halved)::value;
            constexpr int PARTS = HALF ? kTileSplitHalf : SPLIT;       // waves that share a row group
            constexpr int RUNS = HALF ? 1 : (ROWS + kWave - 1) / kWave;
            for (int s = wave; s < n_t; s += kTileWaves) {
                const size_t entry = (size_t)now.b * M + (kPasses ? s0 : 0) + s;
                float* dst = p.z + entry * ROWS + (HALF ? now.half * kWave : 0) + ln;
                float zs[2] = {-INFINITY, -INFINITY};
#pragma unroll
                for (int hf = 0; hf < RUNS; ++hf) {
                    const int tile = hf * 4 + (ln >> 4), row = ln & 15;   // row tile of the unit
                    const int e = (row >> 2) * 68 + (s & 15) * 4 + (row & 3);
                    const int w0 = ((tile >> 1) * PARTS) & (kTileWaves - 1);   // the row group's first wave
                    float z = 0.f;
#pragma unroll
                    for (int q = 0; q < PARTS; ++q)
                        z += red[(w0 + q) * kRedWave + (tile & 1) * kRedTile + (s >> 4) * kRedCt + e];
                    if (ROWS >= kWave || ln < ROWS) {  // (32-row blocks: the lanes above repeat the rows)
                        dst[hf * kWave] = z;
                        zs[hf] = now.first + hf * kWave + ln < now.end ? z : -INFINITY;
                    }
                }
                const float wm = wave_max(fmaxf(zs[0], zs[1]));
                float sum = 0.f;
                if (p.want_lse)                        // block-uniform
                    sum = wave_sum(wm > -INFINITY ? expf(zs[0] - wm) + expf(zs[1] - wm) : 0.f);
                if (ln == 0) {
                    float2* st = p.stat + entry;
                    if (HALF && now.half == 1) st = p.stat_upper + (entry - (size_t)split_from * M);
                    *st = make_float2(wm, sum);
                }
            }
        };
        if constexpr (HALVES) {
            if (now.half >= 0) finish(std::true_type());       // uniform
            else finish(std::false_type());
        } else {
            finish(std::false_type());
        }
        __syncthreads();
        if (kPasses) s0 = last_pass ? 0 : s0 + kPassTokens;
        at = next_at;
        now = next;
    }
}

// The table of the activated groups, then the blocks with the loads that suit the table's rows.
// GENERAL: the general path's form: any storage type, rows of any number of 16-byte vectors (the
// last chunk partly filled, loads and operands past a row's end guarded) and sums as exact as the
// staged kernels'.  Otherwise 16-bit storage and whole chunks.
template <int DT, bool GENERAL, int SPLIT>
__global__ __launch_bounds__(kTileBlock) void k_tiles(TileParams p, int dense) {
    static_assert(SPLIT == kTileSplit || GENERAL, "blocks of 32 rows exist in the general form");
    constexpr int ROWS = tile_rows(SPLIT);
    extern __shared__ uint4 smem[];
    char* lds = reinterpret_cast<char*>(smem);
    const TileLds lay = tile_lds_layout(p.u_max);
    uint4* hbuf = reinterpret_cast<uint4*>(lds + lay.o_hbuf);
    int* ustart = reinterpret_cast<int*>(lds + lay.o_ustart);
    int* uend = reinterpret_cast<int*>(lds + lay.o_uend);
    int* uprefix = reinterpret_cast<int*>(lds + lay.o_uprefix);
    unsigned long long* umask = reinterpret_cast<unsigned long long*>(lds + lay.o_umask);
    int* flags = reinterpret_cast<int*>(lds + lay.o_flags);

    const int lane = threadIdx.x & (kWave - 1);
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x / kWave);
    const int M = p.M;

    // Blocks cost different amounts (one to four token tiles), so they are handed out from
    // a queue, most expensive groups first, rather than dealt round robin.
    unsigned int drawn = 0u;
    if (threadIdx.x == 0)
        drawn = __hip_atomic_fetch_add(p.next_block, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    int total_blocks, rows = p.V;                      // blocks and weight rows of the launch
    if (dense) {
        total_blocks = (p.V + ROWS - 1) / ROWS;
        if (threadIdx.x == 0) {
            flags[1] = (int)drawn;
            flags[2] = M > kTileHalfTokens ? total_blocks : 0;
        }
        __syncthreads();
    } else {
        // The activated groups in the order the workgroups go through them: most token
        // tiles first (a block costs more the more tokens it serves), then ascending group id;
        // each with its row range, token mask and the number of blocks before it.  Every
        // workgroup builds the same table; the scratch arrays lie over the staging buffers,
        // which are free until the first K loop.
        unsigned long long* gmask = reinterpret_cast<unsigned long long*>(hbuf);      // [G]
        int* off_lds = reinterpret_cast<int*>(gmask + p.G);                            // [G + 1]
        int* ulist = off_lds + p.G + 1;                                                // [G]
        int* order = ulist + p.G;                                                      // [G]
        const int n_tt = (M + 15) / 16;
        for (int g0 = threadIdx.x; g0 <= p.G; g0 += kTileBlock) {
            off_lds[g0] = p.offsets[g0];
            if (g0 < p.G) {
                unsigned long long mk = 0ull;
                for (int c = 0; c < n_tt; ++c) mk |= p.tile_mask[(size_t)c * p.G + g0];
                gmask[g0] = mk;
                if (blockIdx.x == 0) p.group_mask[g0] = mk;
            }
        }
        __syncthreads();
        if (wave == 0) {
            int count = 0;
            for (int base = 0; base < p.G; base += kWave) {    // wave-uniform
                const int g0 = base + lane;
                const bool on = g0 < p.G && gmask[g0] != 0ull;
                const unsigned long long bal = __ballot(on);
                if (on) ulist[count + __popcll(bal & ((1ull << lane) - 1ull))] = g0;
                count += __popcll(bal);
            }
            if (count <= kWave) {
                // a group has one to four token tiles (M <= 64): four ballots place it
                const int g0 = lane < count ? ulist[lane] : 0;
                const int w0 = lane < count ? (__popcll(gmask[g0]) + 15) >> 4 : 0;
                int rank = 0;
#pragma unroll
                for (int w = 4; w >= 1; --w) {
                    const unsigned long long bal = __ballot(w0 == w);
                    if (w0 < w) rank += __popcll(bal);
                    if (w0 == w) rank += __popcll(bal & ((1ull << lane) - 1ull));
                }
                if (lane < count) order[rank] = g0;
            } else {
                // (many groups: ascending id; the order only balances the load)
                for (int r = lane; r < count; r += kWave) order[r] = ulist[r];
            }
            int carry = 0, many_end = 0, row_sum = 0;
            for (int base = 0; base < count; base += kWave) {  // wave-uniform
                const int r = base + lane;
                const int g0 = r < count ? order[r] : 0;
                const int n_rows = r < count ? off_lds[g0 + 1] - off_lds[g0] : 0;
                const int nb = (n_rows + ROWS - 1) / ROWS;
                const int incl = wave_scan_inclusive(nb);
                row_sum += __builtin_amdgcn_readlane(wave_scan_inclusive(n_rows), 63);
                if (r < count) {
                    ustart[r] = off_lds[g0];
                    uend[r] = off_lds[g0 + 1];
                    uprefix[r] = carry + incl - nb;
                    umask[r] = gmask[g0];
                    if (blockIdx.x == 0) p.group_first_block[g0] = carry + incl - nb;
                }
                const unsigned long long many = __ballot(r < count && __popcll(gmask[g0]) > kTileHalfTokens);
                if (many) many_end = carry + __builtin_amdgcn_readlane(incl, 63 - __clzll((long long)many));
                carry += __builtin_amdgcn_readlane(incl, 63);
            }
            if (lane == 0) {                           // LDS is in order within a wave
                uprefix[count] = carry;
                flags[0] = count;
                flags[2] = many_end;
                flags[3] = row_sum;
                flags[1] = (int)drawn;
            }
        }
        __syncthreads();
        total_blocks = uni(uprefix[uni(flags[0])]);
        rows = uni(flags[3]);
    }
    const int at = uni(flags[1]);
    if (rows >= p.stream_rows) tile_units<true, DT, GENERAL, SPLIT>(p, dense, at, total_blocks, lay, lds);
    else tile_units<false, DT, GENERAL, SPLIT>(p, dense, at, total_blocks, lay, lds);
}

// Gate and selection for the tile path (Eq. 7's W2 projection, then top-g): one workgroup
// per tile of 16 groups x 16 tokens and half of the columns (two workgroups share a tile: 32
// compute units pull the operands instead of 16), the columns split over its 16 waves in
// blocks of 128 (256 bytes of a row: both operands are loaded four rows x 256 bytes per wave
// load and transposed in registers); the partial tiles are summed in wave order and the two workgroups' sums by
// whoever reads the scores, in a fixed order.  The workgroups of one token tile count
// themselves in on that tile's counter; the one that arrives last has all scores of its 16
// tokens and ranks them by counting, one wave per token, writes the selection and, per
// group, the mask of those of its tokens that selected it.  The tile kernel combines the
// token tiles' masks itself, so the token tiles finish independently of each other.
struct GateSelParams {
    const uint4* hidden;                    // [M, n_vec]
    const uint4* gate_W;                    // [G, n_vec]
    const float* bias;                      // [G] or null
    float* s;                               // [parts, M, G] scores (workspace)
    int32_t* sel;                           // [M, g]
    unsigned long long* tile_mask;          // [token tiles, G] out: tokens of the tile that selected the group
    unsigned int* counters;                 // [token tiles] arrival counters, zero between calls
    int M, G, g, n_vec;
    float* logp_sel;                        // [M, g] out: log p_router of the selected group
                                            // (log-probability mode), else null
};

__device__ __forceinline__ float load_score(const float* p) {
    return __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

template <int DT>
__global__ __launch_bounds__(kFusedBlock) void k_gate_select(GateSelParams p) {
    __shared__ __attribute__((aligned(16))) float part[kFusedWaves][kGateTileFloats];
    __shared__ unsigned long long mask[kMaxG];
    __shared__ __attribute__((aligned(16))) unsigned long long sel_keys[kFusedWaves][kWave];
    __shared__ int is_last;
    const int lane = threadIdx.x & (kWave - 1);
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x / kWave);
    const int n_tt = (p.M + 15) / 16, n_gt = (p.G + 15) / 16;
    const int gt = blockIdx.x / n_tt, tt = blockIdx.x - gt * n_tt;
    float bias_r = 0.f;                                // the bias of the score this thread will sum
    if (threadIdx.x < 256 && p.bias) {
        const int gn = gt * 16 + ((threadIdx.x >> 2) >> 4) * 4 + (threadIdx.x & 3);
        if (gn < p.G) bias_r = p.bias[gn];
    }
    // A wave takes 256-byte blocks of the columns (every kFusedWaves * n_parts-th), two per
    // pass with all loads requested before the first is used: per block four wave loads of
    // four rows x 256 contiguous bytes for each operand, transposed in registers to the
    // operands of four 32-column steps (mfma_operands_from_quad_rows).
    const int q4 = lane >> 4, a4 = (lane >> 2) & 3, c4 = lane & 3;
    f32x4_t acc = f32x4_t{0.f, 0.f, 0.f, 0.f};
    const int cpart = blockIdx.y, n_parts = gridDim.y;              // the columns are split over n_parts workgroups
    const int n_blk = (p.n_vec + 15) / 16, bstride = kFusedWaves * n_parts;
    for (int blk0 = cpart * kFusedWaves + wave; blk0 < n_blk; blk0 += 2 * bstride) {     // wave-uniform
        uint4 a[2][4], b[2][4];
#pragma unroll
        for (int u = 0; u < 2; ++u) {
            const int vec = (blk0 + u * bstride) * 16 + q4 * 4 + c4;
#pragma unroll
            for (int t = 0; t < 4; ++t) {
                const int n = gt * 16 + a4 * 4 + t, m = tt * 16 + a4 * 4 + t;
                a[u][t] = make_uint4(0, 0, 0, 0);
                b[u][t] = make_uint4(0, 0, 0, 0);
                if (vec < p.n_vec) {
                    if (n < p.G) a[u][t] = p.gate_W[(size_t)n * p.n_vec + vec];
                    if (m < p.M) b[u][t] = p.hidden[(size_t)m * p.n_vec + vec];
                }
            }
        }
#pragma unroll
        for (int u = 0; u < 2; ++u) {
            if (blk0 + u * bstride >= n_blk) break;        // wave-uniform
            mfma_operands_from_quad_rows(a[u][0], a[u][1], a[u][2], a[u][3], lane);
            mfma_operands_from_quad_rows(b[u][0], b[u][1], b[u][2], b[u][3], lane);
#pragma unroll
            for (int c = 0; c < 4; ++c) acc = mfma_tile<DT>(a[u][c], b[u][c], acc);
        }
    }
    *reinterpret_cast<f32x4_t*>(&part[wave][lane * 4]) = acc;
    __syncthreads();
    if (threadIdx.x < 256) {
        const int e = threadIdx.x, l = e >> 2, i = e & 3;
        const int gn = gt * 16 + (l >> 4) * 4 + i;
        const int tm = tt * 16 + (l & 15);
        float sum = 0.f;
        for (int w = 0; w < kFusedWaves; ++w) sum += part[w][e];
        if (gn < p.G && tm < p.M)
            __hip_atomic_store(p.s + ((size_t)cpart * p.M + tm) * p.G + gn, cpart == 0 ? sum + bias_r : sum,
                               __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    }
    __builtin_amdgcn_s_waitcnt(0x0F70);                // vmcnt(0): the scores are out
    __syncthreads();
    if (threadIdx.x == 0) {
        const unsigned int old = __hip_atomic_fetch_add(p.counters + tt, 1u, __ATOMIC_RELAXED,
                                                        __HIP_MEMORY_SCOPE_AGENT);
        is_last = old == (unsigned)(n_gt * n_parts - 1) ? 1 : 0;
    }
    __syncthreads();
    if (!uni(is_last)) return;                         // block-uniform

    // the token tile is complete: its tokens tt * 16 .. + 15; a score is the sum of its parts in order
    auto score = [&](int tm, int gn) {
        float v = load_score(p.s + (size_t)tm * p.G + gn);
        for (int q = 1; q < n_parts; ++q) v += load_score(p.s + ((size_t)q * p.M + tm) * p.G + gn);
        return v;
    };
    for (int g0 = threadIdx.x; g0 < p.G; g0 += kFusedBlock) mask[g0] = 0ull;
    __syncthreads();
    if (p.G <= kWave) {
        // one wave per token, group in lane
        const int tm = tt * 16 + wave;
        if (wave < 16 && tm < p.M) {                   // wave-uniform
            float v = lane < p.G ? score(tm, lane) : -INFINITY;
            if (!(v == v)) v = -INFINITY;
            const int rank = wave_rank(sel_keys[wave], v, lane, p.G, lane);
            float lse_s = 0.f;
            if (p.logp_sel) {                          // the router's softmax over all G scores (Eq. 7)
                const float smax = wave_max(v);
                lse_s = smax + logf(wave_sum(lane < p.G ? expf(v - smax) : 0.f));
            }
            if (lane < p.G && rank < p.g) {
                atomicOr(&mask[lane], 1ull << tm);
                p.sel[tm * p.g + rank] = lane;
                if (p.logp_sel) p.logp_sel[tm * p.g + rank] = v - lse_s;
            }
        }
    } else {
        // more groups than lanes: one wave per token, up to 16 scores per lane, the g best cut out
        // by bisection and ranked among themselves.  (Counting over all pairs of groups, every
        // score read back from memory, took 20 us and more.)
        auto select_token = [&](auto regs) {
            constexpr int N = decltype(regs)::value;
            const int tm = tt * 16 + wave;
            if (tm >= p.M) return;                     // wave-uniform
            float v[N];
            unsigned long long key[N];
#pragma unroll
            for (int i = 0; i < N; ++i) {
                const int n = i * kWave + lane;
                v[i] = score(tm, n < p.G ? n : p.G - 1);
            }
            float top = -INFINITY;
#pragma unroll
            for (int i = 0; i < N; ++i) {
                const int n = i * kWave + lane;
                if (!(v[i] == v[i])) v[i] = -INFINITY;
                if (n >= p.G) v[i] = -INFINITY;
                key[i] = n < p.G ? cand_key(v[i], n) : 0ull;
                top = fmaxf(top, v[i]);
            }
            float lse_s = 0.f;
            if (p.logp_sel) {                          // the router's softmax over all G scores (Eq. 7)
                const float smax = wave_max(top);
                float sum = 0.f;
#pragma unroll
                for (int i = 0; i < N; ++i) sum += i * kWave + lane < p.G ? expf(v[i] - smax) : 0.f;
                lse_s = smax + logf(wave_sum(sum));
            }
            auto chosen = [&](int rank, int n, float s) {
                atomicOr(&mask[n], 1ull << tm);
                p.sel[tm * p.g + rank] = n;
                if (p.logp_sel) p.logp_sel[tm * p.g + rank] = s - lse_s;
            };
            if (p.g <= kWave) {                        // uniform
                wave_topk<N>(key, p.g, lane, sel_keys[wave],
                             [&](int rank, unsigned long long kk) { chosen(rank, key_id(kk), key_value(kk)); });
            } else {
                int rank[N];
#pragma unroll
                for (int i = 0; i < N; ++i) rank[i] = 0;
#pragma unroll
                for (int o = 0; o < N; ++o)
                    for (int l = 0; l < kWave; ++l) {  // wave-uniform
                        const unsigned long long other =
                            ((unsigned long long)(unsigned)__builtin_amdgcn_readlane((int)(key[o] >> 32), l) << 32) |
                            (unsigned)__builtin_amdgcn_readlane((int)(unsigned)key[o], l);
#pragma unroll
                        for (int i = 0; i < N; ++i) rank[i] += other > key[i] ? 1 : 0;
                    }
#pragma unroll
                for (int i = 0; i < N; ++i)
                    if (key[i] != 0ull && rank[i] < p.g) chosen(rank[i], i * kWave + lane, v[i]);
            }
        };
        if (p.G <= 2 * kWave) select_token(std::integral_constant<int, 2>());          // uniform
        else if (p.G <= 4 * kWave) select_token(std::integral_constant<int, 4>());
        else select_token(std::integral_constant<int, 16>());
    }
    __syncthreads();
    for (int g0 = threadIdx.x; g0 < p.G; g0 += kFusedBlock) p.tile_mask[(size_t)tt * p.G + g0] = mask[g0];
    if (threadIdx.x == 0)
        __hip_atomic_store(p.counters + tt, 0u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

// Ranking behind k_tiles: one workgroup per token.  Its blocks are those of the groups it
// selected (dense: all), and k_tiles left every block's largest logit.  The k-th largest of
// these block maxima is a lower bound of the token's k-th logit (k blocks hold a logit that
// reaches it), so only blocks whose largest reaches it can hold a result: about k of them,
// out of 128 (wide draft tree) or a thousand (dense).  Their logits, 32 blocks (4096
// candidates, eight per thread) at a time, are filtered by the bound and by the k-th entry
// of the list so far, collected in LDS with the list, and ranked by counting (64-bit
// ordering keys, all distinct).  Should more than 256 pass (k beyond 32, few blocks), a bound
// taken from the threads' best candidates as from the blocks' maxima comes first; should still
// more than 512 pass (equal logits), the same by whole keys, which are distinct.
// Log-probability mode (Eq. 8): log p(x) = log p_router(n) + z[x] - lse_n; lse_n comes from
// the (largest, sum of exp) pieces k_tiles left per block, combined in block order, and
// bounds and keys are formed from z + (log p_router(n) - lse_n).
struct TileSelectParams {
    const float* z;                         // [blocks, M, rows of a block] what k_tiles left
    const float2* stat;                     // [blocks, M]
    const float2* stat_upper;
    const int32_t* split_from;
    const int32_t* sel;                     // [M, g] selected groups (grouped)
    const int32_t* offsets;                 // [G+1]
    const int32_t* rows;                    // [V]
    const int32_t* group_first_block;       // [G] first block of an activated group
    const unsigned long long* group_mask;   // [G] tokens that selected it
    const float* logp_sel;                  // [M, g] log p_router (log-probability mode)
    unsigned int* next_block;               // k_tiles' queue: left at zero for the next call
    int32_t* topk_ids;                      // [M, k]
    float* topk_out;                        // [M, k]
    int M, V, g, k;
    int max_blocks;                         // capacity of the per-block arrays in LDS
};

constexpr int kSelectThreads = 512;
constexpr int kSelectWaves = kSelectThreads / kWave;
constexpr int kSelectKeys = 8;                   // candidates per thread and chunk
constexpr int kSelectFew = 4 * kWave;            // so many are ranked as they are
constexpr int kKeptMax = kSelectKeys * kSelectThreads + kMaxK;   // a chunk's candidates and the list

struct TileSelectLds {
    int o_buf, o_list, o_wkeys, o_start, o_rows, o_fb, o_slot, o_nb, o_pre, o_shift, o_bst, o_binfo,
        o_bval, o_qblk, o_qval, total;
};
__host__ __device__ inline TileSelectLds tile_select_lds_layout(int n_groups, int max_blocks) {
    TileSelectLds L;
    int off = 0;
    auto take = [&](size_t bytes) {
        int at = off;
        off = (int)((off + bytes + 15) / 16 * 16);
        return at;
    };
    L.o_buf = take((size_t)kKeptMax * sizeof(unsigned long long));
    L.o_list = take((size_t)kMaxK * sizeof(unsigned long long));
    L.o_wkeys = take((size_t)kSelectThreads * sizeof(unsigned long long));
    L.o_start = take((size_t)n_groups * sizeof(int));
    L.o_rows = take((size_t)n_groups * sizeof(int));
    L.o_fb = take((size_t)n_groups * sizeof(int));
    L.o_slot = take((size_t)n_groups * sizeof(int));
    L.o_nb = take((size_t)n_groups * sizeof(int));
    L.o_pre = take((size_t)(n_groups + 1) * sizeof(int));
    L.o_shift = take((size_t)n_groups * sizeof(float));
    L.o_bst = take((size_t)max_blocks * sizeof(float2));
    L.o_binfo = take((size_t)max_blocks * sizeof(int));
    L.o_bval = take((size_t)max_blocks * sizeof(unsigned));
    L.o_qblk = take((size_t)max_blocks * sizeof(int));
    L.o_qval = take((size_t)max_blocks * sizeof(unsigned));
    L.total = off;
    return L;
}

// SHIFT: log2 of k_tiles' rows per block.
template <bool DENSE, bool LP, int SHIFT>
__global__ __launch_bounds__(kSelectThreads) void k_tile_select(TileSelectParams p) {
    extern __shared__ uint4 smem[];
    char* lds = reinterpret_cast<char*>(smem);
    const int n_groups = DENSE ? 1 : p.g;
    const TileSelectLds lay = tile_select_lds_layout(n_groups, p.max_blocks);
    unsigned long long* buf = reinterpret_cast<unsigned long long*>(lds + lay.o_buf);
    unsigned long long* list = reinterpret_cast<unsigned long long*>(lds + lay.o_list);
    unsigned long long* wkeys = reinterpret_cast<unsigned long long*>(lds + lay.o_wkeys);
    int* g_start = reinterpret_cast<int*>(lds + lay.o_start);
    int* g_rows = reinterpret_cast<int*>(lds + lay.o_rows);
    int* g_fb = reinterpret_cast<int*>(lds + lay.o_fb);
    int* g_slot = reinterpret_cast<int*>(lds + lay.o_slot);
    int* g_nb = reinterpret_cast<int*>(lds + lay.o_nb);
    int* g_pre = reinterpret_cast<int*>(lds + lay.o_pre);
    float* g_shift = reinterpret_cast<float*>(lds + lay.o_shift);
    float2* bst = reinterpret_cast<float2*>(lds + lay.o_bst);
    int* binfo = reinterpret_cast<int*>(lds + lay.o_binfo);
    int* qblk = reinterpret_cast<int*>(lds + lay.o_qblk);
    unsigned* bval = reinterpret_cast<unsigned*>(lds + lay.o_bval);
    unsigned* qval = reinterpret_cast<unsigned*>(lds + lay.o_qval);
    __shared__ unsigned long long bound_w[kSelectWaves], bound_all_w[kSelectWaves];
    __shared__ unsigned tau_w[kSelectWaves], tau_all_w[kSelectWaves];
    __shared__ int n_kept, n_qual;

    const int lane = threadIdx.x & (kWave - 1);
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x / kWave);
    const int t = blockIdx.x, k = p.k;
    constexpr int rows_per_block = 1 << SHIFT;
    constexpr int chunk_blocks = kSelectKeys * kSelectThreads >> SHIFT;
    const int split_from = rows_per_block == kTileRows ? *p.split_from : 0;
    if (blockIdx.x == 0 && threadIdx.x == 0)
        __hip_atomic_store(p.next_block, 0u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    if (threadIdx.x == 0) {
        n_kept = 0;
        n_qual = 0;
    }

    // 1. the token's groups: row range, first block, the token's slot in the group's blocks
    if (DENSE) {
        if (threadIdx.x == 0) {
            g_start[0] = 0;
            g_rows[0] = p.V;
            g_fb[0] = 0;
            g_slot[0] = t;
            g_nb[0] = (p.V + rows_per_block - 1) >> SHIFT;
            g_shift[0] = 0.f;
        }
    } else {
        for (int j = threadIdx.x; j < p.g; j += kSelectThreads) {
            const int grp = p.sel[t * p.g + j];
            const int lo = p.offsets[grp], hi = p.offsets[grp + 1];
            const unsigned long long mk = p.group_mask[grp];
            g_start[j] = lo;
            g_rows[j] = hi - lo;
            g_fb[j] = p.group_first_block[grp];
            g_slot[j] = __popcll(mk & ((1ull << t) - 1ull));
            g_nb[j] = (hi - lo + rows_per_block - 1) >> SHIFT;
            g_shift[j] = 0.f;
        }
    }
    __syncthreads();
    if (wave == 0) {                                   // blocks before each group, in the token's order
        int carry = 0;
        for (int base = 0; base < n_groups; base += kWave) {   // wave-uniform
            const int j = base + lane;
            const int nb = j < n_groups ? g_nb[j] : 0;
            const int incl = wave_scan_inclusive(nb);
            if (j < n_groups) g_pre[j] = carry + incl - nb;
            carry += __builtin_amdgcn_readlane(incl, kWave - 1);
        }
        if (lane == 0) g_pre[n_groups] = carry;
    }
    __syncthreads();
    const int n_blocks = uni(g_pre[n_groups]);         // <= max_blocks: the groups are distinct

    // 2. the blocks' statistics, one block per thread and trip
    for (int i = threadIdx.x; i < n_blocks; i += kSelectThreads) {
        int lo = 0, hi = n_groups;                     // the group j with g_pre[j] <= i < g_pre[j + 1]
        while (hi - lo > 1) {
            const int mid = (lo + hi) >> 1;
            if (g_pre[mid] <= i) lo = mid; else hi = mid;
        }
        const int lb = i - g_pre[lo];
        binfo[i] = (lo << 16) | lb;
        const size_t entry = (size_t)(g_fb[lo] + lb) * p.M + g_slot[lo];
        float2 st = p.stat[entry];
        if (rows_per_block == kTileRows && g_fb[lo] + lb >= split_from) {      // processed in halves
            const float2 up = p.stat_upper[entry - (size_t)split_from * p.M];
            const float most = fmaxf(st.x, up.x);
            if (LP && most > -INFINITY) st.y = st.y * expf(st.x - most) + up.y * expf(up.x - most);
            st.x = most;
        }
        if (LP) bst[i] = st;
        else bval[i] = ord32(st.x);                    // (no offsets: the block's largest logit as it is)
    }
    __syncthreads();
    if (LP) {
        // lse of every group from its blocks' pieces, a wave per group (block in lane); the
        // offset log p_router(n) - lse_n of its entries
        for (int j = wave; j < n_groups; j += kSelectWaves) {          // wave-uniform
            float m = -INFINITY, sum = 0.f;
            for (int i = g_pre[j] + lane; i < g_pre[j + 1]; i += kWave) {
                const float2 st = bst[i];
                const float nm = fmaxf(m, st.x);
                if (nm > -INFINITY) sum = sum * expf(m - nm) + st.y * expf(st.x - nm);
                m = nm;
            }
            const float wm = wave_max(m);
            const float wsum = wave_sum(wm > -INFINITY ? sum * expf(m - wm) : 0.f);
            if (lane == 0) g_shift[j] = p.logp_sel[t * p.g + j] - (wm + logf(wsum));
        }
        __syncthreads();
    }

    // 3. the bound: a value that k block maxima reach.  Of the workgroup's threads, each with its
    // best of the candidates, two samples say one: the k-th largest of a wave's 64 (k threads of
    // that wave reach it; the largest of the waves' values counts, 0 if fewer than k threads of
    // each have a candidate), and the (k / 8)-th largest of every wave's (so many of each wave
    // reach the smallest of the eight values).  The first is exact for up to 64 candidates and the
    // tighter one for k of about 10; beyond k = 32 it says next to nothing of more (ranking 64 of
    // 3000 candidates took 80 us with it alone, 10 with the second as well).  Blocks that reach the
    // bound are the next round's candidates: 1188 blocks come down to 13 with k = 4, 34 with 10, 77
    // with 64.
    if (LP) {
        for (int i = threadIdx.x; i < n_blocks; i += kSelectThreads)
            bval[i] = ord32(bst[i].x + g_shift[binfo[i] >> 16]);
        __syncthreads();
    }
    unsigned* keys32 = reinterpret_cast<unsigned*>(wkeys) + wave * kWave;
    const int k_wave = (k + kSelectWaves - 1) / kSelectWaves;
    // what the waves' samples say together; every thread of the workgroup calls it
    auto bound_of = [&](unsigned best) {
        const TwoKeys kth = k <= 10 ? TwoKeys{wave_kth_key(keys32, best, k, lane), 0u}         // uniform
                                    : wave_kth_keys(keys32, best, k, k_wave, lane);
        if (lane == 0) {
            tau_w[wave] = kth.first;
            tau_all_w[wave] = kth.second;
        }
        __syncthreads();
        unsigned one = tau_w[0], all = tau_all_w[0];
#pragma unroll
        for (int w = 1; w < kSelectWaves; ++w) {
            one = tau_w[w] > one ? tau_w[w] : one;
            all = tau_all_w[w] < all ? tau_all_w[w] : all;
        }
        return one > all ? one : all;
    };
    unsigned tau = 0u;
    int n_q = n_blocks;
    {
        int* src_i = binfo;
        unsigned* src_v = bval;
        int* dst_i = qblk;
        unsigned* dst_v = qval;
        for (int round = 0; round < 3; ++round) {      // block-uniform
            unsigned best = 0u;
            if (n_q <= kSelectThreads && n_q > 2 * kWave && k > 10) {      // an equal share for every wave
                const int per = (n_q + kSelectWaves - 1) / kSelectWaves;
                const int i = wave * per + lane;
                if (lane < per && i < n_q) best = src_v[i];
            } else {
                for (int i = threadIdx.x; i < n_q; i += kSelectThreads) best = src_v[i] > best ? src_v[i] : best;
            }
            tau = bound_of(best);
            for (int base = 0; base < n_q; base += kSelectThreads) {   // block-uniform
                const int i = base + threadIdx.x;
                const bool on = i < n_q && src_v[i] >= tau;
                const unsigned long long bal = __ballot(on);
                int at = 0;
                if (lane == 0 && bal) at = atomicAdd(&n_qual, __popcll(bal));
                at = __builtin_amdgcn_readfirstlane(at) + __popcll(bal & ((1ull << lane) - 1ull));
                if (on) {
                    dst_i[at] = src_i[i];
                    dst_v[at] = src_v[i];
                }
            }
            __syncthreads();
            const int before = n_q;
            n_q = uni(n_qual);
            int* ti = src_i; src_i = dst_i; dst_i = ti;
            unsigned* tv = src_v; src_v = dst_v; dst_v = tv;
            // done once the candidates fit one chunk, or hardly fewer are left than before
            if (before <= kSelectThreads && (n_q <= chunk_blocks || 4 * n_q > 3 * before)) break;
            __syncthreads();                           // (everyone has the count)
            if (threadIdx.x == 0) n_qual = 0;
        }
        qblk = src_i;                                  // the blocks whose largest reaches the bound
    }

    // 5. their candidates, 4096 at a time, merged with the list so far (buf[0, have))
    int have = 0;                                      // entries of the list so far
    unsigned long long list_kth = 0ull;                // its k-th key once it has k entries
    for (int base = 0; base < n_q; base += chunk_blocks) {       // block-uniform
        unsigned long long key[kSelectKeys];
        {
            float zv[kSelectKeys];
            int idv[kSelectKeys], grp[kSelectKeys];
            bool valid[kSelectKeys];
#pragma unroll
            for (int q = 0; q < kSelectKeys; ++q) {
                const int e = q * kSelectThreads + threadIdx.x;
                const int qb = base + (e >> SHIFT), r = e & (rows_per_block - 1);
                const int info = qblk[qb < n_q ? qb : n_q - 1];
                const int j = info >> 16, lb = info & 0xffff;
                const int row = (lb << SHIFT) + r, n_rows = g_rows[j];
                valid[q] = qb < n_q && row < n_rows;
                grp[q] = j;
                zv[q] = p.z[(((size_t)(g_fb[j] + lb) * p.M + g_slot[j]) << SHIFT) + r];
                idv[q] = DENSE ? row : p.rows[g_start[j] + (row < n_rows ? row : n_rows - 1)];
            }
#pragma unroll
            for (int q = 0; q < kSelectKeys; ++q) {
                const float v = LP ? zv[q] + g_shift[grp[q]] : zv[q];
                const unsigned long long kk = cand_key(v, idv[q]);
                key[q] = valid[q] && ord32(v) >= tau && kk > list_kth ? kk : 0ull;
            }
        }
        unsigned long long pass[kSelectKeys];
        auto reserve = [&](unsigned long long bnd) {
            int mine = 0;
#pragma unroll
            for (int q = 0; q < kSelectKeys; ++q) {
                pass[q] = __ballot(key[q] != 0ull && key[q] >= bnd);
                mine += __popcll(pass[q]);
            }
            int at = 0;
            if (lane == 0 && mine) at = atomicAdd(&n_kept, mine);
            return __builtin_amdgcn_readfirstlane(at);
        };
        int at = reserve(0ull);                        // (n_kept = have: the list comes first)
        __syncthreads();
        int passed = uni(n_kept) - have;
        auto again = [&](unsigned long long bnd) {
            __syncthreads();                           // (every wave has read the count by now)
            if (threadIdx.x == 0) n_kept = have;
            __syncthreads();
            at = reserve(bnd);
            __syncthreads();
            passed = uni(n_kept) - have;
        };
        if (passed > kSelectFew) {                     // block-uniform: the candidates' own bound
            unsigned best = 0u;
#pragma unroll
            for (int q = 0; q < kSelectKeys; ++q) best = (unsigned)(key[q] >> 32) > best ? (unsigned)(key[q] >> 32) : best;
            again((unsigned long long)bound_of(best) << 32);
        }
        if (passed > kSelectThreads) {                 // block-uniform: equal values; the same by whole keys
            unsigned long long best = key[0];
#pragma unroll
            for (int q = 1; q < kSelectKeys; ++q) best = key[q] > best ? key[q] : best;
            unsigned long long* wk = wkeys + wave * kWave;
            wk[lane] = best;
            const int above = count_above(wk, kWave, best);
            auto ranked = [&](int rank) {              // the key of that rank, 0 if there is none
                const unsigned long long hit = __ballot(best != 0ull && above == rank);
                if (!hit) return 0ull;
                const int src = __ffsll((long long)hit) - 1;
                return ((unsigned long long)(unsigned)__builtin_amdgcn_readlane((int)(unsigned)(best >> 32), src) << 32) |
                       (unsigned)__builtin_amdgcn_readlane((int)(unsigned)best, src);
            };
            const unsigned long long one = ranked(k - 1), all = ranked(k_wave - 1);
            if (lane == 0) {
                bound_w[wave] = one;
                bound_all_w[wave] = all;
            }
            __syncthreads();
            unsigned long long bnd = bound_w[0], least = bound_all_w[0];
#pragma unroll
            for (int w = 1; w < kSelectWaves; ++w) {
                bnd = bound_w[w] > bnd ? bound_w[w] : bnd;
                least = bound_all_w[w] < least ? bound_all_w[w] : least;
            }
            again(bnd > least ? bnd : least);
        }
#pragma unroll
        for (int q = 0; q < kSelectKeys; ++q) {
            if ((pass[q] >> lane) & 1ull) buf[at + __popcll(pass[q] & ((1ull << lane) - 1ull))] = key[q];
            at += __popcll(pass[q]);
        }
        __syncthreads();
        const int kept = uni(n_kept);
        for (int i = threadIdx.x; i < kept; i += kSelectThreads) {
            const unsigned long long mine = buf[i];
            const int r = count_above(buf, kept, mine);
            if (r < k) list[r] = mine;
        }
        __syncthreads();
        have = kept < k ? kept : k;
        if (base + chunk_blocks >= n_q) break;   // block-uniform: that was the last chunk
        if ((int)threadIdx.x < have) buf[threadIdx.x] = list[threadIdx.x];
        if (threadIdx.x == 0) n_kept = have;
        list_kth = have == k ? list[k - 1] : 0ull;
        __syncthreads();
    }
    if ((int)threadIdx.x < k) {
        Cand c = sentinel();
        if ((int)threadIdx.x < have) {
            c.v = key_value(list[threadIdx.x]);
            c.id = key_id(list[threadIdx.x]);
        }
        p.topk_ids[(size_t)t * k + threadIdx.x] = c.id;
        p.topk_out[(size_t)t * k + threadIdx.x] = c.v;
    }
}

}  // namespace
