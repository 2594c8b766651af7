// Router pre-mix (section 3.3, Eq. 7): the router's second projection W2 is applied to
// u = act(W1 h) + h, with W1 [d,d] one row per output feature.  A d x d matrix read once per
// step for all tokens: HBM-bound like the LM head itself (33.6 MB at d = 4096 in bf16).
// One wave computes two output features at a time for up to eight tokens whose hidden
// vectors sit in LDS: both weight rows are requested whole (non-temporal, 16 KB per wave in
// flight at d = 4096), dotted with every token's vector (fp32 accumulation), and lane t
// finishes token t: activation, residual, rounding to the storage type.
//
// From a few tokens on the vector units would bound the kernel (a bf16 dot instruction per two
// products of every token), so the contraction goes to the matrix cores: k_premix_wide and
// k_premix_blocks.
#pragma once
#include "device_utils.h"
#include "fused_path.h"

namespace {

constexpr int kPremixTok = 8;                    // tokens of a workgroup (LDS residents)
constexpr int kPremixSegs = 8;                   // 1 KB segments of a row requested together
constexpr int kPremixStage = 8;                  // 16-byte vectors a thread stages through registers

struct PremixParams {
    const uint4* hidden;        // [M, n_vec]
    const uint4* W1;            // [H, n_vec]
    void* out;                  // [M, H] storage type
    int M, H, n_vec, act, tok_per_wg;
};

__device__ __forceinline__ float premix_act(float y, int act) {
    if (act == CORAL_ACT_SILU) return y / (1.0f + expf(-y));
    if (act == CORAL_ACT_RELU) return y > 0.f ? y : 0.f;
    return y;
}

template <int DT>
__global__ __launch_bounds__(kBlock) void k_premix(PremixParams p) {
    extern __shared__ uint4 smem[];                                // [tb][n_vec]
    const int lane = threadIdx.x & (kWave - 1);
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x / kWave);
    const int m0 = blockIdx.y * p.tok_per_wg;
    const int tb = p.M - m0 < p.tok_per_wg ? p.M - m0 : p.tok_per_wg;
    // The tokens' vectors are requested first and written to LDS only after the first weight
    // rows have been requested too: loads complete in order, so the wait for the tokens does
    // not wait for the weights behind them (what does not fit the registers goes directly).
    const int total = tb * p.n_vec;                                // consecutive rows: one block
    const uint4* hsrc = p.hidden + (size_t)m0 * p.n_vec;
    uint4 st[kPremixStage];
#pragma unroll
    for (int j = 0; j < kPremixStage; ++j) {
        const int i = threadIdx.x + j * kBlock;
        if (i < total) st[j] = load_vec(hsrc + i);
    }
    for (int i = threadIdx.x + kPremixStage * kBlock; i < total; i += kBlock) smem[i] = hsrc[i];
    const int n_waves = gridDim.x * kWavesPerBlock;
    const int r_first = (blockIdx.x * kWavesPerBlock + wave) * 2;
    auto commit_tokens = [&]() {                                   // every wave exactly once
        asm volatile("" ::: "memory");
#pragma unroll
        for (int j = 0; j < kPremixStage; ++j) {
            const int i = threadIdx.x + j * kBlock;
            if (i < total) store_vec(smem + i, st[j]);
        }
        __syncthreads();
    };
    bool staged = false;
    if (r_first >= p.H) commit_tokens();                           // a wave without rows (wave-uniform)
    for (int r0 = r_first; r0 < p.H; r0 += n_waves * 2) {          // wave-uniform
        const int r1 = r0 + 1 < p.H ? r0 + 1 : r0;
        float a0[kPremixTok], a1[kPremixTok];
#pragma unroll
        for (int t = 0; t < kPremixTok; ++t) a0[t] = a1[t] = 0.f;
        const uint4* w0p = p.W1 + (size_t)r0 * p.n_vec;
        const uint4* w1p = p.W1 + (size_t)r1 * p.n_vec;
        for (int base = 0; base < p.n_vec; base += kWave * kPremixSegs) {
            uint4 w0[kPremixSegs], w1[kPremixSegs];
#pragma unroll
            for (int j = 0; j < kPremixSegs; ++j) {
                const int vec = base + j * kWave + lane;
                w0[j] = make_uint4(0, 0, 0, 0);
                w1[j] = make_uint4(0, 0, 0, 0);
                if (vec < p.n_vec) {
                    w0[j] = load_stream(w0p + vec);
                    w1[j] = load_stream(w1p + vec);
                }
            }
            if (!staged) {                                         // wave-uniform: the wave's first pass
                commit_tokens();
                staged = true;
            }
#pragma unroll
            for (int j = 0; j < kPremixSegs; ++j) {
                const int vec = base + j * kWave + lane;
                const int hv = vec < p.n_vec ? vec : 0;            // the weights there are zero
#pragma unroll
                for (int t = 0; t < kPremixTok; ++t)
                    if (t < tb) {                                  // uniform
                        const uint4 h = smem[t * p.n_vec + hv];
                        a0[t] = dot_vec<DT>(w0[j], h, a0[t]);
                        a1[t] = dot_vec<DT>(w1[j], h, a1[t]);
                    }
            }
        }
        float y0 = 0.f, y1 = 0.f;                                  // lane t keeps token t's sums
#pragma unroll
        for (int t = 0; t < kPremixTok; ++t)
            if (t < tb) {
                const float s0 = wave_sum(a0[t]), s1 = wave_sum(a1[t]);
                if (lane == t) {
                    y0 = s0;
                    y1 = s1;
                }
            }
        if (lane < tb) {
            const size_t o = (size_t)(m0 + lane) * p.H;
            if (DT != kF32) {
                const unsigned short* hs = reinterpret_cast<const unsigned short*>(smem) + (size_t)lane * p.H;
                unsigned short* out = static_cast<unsigned short*>(p.out);
                out[o + r0] = narrow16<DT>(premix_act(y0, p.act) + widen16<DT>(hs[r0]));
                if (r1 != r0)
                    out[o + r1] = narrow16<DT>(premix_act(y1, p.act) + widen16<DT>(hs[r1]));
            } else {
                const float* hs = reinterpret_cast<const float*>(smem) + (size_t)lane * p.H;
                float* out = static_cast<float*>(p.out);
                out[o + r0] = premix_act(y0, p.act) + hs[r0];
                if (r1 != r0) out[o + r1] = premix_act(y1, p.act) + hs[r1];
            }
        }
    }
}

// Rows of up to 8 KB in whole 512-column chunks: the token vectors are staged in such chunks for all token
// tiles at once, and a workgroup of eight waves
// owns 16 output features: wave w takes the 64 columns w*64.. of every chunk, i.e. one
// 128-byte line of each of the 16 rows per chunk, and requests all its lines up front (the
// whole of W1 is in flight in one round).  A line pair's operands serve every token tile.
// A later chunk's token vectors are requested at the top of a chunk and written to a free
// buffer at its end.  bf16 / fp16, H a multiple of 512, at most 8 chunks, four tokens and more (H beyond
// 3072: nine and more, see coral_router_premix).
constexpr int kPremixWideWaves = 8;
constexpr int kPremixWideBlock = kPremixWideWaves * kWave;
constexpr int kPremixChunkVecs = 64;             // 16-byte vectors per 512-column chunk
constexpr int kPremixMaxChunks = 8;
constexpr int kPremixHbStride = kPremixChunkVecs + 1;            // padded rows: conflict-free B reads
constexpr int kPremixHbVecs = 64 * kPremixHbStride;              // one staging buffer: 64 token slots

__host__ __device__ inline size_t premix_wide_lds_bytes() {
    return ((size_t)2 * kPremixHbVecs + (size_t)kPremixWideWaves * kLinePairSlots) * sizeof(uint4);
}

template <int DT, int NCT, bool RING = false>
__global__ __launch_bounds__(kPremixWideBlock) void k_premix_wide(PremixParams p) {
    // NB staging buffers of 16 NCT token slots.  Loads return in order, so a token chunk
    // requested behind the weight lines would arrive only after the last of them: with one
    // or two token tiles every chunk's tokens are therefore requested first of all (they fit
    // the registers: 16 or 32 vectors per lane), staged as buffers come free, and the chunk
    // loop waits for nothing but its own weight lines.  With more token tiles the next
    // chunk's tokens are requested at the top of a chunk and staged at its end, behind the
    // weight lines (there the tokens' share of the work dominates anyway).
    // RING (three or four token tiles, H = 4096: every loop bound a constant, so that the
    // compiler's wait counts are exact): the tokens do not fit the registers whole, so both
    // streams are issued a few chunks ahead instead, interleaved in the order in which they
    // are wanted: tokens of chunk c + 2, then weight lines of chunk c + 4, at the top of
    // chunk c.  A wait for a chunk's tokens then leaves only younger requests outstanding.
    static_assert(!RING || NCT >= 3, "the ring is for token batches that do not fit the registers");
    constexpr int NB = NCT == 1 ? 8 : NCT == 2 ? 4 : 2;
    constexpr bool kUpFront = NCT <= 2;
    constexpr int D = NB - 1;
    constexpr int kBufVecs = 16 * NCT * kPremixHbStride;
    static_assert(NB * kBufVecs <= 2 * kPremixHbVecs, "the buffers fit the staging space");
    extern __shared__ uint4 smem[];
    const int lane = threadIdx.x & (kWave - 1);
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x / kWave);
    const int r16 = lane & 15, q4 = lane >> 4;
    uint4* hbuf = smem;
    uint4* my_slice = smem + 2 * kPremixHbVecs + (size_t)wave * kLinePairSlots;
    const int r0 = blockIdx.x * 16;
    const int n_chunks = p.n_vec / kPremixChunkVecs;

    // The residual term of the result this thread will write at the very end (feature and
    // token as in the last loop below): requested now, so that no trip to memory is left
    // behind the last weight line.
    constexpr int kOutPerThread = (NCT * 256 + kPremixWideBlock - 1) / kPremixWideBlock;
    unsigned short h_res[kOutPerThread];
#pragma unroll
    for (int j = 0; j < kOutPerThread; ++j) {
        const int e = threadIdx.x + j * kPremixWideBlock;
        const int ct = e >> 8, l = (e & 255) >> 2, i = e & 3;
        const int row = r0 + (l >> 4) * 4 + i, tok = ct * 16 + (l & 15);
        h_res[j] = 0;
        if (e < NCT * 256 && tok < p.M)
            h_res[j] = reinterpret_cast<const unsigned short*>(p.hidden)[(size_t)tok * p.H + row];
    }
    // token of slot wave + 8 i; slots past the last token hold zeros (never stored to u)
    auto fetch = [&](int c, uint4 (&st)[2 * NCT]) {
        const uint4* src = p.hidden + c * kPremixChunkVecs + lane;
#pragma unroll
        for (int i = 0; i < 2 * NCT; ++i) {
            const int s = wave + i * kPremixWideWaves;
            st[i] = make_uint4(0, 0, 0, 0);
            if (s < p.M) st[i] = load_vec(src + (size_t)s * p.n_vec);      // wave-uniform
        }
    };
    auto stage = [&](int c, const uint4 (&st)[2 * NCT]) {
        uint4* dst = hbuf + (size_t)(c % NB) * kBufVecs + (size_t)wave * kPremixHbStride + lane;
#pragma unroll
        for (int i = 0; i < 2 * NCT; ++i) store_vec(dst + (size_t)i * kPremixWideWaves * kPremixHbStride, st[i]);
    };
    if (RING) {
        constexpr int kN = kPremixMaxChunks;
        uint4 tka[2 * NCT], tkb[2 * NCT];              // token chunks: even ones in tka, odd ones in tkb
        uint4 lo[kN], hi[kN];
        const uint4* wlo = p.W1 + (size_t)(r0 + line_load_row(lane)) * p.n_vec + wave * 8 + line_load_chunk(lane);
        const uint4* whi = wlo + (size_t)8 * p.n_vec;
        auto lines = [&](int c) {
            lo[c] = load_stream(wlo + c * kPremixChunkVecs);
            hi[c] = load_stream(whi + c * kPremixChunkVecs);
        };
        fetch(0, tka);
        asm volatile("" ::: "memory");
        lines(0);
        asm volatile("" ::: "memory");
        fetch(1, tkb);
        asm volatile("" ::: "memory");
        lines(1);
        lines(2);
        lines(3);
        asm volatile("" ::: "memory");
        stage(0, tka);
        __syncthreads();
        f32x4_t acc[NCT];
#pragma unroll
        for (int ct = 0; ct < NCT; ++ct) acc[ct] = f32x4_t{0.f, 0.f, 0.f, 0.f};
#pragma unroll
        for (int c = 0; c < kN; ++c) {
            if (c + 2 < kN) {                          // (chunk c's tokens left these registers before the last barrier)
                if (c % 2 == 0) fetch(c + 2, tka); else fetch(c + 2, tkb);
            }
            asm volatile("" ::: "memory");
            if (c + 4 < kN) lines(c + 4);
            asm volatile("" ::: "memory");
            uint4 s0, s1;
            mfma_operands_from_lines(lo[c], hi[c], lane, my_slice, s0, s1);
            const uint4* hb = hbuf + (size_t)(c % NB) * kBufVecs + wave * 8 + q4;
#pragma unroll
            for (int ct = 0; ct < NCT; ++ct) {
                const uint4 b0 = hb[(ct * 16 + r16) * kPremixHbStride];
                const uint4 b1 = hb[(ct * 16 + r16) * kPremixHbStride + 4];
                acc[ct] = mfma_tile<DT>(s0, b0, acc[ct]);
                acc[ct] = mfma_tile<DT>(s1, b1, acc[ct]);
            }
            // buffer (c + 1) % 2 was last read in chunk c - 1, before its barrier
            if (c + 1 < kN) {
                if ((c + 1) % 2 == 0) stage(c + 1, tka); else stage(c + 1, tkb);
                __syncthreads();
            }
        }
        __syncthreads();                               // every wave is done with the staging buffers
        float* red = reinterpret_cast<float*>(hbuf);   // [wave][token tile][256]
#pragma unroll
        for (int ct = 0; ct < NCT; ++ct)
            *reinterpret_cast<f32x4_t*>(red + ((size_t)wave * NCT + ct) * 256 + lane * 4) = acc[ct];
        __syncthreads();
#pragma unroll
        for (int j = 0; j < kOutPerThread; ++j) {
            const int e = threadIdx.x + j * kPremixWideBlock;
            if (e >= NCT * 256) break;
            const int ct = e >> 8, l = (e & 255) >> 2, i = e & 3;
            const int row = r0 + (l >> 4) * 4 + i, tok = ct * 16 + (l & 15);
            float y = 0.f;
#pragma unroll
            for (int w = 0; w < kPremixWideWaves; ++w) y += red[((size_t)w * NCT + ct) * 256 + (e & 255)];
            if (tok < p.M)
                static_cast<unsigned short*>(p.out)[(size_t)tok * p.H + row] =
                    narrow16<DT>(premix_act(y, p.act) + widen16<DT>(h_res[j]));
        }
        return;
    }
    constexpr int kHeld = kUpFront ? kPremixMaxChunks : D;
    uint4 tk[kHeld][2 * NCT];
#pragma unroll
    for (int c = 0; c < kHeld; ++c)
        if (c < n_chunks) fetch(c, tk[c]);             // block-uniform
    asm volatile("" ::: "memory");                     // (keeps the order: tokens first, they return first)
    uint4 lo[kPremixMaxChunks], hi[kPremixMaxChunks];
    const uint4* wlo = p.W1 + (size_t)(r0 + line_load_row(lane)) * p.n_vec + wave * 8 + line_load_chunk(lane);
    const uint4* whi = wlo + (size_t)8 * p.n_vec;
#pragma unroll
    for (int c = 0; c < kPremixMaxChunks; ++c) {
        lo[c] = make_uint4(0, 0, 0, 0);
        hi[c] = make_uint4(0, 0, 0, 0);
        if (c < n_chunks) {                            // block-uniform
            lo[c] = load_stream(wlo + c * kPremixChunkVecs);
            hi[c] = load_stream(whi + c * kPremixChunkVecs);
        }
    }
    asm volatile("" ::: "memory");
#pragma unroll
    for (int c = 0; c < (kUpFront ? NB : D); ++c)
        if (c < n_chunks) stage(c, tk[c]);
    // The memory serves requests in the order it got them, and the other workgroups' weight
    // lines are ahead of a late workgroup's tokens: the last tokens arrive when most of W1
    // has (5 of 6.5 us at 8 tokens).  While the workgroup waits for them at the barrier, every
    // wave moves the weight lines it has got to the operand layout (its own lines, its own
    // LDS slice), so that only operand reads and matrix instructions are left behind it.
    if (kUpFront) {
#pragma unroll
        for (int c = 0; c < kPremixMaxChunks; ++c)
            if (c < n_chunks) {                        // block-uniform
                uint4 s0, s1;
                mfma_operands_from_lines(lo[c], hi[c], lane, my_slice, s0, s1);
                lo[c] = s0;
                hi[c] = s1;
            }
    }
    __syncthreads();
    f32x4_t acc[NCT];
#pragma unroll
    for (int ct = 0; ct < NCT; ++ct) acc[ct] = f32x4_t{0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int c = 0; c < kPremixMaxChunks; ++c) {
        if (c < n_chunks) {                            // block-uniform
            const bool more = kUpFront ? c + NB < n_chunks : c + D < n_chunks;
            uint4 st[2 * NCT];
            if (!kUpFront && more) fetch(c + D, st);
            asm volatile("" ::: "memory");
            uint4 s0 = lo[c], s1 = hi[c];
            if (!kUpFront) mfma_operands_from_lines(lo[c], hi[c], lane, my_slice, s0, s1);
            const uint4* hb = hbuf + (size_t)(c % NB) * kBufVecs + wave * 8 + q4;
#pragma unroll
            for (int ct = 0; ct < NCT; ++ct) {
                const uint4 b0 = hb[(ct * 16 + r16) * kPremixHbStride];
                const uint4 b1 = hb[(ct * 16 + r16) * kPremixHbStride + 4];
                acc[ct] = mfma_tile<DT>(s0, b0, acc[ct]);
                acc[ct] = mfma_tile<DT>(s1, b1, acc[ct]);
            }
            if (kUpFront) {
                // buffer c % NB is free once every wave has read chunk c: its next tenant,
                // chunk c + NB, has been waiting in registers
                if (more) {
                    __syncthreads();
                    if (c + NB < kPremixMaxChunks) stage(c + NB, tk[c + NB < kHeld ? c + NB : 0]);
                    // (the next chunk's barrier, if it has one, also stands between this
                    // write and the reads of chunk c + NB)
                    if (!(c + 1 + NB < n_chunks)) __syncthreads();
                }
            } else {
                // buffer (c + D) % NB = (c - 1) % NB was last read in chunk c - 1, before its barrier
                if (more) stage(c + D, st);
                if (c + 1 < n_chunks) __syncthreads();
            }
        }
    }
    __syncthreads();                                   // every wave is done with the staging buffers
    // the waves' partial tiles, summed in wave order; lane l of a tile holds features
    // 4*(l/16)..+4 of token l%16
    float* red = reinterpret_cast<float*>(hbuf);       // [wave][token tile][256]
#pragma unroll
    for (int ct = 0; ct < NCT; ++ct)
        *reinterpret_cast<f32x4_t*>(red + ((size_t)wave * NCT + ct) * 256 + lane * 4) = acc[ct];
    __syncthreads();
#pragma unroll
    for (int j = 0; j < kOutPerThread; ++j) {
        const int e = threadIdx.x + j * kPremixWideBlock;
        if (e >= NCT * 256) break;
        const int ct = e >> 8, l = (e & 255) >> 2, i = e & 3;
        const int row = r0 + (l >> 4) * 4 + i, tok = ct * 16 + (l & 15);
        float y = 0.f;
#pragma unroll
        for (int w = 0; w < kPremixWideWaves; ++w) y += red[((size_t)w * NCT + ct) * 256 + (e & 255)];
        if (tok < p.M)
            static_cast<unsigned short*>(p.out)[(size_t)tok * p.H + row] =
                narrow16<DT>(premix_act(y, p.act) + widen16<DT>(h_res[j]));
    }
}

// Any width and storage type: a workgroup of eight waves owns 16 output features, its waves share
// the columns in blocks of 256 bytes (every eighth), and both operands of a block are loaded four
// rows x 256 bytes per wave load and transposed in registers: no staging of the tokens, no barrier
// before the sums at the end, two workgroups per compute unit.  The tokens come out of the L2, D
// blocks ahead like the weights (loads return in order: tokens requested later than the next
// block's weights would wait for them).  Bound by the weights' stream and, from two token tiles on,
// the tokens' out of the L2.  us a call, against the forms it replaces (four waves holding 16 lines of
// every row, one token tile at a time; the vector units): bf16 H = 6016, 16 tokens 40.3 -> 20.2, 64 tokens
// 112.5 -> 37.4 (bytes at 6.8 TB/s: 10.6), H = 2568, 16 tokens 13.9 -> 7.3; fp32 H = 4096, 16 tokens
// 60.4 -> 18.3.
// Sums no less exact than theirs: a wave keeps one per 32 columns of a block for at most four blocks (16
// bits), or a block's products with the rounding error kept (fp32).  Values of u that fall on the other
// side of a rounding boundary, vector units / one running sum per wave / this: bf16 H = 4096 6.1e-5, 8.8e-5,
// 6.0e-5 of them, H = 7168 7.2e-5, 1.29e-4, 6.9e-5, H = 10248 8.6e-5, 1.59e-4, 7.5e-5; fp32 H = 4096,
// relative error 1.1e-7, 2e-7, 0.75e-7.  (Every block's sum added with its rounding error, 16 bits: 5.4e-5
// at H = 4096, but 5 to 10 % slower.)
constexpr int kPremixBlockWaves = 8;
constexpr int kPremixBlockThreads = kPremixBlockWaves * kWave;
template <int DT, int NCT, int D>
__global__ __launch_bounds__(kPremixBlockThreads, NCT == 1 ? 4 : 2) void k_premix_blocks(PremixParams p) {
    __shared__ __attribute__((aligned(16))) float red[kPremixBlockWaves * NCT * 256];
    const int lane = threadIdx.x & (kWave - 1);
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x / kWave);
    static_assert(4 % D == 0 || DT == kF32, "the sums are gathered between trips");
    const int q4 = lane >> 4, a4 = (lane >> 2) & 3, c4 = lane & 3;
    const int r0 = blockIdx.x * 16, m0 = blockIdx.y * NCT * 16;
    const int tb = p.M - m0;                                       // tokens from m0 on
    const uint4* hidden = p.hidden + (size_t)m0 * p.n_vec;
    // the residual of the results this thread will write, as in k_premix_wide
    constexpr int kOutPerThread = (NCT * 256 + kPremixBlockThreads - 1) / kPremixBlockThreads;
    float h_res[kOutPerThread];
#pragma unroll
    for (int j = 0; j < kOutPerThread; ++j) {
        const int e = threadIdx.x + j * kPremixBlockThreads;
        const int l = (e & 255) >> 2, row = r0 + (l >> 4) * 4 + (e & 3), tok = (e >> 8) * 16 + (l & 15);
        h_res[j] = 0.f;
        if (e < NCT * 256 && tok < tb && row < p.H) {
            const size_t at = (size_t)tok * p.H + row;
            if (DT == kF32) h_res[j] = reinterpret_cast<const float*>(hidden)[at];
            else h_res[j] = widen16<DT>(reinterpret_cast<const unsigned short*>(hidden)[at]);
        }
    }
    const int n_blk = (p.n_vec + 15) / 16;
    const int n = (n_blk - wave + kPremixBlockWaves - 1) / kPremixBlockWaves;      // this wave's blocks
    uint4 a[D][4], b[D][NCT][4];
    auto load = [&](int i, int slot) {
        const int vec = (wave + i * kPremixBlockWaves) * 16 + q4 * 4 + c4;
        const bool in = vec < p.n_vec;
#pragma unroll
        for (int t = 0; t < 4; ++t) {
            const int row = r0 + a4 * 4 + t;
            a[slot][t] = make_uint4(0, 0, 0, 0);
            if (in && row < p.H) a[slot][t] = load_stream(p.W1 + (size_t)row * p.n_vec + vec);
        }
#pragma unroll
        for (int ct = 0; ct < NCT; ++ct)
#pragma unroll
            for (int t = 0; t < 4; ++t) {
                const int m = ct * 16 + a4 * 4 + t;
                b[slot][ct][t] = make_uint4(0, 0, 0, 0);
                if (in && m < tb) b[slot][ct][t] = load_vec(hidden + (size_t)m * p.n_vec + vec);
            }
    };
#pragma unroll
    for (int k = 0; k < D; ++k)
        if (k < n) load(k, k);                                     // wave-uniform
    // Sums: 16 bits, one per 32 columns of a block, gathered in `total` every four blocks; fp32, acc[0]
    // with its rounding errors in acc[1].
    f32x4_t acc[NCT][4], total[NCT];
    auto gather = [&]() {
#pragma unroll
        for (int ct = 0; ct < NCT; ++ct) {
            total[ct] += (acc[ct][0] + acc[ct][1]) + (acc[ct][2] + acc[ct][3]);
#pragma unroll
            for (int c = 0; c < 4; ++c) acc[ct][c] = f32x4_t{0.f, 0.f, 0.f, 0.f};
        }
    };
#pragma unroll
    for (int ct = 0; ct < NCT; ++ct) {
        total[ct] = f32x4_t{0.f, 0.f, 0.f, 0.f};
#pragma unroll
        for (int c = 0; c < 4; ++c) acc[ct][c] = f32x4_t{0.f, 0.f, 0.f, 0.f};
    }
    for (int i = 0; i < n; i += D) {                               // wave-uniform
        if (DT != kF32 && i > 0 && i % 4 == 0) gather();
#pragma unroll
        for (int k = 0; k < D; ++k) {
            if (i + k < n) {
                mfma_operands_from_quad_rows(a[k][0], a[k][1], a[k][2], a[k][3], lane);
#pragma unroll
                for (int ct = 0; ct < NCT; ++ct) {
                    mfma_operands_from_quad_rows(b[k][ct][0], b[k][ct][1], b[k][ct][2], b[k][ct][3], lane);
                    if (DT == kF32) {
                        // a block's products start from zero and are added with the rounding error
                        // kept (two-sum), as in k_tiles' general form
                        const f32x4_t zero = f32x4_t{0.f, 0.f, 0.f, 0.f};
                        const f32x4_t x = (mfma_tile<DT>(a[k][0], b[k][ct][0], zero) + mfma_tile<DT>(a[k][1], b[k][ct][1], zero)) +
                                          (mfma_tile<DT>(a[k][2], b[k][ct][2], zero) + mfma_tile<DT>(a[k][3], b[k][ct][3], zero));
#pragma unroll
                        for (int q = 0; q < 4; ++q) {
                            const float hi = acc[ct][0][q], sum = hi + x[q], back = sum - hi;
                            acc[ct][1][q] += (hi - (sum - back)) + (x[q] - back);
                            acc[ct][0][q] = sum;
                        }
                    } else {
#pragma unroll
                        for (int c = 0; c < 4; ++c) acc[ct][c] = mfma_tile<DT>(a[k][c], b[k][ct][c], acc[ct][c]);
                    }
                }
                if (i + k + D < n) load(i + k + D, k);
            }
        }
    }
    if (DT != kF32) gather();
#pragma unroll
    for (int ct = 0; ct < NCT; ++ct) {
        if (DT == kF32) {
#pragma unroll
            for (int q = 0; q < 4; ++q) {              // (an infinite sum's error is NaN)
                const float sum = acc[ct][0][q] + acc[ct][1][q];
                total[ct][q] = __builtin_isfinite(sum) ? sum : acc[ct][0][q];
            }
        }
        *reinterpret_cast<f32x4_t*>(red + ((size_t)wave * NCT + ct) * 256 + lane * 4) = total[ct];
    }
    __syncthreads();
#pragma unroll
    for (int j = 0; j < kOutPerThread; ++j) {
        const int e = threadIdx.x + j * kPremixBlockThreads;
        if (e >= NCT * 256) break;
        const int ct = e >> 8, l = (e & 255) >> 2, row = r0 + (l >> 4) * 4 + (e & 3), tok = ct * 16 + (l & 15);
        auto part = [&](int w) { return red[((size_t)w * NCT + ct) * 256 + (e & 255)]; };
        static_assert(kPremixBlockWaves == 8, "");
        const float y = ((part(0) + part(1)) + (part(2) + part(3))) + ((part(4) + part(5)) + (part(6) + part(7)));
        if (tok < tb && row < p.H) {
            const float u = premix_act(y, p.act) + h_res[j];
            const size_t at = (size_t)(m0 + tok) * p.H + row;
            if (DT == kF32) static_cast<float*>(p.out)[at] = u;
            else static_cast<unsigned short*>(p.out)[at] = narrow16<DT>(u);
        }
    }
}

}  // namespace
