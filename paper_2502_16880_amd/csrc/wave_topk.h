// Selections done by one wave: the k largest of keys held in its registers, and the k best of
// many sorted lists.  Keys are 64-bit order keys (cand_key: larger value first, then lower id),
// all distinct; zero stands for "no candidate".
#pragma once
#include "device_utils.h"
#include <type_traits>

namespace {

__device__ __forceinline__ Cand sentinel() {
    Cand c;
    c.v = -INFINITY;
    c.id = INT_MAX;
    return c;
}
__device__ __forceinline__ bool is_real(Cand c) { return c.id != INT_MAX; }

// Candidates that cross workgroups are written and read with agent-scope atomic accesses (they
// go through to memory, past the per-XCD L2), so that publishing needs no L2 write-back fence.
__device__ __forceinline__ void publish_cand(Cand* dst, float v, int id) {
    const unsigned long long bits =
        ((unsigned long long)(unsigned)id << 32) | (unsigned long long)(unsigned)__float_as_int(v);
    __hip_atomic_store(reinterpret_cast<unsigned long long*>(dst), bits, __ATOMIC_RELAXED,
                       __HIP_MEMORY_SCOPE_AGENT);
}
__device__ __forceinline__ Cand fetch_cand(const Cand* src) {
    const unsigned long long bits = __hip_atomic_load(
        reinterpret_cast<const unsigned long long*>(src), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    Cand c;
    c.v = __int_as_float((int)(unsigned)(bits & 0xffffffffull));
    c.id = (int)(unsigned)(bits >> 32);
    return c;
}

__device__ __forceinline__ unsigned long long real_key(Cand c) { return is_real(c) ? cand_key(c.v, c.id) : 0ull; }
__device__ __forceinline__ Cand key_cand(unsigned long long key) {
    Cand c = sentinel();
    if (key != 0ull) {
        c.v = key_value(key);
        c.id = key_id(key);
    }
    return c;
}

// Number of keys[0, n) above `key`.  keys is LDS that this wave wrote itself (a wave's LDS
// accesses complete in order); every lane reads the same address, which LDS broadcasts.
__device__ __forceinline__ int count_above(const unsigned long long* keys, int n, unsigned long long key) {
    int r = 0;
#pragma unroll 8
    for (int j = 0; j < n; ++j) r += keys[j] > key ? 1 : 0;    // wave-uniform trip count
    return r;
}

// Rank of this lane's candidate among the candidates of lanes [0, n), n <= 64: the number
// of those that beat it.  Candidates are distinct under the total order (distinct ids).
__device__ __forceinline__ int wave_rank(unsigned long long* keys, float v, int id, int n, int lane) {
    const unsigned long long key = cand_key(v, id);
    keys[lane] = key;
    return count_above(keys, n, key);
}

template <int CTRL, int ROW_MASK>
__device__ __forceinline__ float dpp_max(float x) {
    const int moved = __builtin_amdgcn_update_dpp(__float_as_int(x), __float_as_int(x), CTRL, ROW_MASK, 0xf, false);
    return fmaxf(x, __int_as_float(moved));
}
// Maximum over the 64 lanes (no NaN among the inputs), wave-uniform.
__device__ __forceinline__ float wave_max(float x) {
    x = dpp_max<0x111, 0xf>(x);   // row_shr:1
    x = dpp_max<0x112, 0xf>(x);   // row_shr:2
    x = dpp_max<0x114, 0xf>(x);   // row_shr:4
    x = dpp_max<0x118, 0xf>(x);   // row_shr:8
    x = dpp_max<0x142, 0xa>(x);   // row_bcast:15
    x = dpp_max<0x143, 0xc>(x);   // row_bcast:31
    return __int_as_float(__builtin_amdgcn_readlane(__float_as_int(x), 63));
}

// Order-preserving 32-bit key of a logit (0 is below every logit, used for padding).
__device__ __forceinline__ unsigned ord32(float v) {
    const unsigned u = __float_as_uint(v + 0.0f);
    return u ^ ((u >> 31) ? 0xffffffffu : 0x80000000u);
}

template <int CTRL, int ROW_MASK>
__device__ __forceinline__ unsigned dpp_min(unsigned x) {
    const unsigned moved = (unsigned)__builtin_amdgcn_update_dpp((int)x, (int)x, CTRL, ROW_MASK, 0xf, false);
    return x < moved ? x : moved;
}
__device__ __forceinline__ unsigned wave_min_u32(unsigned x) {
    x = dpp_min<0x111, 0xf>(x);   // row_shr:1
    x = dpp_min<0x112, 0xf>(x);   // row_shr:2
    x = dpp_min<0x114, 0xf>(x);   // row_shr:4
    x = dpp_min<0x118, 0xf>(x);   // row_shr:8
    x = dpp_min<0x142, 0xa>(x);   // row_bcast:15
    x = dpp_min<0x143, 0xc>(x);   // row_bcast:31
    return (unsigned)__builtin_amdgcn_readlane((int)x, 63);
}
__device__ __forceinline__ unsigned wave_max_u32(unsigned x) { return ~wave_min_u32(~x); }

// e / k for 0 <= e < 4096 and 1 <= k <= 64 without an integer division.
__device__ __forceinline__ int div_small(int e, int inv_k) { return (int)(((unsigned)e * (unsigned)inv_k) >> 20); }
__device__ __forceinline__ int inv_small(int k) { return (1 << 20) / k + 1; }

// ---------------------------------------------------------------- bounds and selection
// How many of the wave's keys (N per lane) reach `bound`; wave-uniform.
template <int N>
__device__ __forceinline__ int count_reach(const unsigned long long (&key)[N], unsigned long long bound) {
    int n = 0;
#pragma unroll
    for (int i = 0; i < N; ++i) n += __popcll(__ballot(key[i] >= bound));
    return n;
}

// k-th largest of the 64 lanes' keys by counting (k <= 64); wave-uniform.  keys32: 64
// wave-private LDS words, 16-byte aligned.
__device__ __forceinline__ unsigned wave_kth_key(unsigned* keys32, unsigned key, int k, int lane) {
    keys32[lane] = key;
    int above = 0;
#pragma unroll 4
    for (int j = 0; j < kWave / 4; ++j) {
        const uint4 q = reinterpret_cast<const uint4*>(keys32)[j];
        above += (q.x > key ? 1 : 0) + (q.y > key ? 1 : 0) + (q.z > key ? 1 : 0) + (q.w > key ? 1 : 0);
    }
    return wave_min_u32(above < k ? key : 0xffffffffu);
}
// The same for two ranks at once.
struct TwoKeys {
    unsigned first, second;
};
__device__ __forceinline__ TwoKeys wave_kth_keys(unsigned* keys32, unsigned key, int k1, int k2, int lane) {
    keys32[lane] = key;
    int above = 0;
#pragma unroll 4
    for (int j = 0; j < kWave / 4; ++j) {
        const uint4 q = reinterpret_cast<const uint4*>(keys32)[j];
        above += (q.x > key ? 1 : 0) + (q.y > key ? 1 : 0) + (q.z > key ? 1 : 0) + (q.w > key ? 1 : 0);
    }
    return {wave_min_u32(above < k1 ? key : 0xffffffffu), wave_min_u32(above < k2 ? key : 0xffffffffu)};
}

// A bound that at least `want` and at most `most` (>= want) of the wave's keys reach; 1 (every
// key reaches it) if there are no more than `most`, or fewer than `want`.  First the want-th
// largest of the lanes' best keys (`want` lanes reach it), tight enough for a `want` of up to
// about 20.  Where it is not (its sample says nothing from want = 33 on; equal values),
// bisection on the key values: a step is N compares whose lane masks are counted on the scalar
// unit, and it ends because the keys are distinct.  (Bisection alone, without the sample, made
// the last merge of a step 1.1 us longer: some ten steps of a dependent compare, count and
// branch.)  keys32: 64 wave-private LDS words, 16-byte aligned.
template <int N>
__device__ __forceinline__ unsigned long long wave_bound(const unsigned long long (&key)[N], int want, int most,
                                                         unsigned* keys32, int lane) {
    const int n = count_reach<N>(key, 1ull);
    if (n <= most || n < want) return 1ull;
    unsigned best = 0u;
#pragma unroll
    for (int i = 0; i < N; ++i) {
        const unsigned h = (unsigned)(key[i] >> 32);
        best = h > best ? h : best;
    }
    unsigned long long lo = 1ull;
    if (want <= kWave / 2) {
        const unsigned kth = wave_kth_key(keys32, best, want, lane);
        if (kth != 0u) lo = (unsigned long long)kth << 32;
        if (count_reach<N>(key, lo) <= most) return lo;
    } else if (want <= kWave) {                                // the least of the lanes' best is reached by all lanes
        const unsigned least = wave_min_u32(best);
        if (least != 0u) lo = (unsigned long long)least << 32;
    }
    const unsigned top = wave_max_u32(best);
    unsigned long long hi = top == 0xffffffffu ? ~0ull : (unsigned long long)(top + 1u) << 32;   // reached by none
    while (hi - lo > 1ull) {                                   // wave-uniform; at most 64 steps
        const unsigned long long mid = lo + ((hi - lo) >> 1);
        const int c = count_reach<N>(key, mid);
        if (c >= want) {
            lo = mid;
            if (c <= most) break;
        } else {
            hi = mid;
        }
    }
    return lo;
}

// Appends the lanes' keys that reach `bound` (>= 1) to buf[n...cap); returns the new count (no more
// than cap, which distinct keys do not exceed: an index with repeated rows must not write past it).
__device__ __forceinline__ int wave_append(unsigned long long* buf, int n, int cap, unsigned long long key,
                                           unsigned long long bound, int lane) {
    const unsigned long long b = __ballot(key >= bound);
    const int at = n + __popcll(b & ((1ull << lane) - 1ull));
    if (key >= bound && at < cap) buf[at] = key;
    n += __popcll(b);
    return n < cap ? n : cap;
}

// The k <= 64 largest of the wave's keys in order: put(rank, key) once for every rank < k (key 0
// past the last one).  buf: 64 wave-private LDS words, 16-byte aligned.
template <int N, class Put>
__device__ __forceinline__ void wave_topk(const unsigned long long (&key)[N], int k, int lane,
                                          unsigned long long* buf, Put put) {
    const unsigned long long bound = N == 1 ? 1ull : wave_bound<N>(key, k, kWave, reinterpret_cast<unsigned*>(buf), lane);
    int n = 0;
#pragma unroll
    for (int i = 0; i < N; ++i) n = wave_append(buf, n, kWave, key[i], bound, lane);
    const unsigned long long mine = lane < n ? buf[lane] : 0ull;
    const int r = count_above(buf, n, mine);
    if (lane < n && r < k) put(r, mine);
    if (lane >= n && lane < k) put(lane, 0ull);
}

// wave_topk for keys[0, n) in LDS (in any order), n <= 1024.
template <class Put>
__device__ __forceinline__ void wave_topk_lds(const unsigned long long* keys, int n, int k, int lane,
                                              unsigned long long* buf, Put put) {
    asm volatile("" : "+v"(lane));     // (see wave_merge_lists)
    auto run = [&](auto regs) {
        constexpr int N = decltype(regs)::value;
        unsigned long long key[N];
#pragma unroll
        for (int i = 0; i < N; ++i) key[i] = i * kWave + lane < n ? keys[i * kWave + lane] : 0ull;
        wave_topk<N>(key, k, lane, buf, put);
    };
    if (n <= kWave) run(std::integral_constant<int, 1>());             // wave-uniform
    else if (n <= 2 * kWave) run(std::integral_constant<int, 2>());
    else if (n <= 4 * kWave) run(std::integral_constant<int, 4>());
    else if (n <= 8 * kWave) run(std::integral_constant<int, 8>());
    else run(std::integral_constant<int, 16>());
}
constexpr int kTopkLdsMax = 16 * kWave;

// Wave-private LDS of a list merge.
constexpr int kMergeKeys = 256;
struct MergeScratch {
    __attribute__((aligned(16))) unsigned long long keys[kMergeKeys];
    int tags[kWave];
    Cand out[kWave];
};

// One wave merges n_lists <= 256 sorted lists of k candidates (get(list, i), padding entries are
// sentinels) into the k best, put(rank, key) for every rank < k.  The lists are far away, in
// memory: few candidates are fetched in one trip.  Else the lists' first entries come first: k of
// them reach a bound, so only the lists whose first entry reaches it (at most 64, one per lane)
// can contribute; of those, entries are fetched three at a time for as long as a list's last one
// reaches the bound.  More than 64 survivors between two trips are cut back to the k best first.
template <class Get, class Put>
__device__ __forceinline__ void wave_merge_lists(int n_lists, int k, int lane, MergeScratch* ms, Get get, Put put) {
    constexpr int kDeep = 3;
    static_assert(kWave + kDeep * kWave <= kMergeKeys, "a trip's candidates fit behind 64 survivors");
    asm volatile("" : "+v"(lane));     // (or what is derived from it is kept in registers from the kernel's start)
    unsigned long long key[4];
    const int n_e = n_lists * k;
    const int inv_k = inv_small(k);
    if (n_e <= kWave) {                                        // wave-uniform
        const int e = lane < n_e ? lane : n_e - 1;
        const int l = div_small(e, inv_k);
        const unsigned long long key0 = real_key(get(l, e - l * k));
        const unsigned long long one[1] = {lane < n_e ? key0 : 0ull};
        wave_topk<1>(one, k, lane, ms->keys, put);
        return;
    }
    // (All fetches are unconditional, from clamped places, and what must not count is dropped
    // afterwards: in a guarded fetch the compiler starts the conversion to a key inside the guard,
    // which waits for that fetch before the next one is issued. Three such fetches in a row cost
    // 1.2 us more than one.)
    auto fetch_all = [&](auto regs) {                          // all entries in one trip
        constexpr int N = decltype(regs)::value;
        Cand c[N];
        unsigned long long key[N];
#pragma unroll
        for (int u = 0; u < N; ++u) {
            int e = u * kWave + lane;
            e = e < n_e ? e : n_e - 1;
            const int l = div_small(e, inv_k);
            c[u] = get(l, e - l * k);
        }
#pragma unroll
        for (int u = 0; u < N; ++u) key[u] = u * kWave + lane < n_e ? real_key(c[u]) : 0ull;
        wave_topk<N>(key, k, lane, ms->keys, put);
    };
    if (n_e <= 4 * kWave) {
        fetch_all(std::integral_constant<int, 4>());
        return;
    }
    if (n_e <= 8 * kWave) {
        fetch_all(std::integral_constant<int, 8>());
        return;
    }
    Cand c[4];
#pragma unroll
    for (int u = 0; u < 4; ++u) {
        const int l = u * kWave + lane;
        c[u] = get(l < n_lists ? l : n_lists - 1, 0);
    }
#pragma unroll
    for (int u = 0; u < 4; ++u) key[u] = u * kWave + lane < n_lists ? real_key(c[u]) : 0ull;
    unsigned long long bound = wave_bound<4>(key, k, kWave, reinterpret_cast<unsigned*>(ms->keys), lane);
    int cnt = 0;
#pragma unroll
    for (int u = 0; u < 4; ++u) {
        const unsigned long long b = __ballot(key[u] >= bound);
        if (key[u] >= bound) {
            const int at = cnt + __popcll(b & ((1ull << lane) - 1ull));
            if (at < kWave) {
                ms->keys[at] = key[u];
                ms->tags[at] = u * kWave + lane;
            }
        }
        cnt += __popcll(b);
    }
    cnt = cnt < kWave ? cnt : kWave;
    bool active = lane < cnt;
    const int tag = cnt > 0 ? ms->tags[active ? lane : 0] : 0;
    auto load_kept = [&]() {
#pragma unroll
        for (int u = 0; u < 4; ++u) key[u] = u * kWave + lane < cnt ? ms->keys[u * kWave + lane] : 0ull;
    };
    for (int d = 1; d < k; d += kDeep) {                       // wave-uniform
#pragma unroll
        for (int u = 0; u < kDeep; ++u) c[u] = get(tag, d + u < k ? d + u : k - 1);
        if (cnt > kWave) {                                     // (the loads above are in flight)
            load_kept();
            bound = wave_bound<4>(key, k, kWave, reinterpret_cast<unsigned*>(ms->keys), lane);
            cnt = 0;
#pragma unroll
            for (int u = 0; u < 4; ++u) cnt = wave_append(ms->keys, cnt, kWave, key[u], bound, lane);
        }
#pragma unroll
        for (int u = 0; u < kDeep; ++u) {
            const unsigned long long q = active && d + u < k ? real_key(c[u]) : 0ull;
            cnt = wave_append(ms->keys, cnt, kMergeKeys, q, bound, lane);
            if (u == kDeep - 1) active = q >= bound;
        }
        if (__ballot(active) == 0ull) break;
    }
    if (cnt <= kWave) {                                        // wave-uniform
        const unsigned long long one[1] = {lane < cnt ? ms->keys[lane] : 0ull};
        wave_topk<1>(one, k, lane, ms->keys, put);
        return;
    }
    load_kept();
    wave_topk<4>(key, k, lane, ms->keys, put);
}

}  // namespace
