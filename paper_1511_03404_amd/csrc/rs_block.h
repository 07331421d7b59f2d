// LDS-resident radix sort of up to CAP = THREADS x ITEMS elements by one
// workgroup: the same stable counting sort per 8-bit digit as the digit-pass
// kernel (paper, Section 2.6), with every pass between registers and LDS and
// only one read and one write of HBM.  Used for a whole sort when n <= CAP
// (one launch) and for the small and medium segments of a segmented sort.
#pragma once

#include <cstddef>

#include "rs_device.h"
#include "rs_runs.h"

namespace rs {

// Block-sort shapes of the segmented sort: kSmall for up to 4096 elements
// (several workgroups per CU), kMedium for up to 16384 (8192 for 64-bit pairs,
// whose staging would not fit otherwise).  A whole sort has one workgroup, so
// its time is a chain of latencies, above all the items that a wave ranks
// one after another: as many threads and as few items as hold it.  Whole
// sorts of uniform keys, one shape for all sizes and a pass for every digit
// -> now, device time: 1000 32-bit keys 22 -> 9.5 us, 12000 32-bit pairs 50 ->
// 29 us, 16384 64-bit keys 75 -> 37 us.
template <typename K, bool HAS_V>
struct BlockShape {
    static constexpr int kSmallThreads = 256;
    static constexpr int kMediumThreads = (sizeof(K) == 8 && HAS_V) ? 512 : 1024;
    static constexpr int kItems = 16;
    static constexpr int kSmallCap = kSmallThreads * kItems;
    static constexpr int kMediumCap = kMediumThreads * kItems;
};

// A run of elements to sort on its own.
struct SegRange {
    uint64_t start;       // first element
    uint32_t size;        // elements
    uint32_t tile_start;  // first tile in a batched tile sequence (large segments)
};

// How workers share a list of `len` segments of uneven size: most of it in
// turn, worker w taking entries w, w + workers, ..., and the last eighth by
// claims from one counter, which evens the workers out.  A claim by every
// entry was what bound the tiny segments: atomics on one address end one
// after another, 14 ns apart (50,000 segments, 8.2M elements: 580 us with a
// bitonic network or a radix sort alike, 176 us with most taken in turn).
struct ListTurn {
    uint32_t workers;
    uint32_t fixed;  // entries taken in turn: whole rounds, at least one
    uint32_t at;     // this worker's next one
    __device__ __forceinline__ ListTurn(uint32_t len, uint32_t workers_, uint32_t worker)
        : workers(workers_), fixed(max(1u, (len - len / 8) / workers_) * workers_), at(worker)
    {
    }
    __device__ __forceinline__ bool own() const { return at < fixed; }
    __device__ __forceinline__ uint32_t take()
    {
        const uint32_t item = at;
        at += workers;
        return item;
    }
};

struct BlockArgs {
    const void *kin;
    const void *vin;
    void *kout;
    void *vout;
    // segmented use: the workgroups claim entries of list (list_len of them,
    // a device count) through *claim.  Single sort: list == nullptr, one
    // range [0, n).
    const SegRange *list;
    const uint32_t *list_len;
    uint32_t *claim;
    uint64_t n;
    uint32_t kmap;  // key order (kMap*): applied on load, undone on store
    // single sort with a caller's workspace: its error word, cleared here so
    // that a status query after this sort does not report an older one
    uint32_t *err_clear;
};

// LDS of a block sort of THREADS x ITEMS elements.
template <typename K, bool HAS_V, int THREADS, int ITEMS>
struct BlockLds {
    static constexpr int W = THREADS / kWave;
    static constexpr size_t kStageBytes = (size_t)THREADS * ITEMS * sizeof(K) * (HAS_V ? 2 : 1);
    // the lane-mask tables live in the staging buffer, which a tile of few
    // elements makes larger than its elements need
    static constexpr size_t kMaskBytes = (size_t)W * kRadix * 8;
    uint32_t wcnt[W * kRadix];
    uint32_t tmp[8];
    uint64_t head[2 * W];  // head words of each wave's first and last chunk
    uint32_t out[W];       // bit j: an element of the wave's chunk j is out of order
    uint64_t diff;         // bits in which the keys differ
    __attribute__((aligned(16))) K before[kRunMax];  // run_move's neighbours of the first keys
    __attribute__((aligned(16))) unsigned char
        stage[(kStageBytes > kMaskBytes ? kStageBytes : kMaskBytes) + kRunMax * sizeof(K)];
};

// How a workgroup holds m elements in registers: item j of lane l of wave w is
// element (w * used + j) * 64 + l, j < used = ceil(m / THREADS) rounded up to
// whole groups of kGroup, so that all waves have about the same number of
// items.  Groups past `used` are skipped (a scalar branch); within a group
// the lanes past m take part without effect, so that its items overlap.
template <int THREADS, int ITEMS>
struct BlockItems {
    static constexpr int kGroup = ITEMS < 4 ? ITEMS : 4;
    uint32_t m;
    uint32_t used;
    uint32_t base;  // this lane's element of item 0
    __device__ __forceinline__ explicit BlockItems(uint32_t m_)
        : m(__builtin_amdgcn_readfirstlane(m_)),
          used((m + THREADS * kGroup - 1) / (THREADS * kGroup) * kGroup),
          base(__builtin_amdgcn_readfirstlane(threadIdx.x / kWave) * used * kWave +
               threadIdx.x % kWave)
    {
    }
    // element of item j; has: there is one (for j < used)
    __device__ __forceinline__ uint32_t at(int j) const { return base + j * kWave; }
    __device__ __forceinline__ bool has(int j) const { return at(j) < m; }
    template <typename F>
    __device__ __forceinline__ void each(F &&f) const
    {
#pragma unroll
        for (int g = 0; g < ITEMS; g += kGroup) {
            if ((uint32_t)g < used) {
#pragma unroll
                for (int i = 0; i < kGroup; ++i)
                    f(g + i);
            }
        }
    }
};

// One stable counting sort of the workgroup's elements by the 8-bit digit at
// bit `shift`.  The sorted keys are also left in L.stage.
template <typename K, typename V, bool HAS_V, int THREADS, int ITEMS>
__device__ __forceinline__ void block_sort_digit(BlockLds<K, HAS_V, THREADS, ITEMS> &L,
                                                 const BlockItems<THREADS, ITEMS> &it,
                                                 K (&key)[ITEMS], V (&val)[HAS_V ? ITEMS : 1],
                                                 int shift)
{
    constexpr int CAP = THREADS * ITEMS;
    constexpr int W = THREADS / kWave;
    K *s_k = (K *)L.stage;
    // behind the keys, or in the place of run_move's guard there: the values
    // are dead when the guard is written
    V *s_v = (V *)(L.stage + (size_t)CAP * sizeof(K));
    uint64_t *s_mask = (uint64_t *)L.stage;
    const uint32_t t = threadIdx.x;
    const uint32_t w = t / kWave;
    const uint32_t lane = t % kWave;
    uint32_t *wc = L.wcnt + w * kRadix;
    uint64_t *wm = s_mask + w * kRadix;
    // a wave's counters and lane-mask table are its own: it clears them itself
    for (uint32_t i = lane; i < (uint32_t)kRadix; i += kWave) {
        wc[i] = 0;
        wm[i] = 0;
    }
    // stable ranks within the wave, as in wave_rank; a lane past m sets no
    // bit and takes a slot of its own, so that those lanes do not meet
    uint32_t rank[ITEMS];
    uint32_t *wm32 = (uint32_t *)wm + (lane >> 5);
    it.each([&](int j) {
        const bool has = it.has(j);
        const uint32_t d = has ? digit_at<kRadixBits>(key[j], shift) : lane;
        atomicOr(&wm32[2 * d], has ? 1u << (lane & 31) : 0u);
        const uint64_t peers = wm[d];
        const uint32_t c = wc[d];
        const uint32_t below = lanes_below(peers);
        rank[j] = c + below;
        if (has && below == 0) {
            wc[d] = c + (uint32_t)__popcll(peers);
            wm[d] = 0;
        }
    });
    __syncthreads();
    // exclusive offsets over (digit, wave): digit-major, so that earlier
    // waves (earlier elements) come first within a digit
    uint32_t cnt = 0;
    if (t < kRadix) {
#pragma unroll
        for (int ww = 0; ww < W; ++ww) {
            const uint32_t c = L.wcnt[ww * kRadix + t];
            L.wcnt[ww * kRadix + t] = cnt;
            cnt += c;
        }
    }
    const uint32_t excl = bins_exclusive_scan<kRadix>(cnt, L.tmp);
    if (t < kRadix) {
#pragma unroll
        for (int ww = 0; ww < W; ++ww)
            L.wcnt[ww * kRadix + t] += excl;
    }
    __syncthreads();
    it.each([&](int j) {
        if (it.has(j)) {
            const uint32_t pos = rank[j] + wc[digit_at<kRadixBits>(key[j], shift)];
            s_k[pos] = key[j];
            if constexpr (HAS_V)
                s_v[pos] = val[j];
        }
    });
    __syncthreads();
    // lanes past m read their stale slots: in range, and never used
    it.each([&](int j) {
        const uint32_t at = min(it.at(j), (uint32_t)CAP - 1);
        key[j] = s_k[at];
        if constexpr (HAS_V)
            val[j] = s_v[at];
    });
    __syncthreads();
}

// The counting sorts of the 8-bit digit positions in `digits` (bit p:
// position p), lowest first.
template <typename K, typename V, bool HAS_V, int THREADS, int ITEMS>
__device__ __forceinline__ void block_sort_digits(BlockLds<K, HAS_V, THREADS, ITEMS> &L,
                                                  const BlockItems<THREADS, ITEMS> &it,
                                                  K (&key)[ITEMS], V (&val)[HAS_V ? ITEMS : 1],
                                                  uint32_t digits)
{
    for (; digits; digits &= digits - 1)
        block_sort_digit<K, V, HAS_V, THREADS, ITEMS>(L, it, key, val,
                                                      __builtin_ctz(digits) * kRadixBits);
}

// Orders the run [start, start + len) of the staged keys, sorted by their high bits
// and out of order below: by one wave, one distinct key after another, each found
// and counted in a scan over the run.  Keys alone are written to kout; with
// values, where each element belongs to s_place.  False, with nothing written to
// kout, if the run has too many distinct keys for that.
constexpr uint32_t kPeelKeys = kWave;    // distinct keys, one a lane
constexpr uint32_t kPeelChunks = 512;    // chunks of 64 read in all
template <typename K, bool HAS_V>
__device__ __forceinline__ bool peel_run(const K *s_k, uint16_t *s_place, K *kout, uint32_t kmap,
                                         uint32_t start, uint32_t len)
{
    const uint32_t lane = threadIdx.x % kWave;
    const uint32_t chunks = (len + kWave - 1) / kWave;
    const auto least = [](K x) {
        for (int s = 1; s < kWave; s *= 2) {
            const K y = sizeof(K) == 8 ? (K)__shfl_xor((unsigned long long)x, s)
                                       : (K)__shfl_xor((unsigned int)x, s);
            x = y < x ? y : x;
        }
        return x;
    };
    K next = KeyTraits<K>::kPad;
    for (uint32_t e = lane; e < len; e += kWave)
        next = min(next, s_k[start + e]);
    K own = 0;             // this lane's distinct key, and how many go before it
    uint32_t own_from = 0;
    uint32_t keys = 0, out = 0, read = chunks;
    while (out < len) {
        read += chunks;
        if (keys == kPeelKeys || read > kPeelChunks)
            return false;
        const K key = least(next);
        if (lane == keys) {
            own = key;
            own_from = out;
        }
        ++keys;
        next = KeyTraits<K>::kPad;
        for (uint32_t c = 0; c < len; c += kWave) {
            const bool in = c + lane < len;
            const K x = s_k[start + min(c + lane, len - 1)];
            const uint64_t same = __ballot(in && x == key);
            if constexpr (HAS_V) {
                if (in && x == key)
                    s_place[start + c + lane] = (uint16_t)(start + out + lanes_below(same));
            }
            out += (uint32_t)__popcll(same);
            next = x > key && x < next ? x : next;
        }
    }
    if constexpr (!HAS_V) {
        for (uint32_t i = 0; i < keys; ++i) {
            const K key = read_lane(own, i);
            const uint32_t end = i + 1 < keys ? read_lane(own_from, i + 1) : len;
            for (uint32_t e = read_lane(own_from, i) + lane; e < end; e += kWave)
                kout[start + e] = map_out(key, kmap);
        }
    }
    return true;
}

// Orders the runs of more than kRunMax elements that are out of order, among m
// staged keys sorted by their bits above low_ones, by every thread of the
// workgroup.  s_word is room for a word a chunk of 64 and a mark; the rest as
// peel_run.
template <typename K, bool HAS_V>
__device__ __forceinline__ bool block_long_runs(const K *s_k, uint64_t *s_word, uint16_t *s_place,
                                                K *kout, uint32_t kmap, uint32_t m, K low_ones)
{
    const uint32_t t = threadIdx.x;
    const uint32_t W = blockDim.x / kWave;
    const uint32_t w = __builtin_amdgcn_readfirstlane(t / kWave);
    const uint32_t lane = t % kWave;
    const uint32_t chunks = (m + kWave - 1) / kWave;
    // every chunk's head word (elements past the last count as heads), and a mark
    // for the chunks where a run to order may start (one at most: it goes on
    // into the next)
    uint64_t *s_head = s_word;
    uint32_t *s_mark = (uint32_t *)(s_word + chunks);
    for (uint32_t i = t; i < (chunks + 31) / 32; i += blockDim.x)
        s_mark[i] = 0;
    for (uint32_t c = w; c < chunks; c += W) {
        const uint32_t at = c * kWave + lane;
        const uint64_t head =
            __ballot(at == 0 || at >= m || (s_k[at] ^ s_k[at - 1]) > low_ones);
        if (lane == 0)
            s_head[c] = head;
    }
    __syncthreads();
    for (uint32_t c = w; c < chunks; c += W) {
        const uint32_t at = c * kWave + lane;
        const uint64_t head = uniform_word(s_head[c]);
        const uint64_t inv = __ballot(at > 0 && at < m && s_k[at] < s_k[at - 1]);
        const uint64_t in = head ? (head & (0 - head)) - 1 : ~0ull;
        const uint64_t last = head ? ~0ull << (kWave - 1 - __builtin_clzll(head)) : 0ull;
        const auto mark = [&](uint32_t chunk) {
            if (lane == 0)
                atomicOr(&s_mark[chunk / 32], 1u << (chunk % 32));
        };
        if (inv & last)
            mark(c);
        if (inv & in) {
            // back to a chunk with a head (the first one has)
            uint32_t back = 1;
            uint64_t found;
            while ((found = __ballot(c < back + lane || s_head[c - back - lane] != 0)) == 0)
                back += kWave;
            mark(c - back - (uint32_t)__builtin_ctzll(found));
        }
    }
    __syncthreads();
    bool all = true;
    for (uint32_t c = w; c < chunks; c += W) {
        if (!(__builtin_amdgcn_readfirstlane(s_mark[c / 32]) >> (c % 32) & 1))
            continue;
        const uint32_t start = c * kWave + kWave - 1 - __builtin_clzll(uniform_word(s_head[c]));
        // ahead to a chunk with a head
        uint32_t ahead = c + 1;
        uint64_t found;
        while ((found = __ballot(ahead + lane >= chunks || s_head[ahead + lane] != 0)) == 0)
            ahead += kWave;
        ahead += (uint32_t)__builtin_ctzll(found);
        const uint32_t end =
            ahead < chunks
                ? ahead * kWave + (uint32_t)__builtin_ctzll(uniform_word(s_head[ahead]))
                : m;
        if (min(end, m) - start > kRunMax)
            all = all && peel_run<K, HAS_V>(s_k, s_place, kout, kmap, start, min(end, m) - start);
    }
    return !__syncthreads_or(!all);
}

// The runs of keys that share their bits from `shift` up, for staged keys that are
// sorted by those: to[j] is where item j then belongs.  False if longer runs are
// out of order: their elements stay where they are.
template <typename K, bool HAS_V, int THREADS, int ITEMS>
__device__ __forceinline__ bool block_sort_runs(BlockLds<K, HAS_V, THREADS, ITEMS> &L,
                                                const BlockItems<THREADS, ITEMS> &it,
                                                const K (&key)[ITEMS], uint32_t (&to)[ITEMS],
                                                int shift)
{
    constexpr int W = THREADS / kWave;
    K *s_k = (K *)L.stage;
    const uint32_t t = threadIdx.x;
    const uint32_t w = __builtin_amdgcn_readfirstlane(t / kWave);
    const uint32_t lane = t % kWave;
    // the runs: head words and neighbours out of order, as in k_finish
    const K low_ones = ((K)1 << shift) - 1;
    uint64_t head[ITEMS];
    uint32_t out = 0;
    K *s_run = L.before + kRunMax;  // the keys, with kRunMax before them
    using Lds = BlockLds<K, HAS_V, THREADS, ITEMS>;
    static_assert(offsetof(Lds, stage) == offsetof(Lds, before) + kRunMax * sizeof(K),
                  "those neighbours lie right before the keys");
    uint64_t last = ~0ull;
#pragma unroll
    for (int j = 0; j < ITEMS; ++j)
        head[j] = ~0ull;
    it.each([&](int j) {
        const uint32_t at = it.at(j);
        const bool has = it.has(j);
        const K prev = s_run[(int32_t)(has ? at : 0u) - 1];
        head[j] = __ballot(at == 0 || !has || (key[j] ^ prev) > low_ones);
        out |= __ballot(has && at > 0 && key[j] < prev) ? 1u << j : 0u;
        last = head[j];
    });
    if (lane == 0) {
        L.head[2 * w] = head[0];
        L.head[2 * w + 1] = last;
        L.out[w] = out;
    }
    if (!__syncthreads_or(out != 0))
        return true;  // every run is in order already
    const uint64_t before = w == 0 ? ~0ull : uniform_word(L.head[2 * w - 1]);
    const uint64_t behind = w == W - 1 ? ~0ull : uniform_word(L.head[2 * w + 2]);
    // chunks next to one with elements out of order: in the others nothing moves
    // (16000 32-bit keys, 32 of each: 54 us with a sweep of them all, 31 so)
    out |= (out << 1) | (out >> 1);
    out |= w == 0 ? 0u : __builtin_amdgcn_readfirstlane(L.out[w - 1]) >> (it.used - 1) & 1;
    out |= w == W - 1 ? 0u : (__builtin_amdgcn_readfirstlane(L.out[w + 1]) & 1) << (it.used - 1);
    // nothing before the first key is larger, nothing after the last smaller
    if (t < kRunMax) {
        L.before[t] = 0;
        s_k[it.m + t] = KeyTraits<K>::kPad;
    }
    __syncthreads();
    bool lost = false;
    it.each([&](int j) {
        // the wave as a whole: run_move takes part with every lane
        if (out >> j & 1 && it.at(j) - lane < it.m) {
            const uint32_t at = min(it.at(j), it.m - 1);
            const uint64_t next = j + 1 < ITEMS && (uint32_t)j + 1 < it.used
                                      ? head[j + 1 < ITEMS ? j + 1 : j]
                                      : behind;
            bool whole;
            const int32_t move = run_move(s_run, at, key[j], lane, head[j],
                                          j ? head[j ? j - 1 : 0] : before, next, &whole);
            if (it.has(j)) {
                to[j] += (uint32_t)move;
                lost = lost || (!whole && key[j] > s_k[at + 1] &&
                                ((key[j] ^ s_k[at + 1]) <= low_ones));
            }
        }
    });
    return !__syncthreads_or(lost);
}

// Sorts the workgroup's elements; to[j] is where item j then belongs.
//
// The keys' highest differing bit is found first, and only the 16 bits from
// there down are sorted by counting sorts, two passes for any key width: up
// to 16384 elements then share those bits with few others, and each such
// run is put in order by counting (run_move), which needs no staging of the
// values.  Where that does not do, block_sort_rest has to follow:
//   * kBlockLost   longer runs are out of order, which comes of repeated keys
//                  (two that share the 16 bits, with 64 elements or more); the
//                  other elements are in place;
//   * kBlockEvery  the keys mostly share those bits (a few large ones set the
//                  highest bit) and nothing has been done.  They are told by
//                  pairs of elements, 64 in each wave: a wave counts the pairs
//                  that differ, but below the 16 bits from its own highest
//                  differing bit, and most waves have to count two or more.
enum BlockResult { kBlockDone, kBlockLost, kBlockEvery };

template <typename K, typename V, bool HAS_V, int THREADS, int ITEMS>
__device__ __forceinline__ BlockResult block_sort(BlockLds<K, HAS_V, THREADS, ITEMS> &L,
                                                  const BlockItems<THREADS, ITEMS> &it,
                                                  K (&key)[ITEMS], V (&val)[HAS_V ? ITEMS : 1],
                                                  uint32_t (&to)[ITEMS])
{
    constexpr int W = THREADS / kWave;
    K *s_k = (K *)L.stage;
    const uint32_t t = threadIdx.x;
    const uint32_t w = __builtin_amdgcn_readfirstlane(t / kWave);
    const uint32_t lane = t % kWave;
#pragma unroll
    for (int j = 0; j < ITEMS; ++j)
        to[j] = it.at(j);
    // the bits in which any key differs from the first one
    if (t == 0) {
        L.diff = 0;
        s_k[0] = key[0];
    }
    __syncthreads();
    const K first = s_k[0];
    {
        K d = 0;
        it.each([&](int j) { d |= it.has(j) ? key[j] ^ first : (K)0; });
        const uint32_t lo = wave_or((uint32_t)d);
        const uint32_t hi = sizeof(K) == 8 ? wave_or((uint32_t)((uint64_t)d >> 32)) : 0u;
        if (lane == kWave - 1 && (lo | hi))
            atomicOr((unsigned long long *)&L.diff, ((uint64_t)hi << 32) | lo);
        // the wave's highest differing bit + 1, and its pairs (elements 64 P apart)
        // that differ below the 16 bits from there down
        constexpr int P = BlockItems<THREADS, ITEMS>::kGroup - 1;
        const uint64_t wave_diff = read_lane(((uint64_t)hi << 32) | lo, kWave - 1);
        const uint32_t bits = wave_diff ? kWave - __builtin_clzll(wave_diff) : 0u;
        const K x = it.has(P) ? key[0] ^ key[P] : (K)0;
        const uint64_t pairs =
            __ballot(x != 0 && bits > 2 * kRadixBits && (x >> (bits - 2 * kRadixBits)) == 0);
        if (lane == 0)
            L.out[w] = bits << 8 | (uint32_t)__popcll(pairs);
    }
    __syncthreads();
    const uint64_t diff = uniform_word(L.diff);
    if (diff == 0)
        return kBlockDone;  // one key only: in place
    const int top = (kWave - 1) - __builtin_clzll(diff);
    const int shift = max(0, top - (2 * kRadixBits - 1));
    // waves whose pairs mostly share the high bits: all of them if the wave's
    // highest differing bit lies below
    const uint32_t seen = lane < (uint32_t)W ? L.out[lane] : 0u;
    const uint64_t alike = __ballot((seen & 255u) > 1 || (seen && (int)(seen >> 8) <= shift));
    const uint32_t waves = (it.m + it.used * kWave - 1) / (it.used * kWave);
    if (2 * (uint32_t)__popcll(alike) > waves)
        return kBlockEvery;
    block_sort_digit<K, V, HAS_V, THREADS, ITEMS>(L, it, key, val, shift);
    if (top >= kRadixBits)
        block_sort_digit<K, V, HAS_V, THREADS, ITEMS>(L, it, key, val, shift + kRadixBits);
    if (shift == 0 || (diff & (((uint64_t)1 << shift) - 1)) == 0)
        return kBlockDone;  // nothing below the sorted bits
    return block_sort_runs<K, HAS_V, THREADS, ITEMS>(L, it, key, to, shift) ? kBlockDone
                                                                            : kBlockLost;
}

// Where a workgroup's elements come from and go to (the same place: in place), and
// the key orders applied on load and undone on store.
template <typename K, typename V>
struct BlockData {
    const K *kin;
    const V *vin;
    K *kout;
    V *vout;
    uint32_t map_load, map_store;
};

template <typename K, typename V, bool HAS_V, int THREADS, int ITEMS>
__device__ __forceinline__ void block_load(const BlockItems<THREADS, ITEMS> &it, const K *kin,
                                           const V *vin, uint32_t kmap, K (&key)[ITEMS],
                                           V (&val)[HAS_V ? ITEMS : 1])
{
    it.each([&](int j) {
        key[j] = it.has(j) ? kin[it.at(j)] : (K)0;
        if constexpr (HAS_V)
            val[j] = it.has(j) ? vin[it.at(j)] : (V)0;
    });
    // mapped once every load is issued (a map between loads would wait
    // for each in turn)
    if (kmap)
        it.each([&](int j) { key[j] = map_in(key[j], kmap); });
}

// What block_sort has left, once its elements are written: the long runs out of
// order, one distinct key after another (two keys in a run, say).  If one has
// too many for that, or nothing has been done, the whole tile is read again
// and sorted by every digit that differs, 64-bit keys by the 32 highest
// differing bits first.
//
// After the elements are written, since nothing is held in registers then: in
// block_sort itself, where the elements are, this made the sorts of 16384
// spill them (64-bit keys 34 -> 49 us).
//
// With every digit sorted from the start, with all of them after the two passes
// whatever the runs, and so: 16000 32-bit keys of 32 copies each 49, 86 and 39 us;
// 16000 keys below 2^15 and one of 2^30 52, 82 and 38.
template <typename K, typename V, bool HAS_V, int THREADS, int ITEMS>
__device__ __forceinline__ void block_sort_rest(BlockLds<K, HAS_V, THREADS, ITEMS> &L, uint32_t m,
                                                const BlockData<K, V> &d, bool every)
{
    constexpr int W = THREADS / kWave;
    const BlockItems<THREADS, ITEMS> it(m);
    const uint64_t diff = uniform_word(L.diff);
    const int top = (kWave - 1) - __builtin_clzll(diff);
    const K *s_k = (const K *)L.stage;
    // the elements have to be there for every thread of the workgroup
    __syncthreads();
    K key[ITEMS];
    V val[HAS_V ? ITEMS : 1];
    if (!every) {
        // the digit counters are free, and the memory of the values, behind the
        // keys and their guard
        static_assert(W * ITEMS * 8 + (W * ITEMS + 31) / 32 * 4 <= sizeof L.wcnt, "words fit");
        uint16_t *s_place =
            (uint16_t *)(L.stage + ((size_t)THREADS * ITEMS + kRunMax) * sizeof(K));
        if constexpr (HAS_V)
            it.each([&](int j) { s_place[it.at(j)] = (uint16_t)it.at(j); });
        const K low_ones = ((K)1 << (top - (2 * kRadixBits - 1))) - 1;
        if (block_long_runs<K, HAS_V>(s_k, (uint64_t *)L.wcnt, s_place, d.kout, d.map_store, m,
                                      low_ones)) {
            if constexpr (HAS_V) {
                it.each([&](int j) {
                    if (it.has(j) && s_place[it.at(j)] != it.at(j))
                        val[j] = d.vout[it.at(j)];
                });
                __syncthreads();  // everything is read before it is overwritten
                it.each([&](int j) {
                    const uint32_t to = s_place[it.at(j)];
                    if (it.has(j) && to != it.at(j)) {
                        d.kout[to] = map_out(s_k[it.at(j)], d.map_store);
                        d.vout[to] = val[j];
                    }
                });
            }
            return;
        }
        __syncthreads();
    }
    block_load<K, V, HAS_V, THREADS, ITEMS>(it, every ? d.kin : d.kout, every ? d.vin : d.vout,
                                            every ? d.map_load : d.map_store, key, val);
    __syncthreads();  // everything is read before it is overwritten
    bool sorted = false;
    if (sizeof(K) == 8 && !every && top >= 4 * kRadixBits) {
        for (int at = top + 1 - 4 * kRadixBits; at <= top; at += kRadixBits)
            block_sort_digit<K, V, HAS_V, THREADS, ITEMS>(L, it, key, val, at);
        bool inv = false;
        it.each([&](int j) {
            const bool has = it.has(j) && it.at(j) > 0;
            inv = inv || (has && key[j] < s_k[has ? it.at(j) - 1 : 0u]);
        });
        sorted = !__syncthreads_or(inv);
    }
    if (!sorted) {
        uint32_t digits = 0;
        for (int p = 0; p < num_passes<K, kRadixBits>(); ++p)
            digits |= ((diff >> (p * kRadixBits)) & (kRadix - 1)) ? 1u << p : 0u;
        block_sort_digits<K, V, HAS_V, THREADS, ITEMS>(L, it, key, val, digits);
    }
    it.each([&](int j) {
        if (it.has(j)) {
            d.kout[it.at(j)] = map_out(key[j], d.map_store);
            if constexpr (HAS_V)
                d.vout[it.at(j)] = val[j];
        }
    });
}

// Sorts m elements of the workgroup, from d's input to its output.
template <typename K, typename V, bool HAS_V, int THREADS, int ITEMS>
__device__ __forceinline__ void block_sort_data(BlockLds<K, HAS_V, THREADS, ITEMS> &L, uint32_t m,
                                                const BlockData<K, V> &d)
{
    const BlockItems<THREADS, ITEMS> it(m);
    K key[ITEMS];
    V val[HAS_V ? ITEMS : 1];
    block_load<K, V, HAS_V, THREADS, ITEMS>(it, d.kin, d.vin, d.map_load, key, val);
    uint32_t to[ITEMS];
    const BlockResult r = block_sort<K, V, HAS_V, THREADS, ITEMS>(L, it, key, val, to);
    if (r != kBlockEvery)
        it.each([&](int j) {
            if (it.has(j)) {
                d.kout[to[j]] = map_out(key[j], d.map_store);
                if constexpr (HAS_V)
                    d.vout[to[j]] = val[j];
            }
        });
    if (__builtin_expect(r != kBlockDone, 0))
        block_sort_rest<K, V, HAS_V, THREADS, ITEMS>(L, m, d, r == kBlockEvery);
}

template <typename K, typename V, bool HAS_V, int THREADS, int ITEMS>
__global__ __launch_bounds__(THREADS) void k_block_sort(BlockArgs a)
{
    __shared__ BlockLds<K, HAS_V, THREADS, ITEMS> L;
    __shared__ uint32_t s_item;
    const uint32_t t = threadIdx.x;
    const K *kin = (const K *)a.kin;
    const V *vin = (const V *)a.vin;
    K *kout = (K *)a.kout;
    V *vout = (V *)a.vout;
    if (a.err_clear && blockIdx.x == 0 && t == 0)
        *a.err_clear = 0;

    const uint32_t len = a.list ? *a.list_len : 1u;
    ListTurn turn(len, gridDim.x, blockIdx.x);
    for (uint32_t iter = 0;; ++iter) {
        if (t == 0)
            s_item = !a.list      ? iter
                     : turn.own() ? turn.take()
                                  : turn.fixed + atomicAdd(a.claim, 1u);
        __syncthreads();
        const uint32_t item = s_item;
        uint64_t start;
        uint32_t m;
        if (a.list) {
            if (item >= len)
                break;
            start = a.list[item].start;
            m = a.list[item].size;
        } else {
            if (item != 0)
                break;
            start = 0;
            m = (uint32_t)a.n;
        }

        const BlockData<K, V> d{kin + start,  HAS_V ? vin + start : nullptr,
                                kout + start, HAS_V ? vout + start : nullptr,
                                a.kmap,       a.kmap};
        block_sort_data<K, V, HAS_V, THREADS, ITEMS>(L, m, d);
        __syncthreads();  // the next range overwrites the LDS
    }
}

}  // namespace rs
