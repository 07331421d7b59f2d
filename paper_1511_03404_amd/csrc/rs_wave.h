// LDS radix sort of up to 1024 elements by one wave: the one-workgroup sort
// (rs_block.h) with a single wave, so that no step needs a barrier.  Used for
// the tiny segments of a segmented sort that are too long for the bitonic
// network to win (rs_bitonic.h), and for runs that a sweep could not order
// (rs_finish.h).
#pragma once

#include <cstddef>

#include "rs_device.h"
#include "rs_runs.h"

namespace rs {

constexpr uint32_t kWaveSortMax = 1024;

// LDS of one wave that sorts up to MAX elements: the digit counters and the
// staged elements, with run_move's neighbours on either side of the keys.  The
// lane-mask table shares the keys' memory; positions need 16 bits.
template <typename K, bool HAS_V, uint32_t MAX = kWaveSortMax>
struct WaveLds {
    static_assert(MAX >= kRadix * 8 / sizeof(K) && MAX <= 1u << 16,
                  "the lane-mask table lives in the staged keys");
    uint32_t wc[kRadix];
    uint16_t pos[HAS_V ? MAX : 2];
    __attribute__((aligned(16))) K before[kRunMax];
    K key[MAX];
    K behind[kRunMax];
};

// One stable counting sort by the 8-bit digit at bit `shift`: item j of lane
// l is element j*64 + l, before and after.  Only elements below m take part.
template <typename K, bool HAS_V, int R, uint32_t MAX>
__device__ __forceinline__ void wave_sort_digit(WaveLds<K, HAS_V, MAX> &L, K (&key)[R],
                                                uint32_t (&pos)[HAS_V ? R : 1], uint32_t m,
                                                uint32_t lane, int shift)
{
    uint64_t *wm = (uint64_t *)L.key;
    wave_lds_fence();
    ((uint4 *)L.wc)[lane] = make_uint4(0, 0, 0, 0);
    ((uint4 *)wm)[lane] = make_uint4(0, 0, 0, 0);
    ((uint4 *)wm)[kWave + lane] = make_uint4(0, 0, 0, 0);
    wave_lds_fence();
    uint32_t rank[R];
    uint32_t *wm32 = (uint32_t *)wm + (lane >> 5);
#pragma unroll
    for (int j = 0; j < R; ++j) {
        if ((uint32_t)j * kWave < m) {
            // a lane past m sets no bit and takes a slot of its own
            const bool has = j * kWave + lane < m;
            const uint32_t d = has ? digit_at<kRadixBits>(key[j], shift) : lane;
            atomicOr(&wm32[2 * d], has ? 1u << (lane & 31) : 0u);
            const uint64_t peers = wm[d];
            const uint32_t c = L.wc[d];
            const uint32_t below = lanes_below(peers);
            rank[j] = c + below;
            if (has && below == 0) {
                L.wc[d] = c + (uint32_t)__popcll(peers);
                wm[d] = 0;
            }
        }
    }
    wave_lds_fence();
    // exclusive offsets, four digits per lane
    uint4 c = ((uint4 *)L.wc)[lane];
    const uint32_t sum = c.x + c.y + c.z + c.w;
    const uint32_t base = wave_inclusive_scan(sum) - sum;
    ((uint4 *)L.wc)[lane] =
        make_uint4(base, base + c.x, base + c.x + c.y, base + c.x + c.y + c.z);
    wave_lds_fence();
#pragma unroll
    for (int j = 0; j < R; ++j) {
        if (j * kWave + lane < m) {
            const uint32_t p = rank[j] + L.wc[digit_at<kRadixBits>(key[j], shift)];
            L.key[p] = key[j];
            if constexpr (HAS_V)
                L.pos[p] = (uint16_t)pos[j];
        }
    }
    wave_lds_fence();
#pragma unroll
    for (int j = 0; j < R; ++j) {
        if ((uint32_t)j * kWave < m) {
            key[j] = L.key[j * kWave + lane];
            if constexpr (HAS_V)
                pos[j] = L.pos[j * kWave + lane];
        }
    }
}

// Sorts a wave's m elements (m >= 1); to[j] is where item j then belongs.
// As block_sort: two passes from the highest differing bit, then the runs.
template <typename K, bool HAS_V, int R, uint32_t MAX>
__device__ __forceinline__ void wave_sort(WaveLds<K, HAS_V, MAX> &L, K (&key)[R],
                                          uint32_t (&pos)[HAS_V ? R : 1], uint32_t m,
                                          uint32_t lane, uint32_t (&to)[R])
{
#pragma unroll
    for (int j = 0; j < R; ++j)
        to[j] = j * kWave + lane;
    K d = 0;
    const K first = read_lane(key[0], 0);
#pragma unroll
    for (int j = 0; j < R; ++j)
        d |= j * kWave + lane < m ? key[j] ^ first : (K)0;
    const uint32_t lo = read_lane(wave_or((uint32_t)d), kWave - 1);
    const uint32_t hi =
        sizeof(K) == 8 ? read_lane(wave_or((uint32_t)((uint64_t)d >> 32)), kWave - 1) : 0u;
    const uint64_t diff = ((uint64_t)hi << 32) | lo;
    if (diff == 0)
        return;
    const int top = (kWave - 1) - __builtin_clzll(diff);
    const int shift = max(0, top - (2 * kRadixBits - 1));
    wave_sort_digit<K, HAS_V, R, MAX>(L, key, pos, m, lane, shift);
    if (top >= kRadixBits)
        wave_sort_digit<K, HAS_V, R, MAX>(L, key, pos, m, lane, shift + kRadixBits);
    if (shift == 0 || (diff & (((uint64_t)1 << shift) - 1)) == 0)
        return;
    const K low_ones = ((K)1 << shift) - 1;
    const K *s_run = L.before + kRunMax;
    using Lds = WaveLds<K, HAS_V, MAX>;
    static_assert(R * kWave <= (int)MAX, "the wave's elements are staged");
    static_assert(offsetof(Lds, key) == offsetof(Lds, before) + kRunMax * sizeof(K),
                  "the neighbours lie right before the keys");
    static_assert(offsetof(Lds, behind) == offsetof(Lds, key) + MAX * sizeof(K),
                  "and right behind them");
    uint64_t head[R];
    bool inv = false;
#pragma unroll
    for (int j = 0; j < R; ++j) {
        const uint32_t e = j * kWave + lane;
        const bool has = e < m;
        const K prev = s_run[(int32_t)(has ? e : 0u) - 1];
        head[j] = __ballot(e == 0 || !has || (key[j] ^ prev) > low_ones);
        inv = inv || (has && e > 0 && key[j] < prev);
    }
    if (__ballot(inv) == 0)
        return;
    wave_lds_fence();
    L.before[lane] = 0;
    L.key[m + lane] = KeyTraits<K>::kPad;  // into `behind` when m is close to the maximum
    wave_lds_fence();
    bool lost = false;
#pragma unroll
    for (int j = 0; j < R; ++j) {
        if ((uint32_t)j * kWave < m) {
            const uint32_t e = min((uint32_t)(j * kWave + lane), m - 1);
            bool whole;
            const int32_t move =
                run_move(s_run, e, key[j], lane, head[j], j ? head[j ? j - 1 : 0] : ~0ull,
                         j + 1 < R ? head[j + 1 < R ? j + 1 : j] : ~0ull, &whole);
            if (j * kWave + lane < m) {
                to[j] += (uint32_t)move;
                lost = lost ||
                       (!whole && key[j] > s_run[e + 1] && (key[j] ^ s_run[e + 1]) <= low_ones);
            }
        }
    }
    if (__ballot(lost) == 0)
        return;
    // long runs out of order: every digit that differs
    for (int p = 0; p < num_passes<K, kRadixBits>(); ++p)
        if ((diff >> (p * kRadixBits)) & (kRadix - 1))
            wave_sort_digit<K, HAS_V, R, MAX>(L, key, pos, m, lane, p * kRadixBits);
#pragma unroll
    for (int j = 0; j < R; ++j)
        to[j] = j * kWave + lane;
}

// Where a wave's elements come from and go to (the same place: in place).
template <typename K, typename V>
struct WaveData {
    const K *kin;
    const V *vin;
    K *kout;
    V *vout;
};

// Sorts m elements, 1 <= m <= 64 R, in R slots of 64; kmap is applied to the keys
// on load and undone on store.
template <typename K, typename V, bool HAS_V, int R, uint32_t MAX>
__device__ __forceinline__ void radix_wave(WaveLds<K, HAS_V, MAX> &L, const WaveData<K, V> &d,
                                           uint32_t m, uint32_t lane, uint32_t kmap)
{
    K key[R];
    uint32_t pos[HAS_V ? R : 1], to[R];
#pragma unroll
    for (int j = 0; j < R; ++j) {
        const uint32_t e = j * kWave + lane;
        key[j] = e < m ? d.kin[e] : (K)0;
        if constexpr (HAS_V)
            pos[j] = e;
    }
    if (kmap) {
#pragma unroll
        for (int j = 0; j < R; ++j)
            key[j] = map_in(key[j], kmap);
    }
    wave_sort<K, HAS_V, R, MAX>(L, key, pos, m, lane, to);
    // every value is read before any is written (in place: vin == vout)
    V val[HAS_V ? R : 1];
    if constexpr (HAS_V) {
#pragma unroll
        for (int j = 0; j < R; ++j)
            val[j] = j * kWave + lane < m ? d.vin[pos[j]] : (V)0;
    }
#pragma unroll
    for (int j = 0; j < R; ++j) {
        if (j * kWave + lane < m) {
            d.kout[to[j]] = map_out(key[j], kmap);
            if constexpr (HAS_V)
                d.vout[to[j]] = val[j];
        }
    }
}

}  // namespace rs
