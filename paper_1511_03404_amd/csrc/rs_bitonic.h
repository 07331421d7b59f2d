// The tiny segments of a segmented sort, one wave per segment of up to 1024
// elements: up to 64 by a bitonic sorting network in registers (paper,
// Section 2.1; Batcher), more by the wave's LDS radix sort (rs_wave.h).
//
// Stage k = 2, 4, ..., 64 of the network builds sorted runs of length k; its
// steps of distance s = k/2, ..., 1 compare element e (in lane e) with e XOR s
// by a cross-lane shuffle and order each pair ascending when bit k of e is
// clear, descending when it is set.
//
// The network alone is not stable; every element is the pair (key, position
// in the segment), compared lexicographically, so all elements differ and
// the sorted order is the stable sort.  Values do not travel through the
// network: each output gathers its value by the position it carries.  Lanes
// past the segment hold a padding element greater than every real one.
//
// The network's steps grow with the square of log2 of the size; from 65
// elements on, two digit passes and a count over short runs take fewer
// (50,000 segments of 2 to 1024 pairs, whole batch: 32-bit 209 us with the
// network up to 64, 218 up to 128, 311 at all sizes; 64-bit 223 and 421 at all
// sizes).
#pragma once

#include "rs_block.h"
#include "rs_device.h"
#include "rs_wave.h"

namespace rs {

// Largest tiny segment.
constexpr uint32_t kTinyMax = kWaveSortMax;

// (key, position) as one comparable word: 32-bit keys pack into a 64-bit
// integer; 64-bit keys keep the position beside the key.
template <typename K>
struct BitonicElem;

template <>
struct BitonicElem<uint32_t> {
    using T = uint64_t;
    static __device__ __forceinline__ T make(uint32_t k, uint32_t pos)
    {
        return ((uint64_t)k << 32) | pos;
    }
    static __device__ __forceinline__ T pad() { return ~0ull; }
    static __device__ __forceinline__ uint32_t key(T e) { return (uint32_t)(e >> 32); }
    static __device__ __forceinline__ uint32_t pos(T e) { return (uint32_t)e; }
    static __device__ __forceinline__ bool less(T a, T b) { return a < b; }
    static __device__ __forceinline__ T sel(bool c, T a, T b) { return c ? a : b; }
    static __device__ __forceinline__ T shfl_xor(T e, uint32_t s)
    {
        return __shfl_xor((unsigned long long)e, (int)s);
    }
};

template <>
struct BitonicElem<uint64_t> {
    struct T {
        uint64_t k;
        uint32_t p;
    };
    static __device__ __forceinline__ T make(uint64_t k, uint32_t pos) { return T{k, pos}; }
    static __device__ __forceinline__ T pad() { return T{~0ull, ~0u}; }
    static __device__ __forceinline__ uint64_t key(T e) { return e.k; }
    static __device__ __forceinline__ uint32_t pos(T e) { return e.p; }
    static __device__ __forceinline__ bool less(T a, T b)
    {
        return a.k < b.k || (a.k == b.k && a.p < b.p);
    }
    // field by field: a select of the whole struct would go through memory
    static __device__ __forceinline__ T sel(bool c, T a, T b)
    {
        return T{c ? a.k : b.k, c ? a.p : b.p};
    }
    static __device__ __forceinline__ T shfl_xor(T e, uint32_t s)
    {
        return T{(uint64_t)__shfl_xor((unsigned long long)e.k, (int)s),
                 (uint32_t)__shfl_xor((int)e.p, (int)s)};
    }
};

struct TinyArgs {
    const void *kin;
    const void *vin;
    void *kout;
    void *vout;
    const SegRange *list;     // the tiny segments (2 .. kTinyMax elements)
    const uint32_t *list_len; // their number (a device counter)
    uint32_t *claim;          // claim counter, zero at launch
    uint32_t kmap;            // key order: applied on load, undone on store
};

template <typename K, typename V, bool HAS_V>
__device__ __forceinline__ void bitonic_wave(const TinyArgs &a, uint64_t start, uint32_t m,
                                             uint32_t lane)
{
    using E = BitonicElem<K>;
    using T = typename E::T;
    const bool in = lane < m;
    const K raw = in ? ((const K *)a.kin)[start + lane] : (K)0;
    T x = E::sel(in, E::make(map_in(raw, a.kmap), lane), E::pad());
    for (uint32_t k = 2; k <= (uint32_t)kWave; k <<= 1) {
        const bool up = (lane & k) == 0;
        for (uint32_t s = k >> 1; s >= 1; s >>= 1) {
            const bool lower = (lane & s) == 0;
            const T y = E::shfl_xor(x, s);
            // the lower element of an ascending pair keeps the smaller
            const bool take_y = (lower == up) == E::less(y, x);
            x = E::sel(take_y, y, x);
        }
    }
    // every value is read before any is written (in place: vin == vout)
    V val = 0;
    if constexpr (HAS_V)
        val = in ? ((const V *)a.vin)[start + E::pos(x)] : (V)0;
    if (in) {
        ((K *)a.kout)[start + lane] = map_out((K)E::key(x), a.kmap);
        if constexpr (HAS_V)
            ((V *)a.vout)[start + lane] = val;
    }
}

// Persistent workgroups of 4 waves; each wave takes one tiny segment at a
// time until the list is exhausted.
template <typename K, typename V, bool HAS_V>
__global__ __launch_bounds__(256) void k_seg_bitonic(TinyArgs a)
{
    __shared__ WaveLds<K, HAS_V> s_lds[4];
    WaveLds<K, HAS_V> &L = s_lds[threadIdx.x / kWave];
    const uint32_t lane = threadIdx.x & (kWave - 1);
    const uint32_t len = *a.list_len;
    ListTurn turn(len, gridDim.x * (blockDim.x / kWave),
                  blockIdx.x * (blockDim.x / kWave) + threadIdx.x / kWave);
    while (true) {
        uint32_t item;
        if (turn.own()) {
            item = turn.take();
        } else {
            uint32_t c = 0;
            if (lane == 0)
                c = atomicAdd(a.claim, 1u);
            item = turn.fixed + __builtin_amdgcn_readfirstlane(c);
        }
        if (item >= len)
            break;
        const uint64_t start = a.list[item].start;
        const uint32_t m = a.list[item].size;
        const WaveData<K, V> in{(const K *)a.kin + start, (const V *)a.vin + (HAS_V ? start : 0),
                                (K *)a.kout + start, (V *)a.vout + (HAS_V ? start : 0)};
        if (m <= (uint32_t)kWave)
            bitonic_wave<K, V, HAS_V>(a, start, m, lane);
        else if (m <= 256)
            radix_wave<K, V, HAS_V, 4>(L, in, m, lane, a.kmap);
        else if (m <= 512)
            radix_wave<K, V, HAS_V, 8>(L, in, m, lane, a.kmap);
        else
            radix_wave<K, V, HAS_V, 16>(L, in, m, lane, a.kmap);
    }
}

}  // namespace rs
