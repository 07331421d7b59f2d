// Ordering the short runs of an array that is stably sorted by its high bits:
// the elements of a run share those bits, and each moves by the number of
// the run's elements that belong on its other side.
#pragma once

#include "rs_device.h"

namespace rs {

// Longest run ordered by counting: with one 64-element chunk on either side
// of its own, every element of such a run sees the whole run.
constexpr uint32_t kRunMax = kWave;
// Distances compared per round.
constexpr int kRunStep = 4;  // (the compares below are written out)
static_assert(kRunMax % kRunStep == 0, "the last round stays within kRunMax elements");

// n += how many of a[0..3] are less (greater) than b, as four compares and
// four adds with carry: written out because the compiler turns the sum of
// compares into selects, shifts and a bit count, twice the instructions
// (2^20 32-bit keys, runs of 16: 12.0 us a sweep, 10.3 us so).  The
// compares come first: a mask is read at least three instructions after it
// is written.
__device__ __forceinline__ void count_less(uint32_t &n, const uint32_t (&a)[kRunStep], uint32_t b)
{
    uint64_t m0, m1, m2, m3;
    asm("v_cmp_lt_u32_e64 %1, %5, %9\n\t"
        "v_cmp_lt_u32_e64 %2, %6, %9\n\t"
        "v_cmp_lt_u32_e64 %3, %7, %9\n\t"
        "v_cmp_lt_u32_e64 %4, %8, %9\n\t"
        "v_addc_co_u32_e64 %0, %1, 0, %0, %1\n\t"
        "v_addc_co_u32_e64 %0, %2, 0, %0, %2\n\t"
        "v_addc_co_u32_e64 %0, %3, 0, %0, %3\n\t"
        "v_addc_co_u32_e64 %0, %4, 0, %0, %4"
        : "+v"(n), "=&s"(m0), "=&s"(m1), "=&s"(m2), "=&s"(m3)
        : "v"(a[0]), "v"(a[1]), "v"(a[2]), "v"(a[3]), "v"(b));
}

__device__ __forceinline__ void count_less(uint32_t &n, const uint64_t (&a)[kRunStep], uint64_t b)
{
    uint64_t m0, m1, m2, m3;
    asm("v_cmp_lt_u64_e64 %1, %5, %9\n\t"
        "v_cmp_lt_u64_e64 %2, %6, %9\n\t"
        "v_cmp_lt_u64_e64 %3, %7, %9\n\t"
        "v_cmp_lt_u64_e64 %4, %8, %9\n\t"
        "v_addc_co_u32_e64 %0, %1, 0, %0, %1\n\t"
        "v_addc_co_u32_e64 %0, %2, 0, %0, %2\n\t"
        "v_addc_co_u32_e64 %0, %3, 0, %0, %3\n\t"
        "v_addc_co_u32_e64 %0, %4, 0, %0, %4"
        : "+v"(n), "=&s"(m0), "=&s"(m1), "=&s"(m2), "=&s"(m3)
        : "v"(a[0]), "v"(a[1]), "v"(a[2]), "v"(a[3]), "v"(b));
}

__device__ __forceinline__ void count_greater(uint32_t &n, const uint32_t (&a)[kRunStep],
                                              uint32_t b)
{
    uint64_t m0, m1, m2, m3;
    asm("v_cmp_gt_u32_e64 %1, %5, %9\n\t"
        "v_cmp_gt_u32_e64 %2, %6, %9\n\t"
        "v_cmp_gt_u32_e64 %3, %7, %9\n\t"
        "v_cmp_gt_u32_e64 %4, %8, %9\n\t"
        "v_addc_co_u32_e64 %0, %1, 0, %0, %1\n\t"
        "v_addc_co_u32_e64 %0, %2, 0, %0, %2\n\t"
        "v_addc_co_u32_e64 %0, %3, 0, %0, %3\n\t"
        "v_addc_co_u32_e64 %0, %4, 0, %0, %4"
        : "+v"(n), "=&s"(m0), "=&s"(m1), "=&s"(m2), "=&s"(m3)
        : "v"(a[0]), "v"(a[1]), "v"(a[2]), "v"(a[3]), "v"(b));
}

__device__ __forceinline__ void count_greater(uint32_t &n, const uint64_t (&a)[kRunStep],
                                              uint64_t b)
{
    uint64_t m0, m1, m2, m3;
    asm("v_cmp_gt_u64_e64 %1, %5, %9\n\t"
        "v_cmp_gt_u64_e64 %2, %6, %9\n\t"
        "v_cmp_gt_u64_e64 %3, %7, %9\n\t"
        "v_cmp_gt_u64_e64 %4, %8, %9\n\t"
        "v_addc_co_u32_e64 %0, %1, 0, %0, %1\n\t"
        "v_addc_co_u32_e64 %0, %2, 0, %0, %2\n\t"
        "v_addc_co_u32_e64 %0, %3, 0, %0, %3\n\t"
        "v_addc_co_u32_e64 %0, %4, 0, %0, %4"
        : "+v"(n), "=&s"(m0), "=&s"(m1), "=&s"(m2), "=&s"(m3)
        : "v"(a[0]), "v"(a[1]), "v"(a[2]), "v"(a[3]), "v"(b));
}

// How far an element moves.  The wave holds a chunk, one element per lane:
// `key` is element `at` of s_k, which holds the chunk's keys and kRunMax
// elements on either side.  here, prev and next are the chunks' head words (a
// bit for every element that starts a run; uniform); whole: whether this
// element's run has at most kRunMax elements (0 is returned if not).
//
// An element moves left by the number of larger keys among the D before it
// and right by the number of smaller keys among the D after it, where D is
// the longest run that touches the chunk, less one.  Neighbours in other
// runs need no test: the array is sorted by the high bits, so those before
// are smaller and those after larger.  Equal keys never pass each other, so
// the order is stable.  Per distance that is two LDS reads at consecutive
// addresses, two compares and two adds with carry, and no address depends on
// data, so the reads of several distances are in flight together.
template <typename K>
__device__ __forceinline__ int32_t run_move(const K *s_k, uint32_t at, K key, uint32_t lane,
                                            uint64_t here, uint64_t prev, uint64_t next,
                                            bool *whole)
{
    // the longest run that touches this chunk: clear bits in a row, across
    // either of its ends (counted here) or inside it (`clear` keeps a bit
    // while d of them are in a row below it)
    const uint32_t into = here ? __builtin_ctzll(here) : kWave;
    const uint32_t outof = here ? __builtin_clzll(here) : kWave;
    const uint32_t left = into + (prev ? __builtin_clzll(prev) : kWave);
    const uint32_t right = outof + (next ? __builtin_ctzll(next) : kWave);
    uint32_t dist = max(left, right);
    uint64_t clear = ~here;
    const uint64_t two = clear & (clear << 1), four = two & (two << 2);
    *whole = true;
    if (dist >= kRunMax) {
        // this element's distance from its run's first and last element
        // (kWave or more where no head is in sight)
        const uint64_t upto = here << (kWave - 1 - lane);
        const uint64_t after = lane < kWave - 1 ? here >> (lane + 1) : 0ull;
        const uint32_t back = upto   ? __builtin_clzll(upto)
                              : prev ? lane + 1 + __builtin_clzll(prev)
                                     : 2 * kWave;
        const uint32_t ahead = after  ? __builtin_ctzll(after)
                               : next ? kWave - 1 - lane + __builtin_ctzll(next)
                                      : 2 * kWave;
        *whole = back + ahead < kRunMax;
        // the longest run ordered here: the others need no distance
        dist = __builtin_amdgcn_readlane(wave_max(*whole ? back + ahead : 0u), kWave - 1);
        clear = 0;
    }
    uint32_t up = 0, down = 0;
    for (uint32_t d = 1; d <= dist || clear != 0; d += kRunStep) {
        K l[kRunStep], r[kRunStep];
#pragma unroll
        for (int i = 0; i < kRunStep; ++i) {
            l[i] = s_k[at - d - i];
            r[i] = s_k[at + d + i];
        }
        count_greater(down, l, key);
        count_less(up, r, key);
        clear &= four << d;
    }
    return *whole ? (int32_t)(up - down) : 0;
}

// A word that is the same in every lane, moved to scalar registers.
__device__ __forceinline__ uint64_t uniform_word(uint64_t x)
{
    const uint32_t hi = __builtin_amdgcn_readfirstlane((uint32_t)(x >> 32));
    const uint32_t lo = __builtin_amdgcn_readfirstlane((uint32_t)x);
    return ((uint64_t)hi << 32) | lo;
}

}  // namespace rs
