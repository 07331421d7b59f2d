// The end of a plain sort whose passes stopped at a high digit position
// (k_plan): the array is sorted by its bits from `shift` up, stably, and what
// is left is to order each run of keys that share those bits.  With n keys
// and about log2(n) - 5 bits sorted the runs are a few elements long, so two
// or three digit passes and one streaming sweep take the place of four or
// eight passes (paper, Section 2.6: a stable counting sort per digit; here
// the digits below `shift` are sorted by counting smaller keys in the run).
//
//   k_finish   one sweep over the array: every element of a run of up to 64
//              counts the run's elements that go before it and is written to
//              that place; a longer run is copied and, where it is out of
//              order, reported;
//   k_last     the last pass slot.  After a sweep that slot is free, and it
//              does what the sweep could not, normally nothing: the reported
//              runs are sorted by a wave or a workgroup each, longer ones by
//              digit passes over the run alone; if there are too many, the
//              whole array is sorted again by every digit.
#pragma once

#include "rs_kernels.h"
#include "rs_runs.h"
#include "rs_wave.h"

namespace rs {

// What the sweep reports and the follow-up works on, in the look-back words of
// the passes, which are done by then (rest_area).
struct RestArea {
    uint32_t *rows;   // look-back words [row][256] of a sort again
    uint32_t *row_run;  // the longer run of each row
    uint32_t max_rows;
    // where runs are out of order: element, segment; once looked up, a run for
    // a wave: start, length (0: none, or listed elsewhere), segment
    uint4 *list;
    uint32_t cap;
    // longer runs: start, length, segment, and its first row if it is longer
    // than a tile
    uint4 *longer;
    uint32_t max_longer;
    uint32_t *words;  // counters (kRest*), then a bit for every 64 elements: the
                      // run that starts among them has been taken
    uint32_t num_words;  // (zero when the follow-up starts)
};
constexpr int kRestFindClaim = 0;   // entries of list claimed
constexpr int kRestFindDone = 1;    // and looked up;
constexpr int kRestShortClaim = 3;  // and claimed to sort the run for a wave
constexpr int kRestLongerClaim = 4; // longer runs claimed
constexpr int kRestItemClaim = 5;   // (stage, row) items claimed
constexpr int kRestRows = 6;        // rows of the runs longer than a tile
constexpr int kRestStageDone = 8;   // [8, 24): items done per stage
constexpr int kRestTaken = 32;

// Lays the area out over the look-back words of `tiles` tiles, 256 a tile for
// each of four or eight digits.  Four digits' words hold it all: 512 a tile for
// the rows (of runs longer than a tile there are fewer than two for every whole
// tile they cover) and 256 for the places; then, in the last quarter, the
// counters, 12 words a tile for the bits (a tile holds at most 24576 elements),
// 192 for the runs of more than 512 elements and 2 for the rows' map.
//
// In a plain sort the counters and bits are zero already: they lie in the words
// of the last pass slot, which k_hist has cleared and no pass has used if a sweep
// follows.  A batch's sweep clears them.
inline RestArea rest_area(uint32_t *look_back, int digits, uint64_t tiles, uint64_t elements)
{
    const auto u32 = [](uint64_t x) { return (uint32_t)std::min<uint64_t>(x, 0xFFFFFFFFu); };
    RestArea a;
    a.rows = look_back;
    a.max_rows = u32(2 * tiles);
    a.cap = u32(64 * tiles);
    a.list = (uint4 *)(a.rows + 2 * tiles * kRadix);
    a.words = look_back + (digits - 1) * tiles * kRadix;
    a.num_words = kRestTaken + (uint32_t)(elements / (32 * kWave)) + 1;
    a.max_longer = u32(48 * tiles);
    a.longer = (uint4 *)(a.words + (a.num_words + 3) / 4 * 4);
    a.row_run = (uint32_t *)(a.longer + a.max_longer);
    return a;
}

struct FinishArgs {
    Bufs b;
    uint32_t n;
    uint32_t *ctrl;
    RestArea rest;
    uint32_t kmap;      // key order undone when the sweep writes the output
};

constexpr int kFinishThreads = 256;
constexpr int kFinishItems = 4;
// Sorts of up to kFinishFused elements sweep in a pass's launch (k_pass_finish).
// The same line for every kind: whole sorts of uniform keys in us, in that launch
// / in one of its own, 2^20 + 1, 1250000 and 1700000 elements: 32-bit keys 57.3 /
// 57.8, 57.9 / 56.1, 69.6 / 64.9; pairs 62.1 / 63.0, 63.7 / 62.5, 74.0 / 71.6;
// 64-bit keys 72.3 / 72.7, 76.6 / 74.1, 88.1 / 84.6; pairs 75.7 / 78.7, 81.1 / 78.8,
// 93.5 / 88.1.
constexpr int kFinishItemsFused = 2;
constexpr uint32_t kFinishFused = 1u << 20;

// Workgroups loop over tiles of THREADS x ITEMS elements; a tile's keys and
// the chunk before and after it are held in LDS.  A chunk is the 64 elements
// of one wave's item; its head word is a ballot, and run_move orders the
// chunk's elements with it and its neighbours' (rs_runs.h).
//
// Counting over each element's own run, found from the head words by every
// lane, was slower: its reads depended on the run bounds, and 64-bit shifts
// per lane cost more than the count (2^25 64-bit keys, runs of 2: 137 us, now
// 117 us, 4.6 TB/s; 2^20 32-bit keys, runs of 16: 17.8 us, now 10.3 us).  It
// is bound by the compares (VALU) for runs of 4 and more, by HBM below.
//
// The sweeps are held to 80 scalar registers: 16 are set aside for
// each wave, and with 96 and those only 7 waves fit a SIMD, not 8, so that the
// grid's last workgroups start when the first have ended (2^25 64-bit keys: 128
// us, 113 with 80).
#define RS_FINISH_SGPRS __attribute__((amdgpu_num_sgpr(80)))
constexpr uint32_t kFinishPend = 16;
template <typename K, int THREADS, int ITEMS>
struct FinishLds {
    static constexpr uint32_t T = THREADS * ITEMS;
    static constexpr uint32_t H = kWave;  // elements held on either side
    static constexpr int W = THREADS / kWave;
    K k[T + 2 * H];
    // per wave: the head words of its first and last chunk; then those of the
    // chunks before and after the tile.  The same for the words of adjacent
    // elements out of order.
    uint64_t head[2 * W + 2], inv[2 * W + 2];
    uint2 pend[W][kFinishPend];  // places that each wave has to report
    uint32_t longs;              // longer runs met, in order or not
};

// The wave reports that element i of segment seg is smaller than the one before
// it, in a run that is too long to be ordered here.  Reports wait in LDS, since
// atomics on one word end one after another, 14 ns apart (2^25 64-bit keys, 100 of
// each: with an atomic for each of 335,000 long runs the sweep took 5 ms).
template <typename K, int THREADS, int ITEMS>
__device__ __forceinline__ void finish_report(FinishLds<K, THREADS, ITEMS> &L, uint32_t &places,
                                              uint32_t i, uint32_t seg)
{
    if (threadIdx.x % kWave == 0)
        L.pend[threadIdx.x / kWave][places] = make_uint2(i, seg);
    ++places;
}

// After a tile: lists the wave's reports if there may be no room for those of
// another tile, or if it was the last one.  After the last one the workgroup's
// longer runs are counted too.
template <typename K, int THREADS, int ITEMS>
__device__ __forceinline__ void finish_list(FinishLds<K, THREADS, ITEMS> &L, uint32_t *ctrl,
                                            const RestArea &rest, uint32_t &places, bool last)
{
    static_assert(2 * 2 * ITEMS <= (int)kFinishPend, "a tile has two places a chunk");
    const uint32_t lane = threadIdx.x % kWave;
    if (__builtin_expect(places > (last ? 0 : kFinishPend - 2 * ITEMS), 0)) {
        uint32_t l = 0;
        if (lane == 0)
            l = atomicAdd(&ctrl[kCtrlUnsorted], places);
        l = __builtin_amdgcn_readfirstlane(l) + lane;
        if (lane < places && l < rest.cap) {
            const uint2 place = L.pend[threadIdx.x / kWave][lane];
            rest.list[l] = make_uint4(place.x, place.y, 0, 0);
        }
        places = 0;
    }
    if (last && threadIdx.x == 0 && L.longs)
        atomicAdd(&ctrl[kCtrlLongLen], L.longs);
}

// The tile of an array of n elements that starts at tb: from sk, sv to dk,
// dv, every short run in order.  report(i) is called where a longer run is out
// of order, at one place at least of every such run.
template <typename K, typename V, bool HAS_V, int THREADS, int ITEMS, typename Report>
__device__ __forceinline__ void finish_tile(FinishLds<K, THREADS, ITEMS> &L, const K *sk,
                                            const V *sv, K *dk, V *dv, uint32_t n, uint32_t tb,
                                            int shift, uint32_t map, Report &&report)
{
    constexpr uint32_t T = THREADS * ITEMS;
    constexpr uint32_t H = kWave;
    constexpr int W = THREADS / kWave;
    K *s_k = L.k;
    uint64_t *s_head = L.head, *s_inv = L.inv;
    const uint32_t t = threadIdx.x;
    const uint32_t lane = t % kWave;
    const uint32_t w = __builtin_amdgcn_readfirstlane(t / kWave);
    const uint32_t e0 = w * (kWave * ITEMS) + lane;  // element of item 0 in the tile
    const bool full = tb + T <= n;
    K key[ITEMS];
    V val[HAS_V ? ITEMS : 1];
    if (full) {
#pragma unroll
        for (int j = 0; j < ITEMS; ++j)
            key[j] = sk[tb + e0 + j * kWave];
        if constexpr (HAS_V) {
#pragma unroll
            for (int j = 0; j < ITEMS; ++j)
                val[j] = sv[tb + e0 + j * kWave];
        }
    } else {
#pragma unroll
        for (int j = 0; j < ITEMS; ++j) {
            const uint32_t i = tb + e0 + j * kWave;
            key[j] = i < n ? sk[i] : KeyTraits<K>::kPad;
            if constexpr (HAS_V)
                val[j] = i < n ? sv[i] : (V)0;
        }
    }
    // the chunks before and after the tile, by the first and last wave
    if (w == 0)
        s_k[lane] = tb > 0 ? sk[tb - H + lane] : (K)0;
    if (w == W - 1) {
        const uint32_t i = tb + T + lane;
        s_k[H + T + lane] = i < n ? sk[i] : KeyTraits<K>::kPad;
    }
#pragma unroll
    for (int j = 0; j < ITEMS; ++j)
        s_k[H + e0 + j * kWave] = key[j];
    __syncthreads();
    // head words; positions from n on count as heads, so the last run
    // ends there.  Of the chunk before the tile only heads after its
    // first element matter (a run from there to the tile is too long).
    const K low_ones = ((K)1 << shift) - 1;
    uint64_t head[ITEMS + 2], inv[ITEMS + 2];
#pragma unroll
    for (int j = 0; j < ITEMS; ++j) {
        const uint32_t e = e0 + j * kWave;
        const K before = s_k[H + e - 1];
        bool h = (key[j] ^ before) > low_ones;
        if (!full)
            h = h || tb + e >= n;
        if (j == 0)
            h = h || tb + e == 0;
        head[j + 1] = __ballot(h);
        inv[j + 1] = __ballot(key[j] < before);
    }
    if (lane == 0) {
        s_head[2 * w] = head[1];
        s_head[2 * w + 1] = head[ITEMS];
        s_inv[2 * w] = inv[1];
        s_inv[2 * w + 1] = inv[ITEMS];
    }
    if (w == 0) {
        const K x = s_k[lane], before = s_k[lane - (lane > 0)];
        const uint64_t m = __ballot((x ^ before) > low_ones), v = __ballot(x < before);
        if (lane == 0) {
            s_head[2 * W] = m;
            s_inv[2 * W] = v;
        }
    }
    if (w == W - 1) {
        const K x = s_k[H + T + lane], before = s_k[H + T + lane - 1];
        const uint64_t m = __ballot((x ^ before) > low_ones || tb + T + lane >= n);
        const uint64_t v = __ballot(x < before);
        if (lane == 0) {
            s_head[2 * W + 1] = m;
            s_inv[2 * W + 1] = v;
        }
    }
    __syncthreads();
    {
        const uint32_t p = w == 0 ? 2 * W : 2 * w - 1;
        const uint32_t q = w == W - 1 ? 2 * W + 1 : 2 * w + 2;
        head[0] = uniform_word(s_head[p]);
        head[ITEMS + 1] = uniform_word(s_head[q]);
        inv[0] = uniform_word(s_inv[p]);
        inv[ITEMS + 1] = uniform_word(s_inv[q]);
    }
    uint32_t longs = 0;
#pragma unroll
    for (int j = 0; j < ITEMS; ++j) {
        const uint32_t e = e0 + j * kWave;
        const uint32_t at = H + e;  // this element's LDS slot
        uint32_t pos = tb + e;
        const uint64_t here = head[j + 1], prev = head[j], next = head[j + 2];
        // nothing adjacent out of order in the three chunks: in place
        if ((inv[j] | inv[j + 1] | inv[j + 2]) != 0) {
            bool whole;
            pos += (uint32_t)run_move(s_k, at, key[j], lane, here, prev, next, &whole);
            // elements of longer runs that are below the one before them: in the
            // run that comes in from the chunk before, unless that chunk has
            // seen one in it too, and in the one that goes on into the next
            const uint64_t low = inv[j + 1] & __ballot(!whole);
            if (__builtin_expect(low != 0, 0)) {
                const uint64_t in = here ? (here & (0 - here)) - 1 : ~0ull;
                const uint64_t tail = prev ? ~0ull << (kWave - 1 - __builtin_clzll(prev)) : ~0ull;
                const uint64_t first = inv[j] & tail ? 0ull : low & in, last = low & ~in;
                const uint32_t c = tb + (w * ITEMS + j) * kWave;
                if (first)
                    report(c + (uint32_t)__builtin_ctzll(first));
                if (last)
                    report(c + (uint32_t)__builtin_ctzll(last));
            }
        }
        if (pos < n && (full || tb + e < n)) {
            store_at(dk, pos, map_out(key[j], map));
            if constexpr (HAS_V)
                store_at(dv, pos, val[j]);
        }
        // runs that are too long, in order or not
        const uint32_t ends = here ? __builtin_clzll(here) : 0;
        if (here && ends + (next ? __builtin_ctzll(next) : kWave) >= kRunMax)
            ++longs;
    }
    if (__builtin_expect(longs, 0) && lane == 0)
        atomicAdd(&L.longs, longs);
    __syncthreads();  // the next tile overwrites the LDS
}

template <typename K, typename V, bool HAS_V, int THREADS, int ITEMS>
__device__ __forceinline__ void finish_all(FinishLds<K, THREADS, ITEMS> &L, FinishArgs a,
                                           uint32_t word)
{
    constexpr uint32_t T = THREADS * ITEMS;
    const uint32_t src = (word >> kFinishSrcShift) & 3u;
    const uint32_t dst = (word >> kFinishDstShift) & 3u;
    const int shift = (int)(word >> kFinishShift);
    const uint32_t map = dst == kBufOut ? a.kmap : 0u;
    const K *sk = pick<const K>(a.b, src, false);
    const V *sv = HAS_V ? pick<const V>(a.b, src, true) : nullptr;
    K *dk = pick<K>(a.b, dst, false);
    V *dv = HAS_V ? pick<V>(a.b, dst, true) : nullptr;
    const uint32_t tiles = (a.n + T - 1) / T;
    uint32_t places = 0;  // reports that wait (uniform)
    if (threadIdx.x == 0)
        L.longs = 0;  // a tile has barriers before and after its use
    for (uint32_t tile = blockIdx.x; tile < tiles; tile += gridDim.x) {
        finish_tile<K, V, HAS_V, THREADS, ITEMS>(
            L, sk, sv, dk, dv, a.n, tile * T, shift, map,
            [&](uint32_t i) { finish_report(L, places, i, 0); });
        finish_list(L, a.ctrl, a.rest, places, tile + gridDim.x >= tiles);
    }
}

template <typename K, typename V, bool HAS_V, int THREADS, int ITEMS>
__global__ __launch_bounds__(THREADS) RS_FINISH_SGPRS void k_finish(FinishArgs a)
{
    __shared__ FinishLds<K, THREADS, ITEMS> L;
    const uint32_t word = __builtin_amdgcn_readfirstlane(a.ctrl[kCtrlFinish]);
    if (word & kFinishRun)
        finish_all<K, V, HAS_V, THREADS, ITEMS>(L, a, word);
}

struct PassFinishArgs {
    PassArgs p;
    FinishArgs f;
    uint32_t pass_grid;  // workgroups that the pass wants; the sweep takes all
};

// The slot before the last of a sort of up to kFinishFused elements: its
// pass, or the sweep (a sort that sweeps has saved two passes at least, so
// that slot's is one of them).  With a launch for each, one of the two did
// nothing, for 2 us: 98304 64-bit pairs 47.6 -> 45.6 us, 2^15 32-bit keys of 64
// values 45 -> 44.  The sweep's own smaller workgroups are the faster ones
// where they fill the chip (2^22 64-bit keys 116 us, in this launch 124).
template <typename K, typename V, bool HAS_V, typename C>
__global__ __launch_bounds__(C::kThreads) void k_pass_finish(PassFinishArgs a)
{
    static_assert(!C::kWide && kFinishSaves >= 2, "8-bit digits; the slot is free when the sweep runs");
    __shared__ union {
        PassLds<K, C, HAS_V> pass;
        FinishLds<K, C::kThreads, kFinishItemsFused> finish;
    } L;
    const uint32_t word = __builtin_amdgcn_readfirstlane(a.p.ctrl[kCtrlFinish]);
    const uint32_t plan = __builtin_amdgcn_readfirstlane(a.p.ctrl[kCtrlPlan + a.p.pass]);
    if (word & kFinishRun)
        finish_all<K, V, HAS_V, C::kThreads, kFinishItemsFused>(L.finish, a.f, word);
    else if (blockIdx.x < a.pass_grid)
        pass_slot<K, V, HAS_V, C>(a.p, plan, L.pass);
}

struct LastArgs {
    PassArgs p;  // of the last slot
    RestArea rest;
};

// Waits until *word >= want; bounded like every wait on other workgroups.
// Called by one thread; false when the bound was reached.
__device__ __forceinline__ bool wait_count(const uint32_t *word, uint32_t want, const PassArgs &a)
{
    uint32_t spins = 0;
    while (__hip_atomic_load(word, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) < want) {
        if (++spins > a.spin_limit) {
            atomicOr(a.err, kErrWait);
            return false;
        }
        __builtin_amdgcn_s_sleep(4);
    }
    return true;
}

// One thread of a workgroup, after a barrier: hands the workgroup's writes on
// (the barrier has put them before this thread's release, which then covers
// them all), counts `add` items as done and waits for `want` of them.  One
// release for a workgroup, not one in every wave, and none without items:
// each writes a cache back.
__device__ __forceinline__ bool hand_on_and_wait(uint32_t *done, uint32_t add, uint32_t want,
                                                 const PassArgs &a)
{
    if (add) {
        __builtin_amdgcn_fence(__ATOMIC_RELEASE, "agent");
        atomicAdd(done, add);
    }
    return wait_count(done, want, a);
}

// An array with runs to sort (the plain sort's, or a large segment): where it
// lies, its length, the bits from `shift` up that the elements of a run share,
// the digit positions below that move data, the key order of the stored
// keys, and its first element's place among all arrays.
template <typename K, typename V>
struct RunArray {
    K *k;
    V *v;
    uint32_t n;
    int shift;
    uint32_t digits;
    uint32_t map;
    uint64_t base;
};

// The ends of element p's run, by the whole wave: 64 probes at a time on either
// side, 8 elements apart at first (one trip finds a run of 512), at distances
// that grow 64-fold until one leaves the run and then shrink.
template <typename K, typename V>
__device__ __forceinline__ uint2 run_ends(const RunArray<K, V> &arr, uint32_t p, uint32_t lane)
{
    const K lead = map_in(arr.k[p], arr.map) >> arr.shift;
    const uint32_t room[2] = {p, arr.n - 1 - p};
    uint32_t far[2] = {0, 0}, step[2] = {8, 8};  // step 0: found
    bool grow[2] = {true, true};
    while (step[0] | step[1]) {
        K x[2];
        bool in[2];
#pragma unroll
        for (int i = 0; i < 2; ++i) {
            const uint64_t d = far[i] + (uint64_t)step[i] * (lane + 1);
            in[i] = step[i] && d <= room[i];
            x[i] = in[i] ? arr.k[i ? p + d : p - d] : (K)0;
        }
#pragma unroll
        for (int i = 0; i < 2; ++i) {
            const uint64_t out = ~__ballot(in[i] && (map_in(x[i], arr.map) >> arr.shift) == lead);
            const uint32_t c = out ? (uint32_t)__builtin_ctzll(out) : (uint32_t)kWave;
            far[i] += step[i] * c;
            grow[i] = grow[i] && c == (uint32_t)kWave;
            step[i] = grow[i] ? step[i] * kWave : step[i] == 1 ? 0u : (step[i] + kWave - 1) / kWave;
        }
    }
    return make_uint2(p - far[0], p + far[1] + 1);
}

// Runs of up to kRestWaveRun elements are sorted by a wave each, in its LDS.
// (In registers, each element counting the run's keys as they are broadcast,
// a run of 200 64-bit keys took 20 us; now 4.)
constexpr uint32_t kRestWaveRun = 512;

// One place where a run is out of order, entry i of the list: finds the run and,
// if no other place of it was first, makes it the wave's entry or lists it with
// the longer ones.  By one wave.  (Listed by an atomic on one word, 11,700 runs
// took 165 us of a batch's 640.)
template <typename K, typename V, typename Resolve>
__device__ __forceinline__ void rest_find(uint32_t i, uint32_t tile, uint32_t *ctrl,
                                          const RestArea &rest, Resolve &&resolve)
{
    const uint32_t lane = threadIdx.x % kWave;
    const uint4 entry = rest.list[i];
    const RunArray<K, V> arr = resolve(entry.y);
    const uint2 ends = run_ends(arr, entry.x, lane);
    uint4 run = make_uint4(ends.x, ends.y - ends.x, entry.y, 0);
    // runs listed are longer than 64, so no two start among the same 64
    const uint64_t bit = (arr.base + run.x) / kWave;
    const uint32_t mask = 1u << (bit % 32);
    uint32_t taken = 0;
    if (lane == 0)
        taken = atomicOr(&rest.words[kRestTaken + bit / 32], mask) & mask;
    taken = __builtin_amdgcn_readfirstlane(taken);
    const bool longer = run.y > kRestWaveRun;
    if (lane == 0)
        rest.list[i] = make_uint4(run.x, taken || longer ? 0u : run.y, run.z, 0);
    if (taken || !longer)
        return;
    uint32_t idx = 0;
    if (lane == 0)
        idx = atomicAdd(&ctrl[kCtrlLongerLen], 1u);
    idx = __builtin_amdgcn_readfirstlane(idx);
    // only overlapping segments can need more room than there is: then such a
    // run is not sorted
    if (idx >= rest.max_longer)
        return;
    const uint32_t rows = run.y > tile ? (run.y + tile - 1) / tile : 0u;
    if (rows) {
        if (lane == 0) {
            run.w = atomicAdd(&rest.words[kRestRows], rows);
            atomicAdd(&ctrl[kCtrlGiant], 1u);
        }
        run.w = __builtin_amdgcn_readfirstlane(run.w);
        if ((uint64_t)run.w + rows > rest.max_rows)
            run.y = 0;
    }
    for (uint32_t j = lane; j < rows && (uint64_t)run.w + j < rest.max_rows; j += kWave)
        rest.row_run[run.w + j] = idx;
    if (lane == 0)
        rest.longer[idx] = run;
}

struct RestShared {
    uint32_t item, ok;
};

// LDS of k_last: of a pass, of a run for a workgroup, of runs for its waves.
template <typename K, typename C, bool HAS_V>
union RestLds {
    PassLds<K, C, HAS_V> pass;
    BlockLds<K, HAS_V, C::kThreads, C::kItems> block;
    WaveLds<K, HAS_V, kRestWaveRun> wave[C::kThreads / kWave];
};

// Hands out [0, len) to the waves of the launch's workgroups, a wave each, from
// the counter *claim: one atomic for all waves of a workgroup (with one for
// each of 4096 waves the follow-up took 30 us for a single run).  Returns, to
// thread 0, how many this workgroup took.
template <int THREADS, typename F>
__device__ __forceinline__ uint32_t rest_by_waves(RestShared &S, uint32_t *claim, uint32_t len,
                                                  F &&f)
{
    constexpr uint32_t W = THREADS / kWave;
    const uint32_t w = __builtin_amdgcn_readfirstlane(threadIdx.x / kWave);
    uint32_t taken = 0;
    while (true) {
        __syncthreads();
        if (threadIdx.x == 0)
            S.item = atomicAdd(claim, W);
        __syncthreads();
        const uint32_t item = __builtin_amdgcn_readfirstlane(S.item);
        if (item >= len)
            return taken;
        taken += min(W, len - item);
        if (item + w < len)
            f(item + w);
    }
}

// The runs out of order, by every workgroup of the launch: all look up where
// the sweep reported one and wait for each other; then waves take the shorter
// runs and workgroups the longer ones, up to a tile.  Returns the rows of the
// runs longer than that, which are left to sort_again, or kRestAll if there
// are too many runs and everything is (every workgroup gets the same answer).
// resolve(segment) is the array that holds a run.
constexpr uint32_t kRestAll = 0xFFFFFFFFu;

template <typename K, typename V, bool HAS_V, typename C, typename Resolve>
__device__ __forceinline__ uint32_t rest_runs(RestLds<K, C, HAS_V> &L, RestShared &S,
                                              uint32_t *ctrl, const RestArea &rest,
                                              const PassArgs &wait, Resolve &&resolve)
{
    constexpr uint32_t T = C::kTile;
    constexpr int THREADS = C::kThreads;
    constexpr int ITEMS = C::kItems;
    const uint32_t t = threadIdx.x;
    const uint32_t len = __builtin_amdgcn_readfirstlane(ctrl[kCtrlUnsorted]);
    if (len > rest.cap)
        return kRestAll;
    const uint32_t found =
        rest_by_waves<THREADS>(S, &rest.words[kRestFindClaim], len, [&](uint32_t i) {
            rest_find<K, V>(i, T, ctrl, rest, resolve);
        });
    if (t == 0) {
        S.ok = hand_on_and_wait(&rest.words[kRestFindDone], found, len, wait) ? 1u : 0u;
        __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "agent");
    }
    __syncthreads();
    if (!S.ok)
        return 0;
    const auto count = [](uint32_t *word) {
        return __builtin_amdgcn_readfirstlane(
            __hip_atomic_load(word, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT));
    };
    const uint32_t longer = min(count(&ctrl[kCtrlLongerLen]), rest.max_longer);
    const uint32_t rows = min(count(&rest.words[kRestRows]), rest.max_rows);
    rest_by_waves<THREADS>(S, &rest.words[kRestShortClaim], len, [&](uint32_t i) {
        const uint4 run = rest.list[i];
        if (__builtin_amdgcn_readfirstlane(run.y) == 0)
            return;
        const RunArray<K, V> arr = resolve(run.z);
        K *rk = arr.k + run.x;
        V *rv = HAS_V ? arr.v + run.x : nullptr;
        const uint32_t m = __builtin_amdgcn_readfirstlane(run.y);
        const WaveData<K, V> in{rk, rv, rk, rv};
        auto &lds = L.wave[__builtin_amdgcn_readfirstlane(t / kWave)];
        if (m <= kRestWaveRun / 2)
            radix_wave<K, V, HAS_V, kRestWaveRun / 2 / kWave>(lds, in, m, t % kWave, arr.map);
        else
            radix_wave<K, V, HAS_V, kRestWaveRun / kWave>(lds, in, m, t % kWave, arr.map);
    });
    while (true) {
        __syncthreads();
        if (t == 0)
            S.item = atomicAdd(&rest.words[kRestLongerClaim], 1u);
        __syncthreads();
        const uint32_t item = __builtin_amdgcn_readfirstlane(S.item);
        if (item >= longer)
            break;
        const uint4 run = rest.longer[item];
        if (__builtin_amdgcn_readfirstlane(run.y) > T)
            continue;
        const RunArray<K, V> arr = resolve(run.z);
        K *rk = arr.k + run.x;
        V *rv = HAS_V ? arr.v + run.x : nullptr;
        const BlockItems<THREADS, ITEMS> it(run.y);
        K key[ITEMS];
        V val[HAS_V ? ITEMS : 1];
        it.each([&](int j) {
            key[j] = it.has(j) ? map_in(rk[it.at(j)], arr.map) : (K)0;
            if constexpr (HAS_V)
                val[j] = it.has(j) ? rv[it.at(j)] : (V)0;
        });
        __syncthreads();  // everything is read before it is overwritten
        block_sort_digits<K, V, HAS_V, THREADS, ITEMS>(L.block, it, key, val, arr.digits);
        it.each([&](int j) {
            if (it.has(j)) {
                rk[it.at(j)] = map_out(key[j], arr.map);
                if constexpr (HAS_V)
                    rv[it.at(j)] = val[j];
            }
        });
    }
    __syncthreads();
    return rows;
}

// The next item of stages of `tiles` items each, or false when there is none
// (or a wait reached its bound).  Called by every thread after a barrier that
// ends its last item; an item waits for the stage before its own.  A workgroup
// counts its items as done when it goes on to another stage: a release writes
// a cache back, so one for every item made a stage take as long as two.
struct RestItem {
    uint32_t stage = 0, tile = 0;
    uint32_t held = 0;  // items of `stage` finished or at work
};

__device__ __forceinline__ bool rest_next(RestItem &it, RestShared &S, uint32_t *words,
                                          uint32_t stages, uint32_t tiles, const PassArgs &wait)
{
    uint32_t *stage_done = words + kRestStageDone;
    // One thread reports the last items, claims the next and waits, in one
    // place: with the report at the end of the caller's loop the compiler
    // sends the other threads of its wave to the barrier ahead of it.
    if (threadIdx.x == 0) {
        const uint32_t item = atomicAdd(&words[kRestItemClaim], 1u);
        const uint32_t st = item / tiles;
        S.item = item;
        S.ok = 1;
        if (st != it.stage || it.held == 0) {
            if (it.held) {
                __builtin_amdgcn_fence(__ATOMIC_RELEASE, "agent");
                atomicAdd(&stage_done[it.stage], it.held);
            }
            S.ok = st == 0 || st >= stages || wait_count(&stage_done[st - 1], tiles, wait);
            __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "agent");
        }
    }
    __syncthreads();
    const uint32_t stage = __builtin_amdgcn_readfirstlane(S.item / tiles);
    it.held = stage == it.stage ? it.held + 1 : 1;
    it.stage = stage;
    it.tile = __builtin_amdgcn_readfirstlane(S.item % tiles);
    return it.stage < stages && S.ok != 0;
}

// An array to sort again by every digit in `digits`: its buffers (it lies in the
// first of each, and ends there), its length, its first row, the digits that
// are skewed, the key order of the stored keys, and every digit's offsets (null:
// they are counted).
template <typename K, typename V>
struct AgainArray {
    K *k[2];
    V *v[2];
    uint32_t n;
    uint32_t first;
    uint32_t digits;
    uint32_t skew;
    uint32_t map;
    const uint32_t *base;  // [digit][256]
};

// Sorts arrays again, in `rows` rows of a tile each; resolve(row) is the array
// of a row.  Two stages a digit, one that clears the rows' look-back words (or
// counts their digits) and a pass; the lowest digit twice if their number is
// odd, so that the result ends where it began (sorting by a digit twice changes
// nothing).
template <typename K, typename V, bool HAS_V, typename C, typename Resolve>
__device__ __forceinline__ void sort_again(PassLds<K, C, HAS_V> &L, RestShared &S,
                                           const RestArea &rest, uint32_t rows,
                                           const PassArgs &wait, Resolve &&resolve)
{
    constexpr uint32_t T = C::kTile;
    constexpr uint32_t NB = C::kBins;
    constexpr int R = C::kRadixBits;
    constexpr int THREADS = C::kThreads;
    constexpr uint32_t D = num_passes<K, R>();
    static_assert(R == kRadixBits && D % 2 == 0 && kRestStageDone + 2 * D <= kRestTaken,
                  "8-bit digits; a word for every stage");
    const uint32_t t = threadIdx.x;
    RestItem it;
    while (rest_next(it, S, rest.words, 2 * D, rows, wait)) {
        const AgainArray<K, V> a = resolve(it.tile);
        const uint32_t q = (uint32_t)__popc(a.digits);
        const uint32_t sets = q + (q & 1), set = it.stage / 2;
        if (set >= sets) {
            __syncthreads();
            continue;
        }
        uint32_t left = a.digits;
        for (uint32_t i = q & 1; i < set; ++i)
            left &= left - 1;
        const uint32_t digit = (uint32_t)__builtin_ctz(left);
        const uint32_t from = set & 1, into = from ^ 1;
        const uint32_t tb = (it.tile - a.first) * T;
        const uint32_t valid = a.n > tb ? min(T, a.n - tb) : 0u;
        const uint32_t map_load = set == 0 ? a.map : 0u;
        if (it.stage % 2 == 0) {
            uint32_t sum = 0;
            if (!a.base) {
                uint32_t *wc = L.wcnt + t / kWave * NB;  // a wave's own
                for (uint32_t i = t % kWave; i < NB; i += kWave)
                    wc[i] = 0;
                wave_lds_fence();
                for (uint32_t e = t; e < valid; e += THREADS)
                    atomicAdd(&wc[digit_of<R>(map_in(a.k[from][tb + e], map_load), digit * R)],
                              1u);
                __syncthreads();
                if (t < NB) {
                    for (uint32_t w = 0; w < THREADS / kWave; ++w)
                        sum += L.wcnt[w * NB + t];
                    sum |= kFlagAgg;
                }
            }
            if (t < NB)
                rest.rows[(uint64_t)it.tile * NB + t] = sum;
            __syncthreads();
            continue;
        }
        uint32_t dbase = 0;
        if (a.base) {
            dbase = t < NB ? a.base[digit * NB + t] : 0u;
        } else {
            // every row has its counts: their sum is the look-back from the end
            const uint32_t end = a.first + (a.n + T - 1) / T;
            const uint32_t total =
                t < NB ? lookback_digit<16, C::kGroup>(rest.rows, nullptr, NB, t, end, a.first, wait)
                       : 0u;
            dbase = bins_exclusive_scan<NB>(total, L.tmp);
        }
        pass_tile<K, V, HAS_V, C>(L, a.k[from] + tb, HAS_V ? a.v[from] + tb : nullptr, a.k[into],
                                  HAS_V ? a.v[into] : nullptr, valid, a.n, it.tile, a.first,
                                  rest.rows, nullptr, dbase, (int)digit * R,
                                  ((a.skew >> digit) & 1u) != 0, map_load,
                                  set + 1 == sets ? a.map : 0u, wait, [](uint32_t) {});
    }
}

// The run of a row of sort_again (uniform).
__device__ __forceinline__ uint4 rest_row(const RestArea &rest, uint32_t row)
{
    const uint4 run = rest.longer[rest.row_run[row]];
    return make_uint4(
        __builtin_amdgcn_readfirstlane(run.x), __builtin_amdgcn_readfirstlane(run.y),
        __builtin_amdgcn_readfirstlane(run.z), __builtin_amdgcn_readfirstlane(run.w));
}

// One launch of persistent workgroups.  Work is claimed in order, (stage,
// tile) after (stage, tile), and an item waits only for the stage before its
// own, whose items are all claimed by running workgroups: no wait depends on
// a workgroup that has not started (nor does the one in rest_runs: a
// workgroup counts what it has looked up as done before it waits for the
// others).  Stages hand their data on through memory within the launch
// (hand_on_and_wait).
template <typename K, typename V, bool HAS_V, typename C>
__global__ __launch_bounds__(C::kThreads) void k_last(LastArgs a)
{
    static_assert(C::kRadixBits == kRadixBits, "8-bit digits");
    __shared__ RestLds<K, C, HAS_V> L;
    __shared__ RestShared S;

    uint32_t *ctrl = a.p.ctrl;
    const uint32_t finish = __builtin_amdgcn_readfirstlane(ctrl[kCtrlFinish]);
    const uint32_t plan = __builtin_amdgcn_readfirstlane(ctrl[kCtrlPlan + a.p.pass]);
    const uint32_t unsorted = __builtin_amdgcn_readfirstlane(ctrl[kCtrlUnsorted]);
    if (!(finish & kFinishRun)) {
        pass_slot<K, V, HAS_V, C>(a.p, plan, L.pass);
        return;
    }
    if (unsorted == 0)
        return;
    const uint32_t n = a.p.n;
    const uint32_t buf = (finish >> kFinishDstShift) & 3u;  // where k_finish wrote
    const uint32_t digits = __builtin_amdgcn_readfirstlane(ctrl[kCtrlDigits]);
    // the output holds unmapped keys, the scratch copy mapped ones
    const uint32_t map = buf == kBufOut ? a.p.kmap : 0u;
    const int shift = (int)(finish >> kFinishShift);
    K *bk = pick<K>(a.p.b, buf, false);
    V *bv = HAS_V ? pick<V>(a.p.b, buf, true) : nullptr;
    const uint32_t low = digits & ((1u << (shift / C::kRadixBits)) - 1u);
    const uint32_t rows =
        rest_runs<K, V, HAS_V, C>(L, S, ctrl, a.rest, a.p, [=](uint32_t) {
            return RunArray<K, V>{bk, bv, n, shift, low, map, 0};
        });
    if (rows == 0)
        return;
    const uint32_t other = buf == kBufOut ? kBufTmp : kBufOut;
    K *ok = pick<K>(a.p.b, other, false);
    V *ov = HAS_V ? pick<V>(a.p.b, other, true) : nullptr;
    const uint32_t skew = __builtin_amdgcn_readfirstlane(ctrl[kCtrlSkew]);
    const bool all = rows == kRestAll;
    const RestArea rest = a.rest;
    const uint32_t *base = a.p.digit_base;
    sort_again<K, V, HAS_V, C>(L.pass, S, rest, all ? a.p.num_tiles : rows, a.p, [=](uint32_t row) {
        if (all)
            return AgainArray<K, V>{{bk, ok}, {bv, ov}, n, 0, digits, skew, map, base};
        const uint4 run = rest_row(rest, row);
        return AgainArray<K, V>{{bk + run.x, ok + run.x},
                                {HAS_V ? bv + run.x : nullptr, HAS_V ? ov + run.x : nullptr},
                                run.y,
                                run.w,
                                low,
                                skew,
                                map,
                                nullptr};
    });
}

// ---------------------------------------------------------------------------
// The same for the large segments of a segmented sort, each with its own
// finish shift (k_seg_scan).  2000 segments of 2^4 to 2^20 32-bit pairs: four
// passes of 738 us each before, two and a sweep of 828 us now; 24 of 2^10 to
// 2^22 64-bit pairs: eight passes of 62 us, now three and a sweep of 48 us.
// With runs of up to 16 the sweep is bound by its compares, not by HBM (590 us).

struct SegFinishArgs {
    Bufs b;
    const SegLarge *large;
    const uint32_t *tile_seg;
    const uint32_t *seg_flags;
    uint32_t *ctrl;
    uint32_t max_tiles;
    uint32_t tile;      // elements per tile of the passes, a multiple of the sweep's
    uint32_t group;     // sweep tiles that a workgroup takes together, of one tile
    RestArea rest;
    uint32_t kmap;
    int in_place;
};

template <typename K, typename V, bool HAS_V, int THREADS, int ITEMS>
__global__ __launch_bounds__(THREADS) RS_FINISH_SGPRS void k_seg_finish(SegFinishArgs a)
{
    constexpr uint32_t T = THREADS * ITEMS;
    __shared__ FinishLds<K, THREADS, ITEMS> L;
    if (!(a.ctrl[kSegPassMask] & kSegAnyFinish))
        return;
    for (uint32_t i = blockIdx.x * THREADS + threadIdx.x; i < a.rest.num_words;
         i += gridDim.x * THREADS)
        a.rest.words[i] = 0;
    uint32_t places = 0;
    if (threadIdx.x == 0)
        L.longs = 0;
    __syncthreads();  // there may be no tile
    const uint32_t tiles = std::min(a.ctrl[kSegTiles], a.max_tiles);
    // groups of sweep tiles: a segment's record takes three dependent loads
    const uint32_t per = a.tile / (T * a.group);
    for (uint32_t item = blockIdx.x; item < tiles * per; item += gridDim.x) {
        const uint32_t tile = item / per;
        const uint32_t seg = a.tile_seg[tile];
        const SegLarge rec = a.large[seg];
        const SegMoves m = seg_moves<K, kRadixBits>(
            __builtin_amdgcn_readfirstlane(a.seg_flags[seg]), a.in_place != 0);
        if (m.low == 0)
            continue;
        const uint32_t src = m.dst(m.moves - 2), dst = m.dst(m.moves - 1);
        const K *sk = pick<const K>(a.b, src, false) + rec.start;
        const V *sv = HAS_V ? pick<const V>(a.b, src, true) + rec.start : nullptr;
        K *dk = pick<K>(a.b, dst, false) + rec.start;
        V *dv = HAS_V ? pick<V>(a.b, dst, true) + rec.start : nullptr;
        const uint32_t size = __builtin_amdgcn_readfirstlane(rec.size);
        uint32_t tb = __builtin_amdgcn_readfirstlane(
            (tile - rec.tile_start) * a.tile + (item - tile * per) * a.group * T);
        for (uint32_t g = 0; g < a.group && tb < size; ++g, tb += T) {
            finish_tile<K, V, HAS_V, THREADS, ITEMS>(
                L, sk, sv, dk, dv, size, tb, (int)(m.low * kRadixBits),
                dst == kBufOut ? a.kmap : 0u,
                [&](uint32_t i) { finish_report(L, places, i, seg); });
            finish_list(L, a.ctrl, a.rest, places, false);
        }
    }
    finish_list(L, a.ctrl, a.rest, places, true);
}

struct SegLastArgs {
    SegPassArgs p;
    RestArea rest;
};

template <typename K, typename V, bool HAS_V, typename C>
__global__ __launch_bounds__(C::kThreads) void k_seg_last(SegLastArgs a)
{
    constexpr uint32_t NB = C::kBins;
    constexpr int R = C::kRadixBits;
    constexpr int D = num_passes<K, R>();
    __shared__ RestLds<K, C, HAS_V> L;
    __shared__ RestShared S;
    uint32_t *ctrl = a.p.ctrl;
    if (ctrl[kCtrlUnsorted] == 0)
        return;
    const bool in_place = a.p.keys_in_place || a.p.vals_in_place;
    const SegLarge *large = a.p.large;
    const uint32_t *seg_flags = a.p.seg_flags;
    const Bufs b = a.p.b;
    const uint32_t kmap = a.p.kmap;
    PassArgs wait{};
    wait.err = ctrl + kSegError;
    wait.spin_limit = a.p.spin_limit;
    wait.stall = a.p.stall;
    const auto uniform = [](uint32_t x) {
        return (uint32_t)__builtin_amdgcn_readfirstlane(x);
    };
    const uint32_t rows =
        rest_runs<K, V, HAS_V, C>(L, S, ctrl, a.rest, wait, [=](uint32_t seg) {
            const SegLarge rec = large[seg];
            const uint32_t flags = seg_flags[seg];
            const SegMoves m = seg_moves<K, R>(flags, in_place);
            const uint32_t buf = m.dst(m.moves - 1);
            return RunArray<K, V>{pick<K>(b, buf, false) + rec.start,
                                  HAS_V ? pick<V>(b, buf, true) + rec.start : nullptr,
                                  uniform(rec.size),
                                  (int)uniform(m.low * R),
                                  uniform(~flags & ((1u << m.low) - 1u)),
                                  buf == kBufOut ? kmap : 0u,
                                  rec.start};
        });
    if (rows == 0)
        return;

    // the runs longer than a tile, or every segment that was swept
    const bool all = rows == kRestAll;
    const uint32_t tiles = std::min(ctrl[kSegTiles], a.p.max_tiles);
    const uint32_t *tile_seg = a.p.tile_seg, *seg_base = a.p.seg_base;
    const RestArea rest = a.rest;
    sort_again<K, V, HAS_V, C>(L.pass, S, rest, all ? tiles : rows, wait, [=](uint32_t row) {
        const uint4 run = all ? make_uint4(0, 0, tile_seg[row], 0) : rest_row(rest, row);
        const uint32_t seg = run.z;
        const SegLarge rec = large[seg];
        const uint32_t flags = uniform(seg_flags[seg]);
        const SegMoves m = seg_moves<K, R>(flags, in_place);
        const uint32_t buf = m.dst(m.moves - 1), other = buf == kBufOut ? kBufTmp : kBufOut;
        const uint64_t at = rec.start + run.x;
        const uint32_t digits = ~flags & ((1u << (all ? D : m.low)) - 1u);
        return AgainArray<K, V>{{pick<K>(b, buf, false) + at, pick<K>(b, other, false) + at},
                                {HAS_V ? pick<V>(b, buf, true) + at : nullptr,
                                 HAS_V ? pick<V>(b, other, true) + at : nullptr},
                                all ? uniform(rec.size) : run.y,
                                all ? uniform(rec.tile_start) : run.w,
                                m.low ? digits : 0u,
                                flags >> kSegSkewShift,
                                buf == kBufOut ? kmap : 0u,
                                all ? seg_base + (uint64_t)seg * D * NB : nullptr};
    });
}

}  // namespace rs
