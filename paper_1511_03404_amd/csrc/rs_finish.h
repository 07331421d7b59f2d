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
//              that place; a longer run is copied and, if it is out of order
//              anywhere, reported;
//   k_last     the last pass slot.  After a sweep that slot is free, and it
//              does what the sweep could not, normally nothing: long runs
//              out of order are sorted by a wave or a workgroup each, and if
//              one is longer than a tile (or there are too many) the whole
//              array is sorted again by every digit.
#pragma once

#include "rs_kernels.h"
#include "rs_runs.h"

namespace rs {

struct FinishArgs {
    Bufs b;
    uint32_t n;
    uint32_t *ctrl;
    uint32_t *list;     // starts of the runs longer than kRunMax
    uint32_t list_cap;
    uint32_t kmap;      // key order undone when the sweep writes the output
};

constexpr int kFinishThreads = 256;
constexpr int kFinishItems = 4;
// sorts of up to kFinishFused elements sweep in a pass's launch
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
};

// The tile of an array of n elements that starts at tb: from sk, sv to dk,
// dv, every short run in order.  *unsorted is set if a longer one is not in
// order; list_run(i) is called for every longer run, which starts at i.
template <typename K, typename V, bool HAS_V, int THREADS, int ITEMS, typename List>
__device__ __forceinline__ void finish_tile(FinishLds<K, THREADS, ITEMS> &L, const K *sk,
                                            const V *sv, K *dk, V *dv, uint32_t n, uint32_t tb,
                                            int shift, uint32_t map, uint32_t *unsorted,
                                            List &&list_run)
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
            if (!whole) {
                const bool in_run =
                    (lane < kWave - 1 ? (here >> (lane + 1)) & 1ull : next & 1ull) == 0;
                if (in_run && key[j] > s_k[at + 1])
                    __hip_atomic_store(unsorted, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            }
        }
        if (pos < n && (full || tb + e < n)) {
            store_at(dk, pos, map_out(key[j], map));
            if constexpr (HAS_V)
                store_at(dv, pos, val[j]);
        }
        // the starts of the runs that are too long, in order or not
        const uint32_t ends = here ? __builtin_clzll(here) : 0;
        if (here && ends + (next ? __builtin_ctzll(next) : kWave) >= kRunMax) {
            const uint32_t i = tb + e;
            if (lane == kWave - 1 - ends && i < n)
                list_run(i);
        }
    }
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
    uint32_t *ctrl = a.ctrl, *list = a.list;
    const uint32_t cap = a.list_cap;
    const uint32_t tiles = (a.n + T - 1) / T;
    for (uint32_t tile = blockIdx.x; tile < tiles; tile += gridDim.x)
        finish_tile<K, V, HAS_V, THREADS, ITEMS>(L, sk, sv, dk, dv, a.n, tile * T, shift, map,
                                                 &ctrl[kCtrlUnsorted], [=](uint32_t i) {
                                                     const uint32_t l =
                                                         atomicAdd(&ctrl[kCtrlLongLen], 1u);
                                                     if (l < cap)
                                                         list[l] = i;
                                                 });
}

template <typename K, typename V, bool HAS_V, int THREADS, int ITEMS>
__global__ __launch_bounds__(THREADS) void k_finish(FinishArgs a)
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
    const uint32_t word = __builtin_amdgcn_readfirstlane(a.f.ctrl[kCtrlFinish]);
    if (word & kFinishRun)
        finish_all<K, V, HAS_V, C::kThreads, kFinishItemsFused>(L.finish, a.f, word);
    else if (blockIdx.x < a.pass_grid)
        pass_slot<K, V, HAS_V, C>(a.p, L.pass);
}

struct LastArgs {
    PassArgs p;        // of the last slot
    uint32_t *status;  // look-back words of every slot
    uint32_t d;        // digit positions (and sets of look-back words)
    uint32_t *list;    // k_finish's long runs
    uint32_t list_cap;
};

// Runs too long for a workgroup are checked for order over this many tiles;
// one that is longer still counts as out of order.
constexpr uint32_t kRestScanTiles = 32;

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

// A listed run: its first element, the elements from there to the end of its
// array, the bits from `shift` up that its elements share, the digit
// positions below that move data, and the key order of the stored keys.
template <typename K, typename V>
struct LongRun {
    K *k;
    V *v;
    uint32_t n;
    int shift;
    uint32_t digits;
    uint32_t map;
};

// Runs of up to kRestWaveRun elements are sorted by a wave each, in
// registers: every element counts the run's elements that go before it, the
// run's keys broadcast one after another.  Longer ones are listed again,
// from the list's end.  Returns how many runs this wave took.
constexpr uint32_t kRestSlots = 8;
constexpr uint32_t kRestWaveRun = kRestSlots * kWave;

// Writes a run of m <= 64 SLOTS elements, in registers (element s*64 + lane
// in slot s), back in order.
template <typename K, typename V, bool HAS_V, uint32_t SLOTS>
__device__ __forceinline__ void rest_place(const LongRun<K, V> &run, uint32_t m,
                                           const K (&x)[kRestSlots],
                                           const V (&v)[HAS_V ? kRestSlots : 1])
{
    const uint32_t lane = threadIdx.x % kWave;
    uint32_t before[SLOTS] = {};
#pragma unroll
    for (uint32_t j = 0; j < SLOTS; ++j) {
        const uint32_t end = m > j * kWave ? min(m - j * kWave, (uint32_t)kWave) : 0u;
        for (uint32_t l = 0; l < end; ++l) {
            const K k = read_lane(x[j], l);
#pragma unroll
            for (uint32_t s = 0; s < SLOTS; ++s) {
                // an equal key goes first if it came first
                const bool first = s > j || (s == j && l < lane);
                before[s] += first ? k <= x[s] : k < x[s];
            }
        }
    }
#pragma unroll
    for (uint32_t s = 0; s < SLOTS; ++s) {
        if (s * kWave + lane < m) {
            run.k[before[s]] = map_out(x[s], run.map);
            if constexpr (HAS_V)
                run.v[before[s]] = v[s];
        }
    }
}

template <typename K, typename V, bool HAS_V, typename E, typename Resolve>
__device__ __forceinline__ uint32_t rest_wave_runs(uint32_t *ctrl, E *list, uint32_t list_cap,
                                                   uint32_t len, Resolve &&resolve)
{
    const uint32_t lane = threadIdx.x % kWave;
    uint32_t taken = 0;
    while (true) {
        uint32_t item = 0;
        if (lane == 0)
            item = atomicAdd(&ctrl[kCtrlLongClaim], 1u);
        item = __builtin_amdgcn_readfirstlane(item);
        if (item >= len)
            return taken;
        ++taken;
        const E entry = list[item];
        const LongRun<K, V> run = resolve(entry);
        K x[kRestSlots];
#pragma unroll
        for (uint32_t s = 0; s < kRestSlots; ++s) {
            const uint32_t e = s * kWave + lane;
            x[s] = e < run.n ? run.k[e] : (K)0;
        }
        if (run.map) {
#pragma unroll
            for (uint32_t s = 0; s < kRestSlots; ++s)
                x[s] = map_in(x[s], run.map);
        }
        const K lead = read_lane(x[0], 0) >> run.shift;
        uint32_t m = 0;  // the run's length, as far as it was read
#pragma unroll
        for (uint32_t s = 0; s < kRestSlots; ++s) {
            const uint64_t in =
                __ballot(s * kWave + lane < run.n && (x[s] >> run.shift) == lead);
            if (m == s * kWave)
                m += ~in ? (uint32_t)__builtin_ctzll(~in) : kWave;
        }
        if (m == kRestWaveRun) {
            if (lane == 0)
                list[list_cap - 1 - atomicAdd(&ctrl[kCtrlLongerLen], 1u)] = entry;
            continue;
        }
        V v[HAS_V ? kRestSlots : 1];
        if constexpr (HAS_V) {
#pragma unroll
            for (uint32_t s = 0; s < kRestSlots; ++s)
                v[s] = s * kWave + lane < m ? run.v[s * kWave + lane] : (V)0;
        }
        if (m <= 2 * kWave)
            rest_place<K, V, HAS_V, 2>(run, m, x, v);
        else if (m <= 4 * kWave)
            rest_place<K, V, HAS_V, 4>(run, m, x, v);
        else
            rest_place<K, V, HAS_V, 8>(run, m, x, v);
    }
}

struct RestShared {
    uint32_t item, len, ok, giant, held;
};

// The listed runs, by every workgroup of the launch: waves take the shorter
// ones, then workgroups the longer ones, up to a tile.  A run longer than a
// tile that is out of order is passed to giant(entry), and then, or if there
// are more than `limit` of the longer ones, the result is true: the whole
// array has to be sorted again (every workgroup gets the same answer, and
// sees what the others wrote).
template <typename K, typename V, bool HAS_V, typename C, typename E, typename Resolve,
          typename Giant>
__device__ __forceinline__ bool rest_long_runs(
    BlockLds<K, HAS_V, C::kThreads, C::kItems> &L, RestShared &S, uint32_t *ctrl, E *list,
    uint32_t list_cap, uint32_t limit, const PassArgs &wait, Resolve &&resolve, Giant &&giant)
{
    constexpr uint32_t T = C::kTile;
    constexpr int THREADS = C::kThreads;
    constexpr int ITEMS = C::kItems;
    const uint32_t t = threadIdx.x;
    const uint32_t len = __builtin_amdgcn_readfirstlane(ctrl[kCtrlLongLen]);
    if (len > list_cap)
        return true;
    if (t == 0)
        S.held = 0;
    __syncthreads();
    const uint32_t held = rest_wave_runs<K, V, HAS_V>(ctrl, list, list_cap, len, resolve);
    if (t % kWave == 0 && held)
        atomicAdd(&S.held, held);
    __syncthreads();
    if (t == 0) {
        S.ok = hand_on_and_wait(&ctrl[kCtrlLongDone], S.held, len, wait) ? 1u : 0u;
        S.len = __hip_atomic_load(&ctrl[kCtrlLongerLen], __ATOMIC_RELAXED,
                                  __HIP_MEMORY_SCOPE_AGENT);
    }
    __syncthreads();
    const uint32_t longer = S.len;
    if (!S.ok || longer == 0)
        return false;
    if (t == 0)
        __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "agent");
    if (longer > limit) {
        __syncthreads();
        return true;
    }
    uint32_t mine = 0;
    while (true) {
        __syncthreads();
        if (t == 0) {
            S.item = atomicAdd(&ctrl[kCtrlLongerClaim], 1u);
            S.len = T;
        }
        __syncthreads();
        if (S.item >= longer)
            break;
        ++mine;
        const E entry = list[list_cap - 1 - S.item];
        const LongRun<K, V> run = resolve(entry);
        const K lead = map_in(run.k[0], run.map) >> run.shift;
        uint32_t end = T;
        for (uint32_t e = t; e < T; e += THREADS)
            if (e >= run.n || (map_in(run.k[e], run.map) >> run.shift) != lead)
                end = min(end, e);
        if (end < T)
            atomicMin(&S.len, end);
        __syncthreads();
        const uint32_t m = S.len;
        if (m == T && run.n > T && (map_in(run.k[T], run.map) >> run.shift) == lead) {
            // longer than a tile: only its order is checked here
            bool bad = true;
            for (uint32_t tl = 0; tl < kRestScanTiles; ++tl) {
                bool out = false, ends = false;
                for (uint32_t e = t; e < T; e += THREADS) {
                    const uint64_t i = (uint64_t)tl * T + e;
                    if (i + 1 >= run.n) {
                        ends = true;
                        continue;
                    }
                    const K x = map_in(run.k[i], run.map), y = map_in(run.k[i + 1], run.map);
                    if ((x >> run.shift) != lead)
                        ends = true;
                    else
                        out = out || ((y >> run.shift) == lead && x > y);
                }
                if (__syncthreads_or(out))
                    break;
                if (__syncthreads_or(ends)) {
                    bad = false;
                    break;
                }
            }
            if (bad && t == 0) {
                giant(entry);
                __hip_atomic_store(&ctrl[kCtrlGiant], 1u, __ATOMIC_RELAXED,
                                   __HIP_MEMORY_SCOPE_AGENT);
            }
        } else {
            const BlockItems<THREADS, ITEMS> it(m);
            K key[ITEMS];
            V val[HAS_V ? ITEMS : 1];
            it.each([&](int j) {
                key[j] = it.has(j) ? map_in(run.k[it.at(j)], run.map) : (K)0;
                if constexpr (HAS_V)
                    val[j] = it.has(j) ? run.v[it.at(j)] : (V)0;
            });
            __syncthreads();  // everything is read before it is overwritten
            block_sort_digits<K, V, HAS_V, THREADS, ITEMS>(L, it, key, val, run.digits);
            it.each([&](int j) {
                if (it.has(j)) {
                    run.k[it.at(j)] = map_out(key[j], run.map);
                    if constexpr (HAS_V)
                        run.v[it.at(j)] = val[j];
                }
            });
        }
    }
    __syncthreads();
    if (t == 0) {
        S.ok = hand_on_and_wait(&ctrl[kCtrlLongerDone], mine, longer, wait) ? 1u : 0u;
        S.giant = __hip_atomic_load(&ctrl[kCtrlGiant], __ATOMIC_RELAXED,
                                    __HIP_MEMORY_SCOPE_AGENT);
    }
    __syncthreads();
    if (!S.ok || S.giant == 0)
        return false;
    if (t == 0)
        __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "agent");
    __syncthreads();
    return true;
}

// The next item of stages of `tiles` items each, or false when there is none
// (or a wait reached its bound).  Called by every thread after a barrier that
// ends its last item, which it counts as done (stage_done: one zeroed word
// per stage); an item waits for the stage before its own.
struct RestItem {
    uint32_t stage = 0, tile = 0;
    bool held = false;
};

__device__ __forceinline__ bool rest_next(RestItem &it, RestShared &S, uint32_t *ctrl,
                                          uint32_t *stage_done, uint32_t stages, uint32_t tiles,
                                          const PassArgs &wait)
{
    // One thread reports the last item, claims the next and waits, in one
    // place: with the report at the end of the caller's loop the compiler
    // sends the other threads of its wave to the barrier ahead of it.
    if (threadIdx.x == 0) {
        __builtin_amdgcn_fence(__ATOMIC_RELEASE, "agent");
        if (it.held)
            atomicAdd(&stage_done[it.stage], 1u);
        const uint32_t item = atomicAdd(&ctrl[kCtrlRestClaim], 1u);
        const uint32_t st = item / tiles;
        S.item = item;
        S.ok = st == 0 || st >= stages || wait_count(&stage_done[st - 1], tiles, wait);
        __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "agent");
    }
    __syncthreads();
    it.held = true;
    it.stage = __builtin_amdgcn_readfirstlane(S.item / tiles);
    it.tile = __builtin_amdgcn_readfirstlane(S.item % tiles);
    return it.stage < stages && S.ok != 0;
}

// One launch of persistent workgroups.  Work is claimed in order, (stage,
// tile) after (stage, tile), and an item waits only for the stage before its
// own, whose items are all claimed by running workgroups: no wait depends on
// a workgroup that has not started (nor do those for the long runs: a
// workgroup counts its runs as done before it waits for the others').
// Stages hand their data on through memory within the launch
// (hand_on_and_wait).
template <typename K, typename V, bool HAS_V, typename C>
__global__ __launch_bounds__(C::kThreads) void k_last(LastArgs a)
{
    constexpr uint32_t T = C::kTile;
    constexpr uint32_t NB = C::kBins;
    constexpr int R = C::kRadixBits;
    constexpr int THREADS = C::kThreads;
    static_assert(R == kRadixBits, "8-bit digits");
    using Block = BlockLds<K, HAS_V, THREADS, C::kItems>;
    using Pass = PassLds<K, C, HAS_V>;
    __shared__ union {
        Pass pass;
        Block block;
    } L;
    __shared__ RestShared S;

    uint32_t *ctrl = a.p.ctrl;
    const uint32_t finish = __builtin_amdgcn_readfirstlane(ctrl[kCtrlFinish]);
    if (!(finish & kFinishRun)) {
        pass_slot<K, V, HAS_V, C>(a.p, L.pass);
        return;
    }
    if (ctrl[kCtrlUnsorted] == 0)
        return;
    const uint32_t t = threadIdx.x;
    const uint32_t n = a.p.n;
    const uint32_t buf = (finish >> kFinishDstShift) & 3u;  // where k_finish wrote
    const uint32_t digits = __builtin_amdgcn_readfirstlane(ctrl[kCtrlDigits]);
    const uint32_t skew = __builtin_amdgcn_readfirstlane(ctrl[kCtrlSkew]);
    const uint32_t tiles = a.p.num_tiles;
    // the output holds unmapped keys, the scratch copy mapped ones
    const uint32_t map = buf == kBufOut ? a.p.kmap : 0u;
    const int run_shift = (int)(finish >> kFinishShift);
    K *bk = pick<K>(a.p.b, buf, false);
    V *bv = HAS_V ? pick<V>(a.p.b, buf, true) : nullptr;
    const uint32_t low = digits & ((1u << (run_shift / R)) - 1u);
    // a longer run takes a workgroup about one tile's time per digit below
    // the finish shift: past this many the whole array is sorted again
    if (!rest_long_runs<K, V, HAS_V, C>(
            L.block, S, ctrl, a.list, a.list_cap, max(512u, a.d * tiles), a.p,
            [=](uint32_t start) {
                return LongRun<K, V>{bk + start, HAS_V ? bv + start : nullptr, n - start,
                                     run_shift, low, map};
            },
            [](uint32_t) {}))
        return;

    // again by every digit: one stage that clears the look-back words, then
    // the digits, the lowest one twice if their number is odd, so that the
    // result ends where k_finish wrote (sorting by a digit twice changes
    // nothing)
    const uint32_t q = (uint32_t)__popc(digits);
    const uint32_t sets = q + (q & 1);
    const uint32_t other = buf == kBufOut ? kBufTmp : kBufOut;
    RestItem it;
    while (rest_next(it, S, ctrl, ctrl + kCtrlStageDone, 1 + sets, tiles, a.p)) {
        if (it.stage == 0) {
            for (uint32_t set = 0; set < sets; ++set)
                for (uint32_t i = t; i < NB; i += THREADS)
                    a.status[((uint64_t)set * tiles + it.tile) * NB + i] = 0;
            __syncthreads();
            continue;
        }
        const uint32_t set = it.stage - 1;
        uint32_t left = digits;
        for (uint32_t i = q & 1; i < set; ++i)
            left &= left - 1;
        const uint32_t digit = (uint32_t)__builtin_ctz(left);
        const uint32_t from = set & 1 ? other : buf;
        const uint32_t into = set & 1 ? buf : other;
        const K *sk = pick<const K>(a.p.b, from, false);
        const V *sv = HAS_V ? pick<const V>(a.p.b, from, true) : nullptr;
        const uint32_t tb = it.tile * T;
        const uint32_t dbase = t < NB ? a.p.digit_base[digit * NB + t] : 0u;
        pass_tile<K, V, HAS_V, C>(
            L.pass, sk + tb, HAS_V ? sv + tb : nullptr, pick<K>(a.p.b, into, false),
            HAS_V ? pick<V>(a.p.b, into, true) : nullptr, min(T, n - tb), n, it.tile, 0,
            a.status + (uint64_t)set * tiles * NB, nullptr, dbase, (int)digit * R,
            (skew >> digit) & 1u, set == 0 ? map : 0u, set + 1 == sets ? map : 0u, a.p,
            [](uint32_t) {});
    }
}

// ---------------------------------------------------------------------------
// The same for the large segments of a segmented sort, each with its own
// finish shift (k_seg_scan).  2000 segments of 2^4 to 2^20 32-bit pairs: four
// passes of 738 us each before, two and a sweep of 1020 us now; 24 of 2^10 to
// 2^22 64-bit pairs: eight passes of 62 us, now three and a sweep of 50 us.
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
    uint2 *list;        // long runs: start within the segment, segment
    uint32_t list_cap;
    uint32_t kmap;
    int in_place;
};

template <typename K, typename V, bool HAS_V, int THREADS, int ITEMS>
__global__ __launch_bounds__(THREADS) void k_seg_finish(SegFinishArgs a)
{
    constexpr uint32_t T = THREADS * ITEMS;
    __shared__ FinishLds<K, THREADS, ITEMS> L;
    if (!(a.ctrl[kSegPassMask] & kSegAnyFinish))
        return;
    uint32_t *ctrl = a.ctrl;
    uint2 *list = a.list;
    const uint32_t cap = a.list_cap;
    const uint32_t tiles = std::min(ctrl[kSegTiles], a.max_tiles);
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
        for (uint32_t g = 0; g < a.group && tb < size; ++g, tb += T)
            finish_tile<K, V, HAS_V, THREADS, ITEMS>(
                L, sk, sv, dk, dv, size, tb, (int)(m.low * kRadixBits),
                dst == kBufOut ? a.kmap : 0u, &ctrl[kCtrlUnsorted], [=](uint32_t i) {
                    const uint32_t l = atomicAdd(&ctrl[kCtrlLongLen], 1u);
                    if (l < cap)
                        list[l] = make_uint2(i, seg);
                });
    }
}

struct SegLastArgs {
    SegPassArgs p;  // status: the look-back words of every pass
    uint64_t status_stride;
    uint2 *list;
    uint32_t list_cap;
};

template <typename K, typename V, bool HAS_V, typename C>
__global__ __launch_bounds__(C::kThreads) void k_seg_last(SegLastArgs a)
{
    constexpr uint32_t T = C::kTile;
    constexpr uint32_t NB = C::kBins;
    constexpr int R = C::kRadixBits;
    constexpr int D = num_passes<K, R>();
    constexpr int THREADS = C::kThreads;
    static_assert(R == kRadixBits && D % 2 == 0, "8-bit digits");
    __shared__ union {
        PassLds<K, C, HAS_V> pass;
        BlockLds<K, HAS_V, THREADS, C::kItems> block;
    } L;
    __shared__ RestShared S;
    uint32_t *ctrl = a.p.ctrl;
    if (ctrl[kCtrlUnsorted] == 0)
        return;
    const uint32_t t = threadIdx.x;
    const bool in_place = a.p.keys_in_place || a.p.vals_in_place;
    const uint32_t tiles = std::min(ctrl[kSegTiles], a.p.max_tiles);
    const SegLarge *large = a.p.large;
    uint32_t *seg_flags = a.p.seg_flags;
    const Bufs b = a.p.b;
    const uint32_t kmap = a.p.kmap;
    PassArgs wait{};
    wait.err = ctrl + kSegError;
    wait.spin_limit = a.p.spin_limit;
    wait.stall = a.p.stall;
    if (!rest_long_runs<K, V, HAS_V, C>(
            L.block, S, ctrl, a.list, a.list_cap, ~0u, wait,
            [=](uint2 entry) {
                const SegLarge rec = large[entry.y];
                const uint32_t flags = seg_flags[entry.y];
                const SegMoves m = seg_moves<K, R>(flags, in_place);
                const uint32_t buf = m.dst(m.moves - 1);
                const uint64_t at = rec.start + entry.x;
                return LongRun<K, V>{
                    pick<K>(b, buf, false) + at,
                    HAS_V ? pick<V>(b, buf, true) + at : nullptr,
                    (uint32_t)__builtin_amdgcn_readfirstlane(rec.size - entry.x),
                    (int)__builtin_amdgcn_readfirstlane(m.low * R),
                    (uint32_t)__builtin_amdgcn_readfirstlane(~flags & ((1u << m.low) - 1u)),
                    buf == kBufOut ? kmap : 0u};
            },
            [=](uint2 entry) { atomicOr(&seg_flags[entry.y], kSegGiant); }))
        return;

    // segments with a giant run: again by every digit, as in k_last
    RestItem it;
    while (rest_next(it, S, ctrl, ctrl + kSegStageDone, 1 + D, tiles, wait)) {
        const uint32_t seg = a.p.tile_seg[it.tile];
        const SegLarge rec = large[seg];
        const uint32_t flags = __builtin_amdgcn_readfirstlane(__hip_atomic_load(
            &seg_flags[seg], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT));
        const SegMoves m = seg_moves<K, R>(flags, in_place);
        const uint32_t digits = ~flags & ((1u << D) - 1u);
        const uint32_t q = (uint32_t)__popc(digits);
        const uint32_t sets = q + (q & 1);
        if (!(flags & kSegGiant) || it.stage > sets) {
            __syncthreads();
            continue;
        }
        if (it.stage == 0) {
            for (uint32_t set = 0; set < sets; ++set)
                for (uint32_t i = t; i < NB; i += THREADS)
                    a.p.status[set * a.status_stride + (uint64_t)it.tile * NB + i] = 0;
            __syncthreads();
            continue;
        }
        const uint32_t set = it.stage - 1;
        uint32_t left = digits;
        for (uint32_t i = q & 1; i < set; ++i)
            left &= left - 1;
        const uint32_t digit = (uint32_t)__builtin_ctz(left);
        const uint32_t buf = m.dst(m.moves - 1);
        const uint32_t other = buf == kBufOut ? kBufTmp : kBufOut;
        const uint32_t from = set & 1 ? other : buf, into = set & 1 ? buf : other;
        const uint32_t map = buf == kBufOut ? kmap : 0u;
        const uint32_t first = (it.tile - rec.tile_start) * T;
        const uint32_t valid = rec.size > first ? min(T, rec.size - first) : 0u;
        const uint64_t off = rec.start + first;
        const uint32_t dbase =
            t < NB ? a.p.seg_base[((uint64_t)seg * D + digit) * NB + t] : 0u;
        pass_tile<K, V, HAS_V, C>(
            L.pass, pick<const K>(b, from, false) + off,
            HAS_V ? pick<const V>(b, from, true) + off : nullptr,
            pick<K>(b, into, false) + rec.start,
            HAS_V ? pick<V>(b, into, true) + rec.start : nullptr, valid, rec.size, it.tile,
            rec.tile_start, a.p.status + set * a.status_stride, nullptr, dbase, (int)digit * R,
            ((flags >> (kSegSkewShift + digit)) & 1u) != 0, set == 0 ? map : 0u,
            set + 1 == sets ? map : 0u, wait, [](uint32_t) {});
    }
}

}  // namespace rs
