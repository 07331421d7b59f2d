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
// sorts of up to kFinishSmall elements take smaller tiles, so that every
// compute unit has one
constexpr int kFinishItemsSmall = 2;
constexpr uint32_t kFinishSmall = 1u << 19;

// Workgroups loop over tiles of THREADS x ITEMS elements; a tile's keys and
// the chunk before and after it are held in LDS.  A chunk is the 64 elements
// of one wave's item; its head word is a ballot, and run_move orders the
// chunk's elements with it and its neighbours' (rs_runs.h).
//
// Counting over each element's own run, found from the head words by every
// lane, was slower: its reads depended on the run bounds, and 64-bit shifts
// per lane cost more than the count (2^25 64-bit keys, runs of 2: 137 us, now
// 119 us, 4.5 TB/s; 2^20 32-bit keys, runs of 16: 17.8 us, now 12.0 us).  It
// is bound by the compares (VALU) for runs of 4 and more, by HBM below.
template <typename K, typename V, bool HAS_V, int THREADS, int ITEMS>
__global__ __launch_bounds__(THREADS) void k_finish(FinishArgs a)
{
    constexpr uint32_t T = THREADS * ITEMS;
    constexpr uint32_t H = kWave;  // elements held on either side
    constexpr int W = THREADS / kWave;
    __shared__ K s_k[T + 2 * H];
    // per wave: the head words of its first and last chunk; then those of the
    // chunks before and after the tile.  Below them the same for the words of
    // adjacent elements out of order.
    __shared__ uint64_t s_head[2 * W + 2], s_inv[2 * W + 2];

    const uint32_t word = __builtin_amdgcn_readfirstlane(a.ctrl[kCtrlFinish]);
    if (!(word & kFinishRun))
        return;
    const uint32_t src = (word >> kFinishSrcShift) & 3u;
    const uint32_t dst = (word >> kFinishDstShift) & 3u;
    const int shift = (int)(word >> kFinishShift);
    const uint32_t map = dst == kBufOut ? a.kmap : 0u;
    const K *sk = pick<const K>(a.b, src, false);
    const V *sv = HAS_V ? pick<const V>(a.b, src, true) : nullptr;
    K *dk = pick<K>(a.b, dst, false);
    V *dv = HAS_V ? pick<V>(a.b, dst, true) : nullptr;
    const uint32_t n = a.n;
    const uint32_t t = threadIdx.x;
    const uint32_t lane = t % kWave;
    const uint32_t w = __builtin_amdgcn_readfirstlane(t / kWave);
    const uint32_t tiles = (n + T - 1) / T;

    for (uint32_t tile = blockIdx.x; tile < tiles; tile += gridDim.x) {
        const uint32_t tb = tile * T;
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
            s_k[lane] = tile > 0 ? sk[tb - H + lane] : (K)0;
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
                        __hip_atomic_store(&a.ctrl[kCtrlUnsorted], 1u, __ATOMIC_RELAXED,
                                           __HIP_MEMORY_SCOPE_AGENT);
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
                if (lane == kWave - 1 - ends && i < n) {
                    const uint32_t l = atomicAdd(&a.ctrl[kCtrlLongLen], 1u);
                    if (l < a.list_cap)
                        a.list[l] = i;
                }
            }
        }
        __syncthreads();  // the next tile overwrites the LDS
    }
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

// Runs of up to kRestWaveRun elements are sorted by a wave each, in
// registers: every element counts the run's elements that go before it, the
// run's keys broadcast one after another.  Longer ones are listed again,
// from the list's end.  Returns how many runs this wave took.
constexpr uint32_t kRestSlots = 8;
constexpr uint32_t kRestWaveRun = kRestSlots * kWave;

// Writes a run of m <= 64 SLOTS elements, in registers (element s*64 + lane
// in slot s), back in order.
template <typename K, typename V, bool HAS_V, uint32_t SLOTS>
__device__ __forceinline__ void rest_place(K *bk, V *bv, uint32_t start, uint32_t m,
                                           const K (&x)[kRestSlots],
                                           const V (&v)[HAS_V ? kRestSlots : 1], uint32_t map)
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
            bk[start + before[s]] = map_out(x[s], map);
            if constexpr (HAS_V)
                bv[start + before[s]] = v[s];
        }
    }
}

template <typename K, typename V, bool HAS_V>
__device__ __forceinline__ uint32_t rest_wave_runs(const LastArgs &a, K *bk, V *bv, uint32_t len,
                                                   int shift, uint32_t map)
{
    const uint32_t n = a.p.n;
    const uint32_t lane = threadIdx.x % kWave;
    uint32_t taken = 0;
    while (true) {
        uint32_t item = 0;
        if (lane == 0)
            item = atomicAdd(&a.p.ctrl[kCtrlLongClaim], 1u);
        item = __builtin_amdgcn_readfirstlane(item);
        if (item >= len)
            return taken;
        ++taken;
        const uint32_t start = __builtin_amdgcn_readfirstlane(a.list[item]);
        K x[kRestSlots];
#pragma unroll
        for (uint32_t s = 0; s < kRestSlots; ++s) {
            const uint32_t e = s * kWave + lane;
            x[s] = e < n - start ? bk[start + e] : (K)0;
        }
        if (map) {
#pragma unroll
            for (uint32_t s = 0; s < kRestSlots; ++s)
                x[s] = map_in(x[s], map);
        }
        const K lead = read_lane(x[0], 0) >> shift;
        uint32_t m = 0;  // the run's length, as far as it was read
#pragma unroll
        for (uint32_t s = 0; s < kRestSlots; ++s) {
            const uint64_t in = __ballot(s * kWave + lane < n - start && (x[s] >> shift) == lead);
            if (m == s * kWave)
                m += ~in ? (uint32_t)__builtin_ctzll(~in) : kWave;
        }
        if (m == kRestWaveRun) {
            if (lane == 0) {
                const uint32_t l = atomicAdd(&a.p.ctrl[kCtrlLongerLen], 1u);
                a.list[a.list_cap - 1 - l] = start;
            }
            continue;
        }
        V v[HAS_V ? kRestSlots : 1];
        if constexpr (HAS_V) {
#pragma unroll
            for (uint32_t s = 0; s < kRestSlots; ++s)
                v[s] = s * kWave + lane < m ? bv[start + s * kWave + lane] : (V)0;
        }
        if (m <= 2 * kWave)
            rest_place<K, V, HAS_V, 2>(bk, bv, start, m, x, v, map);
        else if (m <= 4 * kWave)
            rest_place<K, V, HAS_V, 4>(bk, bv, start, m, x, v, map);
        else
            rest_place<K, V, HAS_V, 8>(bk, bv, start, m, x, v, map);
    }
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
    constexpr int ITEMS = C::kItems;
    static_assert(R == kRadixBits, "8-bit digits");
    using Block = BlockLds<K, HAS_V, THREADS, ITEMS>;
    using Pass = PassLds<K, C, HAS_V>;
    __shared__ union {
        Pass pass;
        Block block;
    } L;
    __shared__ uint32_t s_item, s_len, s_ok, s_giant, s_held;

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

    {
        const uint32_t len = __builtin_amdgcn_readfirstlane(ctrl[kCtrlLongLen]);
        const int shift = (int)(finish >> kFinishShift);
        K *bk = pick<K>(a.p.b, buf, false);
        V *bv = HAS_V ? pick<V>(a.p.b, buf, true) : nullptr;
        if (len <= a.list_cap) {
            if (t == 0)
                s_held = 0;
            __syncthreads();
            const uint32_t held = rest_wave_runs<K, V, HAS_V>(a, bk, bv, len, shift, map);
            if (t % kWave == 0 && held)
                atomicAdd(&s_held, held);
            __syncthreads();
            if (t == 0) {
                s_ok = hand_on_and_wait(&ctrl[kCtrlLongDone], s_held, len, a.p) ? 1u : 0u;
                s_len = __hip_atomic_load(&ctrl[kCtrlLongerLen], __ATOMIC_RELAXED,
                                          __HIP_MEMORY_SCOPE_AGENT);
            }
            __syncthreads();
            const uint32_t longer = s_len;
            if (!s_ok || longer == 0)
                return;
            if (t == 0)
                __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "agent");
            // a run takes a workgroup about one tile's time per digit below the
            // finish shift: past this many the whole array is sorted again
            if (longer <= max(512u, a.d * tiles)) {
                const uint32_t low = digits & ((1u << (shift / R)) - 1u);
                uint32_t mine = 0;
                while (true) {
                    __syncthreads();
                    if (t == 0) {
                        s_item = atomicAdd(&ctrl[kCtrlLongerClaim], 1u);
                        s_len = T;
                    }
                    __syncthreads();
                    if (s_item >= longer)
                        break;
                    ++mine;
                    const uint32_t start = a.list[a.list_cap - 1 - s_item];
                    const K lead = map_in(bk[start], map) >> shift;
                    uint32_t end = T;
                    for (uint32_t e = t; e < T; e += THREADS)
                        if (e >= n - start || (map_in(bk[start + e], map) >> shift) != lead)
                            end = min(end, e);
                    if (end < T)
                        atomicMin(&s_len, end);
                    __syncthreads();
                    const uint32_t m = s_len;
                    if (m == T && n - start > T && (map_in(bk[start + T], map) >> shift) == lead) {
                        // longer than a tile: only its order is checked here
                        bool bad = true;
                        for (uint32_t tl = 0; tl < kRestScanTiles; ++tl) {
                            bool out = false, ends = false;
                            for (uint32_t e = t; e < T; e += THREADS) {
                                const uint64_t i = (uint64_t)start + (uint64_t)tl * T + e;
                                if (i + 1 >= n) {
                                    ends = true;
                                    continue;
                                }
                                const K x = map_in(bk[i], map), y = map_in(bk[i + 1], map);
                                if ((x >> shift) != lead)
                                    ends = true;
                                else
                                    out = out || ((y >> shift) == lead && x > y);
                            }
                            if (__syncthreads_or(out))
                                break;
                            if (__syncthreads_or(ends)) {
                                bad = false;
                                break;
                            }
                        }
                        if (bad && t == 0)
                            __hip_atomic_store(&ctrl[kCtrlGiant], 1u, __ATOMIC_RELAXED,
                                               __HIP_MEMORY_SCOPE_AGENT);
                    } else {
                        const BlockItems<THREADS, ITEMS> it(m);
                        K key[ITEMS];
                        V val[HAS_V ? ITEMS : 1];
                        it.each([&](int j) {
                            key[j] = it.has(j) ? map_in(bk[start + it.at(j)], map) : (K)0;
                            if constexpr (HAS_V)
                                val[j] = it.has(j) ? bv[start + it.at(j)] : (V)0;
                        });
                        __syncthreads();  // everything is read before it is overwritten
                        block_sort_digits<K, V, HAS_V, THREADS, ITEMS>(L.block, it, key, val, low);
                        it.each([&](int j) {
                            if (it.has(j)) {
                                bk[start + it.at(j)] = map_out(key[j], map);
                                if constexpr (HAS_V)
                                    bv[start + it.at(j)] = val[j];
                            }
                        });
                    }
                }
                __syncthreads();
                if (t == 0) {
                    s_ok = hand_on_and_wait(&ctrl[kCtrlLongerDone], mine, longer, a.p) ? 1u : 0u;
                    s_giant = __hip_atomic_load(&ctrl[kCtrlGiant], __ATOMIC_RELAXED,
                                                __HIP_MEMORY_SCOPE_AGENT);
                }
                __syncthreads();
                if (!s_ok || s_giant == 0)
                    return;
                if (t == 0)
                    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "agent");
                __syncthreads();
            }
        }
    }

    // again by every digit: one stage that clears the look-back words, then
    // the digits, the lowest one twice if their number is odd, so that the
    // result ends where k_finish wrote (sorting by a digit twice changes
    // nothing)
    const uint32_t q = (uint32_t)__popc(digits);
    const uint32_t sets = q + (q & 1);
    const uint32_t stages = 1 + sets;
    const uint32_t other = buf == kBufOut ? kBufTmp : kBufOut;
    // One thread reports an item done, claims the next and waits for the
    // stage before it in one place: with the report at the loop's end the
    // compiler sends the other threads of its wave to the barrier ahead of it.
    uint32_t held = 0, stage = 0;
    while (true) {
        if (t == 0) {
            __builtin_amdgcn_fence(__ATOMIC_RELEASE, "agent");
            if (held)
                atomicAdd(&ctrl[kCtrlStageDone + stage], 1u);
            const uint32_t item = atomicAdd(&ctrl[kCtrlRestClaim], 1u);
            const uint32_t st = item / tiles;
            s_item = item;
            s_ok = st == 0 || st >= stages ||
                   wait_count(&ctrl[kCtrlStageDone + st - 1], tiles, a.p);
            __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "agent");
        }
        held = 1;
        __syncthreads();
        stage = s_item / tiles;
        const uint32_t tile = s_item % tiles;
        if (stage >= stages || !s_ok)
            break;
        if (stage == 0) {
            for (uint32_t set = 0; set < sets; ++set)
                for (uint32_t i = t; i < NB; i += THREADS)
                    a.status[((uint64_t)set * tiles + tile) * NB + i] = 0;
            __syncthreads();
        } else {
            const uint32_t set = stage - 1;
            uint32_t left = digits;
            for (uint32_t i = q & 1; i < set; ++i)
                left &= left - 1;
            uint32_t digit = (uint32_t)__builtin_ctz(left);
            const uint32_t from = set & 1 ? other : buf;
            const uint32_t into = set & 1 ? buf : other;
            const uint32_t map_load = set == 0 ? map : 0u;
            const uint32_t map_store = stage == stages - 1 ? map : 0u;
            const bool ballot = (skew >> digit) & 1u;
            digit = __builtin_amdgcn_readfirstlane(digit);
            const K *sk = pick<const K>(a.p.b, from, false);
            const V *sv = HAS_V ? pick<const V>(a.p.b, from, true) : nullptr;
            const uint32_t tb = tile * T;
            const uint32_t dbase = t < NB ? a.p.digit_base[digit * NB + t] : 0u;
            pass_tile<K, V, HAS_V, C>(
                L.pass, sk + tb, HAS_V ? sv + tb : nullptr, pick<K>(a.p.b, into, false),
                HAS_V ? pick<V>(a.p.b, into, true) : nullptr, min(T, n - tb), n, tile, 0,
                a.status + (uint64_t)set * tiles * NB, nullptr, dbase, (int)digit * R, ballot,
                map_load, map_store, a.p, [](uint32_t) {});
        }
    }
}

}  // namespace rs
