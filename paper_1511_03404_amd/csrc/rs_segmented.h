// Batched segmented sort: many independent stable LSD radix sorts (paper,
// Section 2.6) of uneven sizes in one enqueue, classified on the device:
//   * size 0 or 1           -- nothing to sort (a single element is copied);
//   * size <= tiny cap      -- one wave sorts it: up to 64 elements with a
//                              bitonic network on (key, position) pairs
//                              (Section 2.1), more with an LDS radix sort
//                              (k_seg_bitonic in rs_bitonic.h; the cap is a
//                              context setting, 0 turns the class off);
//   * size <= small cap     -- one workgroup sorts it in LDS (k_block_sort,
//                              small shape, several workgroups per CU);
//   * size <= medium cap    -- the same with the medium shape;
//   * larger                -- per-segment digit histograms (k_seg_hist) and
//                              plans (k_seg_scan), then one digit-pass launch
//                              per digit over the tiles of all large segments
//                              (k_seg_pass, in rs_kernels.h), each segment
//                              with its own look-back chain and moving only in
//                              the passes of its plan, then the sweep that
//                              orders the short runs left (rs_finish.h).
// Only device counters decide the work, so the sequence is graph-capturable
// and needs no host round trip.
#pragma once

#include "rs.h"
#include "rs_block.h"
#include "rs_device.h"

namespace rs {

using SegLarge = SegRange;

// Per-XCD claim counters (XCC_ID has 3 bits; gfx950 has 8 XCDs).
constexpr uint32_t kXcdSlots = 8;

// Segmented control block (u32 words).
constexpr int kSegSmallLen = 0;
constexpr int kSegMediumLen = 1;
constexpr int kSegLargeLen = 2;
constexpr int kSegTiles = 3;
constexpr int kSegSmallClaim = 4;
constexpr int kSegMediumClaim = 5;
constexpr int kSegHistClaim = 6;
constexpr int kSegError = kCtrlError;  // kErrSegTooLarge, kErrSegTiles, kErrWait
constexpr int kSegTinyLen = 8;
constexpr int kSegTinyClaim = 9;
constexpr int kSegPassCounter = 32; // [32, 48): group counter per pass
constexpr int kSegChunks = 16;      // histogram chunks of the large segments
constexpr int kSegChunkClaim = 17;
constexpr int kSegPassMask = 49;    // passes in which a segment moves, kSegAnyFinish
constexpr int kSegWords = 64;       // (k_seg_finish and k_seg_last: the words of the plain
                                    // sort's control block from kCtrlUnsorted on)
// Large segments are histogrammed in chunks of this many elements, so that
// one huge segment does not leave a single workgroup reading it alone: at
// most 2^18 (a chunk's end adds its counts to memory), fewer when the batch
// would make less than two chunks per compute unit (7.2M 64-bit elements in
// 24 segments: 74 us with 2^18, 27 us with 2^14).
constexpr uint32_t kSegChunkMax = 1u << 18;
constexpr uint32_t kSegChunkMin = 1u << 14;
inline uint32_t seg_chunk(uint64_t total)
{
    uint32_t c = kSegChunkMax;
    while (c > kSegChunkMin && total / c < 512)
        c /= 2;
    return c;
}

struct SegClassifyArgs {
    const uint64_t *offsets;
    uint32_t num_segments;
    uint64_t total;
    uint32_t max_tiles;
    uint32_t *ctrl;
    SegRange *tiny_list;
    SegRange *small_list;
    SegRange *medium_list;
    SegLarge *large;
    uint32_t *tile_seg;
    uint32_t *chunk_seg;  // large segment of each histogram chunk
    uint32_t max_chunks;
    uint32_t *first_chunk;  // of each large segment (read by k_seg_hist)
    const void *kin;
    const void *vin;
    void *kout;
    void *vout;
    uint32_t tiny_cap;  // 0: no tiny class
    uint32_t small_cap;
    uint32_t medium_cap;
    uint32_t tile;
    uint32_t chunk;  // elements per histogram chunk
};

template <typename K, bool HAS_V>
__global__ __launch_bounds__(256) void k_seg_classify(SegClassifyArgs a)
{
    const uint32_t stride = gridDim.x * blockDim.x;
    const uint32_t lane = threadIdx.x % kWave;
    // whole waves go round, so that all lanes can fill a large segment's maps
    const uint32_t first = blockIdx.x * blockDim.x + threadIdx.x;
    for (uint32_t s = first; s - lane < a.num_segments; s += stride) {
        // clamp to [0, total): a malformed offsets array sorts garbage
        // ranges but never leaves the arrays
        uint64_t start = 0, size = 0;
        if (s < a.num_segments) {
            start = std::min<uint64_t>(a.offsets[s], a.total);
            size = std::min<uint64_t>(std::max<uint64_t>(a.offsets[s + 1], start), a.total) - start;
        }
        uint32_t idx = 0, nt = 0, ts = 0, nc = 0, cs = 0;
        if (size == 0) {
        } else if (size == 1) {
            ((K *)a.kout)[start] = ((const K *)a.kin)[start];
            if constexpr (HAS_V)
                ((K *)a.vout)[start] = ((const K *)a.vin)[start];
        } else if (size <= a.tiny_cap) {
            a.tiny_list[atomicAdd(&a.ctrl[kSegTinyLen], 1u)] = SegRange{start, (uint32_t)size, 0};
        } else if (size <= a.small_cap) {
            a.small_list[atomicAdd(&a.ctrl[kSegSmallLen], 1u)] = SegRange{start, (uint32_t)size, 0};
        } else if (size <= a.medium_cap) {
            a.medium_list[atomicAdd(&a.ctrl[kSegMediumLen], 1u)] = SegRange{start, (uint32_t)size, 0};
        } else if (size >= RS_MAX_ELEMENTS) {
            atomicOr(&a.ctrl[kSegError], kErrSegTooLarge);
        } else {
            idx = atomicAdd(&a.ctrl[kSegLargeLen], 1u);
            nt = (uint32_t)((size + a.tile - 1) / a.tile);
            ts = atomicAdd(&a.ctrl[kSegTiles], nt);
            // overlapping segments can need more tiles than the workspace
            // holds: such a segment keeps its tiles but sorts nothing
            const bool fits = (uint64_t)ts + nt <= a.max_tiles;
            if (!fits)
                atomicOr(&a.ctrl[kSegError], kErrSegTiles);
            a.large[idx] = SegLarge{start, fits ? (uint32_t)size : 0u, ts};
            nc = (uint32_t)((size + a.chunk - 1) / a.chunk);
            cs = atomicAdd(&a.ctrl[kSegChunks], nc);
            a.first_chunk[idx] = cs;
        }
        // the wave fills the maps of its large segments, one after another
        for (uint64_t left = __ballot(nt != 0); left; left &= left - 1) {
            const int l = __builtin_ctzll(left);
            const uint32_t i = __shfl(idx, l), n = __shfl(nt, l), t0 = __shfl(ts, l);
            const uint32_t m = __shfl(nc, l), c0 = __shfl(cs, l);
            for (uint32_t j = lane; j < n && t0 + j < a.max_tiles; j += kWave)
                a.tile_seg[t0 + j] = i;
            for (uint32_t j = lane; j < m && c0 + j < a.max_chunks; j += kWave)
                a.chunk_seg[c0 + j] = i;
        }
    }
}

}  // namespace rs
