// Host-side tables of the compiled digit-pass configurations.  Each entry
// enqueues the kernels of one configuration (digit width, tile shape); the
// entries follow the order of the lists in rs_configs.h.  The kernels are
// instantiated in four translation units (32/64-bit keys x plain/segmented)
// that compile in parallel.
#pragma once

#include "rs_finish.h"
#include "rs_kernels.h"

namespace rs {

struct SortOps {
    int r;        // digit bits
    int threads;  // workgroup size of the digit pass
    int items;    // elements per thread
    int tile;     // threads x items
    int d;        // digit passes
    void (*hist)(const HistArgs &, uint32_t grid, hipStream_t);
    void (*plan)(const PlanArgs &, hipStream_t);
    void (*pass)(const PassArgs &, uint32_t grid, hipStream_t);
    const void *pass_kernel;  // for occupancy queries
    // 8-bit digits only (null otherwise): the end of a sort whose passes stop
    // at a high digit position (rs_finish.h)
    void (*finish)(const FinishArgs &, uint32_t grid, hipStream_t);
    void (*pass_finish)(const PassFinishArgs &, uint32_t grid, hipStream_t);
    void (*last)(const LastArgs &, uint32_t grid, hipStream_t);
    const void *finish_kernel, *pass_finish_kernel;
};

struct SegOps {
    int r, threads, items, tile, d;
    void (*hist)(const SegHistArgs &, uint32_t grid, hipStream_t);
    void (*scan)(const SegHistArgs &, uint32_t grid, hipStream_t);
    void (*pass)(const SegPassArgs &, uint32_t grid, hipStream_t);
    void (*copy)(const SegCopyArgs &, uint32_t grid, hipStream_t);
    const void *hist_kernel, *scan_kernel, *pass_kernel;
    // 8-bit digits only (null otherwise), as SortOps
    void (*finish)(const SegFinishArgs &, uint32_t grid, hipStream_t);
    void (*last)(const SegLastArgs &, uint32_t grid, hipStream_t);
    const void *finish_kernel;
};

// Tables of the plain and segmented sorts for 32- and 64-bit keys.
const SortOps *sort_ops_u32(bool has_values, int *count);
const SortOps *sort_ops_u64(bool has_values, int *count);
const SegOps *seg_ops_u32(bool has_values, int *count);
const SegOps *seg_ops_u64(bool has_values, int *count);

template <typename K, bool HAS_V, int R, int THREADS, int ITEMS>
struct SortLaunch {
    using C = PassCfg<R, THREADS, ITEMS>;
    static void hist(const HistArgs &a, uint32_t grid, hipStream_t s)
    {
        hipLaunchKernelGGL((k_hist<K, R>), dim3(grid), dim3(kHistThreads), 0, s, a);
    }
    static void plan(const PlanArgs &a, hipStream_t s)
    {
        hipLaunchKernelGGL((k_plan<K, R>), dim3(1), dim3(kRadix * plan_groups<K, R>()), 0, s, a);
    }
    static void pass(const PassArgs &a, uint32_t grid, hipStream_t s)
    {
        hipLaunchKernelGGL((k_pass<K, K, HAS_V, C>), dim3(grid), dim3(THREADS), 0, s, a);
    }
    static void finish(const FinishArgs &a, uint32_t grid, hipStream_t s)
    {
        hipLaunchKernelGGL((k_finish<K, K, HAS_V, kFinishThreads, kFinishItems>), dim3(grid),
                           dim3(kFinishThreads), 0, s, a);
    }
    static void pass_finish(const PassFinishArgs &a, uint32_t grid, hipStream_t s)
    {
        hipLaunchKernelGGL((k_pass_finish<K, K, HAS_V, C>), dim3(grid), dim3(THREADS), 0, s, a);
    }
    static void last(const LastArgs &a, uint32_t grid, hipStream_t s)
    {
        hipLaunchKernelGGL((k_last<K, K, HAS_V, C>), dim3(grid), dim3(THREADS), 0, s, a);
    }
    static SortOps ops()
    {
        SortOps o{R, THREADS, ITEMS, C::kTile, num_passes<K, R>(), &hist, &plan, &pass,
                  (const void *)k_pass<K, K, HAS_V, C>, nullptr, nullptr, nullptr, nullptr, nullptr};
        if constexpr (R == kRadixBits) {
            o.finish = &finish;
            o.pass_finish = &pass_finish;
            o.pass_finish_kernel = (const void *)k_pass_finish<K, K, HAS_V, C>;
            o.last = &last;
            o.finish_kernel = (const void *)k_finish<K, K, HAS_V, kFinishThreads, kFinishItems>;
        }
        return o;
    }
};

template <typename K, bool HAS_V, int R, int THREADS, int ITEMS>
struct SegLaunch {
    using C = PassCfg<R, THREADS, ITEMS>;
    static void hist(const SegHistArgs &a, uint32_t grid, hipStream_t s)
    {
        hipLaunchKernelGGL((k_seg_hist<K, R>), dim3(grid), dim3(kSegHistThreads), 0, s, a);
    }
    static void scan(const SegHistArgs &a, uint32_t grid, hipStream_t s)
    {
        hipLaunchKernelGGL((k_seg_scan<K, R>), dim3(grid), dim3(256), 0, s, a);
    }
    static void pass(const SegPassArgs &a, uint32_t grid, hipStream_t s)
    {
        hipLaunchKernelGGL((k_seg_pass<K, K, HAS_V, C>), dim3(grid), dim3(THREADS), 0, s, a);
    }
    static void copy(const SegCopyArgs &a, uint32_t grid, hipStream_t s)
    {
        hipLaunchKernelGGL((k_seg_copy<K, HAS_V, R>), dim3(grid), dim3(256), 0, s, a);
    }
    static void finish(const SegFinishArgs &a, uint32_t grid, hipStream_t s)
    {
        hipLaunchKernelGGL((k_seg_finish<K, K, HAS_V, kFinishThreads, kFinishItems>), dim3(grid),
                           dim3(kFinishThreads), 0, s, a);
    }
    static void last(const SegLastArgs &a, uint32_t grid, hipStream_t s)
    {
        hipLaunchKernelGGL((k_seg_last<K, K, HAS_V, C>), dim3(grid), dim3(THREADS), 0, s, a);
    }
    static SegOps ops()
    {
        SegOps o{R,
                 THREADS,
                 ITEMS,
                 C::kTile,
                 num_passes<K, R>(),
                 &hist,
                 &scan,
                 &pass,
                 &copy,
                 (const void *)k_seg_hist<K, R>,
                 (const void *)k_seg_scan<K, R>,
                 (const void *)k_seg_pass<K, K, HAS_V, C>,
                 nullptr,
                 nullptr,
                 nullptr};
        static_assert(C::kTile % (kFinishThreads * kFinishItems) == 0, "whole sweep tiles");
        if constexpr (R == kRadixBits) {
            o.finish = &finish;
            o.last = &last;
            o.finish_kernel =
                (const void *)k_seg_finish<K, K, HAS_V, kFinishThreads, kFinishItems>;
        }
        return o;
    }
};

}  // namespace rs
