// The list builder of the scheduler (see va_sched.hip), for one workgroup of THREADS threads: shared by the scheduler
// kernel and by the dQ launch of a small backward, which carries the builders of its own lists along.
#pragma once
#include "va_device.h"
#include "va_internal.h"

namespace va {

// Exclusive scan of one value per thread over the block; returns the exclusive prefix and
// writes the block total to *total.  `buf` holds one int per wave.
// Inside a wave the scan runs on lane shuffles; the wave totals meet in LDS (two barriers in all, where a
// scan through LDS alone takes twenty: at a few thousand samples the scans were most of this kernel's time).
template <int THREADS>
__device__ int block_exclusive_scan(int v, int* buf, int* total) {
    const int t = threadIdx.x, lane = t & 63, wave = t >> 6;
    int incl = v;
#pragma unroll
    for (int d = 1; d < 64; d <<= 1) {
        const int up = __shfl_up(incl, d, 64);
        if (lane >= d) incl += up;
    }
    if (lane == 63) buf[wave] = incl;
    __syncthreads();
    int before = 0, all = 0;
#pragma unroll
    for (int w = 0; w < THREADS / 64; ++w) {
        const int x = buf[w];
        before += w < wave ? x : 0;
        all += x;
    }
    *total = all;
    __syncthreads();  // buf may be refilled by the next scan
    return before + incl - v;
}

struct SchedJob {  // one work list
    int R, U, mode, max_items;
    int32_t *hdr, *tile_off;
    WorkItem* items;
};
inline SchedJob sched_job(int tile_rows, int partner_rows, CostMode mode, void* ws, const SchedLayout& lay) {
    char* base = (char*)ws;
    return SchedJob{tile_rows, partner_rows, (int)mode, (int)lay.max_items, (int32_t*)base,
                    (int32_t*)(base + lay.tile_off_ofs), (WorkItem*)(base + lay.items_ofs)};
}

// LDS of a builder.  CACHE: samples whose clamped bounds and tile offsets are kept here (3 x 4 bytes each).  A batch
// with up to three times as many keeps the tile offsets here, which is what the per-tile searches walk, and reads
// the bounds of the sample found from cu_seqlens; beyond that the searches read the workspace (same results, slower).
template <int THREADS, int CACHE>
struct SchedLds {
    int scan_buf[THREADS / 64];
    int bins[SCHED_BINS];
    int cache_l[3 * CACHE + 1];
    int longest;
};

template <int THREADS, int CACHE>
__device__ void build_work_list(const int32_t* __restrict__ cu, int B, int T, const SchedJob& job,
                                SchedLds<THREADS, CACHE>& lds) {
    int* const scan_buf = lds.scan_buf;
    int* const bins = lds.bins;
    int* const cache_l = lds.cache_l;
    int& longest = lds.longest;
    const int R = job.R, U = job.U, mode = job.mode;
    int32_t* __restrict__ const hdr = job.hdr;
    int32_t* __restrict__ const tile_off = job.tile_off;
    WorkItem* __restrict__ const items = job.items;
    const bool cached = B <= CACHE;                              // (uniform) bounds and offsets in LDS
    const bool cached_offsets = !cached && B <= 3 * CACHE;   // (uniform) offsets only
    int* const beg_l = cache_l;
    int* const end_l = cache_l + CACHE;
    int* const toff_l = cached ? cache_l + 2 * CACHE : cache_l;
    const int t = threadIdx.x;
    if (t == 0) longest = 0;
    __syncthreads();

    // 1. tile_off[s] = number of tiles of samples 0..s-1
    int carry = 0;
    for (int base = 0; base < B; base += THREADS) {
        int s = base + t;
        int n = 0;
        if (s < B) {
            int begin, end;
            sched_sample_rows(cu[s], cu[s + 1], T, begin, end);
            if (cached) { beg_l[s] = begin; end_l[s] = end; }
            const int len = end - begin;
            n = (len + R - 1) / R;
            if (len >= kXcdChunkMinLen) longest = len;  // (any such length will do: only the threshold matters)
        }
        int total;
        int ex = block_exclusive_scan<THREADS>(n, scan_buf, &total);
        if (s < B) {
            tile_off[s] = carry + ex;
            if (cached || cached_offsets) toff_l[s] = carry + ex;
        }
        carry += total;
    }
    // (a well-formed batch has at most max_items tiles; one that is not loses the surplus instead of
    // writing past the list)
    const int n_items = min(carry, job.max_items);
    if (t == 0) {
        tile_off[B] = n_items;
        hdr[0] = n_items;
        hdr[1] = longest >= kXcdChunkMinLen ? kXcdChunk : 1;  // work order of the compute kernels (xcd_item_head)
    }
    for (int i = t; i < SCHED_BINS; i += THREADS) bins[i] = 0;
    __syncthreads();  // also makes tile_off (global, written by this block) visible to the block

    // the sample that holds tile idx of the batch (largest s with tile_off[s] <= idx), its rows and the tile's cost
    auto locate = [&](int idx, int& begin, int& end, int& tile) {
        int lo = 0, hi = B;
        if (cached) {
            while (hi - lo > 1) {
                const int mid = (lo + hi) >> 1;
                if (toff_l[mid] <= idx) lo = mid; else hi = mid;
            }
            begin = beg_l[lo]; end = end_l[lo]; tile = idx - toff_l[lo];
        } else if (cached_offsets) {
            while (hi - lo > 1) {
                const int mid = (lo + hi) >> 1;
                if (toff_l[mid] <= idx) lo = mid; else hi = mid;
            }
            sched_sample_rows(cu[lo], cu[lo + 1], T, begin, end);
            tile = idx - toff_l[lo];
        } else {
            while (hi - lo > 1) {
                const int mid = (lo + hi) >> 1;
                if (tile_off[mid] <= idx) lo = mid; else hi = mid;
            }
            sched_sample_rows(cu[lo], cu[lo + 1], T, begin, end);
            tile = idx - tile_off[lo];
        }
        return sched_tile_cost(end - begin, tile, R, U, mode);
    };

    // 2. histogram of costs
    for (int idx = t; idx < n_items; idx += THREADS) {
        int begin, end, tile;
        atomicAdd(&bins[locate(idx, begin, end, tile)], 1);
    }
    __syncthreads();

    // 3. start position of each cost class, heaviest class first
    {
        constexpr int PER = SCHED_BINS / THREADS;
        int loc[PER];
        int sum = 0;
        for (int i = 0; i < PER; ++i) {  // thread t owns descending costs
            loc[i] = bins[SCHED_BINS - 1 - (t * PER + i)];
            sum += loc[i];
        }
        int total;
        int ex = block_exclusive_scan<THREADS>(sum, scan_buf, &total);
        for (int i = 0; i < PER; ++i) {
            bins[SCHED_BINS - 1 - (t * PER + i)] = ex;
            ex += loc[i];
        }
    }
    __syncthreads();

    // 4. scatter (the order inside one cost class is arbitrary; results do not depend on it)
    for (int idx = t; idx < n_items; idx += THREADS) {
        int begin, end, tile;
        const int pos = atomicAdd(&bins[locate(idx, begin, end, tile)], 1);
        items[pos] = make_int4(begin + tile * R, begin, end, tile);
    }
}

}  // namespace va
