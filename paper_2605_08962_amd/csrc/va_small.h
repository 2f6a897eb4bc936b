// Launches too small to fill the chip (few heads of one sample, a handful of short samples): every workgroup works out
// its own tile from cu_seqlens instead of reading it from a work list, which saves the scheduler launch in front
// (4-5 us of work and the gap behind it, a third of a call on a few hundred tokens), and a tile's walk over its
// partner tiles is cut into chunks of equal length, so that the launch has as many workgroups as the chip has room for.
//
// The path is taken when a batch has at most 64 samples (one lane per sample) and no more (tile, head) pairs than
// workgroups of the forward, or of dQ, fit on the chip.  Beyond that the order of the list matters (heaviest tiles first)
// and its launch is lost in the noise.  dK/dV, of which fewer fit, goes along and looks after its order itself (small_tile).
//
// What bounds such a launch: the walk of the longest tile, while most of the chip idles; then, once cut, the memory
// round trips and the fragments of each chunk's start (3-9 us), its fp32 results (64 or 128 KB written and read again
// at 5 TB/s), and that a workgroup alone on its CU steps no faster than 1.5-2 times the rate two of them have together.
// Measured, forward + backward: one sample of 4096 tokens, 2 heads of 128, causal, 223 -> 92 us (dQ 84 -> 27, dK/dV
// 102 -> 31 us, 10 us for their sums); 8191 tokens, 4 query heads on one kv head, 1000 -> 361 us (forward 107 -> 97, dQ
// 167 -> 122, dK/dV 717 -> 146 us); four samples of 246 tokens in all, forward, 16.6 -> 13.3 us.
#pragma once
#include "va_device.h"
#include "va_internal.h"

namespace va {

// Inclusive prefix sum / maximum over the 64 lanes (all of them active; values >= 0) on DPP row shifts.
template <bool MAX>
__device__ __forceinline__ int wave_incl_scan(int x) {
    auto join = [](int a, int b) { return MAX ? max(a, b) : a + b; };
    x = join(x, __builtin_amdgcn_update_dpp(0, x, 0x111, 0xf, 0xf, false));  // row_shr:1
    x = join(x, __builtin_amdgcn_update_dpp(0, x, 0x112, 0xf, 0xf, false));  // row_shr:2
    x = join(x, __builtin_amdgcn_update_dpp(0, x, 0x114, 0xf, 0xf, false));  // row_shr:4
    x = join(x, __builtin_amdgcn_update_dpp(0, x, 0x118, 0xf, 0xf, false));  // row_shr:8
    x = join(x, __builtin_amdgcn_update_dpp(0, x, 0x142, 0xa, 0xf, false));  // row_bcast:15 into rows 1 and 3
    x = join(x, __builtin_amdgcn_update_dpp(0, x, 0x143, 0xc, 0xf, false));  // row_bcast:31 into rows 2 and 3
    return x;
}

// Partner tiles a chunk holds at most so that `total` partner tiles, the longest walk being `longest`, come to at most
// `extra` workgroups more than there are walks: sum ceil(steps / C) <= total / C + walks.
__host__ __device__ inline int chunk_steps(int total, int longest, int extra, int max_chunks) {
    const int least = (longest + max_chunks - 1) / max_chunks;
    if (extra <= 0) return longest > 1 ? longest : 1;
    const int c = (total + extra - 1) / extra;
    return c > least ? c : (least > 1 ? least : 1);
}
// Chunks of a tile with `steps` partner tiles; chunk i covers [steps * i / n, steps * (i + 1) / n).
__host__ __device__ inline int chunk_count(int steps, int chunk, int max_chunks) {
    const int n = (steps + chunk - 1) / chunk;
    return n < max_chunks ? (n > 0 ? n : 1) : max_chunks;
}

// Tiles, of a sample of n tiles of r partner tiles each (nu partner tiles in all), that meet more than `past` of them.
__host__ __device__ inline int tiles_with_chunk(int n, int nu, int r, int mode, int past) {
    if (nu <= past) return 0;
    if (mode == COST_FULL) return n;
    const int k = mode == COST_CAUSAL_QUERY ? n - past / r : (nu - past + r - 1) / r;
    return k < 1 ? 1 : (k < n ? k : n);
}

// Place of sample s among n in decreasing order of length, equal ones in their own order; len_of(i): length of sample i.
template <typename LenOf>
__host__ __device__ inline int length_rank(int n, int s, int len, LenOf len_of) {
    int rank = 0;
    for (int i = 0; i < n; ++i) {
        const int other = len_of(i);
        rank += other > len || (other == len && i < s);
    }
    return rank;
}

// Under the causal masks the v-th tile from a sample's light end costs the same in every sample.  from(v): tiles of the batch
// that cost at least that (never more for a larger v, none above `most`).  The cost of the idx-th tile by falling cost.
template <typename From>
__host__ __device__ inline int cost_level(int idx, int most, From from) {
    int v = 1, hi = most;
    while (v < hi) {
        const int mid = (v + hi + 1) >> 1;
        if (from(mid) > idx) v = mid; else hi = mid - 1;
    }
    return v;
}

struct SmallShape {  // of a launch
    int rows, partner_rows;  // R, U: rows per tile and per partner tile
    int mode;                // CostMode
    int heads, per_pair;     // `heads` workgroups walk each tile, `per_pair` times its partner tiles each
    SmallPlan plan;
    int room;                // workgroups beyond which the order of the samples counts (see small_tile), 0: it does not
};
struct SmallTile {
    int begin, len;  // first packed row and length of the sample
    int tile;        // tile index inside the sample
    int steps;       // partner tiles it meets, times per_pair
    int ch, nch;     // chunk, chunks of the tile
    // (integer division runs on the vector ALU: made scalar again, as nch is, or everything derived from them, the
    // staging pointers of the loops included, would live in vector registers: causal dQ at head_dim 80 spilled nine in its
    // loop, one sample of 1877 tokens, 8 heads, 51 -> 36 us, 3000 tokens, 4 heads, 71 -> 51)
    __device__ __forceinline__ int first_step() const {
        return nch == 1 ? 0 : __builtin_amdgcn_readfirstlane(steps * ch / nch);
    }
    __device__ __forceinline__ int end_step() const {
        return nch == 1 ? steps : __builtin_amdgcn_readfirstlane(steps * (ch + 1) / nch);
    }
};
// The idx-th (tile, chunk) of a batch of B <= 64 samples; false if there are not that many.
// First every tile's chunk 0, then the chunks 1 of the tiles that have one, and so on: no index in between is without
// work.  (Workgroup ids go round-robin over the XCDs and their shader engines, wherever there is room; a launch
// with holes in it leaves some of them with two workgroups per CU, one after the other, and others with none: measured
// twice the time.)  Inside a sample the heaviest tiles come first.  Across samples the order counts where `room`
// workgroups are exceeded (SmallShape), since the last ones share a CU or wait for one:
//   causal, from one workgroup per CU on: tiles by falling cost.  30 samples of 1318 tokens, one head of 128, dQ 49 -> 41 us,
//     dK/dV 72 -> 52, forward 42 -> 39; 9 of 2229, 2 heads, dQ 75 -> 58, dK/dV 91 -> 72.  The forward at head_dim 64, 80 and
//     96 goes without: the search cost it 2-6 % in the launches that have no use for it (at 128 nothing).
//   without the mask, dK/dV beyond what the chip holds at a time (one workgroup per CU at head_dim 96 and 128): the longest
//     sample first.  4 heads of 128, 19 samples of 300 tokens and one of 2000 behind them, 74 -> 61 us; 8 heads, 30 of 100
//     and one of 900, 48 -> 38; 12 of 400 unchanged.  Below that it was no gain (dQ and dK/dV of 41 samples, 8 heads of 64:
//     26.1 / 26.8 us, longest first 26.9 / 30.7).
// Must be reached by all 64 lanes; every result is wave-uniform.
__device__ __forceinline__ bool small_tile(const int32_t* __restrict__ cu, int B, int T, const SmallShape& p, int idx,
                                           SmallTile& out) {
    const int lane = threadIdx.x & 63;
    int begin = 0, end = 0;
    if (lane < B) sched_sample_rows(cu[lane], cu[lane + 1], T, begin, end);
    int len = end - begin;
    const int R = p.rows, r = p.rows / p.partner_rows;
    bool by_cost = false;
    if (p.room > 0 && B > 1 && (T / R + B) * p.heads > p.room) {
        const int tiles = __builtin_amdgcn_readlane(wave_incl_scan<false>((len + R - 1) / R), 63);
        by_cost = p.mode != COST_FULL && tiles * p.heads > p.room;
        const int next = __builtin_amdgcn_update_dpp(0, len, 0x130, 0xf, 0xf, false);  // wave_shl:1
        if (!by_cost && tiles * p.heads > p.room && __builtin_amdgcn_ballot_w64(len < next)) {
            const int place = length_rank(B, lane, len, [&](int i) { return __builtin_amdgcn_readlane(len, i); }) * 4;
            begin = __builtin_amdgcn_ds_permute(place, begin);
            len = __builtin_amdgcn_ds_permute(place, len);
            if (lane >= B) begin = len = 0;
        }
    }
    const int n = (len + R - 1) / R, nu = (len + p.partner_rows - 1) / p.partner_rows;
    int chunk = 1 << 30, count = n, incl = 0, ch = 0;
    for (;; ++ch) {  // count: this lane's tiles that have a chunk ch
        incl = wave_incl_scan<false>(count);
        const int here = __builtin_amdgcn_readlane(incl, 63);
        if (ch == 0 && p.plan.max_chunks > 1) {
            chunk = p.plan.chunk;
            if (chunk == 0) {
                // partner tiles of a sample: n tiles of nu, minus what the causal masks take off (r of them per tile)
                const int off = p.mode == COST_FULL ? 0 : n * (n - 1) / 2 * r;
                const int sum = p.mode == COST_CAUSAL_QUERY ? (n > 0 ? off + nu : 0) : n * nu - off;
                const int total = __builtin_amdgcn_readlane(wave_incl_scan<false>(sum), 63) * p.heads * p.per_pair;
                const int longest = __builtin_amdgcn_readlane(wave_incl_scan<true>(nu), 63) * p.per_pair;
                chunk = max(longest, 1);
                // Uncut where no walk is longer than the work there is for a CU anyway (6 steps: a tile's start), unless the
                // walks are long: more and shorter ones side by side on a CU step faster together.  Without the hint, cut /
                // uncut: two samples of 7724 tokens, 2 heads of 96, 115 / 129 us; 12 of 640, 5 heads of 64, 30 / 22 us.
                const int tiles = here * p.heads, load = (total + 6 * tiles) / max(tiles, 256);
                if ((longest > load || longest >= 32) && longest * p.partner_rows > VA_SMALL_UNCUT_LEN * p.per_pair)
                    chunk = __builtin_amdgcn_readfirstlane(
                        chunk_steps(total, longest, p.plan.extra, p.plan.max_chunks));
            }
        }
        if (idx < here) break;
        if (ch + 1 >= p.plan.max_chunks) return false;
        idx -= here;
        count = tiles_with_chunk(n, nu, r, p.mode, (ch + 1) * chunk / p.per_pair);
    }
    int s, t;
    if (by_cost && ch == 0) {
        auto from = [&](int v) { return __builtin_amdgcn_readlane(wave_incl_scan<false>(max(n - v + 1, 0)), 63); };
        const int v = cost_level(idx, __builtin_amdgcn_readlane(wave_incl_scan<true>(n), 63), from);
        const int place = idx - from(v + 1);  // among the tiles of that cost (all lanes at work here: a lane operation)
        const unsigned long long has = __builtin_amdgcn_ballot_w64(n >= v);
        const int before = __builtin_popcountll(has & ((1ull << lane) - 1));
        const int hit = (n >= v ? 1 : 0) & (before == place ? 1 : 0);
        s = __builtin_ctzll(__builtin_amdgcn_ballot_w64(hit != 0));
        t = __builtin_amdgcn_readlane(n, s) - v;
    } else {
        s = __builtin_popcountll(__builtin_amdgcn_ballot_w64(incl <= idx));  // samples before the one that holds idx
        t = idx - (__builtin_amdgcn_readlane(incl, s) - __builtin_amdgcn_readlane(count, s));
    }
    const int ns = __builtin_amdgcn_readlane(n, s), us = __builtin_amdgcn_readlane(nu, s);
    out.begin = __builtin_amdgcn_readlane(begin, s);
    out.len = __builtin_amdgcn_readlane(len, s);
    out.tile = p.mode == COST_CAUSAL_QUERY ? ns - 1 - t : t;
    out.steps = (p.mode == COST_FULL ? us : p.mode == COST_CAUSAL_QUERY ? min(us, (out.tile + 1) * r) : us - out.tile * r) *
                p.per_pair;
    out.ch = ch;
    out.nch = __builtin_amdgcn_readfirstlane(chunk_count(out.steps, chunk, p.plan.max_chunks));
    return true;
}

}  // namespace va
