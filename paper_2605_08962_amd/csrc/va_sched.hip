// Length-aware tile scheduler.
//
// The paper's motivation is the imbalance that mixed long and short samples cause (Section 2.2,
// Section 4.1.1) and it picks its attention algorithm for its work partitioning on long inputs
// (Section 6, "Efficient Operators").  On one GPU the same problem shows up inside a single
// launch: a 64k-token sample packed with hundreds of short ones.  This kernel turns cu_seqlens
// into a list of row tiles sorted by decreasing cost (the number of partner tiles a tile loops
// over), entirely on the device.  The compute kernels launch one workgroup per (list entry,
// head) in list order, so the hardware dispatcher hands out the heaviest tiles first and the
// light ones fill the tail (longest-processing-time-first list scheduling).
#include <vector>

#include "va_device.h"
#include "va_internal.h"
#include "va_sched.h"

namespace va {

constexpr int SCHED_THREADS = 1024;

SchedLayout sched_layout(int64_t total_tokens, int64_t num_seqs, int tile_rows) {
    SchedLayout lay;
    lay.max_items = total_tokens / tile_rows + num_seqs;  // >= sum_s ceil(L_s / tile_rows)
    lay.tile_off_ofs = 16 * sizeof(int32_t);
    size_t p = lay.tile_off_ofs + (size_t)(num_seqs + 1) * sizeof(int32_t);
    lay.items_ofs = (p + 15) / 16 * 16;
    p = lay.items_ofs + (size_t)lay.max_items * sizeof(WorkItem);
    lay.end_ofs = (p + 255) / 256 * 256;
    return lay;
}

// Samples whose bounds and tile offsets the kernel keeps in LDS (see SchedLds).
constexpr int SCHED_CACHE = 8192;

// One workgroup per work list (the backward builds two at a time).
__global__ void __launch_bounds__(SCHED_THREADS)
sched_kernel(const int32_t* __restrict__ cu, int B, int T, SchedJob job0, SchedJob job1) {
    __shared__ SchedLds<SCHED_THREADS, SCHED_CACHE> lds;
    build_work_list(cu, B, T, blockIdx.x == 0 ? job0 : job1, lds);
}

hipError_t launch_scheduler(const int32_t* cu_seqlens, int num_seqs, int total_tokens, int tile_rows,
                            int partner_rows, CostMode mode, void* ws, const SchedLayout& lay, hipStream_t stream) {
    const SchedJob job = sched_job(tile_rows, partner_rows, mode, ws, lay);
    hipLaunchKernelGGL(sched_kernel, dim3(1), dim3(SCHED_THREADS), 0, stream, cu_seqlens, num_seqs, total_tokens,
                       job, job);
    return hipGetLastError();
}

hipError_t launch_scheduler_pair(const int32_t* cu_seqlens, int num_seqs, int total_tokens, int tile_rows_a,
                                 int partner_rows_a, CostMode mode_a, void* ws_a, const SchedLayout& lay_a,
                                 int tile_rows_b, int partner_rows_b, CostMode mode_b, void* ws_b,
                                 const SchedLayout& lay_b, hipStream_t stream) {
    hipLaunchKernelGGL(sched_kernel, dim3(2), dim3(SCHED_THREADS), 0, stream, cu_seqlens, num_seqs, total_tokens,
                       sched_job(tile_rows_a, partner_rows_a, mode_a, ws_a, lay_a),
                       sched_job(tile_rows_b, partner_rows_b, mode_b, ws_b, lay_b));
    return hipGetLastError();
}

int64_t schedule_on_host(const int32_t* cu, int B, int T, int R, int U, CostMode mode, int64_t max_items,
                         WorkItem* items) {
    // counting sort by cost class, heaviest first; inside a class the tiles keep their (sample, tile) order
    std::vector<int64_t> start(SCHED_BINS + 1, 0);
    int64_t n = 0;
    for (int pass = 0; pass < 2; ++pass) {
        int64_t seen = 0;
        for (int s = 0; s < B && seen < max_items; ++s) {
            int begin, end;
            sched_sample_rows(cu[s], cu[s + 1], T, begin, end);
            const int L = end - begin;
            for (int t = 0; t * (int64_t)R < L && seen < max_items; ++t, ++seen) {
                const int c = sched_tile_cost(L, t, R, U, (int)mode);
                if (pass == 0) ++start[SCHED_BINS - 1 - c + 1];
                else items[start[SCHED_BINS - 1 - c]++] = make_int4(begin + t * R, begin, end, t);
            }
        }
        if (pass == 0) {
            n = seen;
            for (int i = 0; i < SCHED_BINS; ++i) start[i + 1] += start[i];
        }
    }
    return n;
}

// One workgroup walks cu_seqlens; every thread notes what it sees wrong, the block ORs the notes.
__global__ void __launch_bounds__(SCHED_THREADS)
check_cu_seqlens_kernel(const int32_t* __restrict__ cu, int B, int T, int32_t* __restrict__ verdict) {
    int bad = 0;
    for (int s = threadIdx.x; s < B; s += SCHED_THREADS) bad |= cu[s] > cu[s + 1];
    if (threadIdx.x == 0) bad |= cu[0] != 0 || cu[B] != T;
    bad = __syncthreads_or(bad);
    if (threadIdx.x == 0) *verdict = bad ? 1 : 0;
}

hipError_t launch_check_cu_seqlens(const int32_t* cu_seqlens, int num_seqs, int total_tokens, int32_t* verdict,
                                   hipStream_t stream) {
    hipLaunchKernelGGL(check_cu_seqlens_kernel, dim3(1), dim3(SCHED_THREADS), 0, stream, cu_seqlens, num_seqs,
                       total_tokens, verdict);
    return hipGetLastError();
}

}  // namespace va
