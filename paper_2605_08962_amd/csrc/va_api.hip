// C-ABI entry points of libvarlen_attn.so: argument validation, workspace carving, launches.
#include <algorithm>
#include <cmath>
#include <cstring>
#include <mutex>
#include <vector>

#include "../../include/varlen_attn.h"
#include "va_internal.h"
#include "va_small.h"

// Scratch of varlen_attn_fwd_static_scratch: device memory that belongs to the library's code object, one
// copy per GPU.  In host code this name is only a handle for hipGetSymbolAddress, never an address.
static __device__ __align__(256) unsigned char scratch[VA_STATIC_SCRATCH_BYTES];

namespace {

thread_local int g_last_hip_error = 0;

int hip_fail(hipError_t e) {
    g_last_hip_error = (int)e;
    return VA_ERR_HIP;
}

// Optional per-kernel timing: while enabled, each kernel launch is bracketed by two events recorded
// on the caller's stream.  Nothing synchronises until varlen_attn_profile_read().
struct ProfSample { int kernel; hipEvent_t a, b; };
std::mutex g_prof_mutex;
bool g_prof_on = false;
std::vector<ProfSample> g_prof_samples;
unsigned long long* g_clock_probe = nullptr;  // device, 6 counters, caller-owned (see the header)

unsigned long long* clock_probe_slot(int pair) {
    std::lock_guard<std::mutex> lock(g_prof_mutex);
    return g_clock_probe ? g_clock_probe + 2 * pair : nullptr;
}

struct ProfScope {
    bool on = false;
    ProfSample s{};
    hipStream_t stream;
    ProfScope(int kernel, hipStream_t st) : stream(st) {
        std::lock_guard<std::mutex> lock(g_prof_mutex);
        if (!g_prof_on) return;
        if (hipEventCreate(&s.a) != hipSuccess) return;
        if (hipEventCreate(&s.b) != hipSuccess) { (void)hipEventDestroy(s.a); return; }
        s.kernel = kernel;
        on = hipEventRecord(s.a, stream) == hipSuccess;
    }
    ~ProfScope() {
        if (!on) return;
        (void)hipEventRecord(s.b, stream);
        std::lock_guard<std::mutex> lock(g_prof_mutex);
        g_prof_samples.push_back(s);
    }
};

void prof_clear_locked() {
    for (auto& s : g_prof_samples) { (void)hipEventDestroy(s.a); (void)hipEventDestroy(s.b); }
    g_prof_samples.clear();
}

bool aligned16(const void* p) { return ((uintptr_t)p & 15u) == 0; }

int check_params(const varlen_attn_params* p) {
    if (!p) return VA_ERR_NULL_PTR;
    if (p->total_tokens < 0 || p->num_seqs < 0 || p->num_q_heads < 1 || p->num_kv_heads < 1 ||
        p->num_q_heads % p->num_kv_heads != 0 || (p->causal != 0 && p->causal != 1) || p->max_seqlen < 0 ||
        p->kv_splits < 0 || p->kv_splits > VA_MAX_KV_SPLITS)
        return VA_ERR_BAD_SHAPE;
    if (p->head_dim != 64 && p->head_dim != 80 && p->head_dim != 96 && p->head_dim != 128)
        return VA_ERR_UNSUPPORTED;
    if (!std::isfinite(p->softmax_scale) || p->softmax_scale < 0.f) return VA_ERR_BAD_SCALE;
    // grid sizes and packed offsets are 32-bit in places: keep the launch within them
    int64_t items = (int64_t)p->total_tokens / 64 + p->num_seqs;
    if (items * p->num_q_heads * std::max(p->kv_splits, 1) >= (int64_t)1 << 31) return VA_ERR_BAD_SHAPE;
    return VA_OK;
}

// The current device must be a gfx950; checked once per device.
int check_device() {
    static thread_local int checked_dev = -1;
    static thread_local int checked_rc = VA_OK;
    int dev = 0;
    hipError_t e = hipGetDevice(&dev);
    if (e != hipSuccess) return hip_fail(e);
    if (dev == checked_dev) return checked_rc;
    hipDeviceProp_t prop;
    e = hipGetDeviceProperties(&prop, dev);
    if (e != hipSuccess) return hip_fail(e);
    checked_dev = dev;
    checked_rc = std::strncmp(prop.gcnArchName, "gfx950", 6) == 0 ? VA_OK : VA_ERR_UNSUPPORTED;
    return checked_rc;
}

bool short_batch(const varlen_attn_params* p) { return p->max_seqlen > 0 && p->max_seqlen <= va::kShortBatchMaxSeqlen; }

// Sample length to reckon with before the device has seen the lengths: the caller's max_seqlen if it gave one, else
// the average.
int64_t expected_len(const varlen_attn_params* p) {
    return p->max_seqlen > 0 ? std::min(p->max_seqlen, p->total_tokens) : p->total_tokens / p->num_seqs;
}

// A launch whose (tile, head) pairs do not fill the `slots` workgroups the chip holds at once (va_small.h).
bool small_launch(const varlen_attn_params* p, int tile_rows, int heads, int slots) {
    return p->num_seqs <= va::VA_SMALL_MAX_SEQS &&
           ((int64_t)p->total_tokens / tile_rows + p->num_seqs) * heads <= slots;
}

// What a small launch's kernel costs, in the time of one of its steps on a CU that runs nothing else.
struct SmallCost {
    int wgs_per_cu;  // workgroups of the kernel a CU holds
    float share;     // with w workgroups on a CU a step takes 1 + share * (w - 1)
    float fixed;     // prologue and epilogue
    float parts;     // fp32 results of 256 chunks, written and read again
    float combine;   // the launch that combines them (the backward's two plans share one)
    int others;      // workgroups of the launch that do something else
};

// How many workgroups share the keys of one query tile in the forward when the launch goes by a work list.
// Splitting only pays when the launch cannot fill the chip: fewer workgroups than the 256 CUs can hold at once (3 per
// CU at head_dim <= 80, else 2), and samples long enough that every chunk still gets two key tiles.
int fwd_kv_splits(const varlen_attn_params* p) {
    if (p->kv_splits >= 1) return p->kv_splits;
    const int64_t wgs = ((int64_t)p->total_tokens / va::FWD_TILE_Q + p->num_seqs) * p->num_q_heads;
    const int64_t slots = 256 * (p->head_dim <= 80 ? 3 : 2);
    const int64_t tiles_per_sample = expected_len(p) / va::FWD_TILE_KV;
    int64_t s = std::min<int64_t>(std::min<int64_t>(slots / std::max<int64_t>(wgs, 1), tiles_per_sample / 2), VA_MAX_KV_SPLITS);
    return (int)std::max<int64_t>(s, 1);
}

// How the walks of a small launch are cut: for the samples the caller's sizes lead to expect, the number of workgroups
// per CU, up to twice what it holds at a time, for which the chunks come out cheapest.  With several samples it is how
// many workgroups that is beyond one per tile that goes to the device, which finds the chunk that gives as many: what is
// expected leaves out the short samples beside the long ones (eight of up to 150 tokens and one of 1877, 8 heads of 80,
// causal, with a hint: forward 36 us where the number was one for all workgroups, 27 so).
// Several samples without max_seqlen are reckoned with as one that holds all tokens, and the device cuts by the lengths it
// finds: 8192 tokens and ten or twenty samples of 16, 2 heads of 64, forward, 107 us where the average was reckoned with,
// 55 us so.  Four even samples of 400 pay for a merge launch that finds nothing to do, 10.6 -> 13.2 us; so that is done only
// where the chip has room for twice the workgroups and the average is 256 tokens: below that a sample worth cutting is less
// likely and such a call shorter yet.
// Samples of up to 512 tokens are not: uncut here / in 2 to 4 chunks by the work list, one of 512 tokens, 2 heads, took
// 10.8 / 15.4 us at head_dim 64, 11.6 / 15.8 at 80, 17.0 / 17.0 at 128 (causal 18.3 / 17.8); four of 400 10.6 / 16.0.
va::SmallPlan small_plan(const varlen_attn_params* p, int tile_rows, int partner_rows, va::CostMode mode, int heads,
                         int per_pair, const SmallCost& cost) {
    const bool unknown = p->max_seqlen == 0 && p->num_seqs > 1;
    const int len = unknown ? p->total_tokens : (int)expected_len(p), R = tile_rows / partner_rows;
    const int nu = (len + partner_rows - 1) / partner_rows, n = (len + tile_rows - 1) / tile_rows;
    const int samples = std::max(p->total_tokens / std::max(len, 1), 1);
    va::SmallPlan best{1, 0, 0};
    if (nu * per_pair < 8 || len <= va::VA_SMALL_UNCUT_LEN || (unknown && fwd_kv_splits(p) < 2)) return best;
    const int longest = nu * per_pair, least = (longest + va::VA_SMALL_CHUNKS - 1) / va::VA_SMALL_CHUNKS;
    auto workgroups = [&](int chunk) {
        int64_t k = 0;
        for (int ch = 0; ch < va::VA_SMALL_CHUNKS && ch * chunk < longest; ++ch)
            k += va::tiles_with_chunk(n, nu, R, mode, ch * chunk / per_pair);
        return k * samples * heads;
    };
    // w workgroups per CU: as many as it holds side by side, then one round after the other.
    auto time = [&](float w, int chunk) {
        const float beside = std::min(w, (float)cost.wgs_per_cu);
        return (1.f + cost.share * (beside - 1.f)) * (chunk + cost.fixed) * w / beside;
    };
    // Uncut: walks of one length take as long as the CUs with one more of them; under a causal mask the light tiles, which
    // come last, fill up.
    const float whole = workgroups(longest) / 256.f;
    float least_time = time(std::max(mode == va::COST_FULL ? std::ceil(whole) : whole, 1.f), longest);
    for (int w = 1; w <= (unknown ? 1 : 2) * cost.wgs_per_cu; ++w) {
        const int target = 256 * w - cost.others;
        int lo = least, hi = longest;  // smallest chunk that gives at most that many workgroups
        if (workgroups(hi) > target) continue;
        while (lo < hi) {
            const int mid = (lo + hi) / 2;
            if (workgroups(mid) <= target) hi = mid; else lo = mid + 1;
        }
        if (lo == longest) continue;
        const float t = time((float)w, lo) + cost.parts * w + cost.combine;
        if (t < least_time) {
            least_time = t;
            best.extra = target - (int)workgroups(longest);
            best.chunk = p->num_seqs == 1 ? lo : 0;
            const int k = va::chunk_count(longest, lo, va::VA_SMALL_CHUNKS);
            best.max_chunks = p->num_seqs == 1 ? k : std::min(k + 1, (int)va::VA_SMALL_CHUNKS);
        }
    }
    return best;
}
// Time stamps inside the kernels, samples of 4096 and 8192 tokens: a step of the forward at head_dim 128 (32 keys) takes
// 0.8 / 1.1 / 1.4 us with one, two, three workgroups on the CU, of dQ 1.6 / 2.8 us, of dK/dV 1.5-2 us; prologue and
// epilogue together 6-8 us each; parts at 5 TB/s.  Fitted to the times of 460 random batches at every head_dim, uncut and
// cut into 256 to 1536 workgroups, the steps take 0.65-0.9 us (forward), 0.75-1.2 (dQ) and 0.85-1.4 (dK/dV), share 0.3-0.6,
// fixed 5-8 (forward at 128: 15); with these constants the choice is on average 3 % off the best one tried, and in 1 of 60
// cases more than 5 % behind the uncut launch.  Fitted before the kernels' mask-free steps lost their bounds and branches, and the
// merges half their rows; since then 240 random launches of samples above 1024 tokens, planned against kv_splits = 1: forward 0.68,
// backward 0.60 of the time on average, 8 of the 480 more than 5 % behind (at worst a forward of five samples of 5528 tokens, 3
// heads of 128, causal, 138 -> 166 us; a backward of five samples of up to 1085, 8 heads of 128, 61 -> 70).
SmallCost fwd_cost(int head_dim) {
    return head_dim == 128 ? SmallCost{va::fwd_small_slots(128) / 256, 0.37f, 8.f, 8.f, 4.f, 0}
                           : SmallCost{va::fwd_small_slots(head_dim) / 256, 0.37f, 6.f, 4.f, 4.f, 0};
}
SmallCost dq_cost(int head_dim) {
    return SmallCost{va::bwd_dq_slots(head_dim) / 256, 0.5f, 5.f, 4.f * head_dim / 128, 3.f, 2};
}
SmallCost dkdv_cost(int head_dim) {
    return SmallCost{va::bwd_dkdv_slots(head_dim) / 256, 0.5f, 5.f, 8.f * head_dim / 128, 3.f, 0};
}

// Causal batches of several long samples with many tiles to a CU: what they gain by the list's order (tiles by falling
// cost) is more than its launch, unless the small kernel keeps that order itself, at head_dim 128 (see small_tile).  Small
// kernel / list, with the hint, 2 heads of 64 and 80: 20 samples of 2047 tokens 54 / 42 and 66 / 48 us, 14 of 3000 62 / 55 and
// 76 / 65; about even at 1300 tokens (20 samples, 27 / 27 and 32 / 31) and at 280 pairs (8 of 2047, 31 / 31 and 36 / 35); 35
// samples of 700 18 / 21 and 21 / 25.  At head_dim 96, where two workgroups fit a CU and not three, 11 of 2047 52 / 44.
bool fwd_wants_order(const varlen_attn_params* p) {
    const int64_t pairs = ((int64_t)p->total_tokens / va::FWD_TILE_Q + p->num_seqs) * p->num_q_heads;
    return p->causal && p->num_seqs > 1 && p->head_dim != 128 && pairs > (p->head_dim == 96 ? 320 : 384) &&
           p->total_tokens / p->num_seqs >= 1000;
}

struct FwdLayout {
    va::SchedLayout sched;
    bool small;
    int splits;
    va::SmallPlan plan;
    size_t part_o_ofs, part_lse_ofs, end;
};

// `room`: bytes the work list and the parts may take.  Automatic chunks become fewer, down to none, until they fit; what
// does not fit then, or is asked for by kv_splits, is the caller's error.
FwdLayout fwd_layout(const varlen_attn_params* p, size_t room = SIZE_MAX) {
    FwdLayout f;
    f.sched = va::sched_layout(p->total_tokens, p->num_seqs, va::FWD_TILE_Q);
    f.small = p->kv_splits == 0 && small_launch(p, va::FWD_TILE_Q, p->num_q_heads, va::fwd_small_slots(p->head_dim)) &&
              !fwd_wants_order(p);
    f.plan = va::SmallPlan{1, 0, 0};
    if (f.small)
        f.plan = small_plan(p, va::FWD_TILE_Q, va::fwd_tile_kv(p->head_dim), p->causal ? va::COST_CAUSAL_QUERY : va::COST_FULL,
                            p->num_q_heads, 1, fwd_cost(p->head_dim));
    f.splits = f.small ? f.plan.max_chunks : fwd_kv_splits(p);
    const size_t rows = (size_t)p->total_tokens * p->num_q_heads;
    f.part_o_ofs = f.sched.end_ofs;
    for (;; --f.splits) {
        f.part_lse_ofs = f.end = f.sched.end_ofs;
        if (f.splits > 1) {
            f.part_lse_ofs = f.part_o_ofs + (size_t)f.splits * rows * p->head_dim * sizeof(float);
            f.end = (f.part_lse_ofs + (size_t)f.splits * rows * sizeof(float) + 255) / 256 * 256;
        }
        if (f.end <= room || p->kv_splits != 0 || f.splits == 1) break;
    }
    if (f.splits < f.plan.max_chunks) f.plan = va::SmallPlan{f.splits, f.plan.extra, 0};
    return f;
}

struct BwdLayout {
    va::SchedLayout kv, q;
    bool small;
    va::SmallPlan plan_q, plan_kv;
    size_t kv_ofs, q_ofs, stats_ofs, part_dq_ofs, part_dk_ofs, part_dv_ofs, end;
};

// `room`: bytes the workspace may take; the chunks become fewer, down to none, until they fit (see fwd_layout).
BwdLayout bwd_layout(const varlen_attn_params* p, size_t room = SIZE_MAX) {
    BwdLayout b;
    b.kv = va::sched_layout(p->total_tokens, p->num_seqs, va::BWD_TILE_KV);
    b.q = va::sched_layout(p->total_tokens, p->num_seqs, va::BWD_TILE_Q);
    b.kv_ofs = 0;
    b.q_ofs = b.kv.end_ofs;
    b.stats_ofs = b.q_ofs + b.q.end_ofs;
    b.end = b.stats_ofs + ((size_t)p->total_tokens * p->num_q_heads * 2 * sizeof(float) + 255) / 256 * 256;
    b.small = p->num_seqs > 0 && small_launch(p, va::BWD_TILE_Q, p->num_q_heads, va::bwd_dq_slots(p->head_dim));
    b.plan_q = b.plan_kv = va::SmallPlan{1, 0, 0};
    // Tiles are cut only where the caller has said that samples are long: without max_seqlen (or kv_splits = 1) a
    // sample's gradients are the same bits whatever it is launched with.
    if (b.small && p->kv_splits == 0 && p->max_seqlen > va::kShortBatchMaxSeqlen) {
        b.plan_q = small_plan(p, va::BWD_TILE_Q, va::BWD_STEP_KV, p->causal ? va::COST_CAUSAL_QUERY : va::COST_FULL,
                              p->num_q_heads, 1, dq_cost(p->head_dim));
        b.plan_kv = small_plan(p, va::BWD_TILE_KV, va::BWD_STEP_Q, p->causal ? va::COST_CAUSAL_KEY : va::COST_FULL,
                               p->num_kv_heads, p->num_q_heads / p->num_kv_heads, dkdv_cost(p->head_dim));
    }
    auto part = [&](int splits, int heads) {
        return splits > 1 ? ((size_t)splits * p->total_tokens * heads * p->head_dim * sizeof(float) + 255) / 256 * 256 : 0;
    };
    b.part_dq_ofs = b.end;
    for (;;) {
        b.part_dk_ofs = b.part_dq_ofs + part(b.plan_q.max_chunks, p->num_q_heads);
        b.part_dv_ofs = b.part_dk_ofs + part(b.plan_kv.max_chunks, p->num_kv_heads);
        b.end = b.part_dv_ofs + part(b.plan_kv.max_chunks, p->num_kv_heads);
        va::SmallPlan& more = b.plan_q.max_chunks >= b.plan_kv.max_chunks ? b.plan_q : b.plan_kv;
        if (b.end <= room || more.max_chunks == 1) return b;
        more = va::SmallPlan{more.max_chunks - 1, more.extra, 0};
    }
}

}  // namespace

extern "C" {

size_t varlen_attn_fwd_workspace_bytes(const varlen_attn_params* p) {
    if (check_params(p) != VA_OK) return 0;
    if (p->total_tokens == 0 || p->num_seqs == 0) return va::sched_layout(0, 0, va::FWD_TILE_Q).end_ofs;
    return fwd_layout(p).end;
}

size_t varlen_attn_bwd_workspace_bytes(const varlen_attn_params* p) {
    if (check_params(p) != VA_OK) return 0;
    return bwd_layout(p).end;
}

int64_t varlen_attn_max_work_items(const varlen_attn_params* p, int which) {
    if (check_params(p) != VA_OK) return 0;
    int rows = which == 0 ? va::FWD_TILE_Q : which == 1 ? va::BWD_TILE_KV : va::BWD_TILE_Q;
    return va::sched_layout(p->total_tokens, p->num_seqs, rows).max_items;
}

int64_t varlen_attn_schedule_host(const varlen_attn_params* p, int which, const int32_t* cu_seqlens_host,
                                  int32_t* items, int64_t items_capacity) {
    if (check_params(p) != VA_OK || which < 0 || which > 2 || !cu_seqlens_host || !items) return -1;
    const int rows = which == 0 ? va::FWD_TILE_Q : which == 1 ? va::BWD_TILE_KV : va::BWD_TILE_Q;
    const int partner = which == 0 ? va::FWD_TILE_KV : which == 1 ? va::BWD_STEP_Q : va::BWD_STEP_KV;
    const va::CostMode mode = !p->causal ? va::COST_FULL : which == 1 ? va::COST_CAUSAL_KEY : va::COST_CAUSAL_QUERY;
    const int64_t max_items = va::sched_layout(p->total_tokens, p->num_seqs, rows).max_items;
    if (items_capacity < max_items) return -1;
    static_assert(sizeof(va::WorkItem) == 4 * sizeof(int32_t), "work items are four int32");
    return va::schedule_on_host(cu_seqlens_host, p->num_seqs, p->total_tokens, rows, partner, mode, max_items,
                                (va::WorkItem*)items);
}

namespace {
int fwd_impl(const varlen_attn_params* p, const void* q, const void* k, const void* v, const int32_t* cu_seqlens, void* o,
             float* lse, const FwdLayout& fl, void* workspace, size_t workspace_bytes, void* hip_stream) {
    if (!q || !k || !v || !cu_seqlens || !o || !lse || !workspace) return VA_ERR_NULL_PTR;
    if (!aligned16(q) || !aligned16(k) || !aligned16(v) || !aligned16(o) || !aligned16(workspace) ||
        ((uintptr_t)lse & 3u) || ((uintptr_t)cu_seqlens & 3u))
        return VA_ERR_MISALIGNED;
    const va::SchedLayout& lay = fl.sched;
    if (workspace_bytes < fl.end) return VA_ERR_WORKSPACE_TOO_SMALL;
    const int rc = check_device();
    if (rc != VA_OK) return rc;
    hipStream_t stream = (hipStream_t)hip_stream;

    hipError_t e = hipSuccess;
    if (!fl.small) {
        ProfScope ps(VA_KERNEL_SCHED, stream);
        e = va::launch_scheduler(cu_seqlens, p->num_seqs, p->total_tokens, va::FWD_TILE_Q, va::FWD_TILE_KV,
                                 p->causal ? va::COST_CAUSAL_QUERY : va::COST_FULL, workspace, lay, stream);
    }
    if (e != hipSuccess) return hip_fail(e);
    va::FwdArgs a;
    a.q = q; a.k = k; a.v = v; a.o = o; a.lse = lse;
    a.sched_hdr = (const int32_t*)workspace;
    a.items = (const va::WorkItem*)((const char*)workspace + lay.items_ofs);
    a.max_items = lay.max_items;
    a.total_tokens = p->total_tokens; a.num_q_heads = p->num_q_heads; a.num_kv_heads = p->num_kv_heads;
    a.head_dim = p->head_dim; a.causal = p->causal; a.scale = p->softmax_scale;
    a.kv_splits = fl.splits;
    a.part_o = (float*)((char*)workspace + fl.part_o_ofs);
    a.part_lse = (float*)((char*)workspace + fl.part_lse_ofs);
    a.clock_probe = clock_probe_slot(0);
    a.lean = short_batch(p) && fl.splits == 1;
    a.small = fl.small;
    a.cu_seqlens = cu_seqlens;
    a.num_seqs = p->num_seqs;
    a.plan = fl.plan;
    {
        ProfScope ps(VA_KERNEL_FWD, stream);
        e = va::launch_fwd(a, stream);
    }
    if (e != hipSuccess) return hip_fail(e);
    if (fl.splits > 1) {
        ProfScope ps(VA_KERNEL_MERGE, stream);
        e = fl.small ? va::launch_fwd_merge_small(a, stream)
                     : va::launch_merge(a.part_o, true, a.part_lse, fl.splits, p->total_tokens, p->num_q_heads,
                                        p->head_dim, o, lse, stream);
        if (e != hipSuccess) return hip_fail(e);
    }
    return VA_OK;
}
}  // namespace

int varlen_attn_fwd(const varlen_attn_params* p, const void* q, const void* k, const void* v,
                    const int32_t* cu_seqlens, void* o, float* lse, void* workspace,
                    size_t workspace_bytes, void* hip_stream) {
    const int rc = check_params(p);
    if (rc != VA_OK) return rc;
    if (p->total_tokens == 0 || p->num_seqs == 0) return VA_OK;
    return fwd_impl(p, q, k, v, cu_seqlens, o, lse, fwd_layout(p, workspace_bytes), workspace, workspace_bytes,
                    hip_stream);
}

namespace {
// Address of `scratch` on the current device, looked up once per device (with that device current).
constexpr int kMaxDevices = 64;
std::mutex g_scratch_mutex;
void* g_scratch_ptr[kMaxDevices] = {};

int static_scratch_ptr(void** out) {
    int dev = 0;
    hipError_t e = hipGetDevice(&dev);
    if (e != hipSuccess) return hip_fail(e);
    if (dev < 0 || dev >= kMaxDevices) return VA_ERR_UNSUPPORTED;
    std::lock_guard<std::mutex> lock(g_scratch_mutex);
    if (!g_scratch_ptr[dev]) {
        void* ptr = nullptr;
        e = hipGetSymbolAddress(&ptr, HIP_SYMBOL(scratch));
        if (e != hipSuccess) return hip_fail(e);
        if (!ptr) return hip_fail(hipErrorInvalidSymbol);
        g_scratch_ptr[dev] = ptr;
    }
    *out = g_scratch_ptr[dev];
    return VA_OK;
}
}  // namespace

int varlen_attn_fwd_static_scratch(const varlen_attn_params* p, const void* q, const void* k, const void* v,
                                   const int32_t* cu_seqlens, void* o, float* lse, void* hip_stream) {
    int rc = check_params(p);
    if (rc != VA_OK) return rc;
    if (p->total_tokens == 0 || p->num_seqs == 0) return VA_OK;
    const FwdLayout fl = fwd_layout(p, (size_t)VA_STATIC_SCRATCH_BYTES);
    if (fl.end > (size_t)VA_STATIC_SCRATCH_BYTES) return VA_ERR_SCRATCH_LIMIT;
    rc = check_device();
    if (rc != VA_OK) return rc;
    void* ptr = nullptr;
    rc = static_scratch_ptr(&ptr);
    if (rc != VA_OK) return rc;
    return fwd_impl(p, q, k, v, cu_seqlens, o, lse, fl, ptr, (size_t)VA_STATIC_SCRATCH_BYTES, hip_stream);
}

int varlen_attn_merge(const varlen_attn_params* p, int32_t num_parts, const void* o_parts, const float* lse_parts,
                      void* o, float* lse, void* hip_stream) {
    int rc = check_params(p);
    if (rc != VA_OK) return rc;
    if (num_parts < 1 || num_parts > VA_MAX_MERGE_PARTS) return VA_ERR_BAD_SHAPE;
    if (p->total_tokens == 0) return VA_OK;
    if (!o_parts || !lse_parts || !o || !lse) return VA_ERR_NULL_PTR;
    if (!aligned16(o_parts) || !aligned16(o) || ((uintptr_t)lse & 3u) || ((uintptr_t)lse_parts & 3u))
        return VA_ERR_MISALIGNED;
    rc = check_device();
    if (rc != VA_OK) return rc;
    hipStream_t stream = (hipStream_t)hip_stream;
    ProfScope ps(VA_KERNEL_MERGE, stream);
    hipError_t e = va::launch_merge(o_parts, false, lse_parts, num_parts, p->total_tokens, p->num_q_heads,
                                    p->head_dim, o, lse, stream);
    if (e != hipSuccess) return hip_fail(e);
    return VA_OK;
}

int varlen_attn_check_cu_seqlens(const varlen_attn_params* p, const int32_t* cu_seqlens, void* workspace,
                                 size_t workspace_bytes, void* hip_stream) {
    int rc = check_params(p);
    if (rc != VA_OK) return rc;
    if (p->num_seqs == 0) return p->total_tokens == 0 ? VA_OK : VA_ERR_BAD_CU_SEQLENS;
    if (!cu_seqlens || !workspace) return VA_ERR_NULL_PTR;
    if (((uintptr_t)cu_seqlens & 3u) || !aligned16(workspace)) return VA_ERR_MISALIGNED;
    if (workspace_bytes < 16) return VA_ERR_WORKSPACE_TOO_SMALL;
    rc = check_device();
    if (rc != VA_OK) return rc;
    hipStream_t stream = (hipStream_t)hip_stream;
    hipError_t e = va::launch_check_cu_seqlens(cu_seqlens, p->num_seqs, p->total_tokens, (int32_t*)workspace, stream);
    if (e != hipSuccess) return hip_fail(e);
    int32_t verdict = 1;
    e = hipMemcpyAsync(&verdict, workspace, sizeof(verdict), hipMemcpyDeviceToHost, stream);
    if (e != hipSuccess) return hip_fail(e);
    e = hipStreamSynchronize(stream);
    if (e != hipSuccess) return hip_fail(e);
    return verdict == 0 ? VA_OK : VA_ERR_BAD_CU_SEQLENS;
}

int varlen_attn_bwd(const varlen_attn_params* p, const void* dout, const void* q, const void* k,
                    const void* v, const void* o, const float* lse, const int32_t* cu_seqlens,
                    void* dq, void* dk, void* dv, void* workspace, size_t workspace_bytes,
                    void* hip_stream) {
    int rc = check_params(p);
    if (rc != VA_OK) return rc;
    if (p->total_tokens == 0 || p->num_seqs == 0) return VA_OK;
    if (!dout || !q || !k || !v || !o || !lse || !cu_seqlens || !dq || !dk || !dv || !workspace)
        return VA_ERR_NULL_PTR;
    if (!aligned16(dout) || !aligned16(q) || !aligned16(k) || !aligned16(v) || !aligned16(o) ||
        !aligned16(dq) || !aligned16(dk) || !aligned16(dv) || !aligned16(workspace) ||
        ((uintptr_t)lse & 3u) || ((uintptr_t)cu_seqlens & 3u))
        return VA_ERR_MISALIGNED;
    const BwdLayout lay = bwd_layout(p, workspace_bytes);
    if (workspace_bytes < lay.end) return VA_ERR_WORKSPACE_TOO_SMALL;
    rc = check_device();
    if (rc != VA_OK) return rc;
    hipStream_t stream = (hipStream_t)hip_stream;
    char* ws = (char*)workspace;

    hipError_t e = hipSuccess;
    if (!lay.small) {   // both work lists (key tiles for dK/dV, query tiles for dQ) in one launch, one workgroup each
        ProfScope ps(VA_KERNEL_SCHED, stream);
        e = va::launch_scheduler_pair(cu_seqlens, p->num_seqs, p->total_tokens, va::BWD_TILE_KV, va::BWD_STEP_Q,
                                      p->causal ? va::COST_CAUSAL_KEY : va::COST_FULL, ws + lay.kv_ofs, lay.kv,
                                      va::BWD_TILE_Q, va::BWD_STEP_KV,
                                      p->causal ? va::COST_CAUSAL_QUERY : va::COST_FULL, ws + lay.q_ofs, lay.q, stream);
    }
    if (e != hipSuccess) return hip_fail(e);

    va::BwdArgs a;
    a.dout = dout; a.q = q; a.k = k; a.v = v; a.o = o; a.lse = lse;
    a.stats = (float*)(ws + lay.stats_ofs);
    a.dq = dq; a.dk = dk; a.dv = dv;
    a.sched_hdr_kv = (const int32_t*)(ws + lay.kv_ofs);
    a.items_kv = (const va::WorkItem*)(ws + lay.kv_ofs + lay.kv.items_ofs);
    a.max_items_kv = lay.kv.max_items;
    a.sched_hdr_q = (const int32_t*)(ws + lay.q_ofs);
    a.items_q = (const va::WorkItem*)(ws + lay.q_ofs + lay.q.items_ofs);
    a.max_items_q = lay.q.max_items;
    a.total_tokens = p->total_tokens; a.num_q_heads = p->num_q_heads; a.num_kv_heads = p->num_kv_heads;
    a.head_dim = p->head_dim; a.causal = p->causal; a.scale = p->softmax_scale;
    a.small = lay.small;
    a.cu_seqlens = cu_seqlens;
    a.num_seqs = p->num_seqs;
    a.plan_q = lay.plan_q; a.plan_kv = lay.plan_kv;
    a.part_dq = (float*)(ws + lay.part_dq_ofs);
    a.part_dk = (float*)(ws + lay.part_dk_ofs);
    a.part_dv = (float*)(ws + lay.part_dv_ofs);
    a.ws_kv = ws + lay.kv_ofs; a.ws_q = ws + lay.q_ofs;
    a.lay_kv = lay.kv; a.lay_q = lay.q;
    a.clock_probe_dkdv = clock_probe_slot(1);
    a.clock_probe_dq = clock_probe_slot(2);
    // dQ first: it also writes the row statistics {LSE * log2 e, -Delta} that dK/dV reads
    {
        ProfScope ps(VA_KERNEL_DQ, stream);
        e = va::launch_bwd_dq(a, stream);
    }
    if (e != hipSuccess) return hip_fail(e);
    {
        ProfScope ps(VA_KERNEL_DKDV, stream);
        e = va::launch_bwd_dkdv(a, stream);
    }
    if (e != hipSuccess) return hip_fail(e);
    if (lay.plan_q.max_chunks > 1 || lay.plan_kv.max_chunks > 1) {
        ProfScope ps(VA_KERNEL_MERGE, stream);
        e = va::launch_bwd_sum_small(a, stream);
        if (e != hipSuccess) return hip_fail(e);
    }
    return VA_OK;
}

const char* varlen_attn_status_string(int status) {
    switch (status) {
        case VA_OK: return "ok";
        case VA_ERR_NULL_PTR: return "a required pointer is NULL";
        case VA_ERR_BAD_SHAPE: return "bad shape: negative size or count, head counts, causal flag, kv_splits, or launch too large";
        case VA_ERR_UNSUPPORTED: return "unsupported: head_dim must be 64, 80, 96 or 128 and the device gfx950";
        case VA_ERR_WORKSPACE_TOO_SMALL: return "workspace too small";
        case VA_ERR_BAD_SCALE: return "softmax_scale must be finite and >= 0";
        case VA_ERR_HIP: return "a HIP call failed";
        case VA_ERR_MISALIGNED: return "a tensor or workspace pointer is not 16-byte aligned";
        case VA_ERR_BAD_CU_SEQLENS: return "cu_seqlens must start at 0, never decrease and end at total_tokens";
        case VA_ERR_SCRATCH_LIMIT: return "the call needs more scratch than the library's static array holds (VA_STATIC_SCRATCH_BYTES)";
        default: return "unknown status";
    }
}

int varlen_attn_last_hip_error(void) { return g_last_hip_error; }

int varlen_attn_profile_enable(int on) {
    std::lock_guard<std::mutex> lock(g_prof_mutex);
    if (on) prof_clear_locked();
    g_prof_on = on != 0;
    return VA_OK;
}

int varlen_attn_profile_read(int kernel, double* total_ms, int64_t* launches) {
    if (!total_ms || !launches) return VA_ERR_NULL_PTR;
    std::lock_guard<std::mutex> lock(g_prof_mutex);
    double sum = 0.0;
    int64_t n = 0;
    for (auto& s : g_prof_samples) {
        if (s.kernel != kernel) continue;
        hipError_t e = hipEventSynchronize(s.b);
        if (e != hipSuccess) return hip_fail(e);
        float ms = 0.f;
        e = hipEventElapsedTime(&ms, s.a, s.b);
        if (e != hipSuccess) return hip_fail(e);
        sum += ms;
        ++n;
    }
    *total_ms = sum;
    *launches = n;
    return VA_OK;
}

int varlen_attn_profile_clock_probe(unsigned long long* device_counters) {
    if (((uintptr_t)device_counters & 7u) != 0) return VA_ERR_MISALIGNED;
    std::lock_guard<std::mutex> lock(g_prof_mutex);
    g_clock_probe = device_counters;
    return VA_OK;
}

}  // extern "C"
