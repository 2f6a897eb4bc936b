// Merge of partial attention results over disjoint key/value shards (HBM-bound, elementwise):
//     LSE = ln sum_p exp(LSE_p),   O = sum_p exp(LSE_p - LSE) O_p,
// the combination that context parallelism over key shards needs (Section 4.1.2 selects it for
// overlong contexts, Section 5.2 shards long samples for it) and that the forward uses itself when it
// splits the keys of a small launch over several workgroups.  A part with LSE_p = -inf is empty and
// its O_p is never multiplied (it may hold anything).
#include "va_device.h"
#include "va_internal.h"

namespace va {

// One thread per (token, head, 8 consecutive channels).  Parts: PartT [P, T, H, D], lse [P, H, T].
// NP > 0: the number of parts is known at compile time, so that all loads of a thread are in flight
// together (the kernel is bound by HBM latency x bytes in flight otherwise); NP = 0: any P.
// STREAM: the parts and the result go past the caches (every byte is touched once), for merges larger than what the
// caches hold.  Measured on bf16 parts: 4 x 178572 tokens x 16 heads of 64 347 -> 330 us (5.4 -> 5.7 TB/s), 8 x 60000 x
// 16 heads of 80 269 -> 248 us, 6 x 150000 x 8 heads of 128 400 -> 360 us; 3 x 20001 x 4 heads of 96 (62 MB in all)
// 13.8 -> 14.2 us.  Reading the LSE from the XCD's own eighth of the rows, 32-bit index arithmetic and loads issued
// ahead of the LSE's made no difference.
template <typename PartT, int NP, bool STREAM>
__global__ void __launch_bounds__(256)
merge_kernel(const PartT* __restrict__ o_parts, const float* __restrict__ lse_parts, int P_rt, int T, int H, int D,
             __bf16* __restrict__ o, float* __restrict__ lse) {
    const int P = NP > 0 ? NP : P_rt;
    const int cpr = D / 8;  // chunks per (token, head) row
    const int64_t idx = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (idx >= (int64_t)T * H * cpr) return;
    const int c = (int)(idx % cpr);
    const int64_t row = idx / cpr;  // token * H + head
    const int h = (int)(row % H);
    const int64_t t = row / H;
    const size_t lse_stride = (size_t)H * T, o_stride = (size_t)T * H * D;
    const float* lp = lse_parts + (size_t)h * T + t;

    float mx = -INFINITY;
#pragma unroll
    for (int p = 0; p < P; ++p) mx = fmaxf(mx, lp[p * lse_stride]);
    float acc[8] = {0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f};
    float total = -INFINITY;
    if (mx != -INFINITY) {
        float den = 0.f;
#pragma unroll
        for (int p = 0; p < P; ++p) den += __expf(lp[p * lse_stride] - mx);
        total = mx + __logf(den);
        const float inv = 1.f / den;
        const PartT* op = o_parts + (size_t)row * D + 8 * c;
#pragma unroll
        for (int p = 0; p < P; ++p) {
            const float x = lp[p * lse_stride];
            if (x == -INFINITY) continue;  // empty part: its O is not read
            const float wgt = __expf(x - mx) * inv;
            if constexpr (sizeof(PartT) == 2) {
                const u32x4* vp = (const u32x4*)(op + p * o_stride);
                const bf16x8 v = __builtin_bit_cast(bf16x8, STREAM ? __builtin_nontemporal_load(vp) : *vp);
#pragma unroll
                for (int e = 0; e < 8; ++e) acc[e] += wgt * (float)v[e];
            } else {
                const float4 v0 = *(const float4*)(op + p * o_stride), v1 = *(const float4*)(op + p * o_stride + 4);
                acc[0] += wgt * v0.x; acc[1] += wgt * v0.y; acc[2] += wgt * v0.z; acc[3] += wgt * v0.w;
                acc[4] += wgt * v1.x; acc[5] += wgt * v1.y; acc[6] += wgt * v1.z; acc[7] += wgt * v1.w;
            }
        }
    }
    bf16x8 out;
#pragma unroll
    for (int e = 0; e < 8; ++e) out[e] = (__bf16)acc[e];
    u32x4* const dst = (u32x4*)(o + (size_t)row * D + 8 * c);
    if (STREAM) __builtin_nontemporal_store(__builtin_bit_cast(u32x4, out), dst);
    else *dst = __builtin_bit_cast(u32x4, out);
    if (c == 0) lse[(size_t)h * T + t] = total;
}

hipError_t launch_merge(const void* o_parts, bool parts_fp32, const float* lse_parts, int P, int T, int H, int D,
                        void* o, float* lse, hipStream_t stream) {
    const int64_t n = (int64_t)T * H * (D / 8);
    if (n == 0) return hipSuccess;
    dim3 grid((unsigned)((n + 255) / 256)), block(256);
    // beyond the 256 MB of the last-level cache nothing written or read here is found there again
    const bool stream_past = !parts_fp32 && (int64_t)(P + 1) * n * 16 > (int64_t)256 << 20;
#define VA_MERGE_LAUNCH(PT, NP, STREAM)                                                                      \
    hipLaunchKernelGGL((merge_kernel<PT, NP, STREAM>), grid, block, 0, stream, (const PT*)o_parts, lse_parts, P, T, H, D, \
                       (__bf16*)o, lse)
#define VA_MERGE_DISPATCH(PT, STREAM)                                        \
    switch (P) {                                                             \
        case 1: VA_MERGE_LAUNCH(PT, 1, STREAM); break;                       \
        case 2: VA_MERGE_LAUNCH(PT, 2, STREAM); break;                       \
        case 3: VA_MERGE_LAUNCH(PT, 3, STREAM); break;                       \
        case 4: VA_MERGE_LAUNCH(PT, 4, STREAM); break;                       \
        case 5: VA_MERGE_LAUNCH(PT, 5, STREAM); break;                       \
        case 6: VA_MERGE_LAUNCH(PT, 6, STREAM); break;                       \
        case 7: VA_MERGE_LAUNCH(PT, 7, STREAM); break;                       \
        case 8: VA_MERGE_LAUNCH(PT, 8, STREAM); break;                       \
        default: VA_MERGE_LAUNCH(PT, 0, STREAM); break;                      \
    }
    if (parts_fp32) { VA_MERGE_DISPATCH(float, false) }
    else if (stream_past) { VA_MERGE_DISPATCH(__bf16, true) }
    else { VA_MERGE_DISPATCH(__bf16, false) }
#undef VA_MERGE_DISPATCH
#undef VA_MERGE_LAUNCH
    return hipGetLastError();
}

}  // namespace va
