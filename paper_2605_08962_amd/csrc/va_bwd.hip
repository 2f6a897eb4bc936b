// Backward kernels.  P is recomputed from Q, K and the saved LSE (the paper recomputes core
// attention in the backward pass, Section 6 "Selective Activation Offloading").
//
//   (row statistics: per (head, row) LSE * log2(e) and -Delta = -sum_d dO * O; every dQ workgroup
//    computes them for its own 128 rows while it loads its fragments and writes them to the workspace,
//    where the dK/dV kernel, launched after it, finds them.  Delta is stored negated so that the dK/dV
//    kernel can load it straight into the accumulator of dP = dO V^T and get dP - Delta for free.)
//   dkdv   : one workgroup per (128-row key tile, kv head); loops over the query heads of the
//            group and over 64-row query steps; S = Q K^T is kept with one KEY per lane, so
//            that P and dS are directly the B operands of dV^T += dO^T P and dK^T += Q^T dS
//            (contraction over query rows).
//   dq     : one workgroup per (128-row query tile, query head); loops over 64-row key steps;
//            S^T = K Q^T is kept with one QUERY per lane (as in the forward), so that dS^T is the
//            B operand of dQ^T += K^T dS^T (contraction over key rows).
// Splitting the backward this way needs no atomics and no fp32 dQ buffer, and the result does not
// depend on scheduling order; it recomputes S and dP once more than a fused kernel would.
//
// Staging is the forward's: 64-row tiles go straight from HBM/L2 into XOR-swizzled LDS tiles with
// direct-to-LDS loads, two (dQ), three or four (dK/dV) stages deep, one barrier per step, completion tracked with vmcnt.
//
// The file is compiled in five parts (VA_BWD_PART), each under the instruction-scheduling strategy of the compiler that
// measured best for its kernels (build.py): 1 dK/dV at head_dim 128, causal; 2 dQ; 3 dK/dV at 80; 4 dK/dV at 96, and at 128
// without the mask; 0 the rest.
#include "va_device.h"
#include "va_internal.h"
#include "va_sched.h"
#include "va_small.h"

#ifndef VA_BWD_PART
#define VA_BWD_PART 0
#endif

namespace va {
hipError_t launch_dkdv_128_causal(const BwdArgs& a, hipStream_t stream);  // part 1
hipError_t launch_dkdv_80(const BwdArgs& a, hipStream_t stream);          // part 3
hipError_t launch_dkdv_96(const BwdArgs& a, hipStream_t stream);          // part 4
hipError_t launch_dkdv_128_full(const BwdArgs& a, hipStream_t stream);    // part 4

template <int D>
struct BwdCfg {
    using T = LdsTile<D>;
    static constexpr int KS = D / 16;
    static constexpr int DB = (D + 31) / 32;
    static constexpr int TILE = 64 * T::ROWB;        // one 64-row tile in LDS
    static constexpr int NI = TileDma<D, 64>::NI;    // load instructions per wave per tile
    static constexpr int EXTRA = TileDma<D, 64>::EXTRA;  // and per pair of tiles
    static constexpr int STAT_BYTES = 4 * 128;       // per wave: 16 x lse2, 16 x delta
};

__device__ __forceinline__ bf16x8 pack_regs(const f32x16& x, int st) {
    return pack8(x[8 * st + 0], x[8 * st + 1], x[8 * st + 2], x[8 * st + 3], x[8 * st + 4], x[8 * st + 5],
                 x[8 * st + 6], x[8 * st + 7]);
}
__device__ __forceinline__ bf16x8 pack_regs_lo(const f32x16& x, int st, bf16x8 hi) {
    bf16x8 r;
#pragma unroll
    for (int e = 0; e < 8; ++e) r[e] = (__bf16)(x[8 * st + e] - bf16_as_float(hi, e));
    return r;
}

// ------------------------------------------------------------------------------------------------
// dK, dV
// ------------------------------------------------------------------------------------------------
// One 64-query step for one wave (32 keys).  MASKED steps apply the causal / sample-end mask and, where
// `lo` is set (wave-uniform), carry P and dS as bf16 hi + lo (see the forward kernel for why).
//   qt, dot : LDS tiles of Q and dO (64 rows);  stat: per 16 rows {16 x lse2, 16 x delta}
//   aaddr   : per-lane offsets of the row-wise 16-byte reads, taddr: of the transposing reads
template <int D, bool CAUSAL, bool MASKED, int OB>
__device__ __forceinline__ void dkdv_step(const unsigned char* qt, const unsigned char* dot,
                                          const unsigned char* stat, const int (&aaddr)[BwdCfg<D>::KS],
                                          const int (&taddr)[OB][2],
                                          const bf16x8 (&kf)[BwdCfg<D>::KS], const bf16x8 (&vf)[BwdCfg<D>::KS],
                                          f32x16 (&dkacc)[OB], f32x16 (&dvacc)[OB],
                                          float c2, int q0, int kv, int L, int hh, bool lo, int wk_lo) {
    using C = BwdCfg<D>;
    constexpr int ROWB = C::T::ROWB;
    // without the causal mask every masked step carries lo parts, next to the hi parts' MFMAs; under it few
    // steps do (`lo`), in a pass of their own behind one wave-uniform branch
    constexpr bool LO_INLINE = MASKED && !CAUSAL;
    // rows that exist and see this lane's key, counted from the lane's first: comparisons with constants (what a key beyond
    // the sample makes of them stays in its lane and is not stored)
    const int end_row = L - q0 - 4 * hh, first_row = kv - q0 - 4 * hh;
    // The two 32-query halves of the step are handled one after the other, so that only one half's
    // scores and dP (2 x 16 registers) are live at a time.
#pragma unroll
    for (int qb = 0; qb < 2; ++qb) {
        // The sample ends in the first half: the second adds zeros (half of all samples end so).  With the same in dQ:
        // 256 samples of 64..1024 tokens, 16 heads of 80, dK/dV 758 -> 736 us, dQ 628 -> 618; the ViT batch 5040 -> 5008
        // and 3710 -> 3691; the LLM batch's dK/dV 2421 -> 2381 (four runs of each in turn, apart by 3, 5 and 25 us).
        if (MASKED && qb && q0 + 32 >= L) break;
        // Under the causal mask: no row of the first half sees a key of this wave (16 heads of 64, 64..1024 tokens, 417 -> 409 us,
        // LLM batch 2397 -> 2374; slices, alone on their SIMDs, wait for the other waves anyway).
        if (MASKED && CAUSAL && OB == C::DB && qb == 0 && q0 + 31 < wk_lo) continue;
        // keep the instruction scheduler from hoisting the second half's LDS reads over the first
        // half: it would hold both halves' operands in registers and spill
        // (a slice has the registers, and nothing else on its SIMD to hide one half's latencies behind)
        if (qb && OB == C::DB) __builtin_amdgcn_sched_barrier(0);
        f32x16 s, dp;
        float lv[16];
#pragma unroll
        for (int r4 = 0; r4 < 4; ++r4) {
            const int qoff = 32 * qb + 8 * r4 + 4 * hh;  // 4 consecutive query rows, inside one 16-row block
            const unsigned char* sp = stat + (qoff >> 4) * 128 + (qoff & 15) * 4;
            const float4 l4 = *(const float4*)(sp);
            const float4 d4 = *(const float4*)(sp + 64);
            lv[4 * r4 + 0] = l4.x; lv[4 * r4 + 1] = l4.y; lv[4 * r4 + 2] = l4.z; lv[4 * r4 + 3] = l4.w;
            // dP accumulates on top of -Delta
            dp[4 * r4 + 0] = d4.x; dp[4 * r4 + 1] = d4.y; dp[4 * r4 + 2] = d4.z; dp[4 * r4 + 3] = d4.w;
        }
#pragma unroll
        for (int r = 0; r < 16; ++r) s[r] = 0.f;
#pragma unroll
        for (int ks = 0; ks < C::KS; ++ks) {
            bf16x8 aq = *(const bf16x8*)(qt + aaddr[ks] + qb * 32 * ROWB);
            s = mfma32(aq, kf[ks], s);
            bf16x8 ad = *(const bf16x8*)(dot + aaddr[ks] + qb * 32 * ROWB);
            dp = mfma32(ad, vf[ks], dp);
        }
#pragma unroll
        for (int r = 0; r < 16; ++r) {
            float p = fast_exp2(__builtin_fmaf(s[r], c2, -lv[r]));
            if (MASKED) {
                const int c = 32 * qb + 8 * (r / 4) + (r % 4);
                p = c < end_row && (!CAUSAL || c >= first_row) ? p : 0.f;
            }
            s[r] = p;
            dp[r] = p * dp[r];
        }
        bf16x8 pk[2], dsk[2];
#pragma unroll
        for (int st = 0; st < 2; ++st) {
            const bf16x8 pb = pk[st] = pack_regs(s, st);
            const bf16x8 dsb = dsk[st] = pack_regs(dp, st);
            bf16x8 pl, dsl;
            if (LO_INLINE) { pl = pack_regs_lo(s, st, pb); dsl = pack_regs_lo(dp, st, dsb); }
            const int rowoff = (32 * qb + 16 * st) * ROWB;
#pragma unroll
            for (int db = 0; db < OB; ++db) {
                bf16x8 ado = cat4(lds_read_tr(dot + rowoff + taddr[db][0]), lds_read_tr(dot + rowoff + taddr[db][1]));
                dvacc[db] = mfma32(ado, pb, dvacc[db]);
                if (LO_INLINE) dvacc[db] = mfma32(ado, pl, dvacc[db]);
                bf16x8 aq = cat4(lds_read_tr(qt + rowoff + taddr[db][0]), lds_read_tr(qt + rowoff + taddr[db][1]));
                dkacc[db] = mfma32(aq, dsb, dkacc[db]);
                if (LO_INLINE) dkacc[db] = mfma32(aq, dsl, dkacc[db]);
            }
        }
        if (MASKED && CAUSAL && lo) {
#pragma unroll
            for (int st = 0; st < 2; ++st) {
                const bf16x8 pl = pack_regs_lo(s, st, pk[st]);
                const bf16x8 dsl = pack_regs_lo(dp, st, dsk[st]);
                const int rowoff = (32 * qb + 16 * st) * ROWB;
#pragma unroll
                for (int db = 0; db < OB; ++db) {
                    bf16x8 ado = cat4(lds_read_tr(dot + rowoff + taddr[db][0]), lds_read_tr(dot + rowoff + taddr[db][1]));
                    dvacc[db] = mfma32(ado, pl, dvacc[db]);
                    bf16x8 aq = cat4(lds_read_tr(qt + rowoff + taddr[db][0]), lds_read_tr(qt + rowoff + taddr[db][1]));
                    dkacc[db] = mfma32(aq, dsl, dkacc[db]);
                }
            }
        }
    }
}

// ---- the mask-free step, cut into phases whose LDS operands are fetched one phase ahead ----
// An LDS read takes a few hundred cycles to return while an MFMA issues every 32; left to itself
// the compiler puts each read right in front of the MFMA that consumes it and the matrix pipe
// waits most of the time.  Here every phase first ISSUES the reads of the next phase into a second
// set of registers and then runs its own MFMAs / vector work on operands that arrived long ago;
// sched_barriers keep the phases apart.
template <int D>
struct DkdvOpsA {  // operands of S = Q K^T and dP = dO V^T for one 32-query half
    bf16x8 q[BwdCfg<D>::KS], d[BwdCfg<D>::KS];
};
template <int D, int OB>
struct DkdvOpsC {  // operands of dV^T += dO^T P and dK^T += Q^T dS for one half
    bf16x8 o[2][OB], q[2][OB];
};
template <int D, int HALF>
__device__ __forceinline__ void dkdv_load_A(const unsigned char* stage, const int (&aaddr)[BwdCfg<D>::KS],
                                            DkdvOpsA<D>& f, f32x16& dp, int hh) {
    using C = BwdCfg<D>;
    constexpr int ROWB = C::T::ROWB;
    const unsigned char* stat = stage + 2 * C::TILE;
#pragma unroll
    for (int ks = 0; ks < C::KS; ++ks) {
        f.q[ks] = *(const bf16x8*)(stage + aaddr[ks] + HALF * 32 * ROWB);
        f.d[ks] = *(const bf16x8*)(stage + C::TILE + aaddr[ks] + HALF * 32 * ROWB);
    }
#pragma unroll
    for (int r4 = 0; r4 < 4; ++r4) {  // dP accumulates on top of -Delta
        const int qoff = 32 * HALF + 8 * r4 + 4 * hh;
        const float4 d4 = *(const float4*)(stat + (qoff >> 4) * 128 + (qoff & 15) * 4 + 64);
        dp[4 * r4 + 0] = d4.x; dp[4 * r4 + 1] = d4.y; dp[4 * r4 + 2] = d4.z; dp[4 * r4 + 3] = d4.w;
    }
}
template <int D, int HALF>
__device__ __forceinline__ void dkdv_load_lse(const unsigned char* stage, float (&lv)[16], int hh) {
    const unsigned char* stat = stage + 2 * BwdCfg<D>::TILE;
#pragma unroll
    for (int r4 = 0; r4 < 4; ++r4) {
        const int qoff = 32 * HALF + 8 * r4 + 4 * hh;
        const float4 l4 = *(const float4*)(stat + (qoff >> 4) * 128 + (qoff & 15) * 4);
        lv[4 * r4 + 0] = l4.x; lv[4 * r4 + 1] = l4.y; lv[4 * r4 + 2] = l4.z; lv[4 * r4 + 3] = l4.w;
    }
}
template <int D, int HALF, int OB>
__device__ __forceinline__ void dkdv_load_C(const unsigned char* stage, const int (&taddr)[OB][2],
                                            DkdvOpsC<D, OB>& f) {
    using C = BwdCfg<D>;
    constexpr int ROWB = C::T::ROWB;
#pragma unroll
    for (int st = 0; st < 2; ++st) {
        const unsigned char* qt = stage + (32 * HALF + 16 * st) * ROWB;
        const unsigned char* dot = qt + C::TILE;
#pragma unroll
        for (int db = 0; db < OB; ++db) {
            f.o[st][db] = cat4(lds_read_tr(dot + taddr[db][0]), lds_read_tr(dot + taddr[db][1]));
            f.q[st][db] = cat4(lds_read_tr(qt + taddr[db][0]), lds_read_tr(qt + taddr[db][1]));
        }
    }
}
template <int D>
__device__ __forceinline__ void dkdv_run_A(const DkdvOpsA<D>& f, const bf16x8 (&kf)[BwdCfg<D>::KS],
                                           const bf16x8 (&vf)[BwdCfg<D>::KS], f32x16& s, f32x16& dp) {
#pragma unroll
    for (int r = 0; r < 16; ++r) s[r] = 0.f;
#pragma unroll
    for (int ks = 0; ks < BwdCfg<D>::KS; ++ks) {
        s = mfma32(f.q[ks], kf[ks], s);
        dp = mfma32(f.d[ks], vf[ks], dp);
    }
}
// P = exp2(S c2 - lse2) and dS = P (dP - Delta), rounded to bf16 (vector ALU only)
__device__ __forceinline__ void dkdv_run_B(const f32x16& s, const f32x16& dp, const float (&lv)[16], float c2,
                                           bf16x8 (&pb)[2], bf16x8 (&dsb)[2]) {
    f32x16 p, ds;
#pragma unroll
    for (int r = 0; r < 16; ++r) {
        p[r] = fast_exp2(__builtin_fmaf(s[r], c2, -lv[r]));
        ds[r] = p[r] * dp[r];
    }
#pragma unroll
    for (int st = 0; st < 2; ++st) {
        pb[st] = pack_regs(p, st);
        dsb[st] = pack_regs(ds, st);
    }
}
template <int D, int OB>
__device__ __forceinline__ void dkdv_run_C(const DkdvOpsC<D, OB>& f, const bf16x8 (&pb)[2], const bf16x8 (&dsb)[2],
                                           f32x16 (&dkacc)[OB], f32x16 (&dvacc)[OB]) {
#pragma unroll
    for (int st = 0; st < 2; ++st)
#pragma unroll
        for (int db = 0; db < OB; ++db) {
            dvacc[db] = mfma32(f.o[st][db], pb[st], dvacc[db]);
            dkacc[db] = mfma32(f.q[st][db], dsb[st], dkacc[db]);
        }
}

// The same work cut differently: S alone, then dP, dV and dK with the vector work in their shadow.
// A wave that has just issued an MFMA cannot issue anything for about 16 cycles and is then free for
// about 16 more before the matrix pipe takes the next one (measured: up to 3 vector instructions per
// MFMA cost nothing, further ones about 4.5 cycles each).  Vector work that does not depend on the
// MFMAs around it is therefore cheapest when spread between them.
template <int D>
__device__ __forceinline__ void dkdv_run_S(const DkdvOpsA<D>& f, const bf16x8 (&kf)[BwdCfg<D>::KS], f32x16& s) {
#pragma unroll
    for (int r = 0; r < 16; ++r) s[r] = 0.f;
#pragma unroll
    for (int ks = 0; ks < BwdCfg<D>::KS; ++ks) s = mfma32(f.q[ks], kf[ks], s);
}
template <int D>
__device__ __forceinline__ void dkdv_run_dP(const DkdvOpsA<D>& f, const bf16x8 (&vf)[BwdCfg<D>::KS], f32x16& dp) {
#pragma unroll
    for (int ks = 0; ks < BwdCfg<D>::KS; ++ks) dp = mfma32(f.d[ks], vf[ks], dp);
}
// rounds of {1 MFMA, DS_PER LDS reads, VALU_PER vector instructions} for the region that ends here
template <int N_MFMA, int DS_PER, int VALU_PER>
__device__ __forceinline__ void dkdv_interleave() {
#pragma unroll
    for (int i = 0; i < N_MFMA; ++i) {
        __builtin_amdgcn_sched_group_barrier(0x008, 1, 0);
        if (DS_PER) __builtin_amdgcn_sched_group_barrier(0x100, DS_PER, 0);
        __builtin_amdgcn_sched_group_barrier(0x002, VALU_PER, 0);
    }
}

// Load K of the 2*NI + EXTRA + 1 direct-to-LDS loads of one dK/dV step: K = 0 the stats, then NI loads of the Q
// tile, NI of the dO tile, and what is left of the two.  K beyond that is a no-op, so callers can name slots freely.
template <int D, int K>
__device__ __forceinline__ void dkdv_issue_part(bool ragged, const TileDma<D, 64>& dma, const unsigned char* q,
                                                const unsigned char* dO, const unsigned char* st,
                                                uint32_t stat_off, uint32_t lds, int wave) {
    constexpr int NI = BwdCfg<D>::NI;
    if constexpr (K == 0) {
        dma4(st, stat_off, lds + 2 * BwdCfg<D>::TILE + (wave & 1) * 256);
    } else if constexpr (K <= NI) {
        dma.issue_one(K - 1, q, ragged, lds, wave);
    } else if constexpr (K <= 2 * NI) {
        dma.issue_one(K - 1 - NI, dO, ragged, lds + BwdCfg<D>::TILE, wave);
    } else if constexpr (K == 2 * NI + 1) {
        dma.issue_extra(q, dO, ragged, ragged, lds, lds + BwdCfg<D>::TILE, wave);
    }
}

// Chunks of the walks of a small launch (va_small.h).
struct DkdvSmall {
    const int32_t* cu;
    int num_seqs;
    SmallPlan plan;
    float *part_dk, *part_dv;  // fp32 [chunks, T, Hkv, D]
};
// (Spilled: at 128 under the causal mask one vector register, into the accumulation half, read back three times a step; at 80
// five in the small form without the mask and two in the general one under it, outside the loops.)
template <int D>
constexpr int kDkdvWgsPerCu = D <= 80 ? 2 : 1;

template <bool CAUSAL>
__device__ __forceinline__ SmallShape dkdv_small_shape(int Hq, int Hkv, const SmallPlan& plan, int room = 0) {
    return SmallShape{BWD_TILE_KV, BWD_STEP_Q, CAUSAL ? COST_CAUSAL_KEY : COST_FULL, Hkv, Hq / Hkv, plan, room};
}

// OB: 32-column blocks of dK and dV a workgroup computes.  All of them, or one (SMALL only): then C::DB workgroups share
// a tile, each forms S and dP in full and its own columns of the results, in the same order of additions (the same
// bits).  More work in all, for launches that leave most CUs idle while one wave walks a tile alone: it is for such
// walks that are not cut into chunks (dkdv_sliced).  Six causal samples of 30..200 tokens, 4 query heads on one kv head of
// 128, forward + backward: 65.0 -> 53.7 us (dK/dV, 16 steps one after the other, 43 -> 31 us).
// SMALL: the walk of a key tile (the steps of all query heads of its group, one after the other) may be cut into
// chunks, one workgroup each, which leave fp32 results for bwd_sum_small.
template <int D, bool CAUSAL, bool SMALL, int OB = BwdCfg<D>::DB>
__global__ void __launch_bounds__(256, (kDkdvWgsPerCu<D>))
dkdv_kernel(const __bf16* __restrict__ Q, const __bf16* __restrict__ K, const __bf16* __restrict__ V,
            const __bf16* __restrict__ dO, const float2* __restrict__ stats,
            __bf16* __restrict__ dK, __bf16* __restrict__ dV, const int32_t* __restrict__ hdr,
            const WorkItem* __restrict__ items, int max_items, int T, int Hq, int Hkv, float scale, DkdvSmall small,
            unsigned long long* __restrict__ clock_probe) {
    using C = BwdCfg<D>;
    using LT = LdsTile<D>;
    constexpr int STAGE = 2 * C::TILE + C::STAT_BYTES;  // Q tile, dO tile, stats
    constexpr int PER = 2 * C::NI + C::EXTRA + 1;       // loads per wave per step
    // LDS stages: four where two workgroups per CU are out of reach anyway or still fit (head_dim 64),
    // three at head_dim 80, where the fourth would cost the second workgroup
    constexpr int NST = D == 80 ? 3 : 4;
    // Mask-free steps whose loads stay inside the head take pointers by addition and no choice of offsets (15 scalar and 6
    // vector instructions fewer per step; head_dim 80 spills 11 registers in the loop's second copy and goes without); at
    // head_dim 64 whole rounds of the stages are written out besides, their LDS addresses constants (elsewhere the copies cost
    // registers the kernel does not have; slices take a handful of steps, for which less code is better).  Measured: 64 ViT
    // samples, 16 heads of 64 5149 -> 5071 us, of 96 8453 -> 8385; LLM batch at 96 1926 -> 1895; at 128 even.
    constexpr bool UNROLLED = D == 64 && OB == C::DB;
    constexpr bool STEADY = D != 80 && OB == C::DB;
    __shared__ __attribute__((aligned(1024))) unsigned char lds[NST * STAGE];

    constexpr unsigned SLICES = C::DB / OB;
    static_assert(SLICES == 1 || (SMALL && OB == 1), "slices of one 32-column block, of small launches");
    const int db0 = SLICES > 1 ? (int)(blockIdx.x % SLICES) : 0;  // first of this workgroup's 32-column blocks
    int item, c;  // work item and kv head (see xcd_item_head)
    WorkItem it;
    SmallTile tl = {};
    if constexpr (SMALL) {
        const unsigned bid = blockIdx.x / SLICES;
        c = __builtin_amdgcn_readfirstlane((int)(bid % (unsigned)Hkv));
        if (!small_tile(small.cu, small.num_seqs, T, dkdv_small_shape<CAUSAL>(Hq, Hkv, small.plan, CAUSAL ? 256 : 256 * kDkdvWgsPerCu<D>),
                        __builtin_amdgcn_readfirstlane((int)(bid / (unsigned)Hkv)), tl))
            return;
    } else {
        if (hdr[1] == 1) short_item_head(blockIdx.x, max_items, Hkv, Hkv, D, item, c);
        else xcd_item_head(blockIdx.x, max_items, Hkv, Hkv, kXcdChunk, item, c);
        // (integer division runs on the vector ALU: without this, everything derived from the two, the
        // staging pointers included, would be kept in vector registers and advanced there)
        item = __builtin_amdgcn_readfirstlane(item); c = __builtin_amdgcn_readfirstlane(c);
        if (item >= hdr[0]) return;
    }
    ClockProbe wg_clock;
    wg_clock.begin(clock_probe);
    stagger_wave_priority();
    const int g = Hq / Hkv;
    if constexpr (!SMALL) {
        it = items[item];
        if (hdr[1] == 1)
            c = __builtin_amdgcn_readfirstlane(
                short_rotated_head(c, item, __builtin_amdgcn_readfirstlane(it.y), Hkv, Hkv, D));
    }
    // same for the whole workgroup: tell the compiler, so that everything derived stays in SGPRs
    const int sb = SMALL ? tl.begin : __builtin_amdgcn_readfirstlane(it.y),
              L = SMALL ? tl.len : __builtin_amdgcn_readfirstlane(it.z - it.y),
              kv0 = SMALL ? tl.tile * BWD_TILE_KV : __builtin_amdgcn_readfirstlane(it.x - it.y);

    const int tid = threadIdx.x, w = uniform_wave_id(), l = tid & 63, ln = l & 31, hh = l >> 5;
    const int kv = kv0 + 32 * w + ln;  // this lane's key row inside the sample
    const bool kvalid = kv < L;

    const int first = CAUSAL ? kv0 / BWD_STEP_Q : 0;               // first query step that can see this tile
    const int nsteps = (L + BWD_STEP_Q - 1) / BWD_STEP_Q - first;  // >= 1 because kv0 < L
    // Steps [0, n_head) sit on the causal diagonal, steps [n_tail, nsteps) hold the sample's ragged
    // end (its out-of-range rows are staged as copies of the last row and must be masked); samples
    // shorter than one step are all "careful".  Steps in between need no mask in any wave.
    const int n_head = (L < BWD_STEP_Q) ? nsteps : (CAUSAL ? min(2, nsteps) : 0);
    const int n_tail = max(n_head, nsteps - ((L % BWD_STEP_Q) ? 1 : 0));

    // Staging state: pointers to the next (head, step) to issue, advanced by additions only.  Every
    // quantity here is wave-uniform (scalar registers).  Loads are issued unconditionally: once the
    // last step has been issued the state stops advancing and later calls fetch that step again into
    // a stage nobody will read, so that the loop needs no branches around its loads and the count of
    // outstanding loads per step is the same everywhere.
    const uint32_t q_row_bytes = (uint32_t)Hq * D * 2;
    TileDma<D, 64> dma;  // Q and dO share the offsets
    dma.init(q_row_bytes, L, w, l);
    // stats: a wave fetches {lse2, -Delta} of 32 rows (waves w and w + 2 fetch the same ones): lanes
    // [0,16) lse2 and [16,32) -Delta of the first 16 rows, lanes [32,64) the same of the next 16
    const int srow = 32 * (w & 1) + 16 * (l >> 5) + (l & 15);
    const int last_q0 = (L - 1) / BWD_STEP_Q * BWD_STEP_Q;
    const uint32_t stat_full = (uint32_t)srow * 8 + ((l >> 4) & 1) * 4;
    const uint32_t stat_last = (uint32_t)min(srow, L - 1 - last_q0) * 8 + ((l >> 4) & 1) * 4;
    const uint32_t lds0 = lds_address(lds);
    // this workgroup's part of the g * nsteps steps: all of them, or one chunk
    int total = g * nsteps, head0 = 0, step0 = 0;
    const int ch = tl.ch, nch = SMALL ? tl.nch : 1;
    if constexpr (SMALL) {
        const int nb = tl.first_step();
        total = tl.end_step() - nb;
        head0 = __builtin_amdgcn_readfirstlane(nb / nsteps);
        step0 = nb - head0 * nsteps;
    }
    const bool ragged_sample = (L % BWD_STEP_Q) != 0;
    const int64_t step_q = (int64_t)BWD_STEP_Q * q_row_bytes, step_st = (int64_t)BWD_STEP_Q * 8;
    const int64_t wrap_q = (int64_t)D * 2 - (int64_t)(nsteps - 1) * step_q;       // last step of a head -> first of the next
    const int64_t wrap_st = (int64_t)T * 8 - (int64_t)(nsteps - 1) * step_st;
    const size_t qoff0 = ((size_t)(sb + (first + step0) * BWD_STEP_Q) * Hq + (size_t)c * g + head0) * D * 2;
    const unsigned char* nxt_q = (const unsigned char*)Q + qoff0;
    const unsigned char* nxt_do = (const unsigned char*)dO + qoff0;
    const unsigned char* nxt_st = (const unsigned char*)(stats + ((size_t)c * g + head0) * T + sb + (first + step0) * BWD_STEP_Q);
    int nxt_s = step0, nxt_n = 0, iss_stage = 0;
    // the step the current round of loads belongs to (set by begin_issue)
    bool iss_ragged = false;
    const unsigned char *iss_q = nullptr, *iss_do = nullptr, *iss_st = nullptr;
    uint32_t iss_lds = 0;
    auto begin_issue = [&]() {
        iss_q = nxt_q; iss_do = nxt_do; iss_st = nxt_st;
        iss_ragged = ragged_sample && nxt_s == nsteps - 1;
        iss_lds = lds0 + iss_stage * STAGE;
        iss_stage = iss_stage == NST - 1 ? 0 : iss_stage + 1;
        const bool more = nxt_n + 1 < total;
        const bool wrap = nxt_s == nsteps - 1;
        const int64_t aq = more ? (wrap ? wrap_q : step_q) : 0, as = more ? (wrap ? wrap_st : step_st) : 0;
        nxt_q += aq; nxt_do += aq; nxt_st += as;
        nxt_s = more ? (wrap ? 0 : nxt_s + 1) : nxt_s;
        nxt_n += more ? 1 : 0;
    };
    auto issue_stat = [&]() {
        dma4(iss_st, iss_ragged ? stat_last : stat_full, iss_lds + 2 * C::TILE + (w & 1) * 256);
    };
    // slot S of 6 per step carries loads S and S + 6
#define VA_DKDV_ISSUE_SLOT(S)                                                                             \
    dkdv_issue_part<D, (S)>(ragged, dma, iss_q, iss_do, iss_st, ragged ? stat_last : stat_full, iss_lds, w); \
    dkdv_issue_part<D, (S) + 6>(ragged, dma, iss_q, iss_do, iss_st, 0, iss_lds, w);
    auto issue_all = [&]() {
        begin_issue();
        issue_stat();
        dma.issue_tile(iss_q, iss_ragged, iss_lds, w, false);
        dma.issue_tile(iss_do, iss_ragged, iss_lds + C::TILE, w, true);
    };

    int aaddr[C::KS], taddr[OB][2];
#pragma unroll
    for (int ks = 0; ks < C::KS; ++ks) aaddr[ks] = LT::off(ln, 2 * ks + hh);
#pragma unroll
    for (int db = 0; db < OB; ++db) {
        taddr[db][0] = LT::tr_off(l, 0, db0 + db);
        taddr[db][1] = LT::tr_off(l, 8, db0 + db);
    }

    // Prologue: the first step and this lane's K and V fragments, all waited for (see the forward kernel for why the register
    // loads must not be left pending at loop entry); only then the next NST - 2 steps, which the first one's work covers.
    // Waiting for those too made every workgroup start with three times the data: 64..1024-token samples, 16 heads of 80 715 ->
    // 706 us, of 96 941 -> 913, of 128 causal 964 -> 920; 64..384 tokens, heads of 64, 391 -> 383; long samples even.
    issue_all();
    bf16x8 kf[C::KS], vf[C::KS];
    {
        const size_t off = ((size_t)(sb + (kvalid ? kv : 0)) * Hkv + c) * D + 8 * hh;
#pragma unroll
        for (int ks = 0; ks < C::KS; ++ks) {
            bf16x8 z = {};
            kf[ks] = kvalid ? *(const bf16x8*)(K + off + 16 * ks) : z;
            vf[ks] = kvalid ? *(const bf16x8*)(V + off + 16 * ks) : z;
        }
    }
    wait_vmcnt<0>();
    wg_barrier();
#pragma unroll
    for (int i = 1; i < NST - 1; ++i) issue_all();
    if constexpr (D > 80) {  // one wave per SIMD: see park_in_acc_registers
#pragma unroll
        for (int ks = 0; ks < C::KS; ++ks) { park_in_acc_registers(kf[ks]); park_in_acc_registers(vf[ks]); }
    }

    f32x16 dkacc[OB], dvacc[OB];
#pragma unroll
    for (int db = 0; db < OB; ++db)
#pragma unroll
        for (int r = 0; r < 16; ++r) { dkacc[db][r] = 0.f; dvacc[db][r] = 0.f; }
    const float c2 = scale * kLog2e;
    const int wk_lo = kv0 + 32 * w;
    // causal: only rows near a sample's start hold few terms, and those meet key tile 0 only
    const bool lo_steps = !CAUSAL || kv0 == 0;

    // Stage protocol.  Step i lives in stage i % NST.  VA_DKDV_SYNC() ends the part of step idx that
    // reads stage idx - 1: it waits until step idx + 1 has landed (with four stages step idx + 2,
    // issued one sync earlier, may stay in flight), passes the barrier, after which every wave is done
    // with stage idx - 1, and refills that stage with step idx + NST - 1.
    int stage_i = 0;  // stage of the current step ("idx" in the comment above)
#define VA_DKDV_SYNC()                                                               \
        wait_vmcnt<(NST - 3) * PER>();                                                   \
        wg_barrier();
#define VA_DKDV_ADVANCE()                                                            \
        stage_i = stage_i == NST - 1 ? 0 : stage_i + 1;
#define VA_DKDV_CAREFUL(st)                                                          \
    {                                                                                    \
        const unsigned char* b = lds + stage_i * STAGE;                                  \
        const int q0 = (first + (st)) * BWD_STEP_Q;                                      \
        /* causal: a query step entirely above this wave's keys sees none of them; every other  \
           step here takes the masked variant (a superset of the plain one) to keep code small */ \
        if (!CAUSAL || q0 + BWD_STEP_Q - 1 >= wk_lo)                                     \
            dkdv_step<D, CAUSAL, true, OB>(b, b + C::TILE, b + 2 * C::TILE, aaddr, taddr, kf, vf, dkacc, dvacc, \
                                       c2, q0, kv, L, hh, lo_steps, wk_lo);              \
        VA_DKDV_SYNC()                                                                   \
        issue_all();                                                                     \
        VA_DKDV_ADVANCE()                                                                \
    }

    // The mask-free step in phases.  Per half: phase A (S, dP MFMAs), phase B (vector ALU), phase C (dV, dK
    // MFMAs); each phase also issues the LDS reads of the phase after it.  The step's sync
    // sits at its start: it only has to retire stage idx - 1, and having stage idx + 1
    // published early lets the last phase fetch the next step's first operands.
    DkdvOpsA<D> fa;
    DkdvOpsC<D, OB> fc;
    f32x16 s, dpa, dpb;  // dP accumulators of the even / odd half, preloaded with -Delta
    float lv[16];
    bf16x8 pb[2], dsb[2];
    // STAGE_TAG: the step's stage where the caller knows it (-1 otherwise); with it the LDS addresses of the
    // operand reads are per-lane offsets plus immediates instead of vector additions per step
    // steady_tag: the step it loads is neither the last of its head nor of the chunk
    auto phased = [&](auto stage_tag, auto steady_tag) {
        constexpr int KNOWN = decltype(stage_tag)::value;
        constexpr bool IN_HEAD = decltype(steady_tag)::value;
        VA_DKDV_SYNC()
        const int si = KNOWN >= 0 ? KNOWN : stage_i;
        const unsigned char* cur = lds + si * STAGE;
        const unsigned char* nxt = lds + (si == NST - 1 ? 0 : si + 1) * STAGE;
        // half 0 (the scalar bookkeeping of this step's loads runs behind its MFMAs)
        dkdv_load_lse<D, 0>(cur, lv, hh);
        dkdv_run_S<D>(fa, kf, s);
        if constexpr (IN_HEAD) {
            iss_q = nxt_q; iss_do = nxt_do; iss_st = nxt_st;
            iss_lds = lds0 + (KNOWN >= 0 ? (KNOWN + NST - 1) % NST : stage_i == 0 ? NST - 1 : stage_i - 1) * STAGE;
            nxt_q += step_q; nxt_do += step_q; nxt_st += step_st;
        } else {
            begin_issue();
        }
        const bool ragged = !IN_HEAD && iss_ragged;
        __builtin_amdgcn_sched_barrier(0);
        VA_DKDV_ISSUE_SLOT(0)
        VA_DKDV_ISSUE_SLOT(1)
        dkdv_load_C<D, 0, OB>(cur, taddr, fc);
        dkdv_run_dP<D>(fa, vf, dpa);
        dkdv_run_B(s, dpa, lv, c2, pb, dsb);
        dkdv_run_C<D, OB>(fc, pb, dsb, dkacc, dvacc);
        dkdv_load_A<D, 1>(cur, aaddr, fa, dpb, hh);
        dkdv_interleave<C::KS, 8 * OB / C::KS, 14>();   // dP; dV/dK operand reads; P
        dkdv_interleave<4 * OB, 2, 2>();                // dV, dK; next half's S/dP operand reads; dS
        __builtin_amdgcn_sched_barrier(0);
        VA_DKDV_ISSUE_SLOT(2)
        // half 1
        dkdv_load_lse<D, 1>(cur, lv, hh);
        dkdv_run_S<D>(fa, kf, s);
        __builtin_amdgcn_sched_barrier(0);
        VA_DKDV_ISSUE_SLOT(3)
        VA_DKDV_ISSUE_SLOT(4)
        dkdv_load_C<D, 1, OB>(cur, taddr, fc);
        dkdv_run_dP<D>(fa, vf, dpb);
        dkdv_run_B(s, dpb, lv, c2, pb, dsb);
        dkdv_run_C<D, OB>(fc, pb, dsb, dkacc, dvacc);
        dkdv_load_A<D, 0>(nxt, aaddr, fa, dpa, hh);  // next step (dropped after the last one)
        dkdv_interleave<C::KS, 8 * OB / C::KS, 14>();   // dP; dV/dK operand reads; P
        dkdv_interleave<4 * OB, 2, 2>();                // dV, dK; next half's S/dP operand reads; dS
        __builtin_amdgcn_sched_barrier(0);
        VA_DKDV_ISSUE_SLOT(5)
        if (KNOWN < 0) VA_DKDV_ADVANCE()
    };

    // A wave whose keys all lie beyond the sample keeps up the loads and the barriers only (see the forward kernel).
    if (wk_lo >= L) {
        for (int i = 0; i < total; ++i) {
            VA_DKDV_SYNC()
            issue_all();
        }
        wait_vmcnt<0>();
        return;
    }
    // Masked steps (the causal diagonal, the one that holds the sample's end) take the simple form: in
    // phases, with the mask and the lo parts on top, they were measured no faster even at one wave per SIMD.
    int left = total;
    for (int hg = 0; SMALL ? left > 0 : hg < g; ++hg) {
        int st = SMALL && hg == 0 ? step0 : 0;
        const int end = SMALL ? min(nsteps, st + left) : nsteps;  // (a chunk may end inside a head)
        left -= end - st;
        const int head_end = SMALL ? min(n_head, end) : n_head, plain_end = SMALL ? min(n_tail, end) : n_tail;
        for (; st < head_end; ++st) VA_DKDV_CAREFUL(st)
        if (st < plain_end) {
            dkdv_load_A<D, 0>(lds + stage_i * STAGE, aaddr, fa, dpa, hh);
            using Unknown = std::integral_constant<int, -1>;
            const int steady_end = STEADY ? min(plain_end, end - NST) : st, st0 = st;
            auto rounds = [&](int until, auto steady) {  // whole rounds of the stages, each stage a constant
                for (; st < until && stage_i != 0; ++st) phased(Unknown{}, steady);
                for (; st + NST <= until; st += NST) {
                    phased(std::integral_constant<int, 0>{}, steady);
                    phased(std::integral_constant<int, 1>{}, steady);
                    phased(std::integral_constant<int, 2>{}, steady);
                    if constexpr (NST == 4) phased(std::integral_constant<int, 3>{}, steady);
                }
            };
            if constexpr (UNROLLED) rounds(steady_end, std::true_type{});
            for (; st < steady_end; ++st) phased(Unknown{}, std::true_type{});
            nxt_s += st - st0; nxt_n += st - st0;
            iss_stage = stage_i == 0 ? NST - 1 : stage_i - 1;
            // (a walk too short for steady steps: short samples)
            if constexpr (UNROLLED) if (st == st0) rounds(plain_end, std::false_type{});
            for (; st < plain_end; ++st) phased(Unknown{}, std::false_type{});
        }
        for (; st < end; ++st) VA_DKDV_CAREFUL(st)
    }
    wait_vmcnt<0>();  // the surplus loads issued near the end must land before this LDS is given away
#undef VA_DKDV_SYNC
#undef VA_DKDV_ISSUE_SLOT
#undef VA_DKDV_ADVANCE
#undef VA_DKDV_CAREFUL

    if (SMALL && nch > 1) {
        if (kvalid) {
            const size_t off = (((size_t)ch * T + sb + kv) * Hkv + c) * D;
#pragma unroll
            for (int db = 0; db < OB; ++db)
#pragma unroll
                for (int r4 = 0; r4 < 4; ++r4) {
                    const int d0 = 32 * (db0 + db) + 8 * r4 + 4 * hh;
                    if (d0 < D) {
                        *(float4*)(small.part_dk + off + d0) = make_float4(dkacc[db][4 * r4 + 0], dkacc[db][4 * r4 + 1],
                                                                           dkacc[db][4 * r4 + 2], dkacc[db][4 * r4 + 3]);
                        *(float4*)(small.part_dv + off + d0) = make_float4(dvacc[db][4 * r4 + 0], dvacc[db][4 * r4 + 1],
                                                                           dvacc[db][4 * r4 + 2], dvacc[db][4 * r4 + 3]);
                    }
                }
        }
    } else if (kvalid) {
        __bf16* dkp = dK + ((size_t)(sb + kv) * Hkv + c) * D;
        __bf16* dvp = dV + ((size_t)(sb + kv) * Hkv + c) * D;
#pragma unroll
        for (int db = 0; db < OB; ++db) {
            const int d0 = 32 * (db0 + db);
            if (D % 32 == 0 || d0 + 32 <= D) {
                store_channels<32>(dkp + d0, dkacc[db], scale, hh);
                store_channels<32>(dvp + d0, dvacc[db], 1.f, hh);
            } else {
                store_channels<16>(dkp + d0, dkacc[db], scale, hh);
                store_channels<16>(dvp + d0, dvacc[db], 1.f, hh);
            }
        }
    }
    wg_clock.end(clock_probe);
}

// Slices (see dkdv_kernel) where every one of them still finds a CU of its own and the walks are not cut.
template <int D>
static bool dkdv_sliced(const BwdArgs& a) {
    return a.plan_kv.max_chunks == 1 && a.max_items_kv * a.num_kv_heads * BwdCfg<D>::DB <= 256;
}
template <int D, bool CAUSAL>
static hipError_t launch_dkdv_dc(const BwdArgs& a, hipStream_t stream) {
    dim3 grid((unsigned)(a.max_items_kv * a.num_kv_heads * a.plan_kv.max_chunks)), block(256);
    auto q = (const __bf16*)a.q; auto k = (const __bf16*)a.k; auto v = (const __bf16*)a.v;
    auto dO = (const __bf16*)a.dout;
    auto st = (const float2*)a.stats;
    auto dk = (__bf16*)a.dk; auto dv = (__bf16*)a.dv;
    const DkdvSmall sm{a.cu_seqlens, a.num_seqs, a.plan_kv, a.part_dk, a.part_dv};
    if (a.small && dkdv_sliced<D>(a)) {
        grid.x *= BwdCfg<D>::DB;
        hipLaunchKernelGGL((dkdv_kernel<D, CAUSAL, true, 1>), grid, block, 0, stream, q, k, v, dO, st, dk, dv, a.sched_hdr_kv,
                           a.items_kv, (int)a.max_items_kv, a.total_tokens, a.num_q_heads, a.num_kv_heads, a.scale, sm,
                           a.clock_probe_dkdv);
    } else if (a.small)
        hipLaunchKernelGGL((dkdv_kernel<D, CAUSAL, true>), grid, block, 0, stream, q, k, v, dO, st, dk, dv, a.sched_hdr_kv,
                           a.items_kv, (int)a.max_items_kv, a.total_tokens, a.num_q_heads, a.num_kv_heads, a.scale, sm,
                           a.clock_probe_dkdv);
    else
        hipLaunchKernelGGL((dkdv_kernel<D, CAUSAL, false>), grid, block, 0, stream, q, k, v, dO, st, dk, dv, a.sched_hdr_kv,
                           a.items_kv, (int)a.max_items_kv, a.total_tokens, a.num_q_heads, a.num_kv_heads, a.scale, sm,
                           a.clock_probe_dkdv);
    return hipGetLastError();
}
template <int D>
static hipError_t launch_dkdv_d(const BwdArgs& a, hipStream_t stream) {
    return a.causal ? launch_dkdv_dc<D, true>(a, stream) : launch_dkdv_dc<D, false>(a, stream);
}

#if VA_BWD_PART == 0
int bwd_dkdv_slots(int head_dim) { return 256 * (head_dim <= 80 ? kDkdvWgsPerCu<80> : kDkdvWgsPerCu<128>); }
hipError_t launch_bwd_dkdv(const BwdArgs& a, hipStream_t stream) {
    switch (a.head_dim) {
        case 64: return launch_dkdv_d<64>(a, stream);
        case 80: return launch_dkdv_80(a, stream);
        case 96: return launch_dkdv_96(a, stream);
        case 128: return a.causal ? launch_dkdv_128_causal(a, stream) : launch_dkdv_128_full(a, stream);
        default: return hipErrorInvalidValue;
    }
}
#elif VA_BWD_PART == 1
hipError_t launch_dkdv_128_causal(const BwdArgs& a, hipStream_t stream) { return launch_dkdv_dc<128, true>(a, stream); }
#elif VA_BWD_PART == 3
hipError_t launch_dkdv_80(const BwdArgs& a, hipStream_t stream) { return launch_dkdv_d<80>(a, stream); }
#elif VA_BWD_PART == 4
hipError_t launch_dkdv_96(const BwdArgs& a, hipStream_t stream) { return launch_dkdv_d<96>(a, stream); }
hipError_t launch_dkdv_128_full(const BwdArgs& a, hipStream_t stream) { return launch_dkdv_dc<128, false>(a, stream); }
#endif

// ------------------------------------------------------------------------------------------------
// dQ
// ------------------------------------------------------------------------------------------------
// A small launch's dQ (va_small.h): every workgroup finds its tile, or chunk of a tile, from cu_seqlens.  The first two
// build the work lists on the side, which no kernel of the call reads: the workspace holds them after every backward, for
// comparison with the lists computed on the host.  Measured with and without, backward: four samples of 246 tokens in all
// 15.6 / 15.6 us, one of 20 8.6 / 8.6, 64 of 10 9.8 / 9.8.
struct DqSmall {
    const int32_t* cu;
    int num_seqs;
    SmallPlan plan;
    float* part;  // fp32 [chunks, T, Hq, D], without the scale
    SchedJob kv, q;
};
template <int D>
constexpr int kDqWgsPerCu = D == 64 ? 3 : 2;
template <bool CAUSAL>
__device__ __forceinline__ SmallShape dq_small_shape(int Hq, const SmallPlan& plan) {
    return SmallShape{BWD_TILE_Q, BWD_STEP_KV, CAUSAL ? COST_CAUSAL_QUERY : COST_FULL, Hq, 1, plan, CAUSAL ? 256 : 0};
}
// What a dQ workgroup works on: false if there is nothing left for it to do.
struct DqWork {
    int sb, L, q0, h, kvh;
    int ch, nch, jb, je;  // chunk, chunks of the tile, key steps [jb, je) of this one
};
template <int D, bool CAUSAL, bool SMALL>
__device__ __forceinline__ bool dq_find_work(const int32_t* __restrict__ hdr, const WorkItem* __restrict__ items,
                                             int max_items, int T, int Hq, int Hkv, const DqSmall& small,
                                             unsigned char* lds, DqWork& wk) {
    int item, hp;
    wk.ch = 0;
    if constexpr (SMALL) {
        if (blockIdx.x < 2) {
            build_work_list(small.cu, small.num_seqs, T, blockIdx.x == 0 ? small.kv : small.q,
                            *(SchedLds<256, VA_SMALL_MAX_SEQS>*)lds);
            return false;
        }
        const unsigned bid = blockIdx.x - 2;
        hp = __builtin_amdgcn_readfirstlane((int)(bid % (unsigned)Hq));
        SmallTile tl;
        if (!small_tile(small.cu, small.num_seqs, T, dq_small_shape<CAUSAL>(Hq, small.plan),
                        __builtin_amdgcn_readfirstlane((int)(bid / (unsigned)Hq)), tl))
            return false;
        wk.sb = tl.begin; wk.L = tl.len; wk.q0 = tl.tile * BWD_TILE_Q;
        wk.ch = tl.ch; wk.nch = tl.nch;
        wk.jb = tl.first_step(); wk.je = tl.end_step();
    } else {
        const bool short_order = hdr[1] == 1;
        if (short_order) short_item_head(blockIdx.x, max_items, Hq, Hkv, D, item, hp);
        else xcd_item_head(blockIdx.x, max_items, Hq, Hkv, kXcdChunk, item, hp);
        item = __builtin_amdgcn_readfirstlane(item); hp = __builtin_amdgcn_readfirstlane(hp);  // see dkdv_kernel
        if (item >= hdr[0]) return false;
        const WorkItem it = items[item];
        // same for the whole workgroup: tell the compiler, so that everything derived stays in SGPRs
        wk.sb = __builtin_amdgcn_readfirstlane(it.y); wk.L = __builtin_amdgcn_readfirstlane(it.z - it.y);
        wk.q0 = __builtin_amdgcn_readfirstlane(it.x - it.y);
        if (short_order) hp = __builtin_amdgcn_readfirstlane(short_rotated_head(hp, item, wk.sb, Hq, Hkv, D));
        wk.nch = 1; wk.jb = 0;
        wk.je = ((CAUSAL ? min(wk.L, wk.q0 + BWD_TILE_Q) : wk.L) + BWD_STEP_KV - 1) / BWD_STEP_KV;
    }
    wk.kvh = hp % Hkv;
    wk.h = wk.kvh * (Hq / Hkv) + hp / Hkv;
    return true;
}
// A chunk's fp32 results of this lane's query row.
template <int D>
__device__ __forceinline__ void dq_store_part(const f32x16 (&dqacc)[BwdCfg<D>::DB], float* __restrict__ dst, int hh) {
#pragma unroll
    for (int db = 0; db < BwdCfg<D>::DB; ++db)
#pragma unroll
        for (int r4 = 0; r4 < 4; ++r4) {
            const int d0 = 32 * db + 8 * r4 + 4 * hh;
            if (d0 < D)
                *(float4*)(dst + d0) = make_float4(dqacc[db][4 * r4 + 0], dqacc[db][4 * r4 + 1], dqacc[db][4 * r4 + 2],
                                                   dqacc[db][4 * r4 + 3]);
        }
}

// ------------------------------------------------------------------------------------------------
// The dQ kernel.  What bounds it is instruction issue, and at a workgroup's start (Q, dO, O, LSE and the first K/V tiles, all
// waited for) and end memory latency, about 8 key steps' worth of it, which only another workgroup on the CU can cover.  So
// K/V are double-buffered in two LDS stages, every operand is read right before its MFMAs, and two workgroups (three at
// head_dim 64) fit a CU: 150 registers and 32 KB at head_dim 64, 246 and 64 KB at 128.
// A form with four stages and the operands of a phase read one phase ahead (400 registers at 128, one workgroup per CU) took
// 2.23 ms for the LLM batch's dQ against 1.79, 0.63 against 0.44 for 512-token causal samples, 3.89 against 3.81 for the ViT
// batch.  At head_dim 80 it lost its lead with the loads without idle lanes and the compiler's strategy for this file's part 2
// (iterative-ilp), and both blocks of a step scheduled together there: four stages -> two, 65536 tokens and 256 short samples,
// 16 heads, 30.6 -> 30.1 ms; 256 samples of 64..1024 tokens 605 -> 549 us, causal 581 -> 500; LLM batch 1283 -> 1241.
// (The operands that only the matrix cores touch are left to the compiler here: parked in the accumulation
// half they pin 128 of the 256 registers there and the vector half spills.)
// ------------------------------------------------------------------------------------------------
template <int D, bool CAUSAL, bool MASKED>
__device__ __forceinline__ void dq_plain_step(const unsigned char* kt, const unsigned char* vt,
                                              const int (&aaddr)[BwdCfg<D>::KS], const int (&taddr)[BwdCfg<D>::DB][2],
                                              const bf16x8 (&qf)[BwdCfg<D>::KS], const bf16x8 (&dof)[BwdCfg<D>::KS],
                                              f32x16 (&dqacc)[BwdCfg<D>::DB], float c2, float lse2,
                                              const f32x16& ndelta16, int kv0, int qrow, int L, int hh, bool lo) {
    using C = BwdCfg<D>;
    constexpr int ROWB = C::T::ROWB;
    // the last key this lane's row sees, counted from the lane's first (a row beyond the sample is not stored)
    const int last_key = (CAUSAL ? min(L - 1, qrow) : L - 1) - kv0 - 4 * hh;
#pragma unroll
    for (int b = 0; b < 2; ++b) {
        if (MASKED && b && kv0 + 32 >= L) break;   // the sample ends in the first block: the second adds zeros
        // Above the diagonal no row of this wave sees a key of the block, nor of the next (LLM batch 1693 -> 1662 us, 16 heads of
        // 64, 64..1024 tokens, 313 -> 310; six causal samples of 30..200 tokens 13.8 -> 12.6).
        if (MASKED && CAUSAL && kv0 + 32 * b > __builtin_amdgcn_readfirstlane(qrow) + 31) break;
        // The second block's operand reads stay behind the first block: mixed, dQ took 8 % longer at head_dim 128, 3 % at 64
        // (three workgroups per CU), about the same at 96.  Head_dim 80 has the registers (240 of 256): 0.6 % faster mixed on
        // 65536 tokens, 1.5 % on 64..1024.
        if (b && D != 80) __builtin_amdgcn_sched_barrier(0);
        f32x16 s, dp;
#pragma unroll
        for (int r = 0; r < 16; ++r) s[r] = 0.f;
#pragma unroll
        for (int ks = 0; ks < C::KS; ++ks) {
            bf16x8 ak = *(const bf16x8*)(kt + aaddr[ks] + b * 32 * ROWB);
            s = mfma32(ak, qf[ks], s);
            bf16x8 av = *(const bf16x8*)(vt + aaddr[ks] + b * 32 * ROWB);
            // -Delta is where the dP accumulation starts: a 16-register constant read as the first MFMA's addend
            dp = mfma32(av, dof[ks], ks == 0 ? ndelta16 : dp);
        }
#pragma unroll
        for (int r = 0; r < 16; ++r) {
            float p = fast_exp2(__builtin_fmaf(s[r], c2, -lse2));
            if (MASKED) p = 32 * b + 8 * (r / 4) + (r % 4) <= last_key ? p : 0.f;
            dp[r] *= p;
        }
#pragma unroll
        for (int st = 0; st < 2; ++st) {
            const bf16x8 dsb = pack_regs(dp, st);
            const int rowoff = (32 * b + 16 * st) * ROWB;
#pragma unroll
            for (int db = 0; db < C::DB; ++db) {
                bf16x8 ak = cat4(lds_read_tr(kt + rowoff + taddr[db][0]), lds_read_tr(kt + rowoff + taddr[db][1]));
                dqacc[db] = mfma32(ak, dsb, dqacc[db]);
            }
        }
        if (MASKED && lo) {  // wave-uniform: the lo parts of dS, in a pass of their own
#pragma unroll
            for (int st = 0; st < 2; ++st) {
                const bf16x8 dsl = pack_regs_lo(dp, st, pack_regs(dp, st));
                const int rowoff = (32 * b + 16 * st) * ROWB;
#pragma unroll
                for (int db = 0; db < C::DB; ++db) {
                    bf16x8 ak = cat4(lds_read_tr(kt + rowoff + taddr[db][0]), lds_read_tr(kt + rowoff + taddr[db][1]));
                    dqacc[db] = mfma32(ak, dsl, dqacc[db]);
                }
            }
        }
    }
}

template <int D, bool CAUSAL, bool SMALL>
__global__ void __launch_bounds__(256, (kDqWgsPerCu<D>))
dq_kernel(const __bf16* __restrict__ Q, const __bf16* __restrict__ K, const __bf16* __restrict__ V,
              const __bf16* __restrict__ dO, const __bf16* __restrict__ O, const float* __restrict__ LSE,
              float2* __restrict__ stats, __bf16* __restrict__ dQ, const int32_t* __restrict__ hdr,
              const WorkItem* __restrict__ items, int max_items, int T, int Hq, int Hkv, float scale, DqSmall small,
              unsigned long long* __restrict__ clock_probe) {
    using C = BwdCfg<D>;
    using LT = LdsTile<D>;
    constexpr int STAGE = 2 * C::TILE;  // K tile, V tile
    // two LDS stages: step j + 1 loads while step j computes (a third stage, tried at head_dim 64, was slower:
    // 16 more registers for nothing that the other workgroups on the CU do not already cover)
    __shared__ __attribute__((aligned(1024))) unsigned char lds[2 * STAGE];

    DqWork wk;
    ClockProbe wg_clock;
    wg_clock.begin(clock_probe);
    if (!dq_find_work<D, CAUSAL, SMALL>(hdr, items, max_items, T, Hq, Hkv, small, lds, wk)) return;
    const int sb = wk.sb, L = wk.L, q0 = wk.q0, h = wk.h, kvh = wk.kvh;
    const int tid = threadIdx.x, w = uniform_wave_id(), l = tid & 63, ln = l & 31, hh = l >> 5;
    const int qrow = q0 + 32 * w + ln;
    const bool qvalid = qrow < L;

    // Steps are counted from the first of this workgroup's: step j holds keys (jb + j) * BWD_STEP_KV and on.
    const int jb = wk.jb, nsteps = wk.je - jb;
    const int n_plain = min(nsteps, (CAUSAL ? min(L, q0 + 1) : L) / BWD_STEP_KV - jb);
    const unsigned char* kbase = (const unsigned char*)(K + ((size_t)(sb + jb * BWD_STEP_KV) * Hkv + kvh) * D);
    const unsigned char* vbase = (const unsigned char*)(V + ((size_t)(sb + jb * BWD_STEP_KV) * Hkv + kvh) * D);
    const uint32_t row_bytes = (uint32_t)Hkv * D * 2;
    TileDma<D, 64> dma;
    dma.init(row_bytes, L, w, l);
    const uint32_t lds0 = lds_address(lds);
    const int64_t step_bytes = (int64_t)BWD_STEP_KV * row_bytes;
    const bool ragged_sample = (L % BWD_STEP_KV) != 0;
    const int last_step = (L + BWD_STEP_KV - 1) / BWD_STEP_KV - 1 - jb;  // the one holding the sample's end
    // loads of step j into stage j % 2; a step past the item's last one is not loaded
    // (the ragged step in a branch of its own, with the flag a constant on either side: a select between the two
    // offset tables on a run-time flag makes the compiler index them through memory, and it then moves them into
    // LDS, at 32 bytes per lane: bank conflicts in every load that reads them)
    auto issue_step = [&](int j) {
        if (j < nsteps) {
            const uint32_t st = lds0 + (j & 1) * STAGE;
            if (ragged_sample && j == last_step) {
                dma.issue_tile(kbase + (size_t)j * step_bytes, true, st, w, false);
                dma.issue_tile(vbase + (size_t)j * step_bytes, true, st + C::TILE, w, true);
            } else {
                dma.issue_tile(kbase + (size_t)j * step_bytes, false, st, w, false);
                dma.issue_tile(vbase + (size_t)j * step_bytes, false, st + C::TILE, w, true);
            }
        }
    };
    int aaddr[C::KS], taddr[C::DB][2];
#pragma unroll
    for (int ks = 0; ks < C::KS; ++ks) aaddr[ks] = LT::off(ln, 2 * ks + hh);
#pragma unroll
    for (int db = 0; db < C::DB; ++db) {
        taddr[db][0] = LT::tr_off(l, 0, db);
        taddr[db][1] = LT::tr_off(l, 8, db);
    }

    issue_step(0);
    bf16x8 qf[C::KS], dof[C::KS];
    float lse2 = 0.f, ndelta = 0.f;  // ndelta = -Delta
    {
        const size_t off = ((size_t)(sb + (qvalid ? qrow : 0)) * Hq + h) * D + 8 * hh;
#pragma unroll
        for (int ks = 0; ks < C::KS; ++ks) {
            bf16x8 z = {};
            qf[ks] = qvalid ? *(const bf16x8*)(Q + off + 16 * ks) : z;
            dof[ks] = qvalid ? *(const bf16x8*)(dO + off + 16 * ks) : z;
        }
        // Row statistics of this lane's row: Delta = sum_d dO * O (each half of the wave sums its 8 of
        // every 16 columns), and the saved LSE in base 2.  Written out for the dK/dV kernel.
        float part = 0.f;
#pragma unroll
        for (int ks = 0; ks < C::KS; ++ks) {
            bf16x8 z = {};
            const bf16x8 of = qvalid ? *(const bf16x8*)(O + off + 16 * ks) : z;
#pragma unroll
            for (int e = 0; e < 8; ++e) part = __builtin_fmaf((float)dof[ks][e], (float)of[e], part);
        }
        ndelta = -xhalf_sum(part);
        if (qvalid) {
            lse2 = LSE[(size_t)h * T + sb + qrow] * kLog2e;
            if (hh == 0 && wk.ch == 0) stats[(size_t)h * T + sb + qrow] = make_float2(lse2, ndelta);
        }
    }
    // (everything waited for here, once: see the forward kernel for why the register loads must not be left
    // pending at loop entry)
    wait_vmcnt<0>();

    f32x16 dqacc[C::DB];
#pragma unroll
    for (int db = 0; db < C::DB; ++db)
#pragma unroll
        for (int r = 0; r < 16; ++r) dqacc[db][r] = 0.f;
    const float c2 = scale * kLog2e;
    // causal: only a sample's first rows hold few terms.  Without the mask every masked step (the one holding the
    // sample's end) carries lo parts; the flag is hidden from the compiler all the same, so that the lo pass stays
    // behind a branch of its own: folded into the step it costs the kernel 10 registers it does not have.
    f32x16 ndelta16;
#pragma unroll
    for (int r = 0; r < 16; ++r) ndelta16[r] = ndelta;
    asm volatile("" : "+v"(ndelta16));  // one set of registers for the whole kernel, not a refill per block
    int always = 1;
    asm volatile("" : "+s"(always));
    const bool lo_steps = CAUSAL ? q0 == 0 : always != 0;

    if (q0 + 32 * w >= L) {  // no row of this wave exists: loads and barriers only (see the forward kernel)
        for (int j = 0; j < nsteps; ++j) {
            wait_vmcnt<0>();
            wg_barrier();
            issue_step(j + 1);
        }
        wait_vmcnt<0>();
        return;
    }
    // Step j: its loads (issued during step j - 1) have landed; the barrier publishes them and tells that every
    // wave is done with step j - 1, whose stage the loads of step j + 1 may now overwrite.
    // PARITY: j % 2 where the caller knows it (-1 otherwise).  The mask-free loop runs two steps per iteration with
    // the stage a constant in each, so that the LDS addresses of the operand reads are the per-lane offsets plus an
    // immediate instead of one vector addition per address and step.
    auto step = [&](int j, auto masked_tag, auto parity_tag) {
        constexpr bool MASKED = decltype(masked_tag)::value;
        constexpr int PARITY = decltype(parity_tag)::value;
        wait_vmcnt<0>();
        wg_barrier();
        issue_step(j + 1);
        const unsigned char* st = lds + (PARITY >= 0 ? PARITY : (j & 1)) * STAGE;
        dq_plain_step<D, CAUSAL, MASKED>(st, st + C::TILE, aaddr, taddr, qf, dof, dqacc, c2, lse2, ndelta16,
                                         (jb + j) * BWD_STEP_KV, qrow, L, hh, lo_steps);
    };
    using Unknown = std::integral_constant<int, -1>;
    int j = 0;
    for (; j + 1 < n_plain; j += 2) {
        step(j, std::false_type{}, std::integral_constant<int, 0>{});
        step(j + 1, std::false_type{}, std::integral_constant<int, 1>{});
    }
    for (; j < n_plain; ++j) step(j, std::false_type{}, Unknown{});
    for (; j < nsteps; ++j) step(j, std::true_type{}, Unknown{});
    wait_vmcnt<0>();

    if (SMALL && wk.nch > 1) {
        if (qvalid) dq_store_part<D>(dqacc, small.part + (((size_t)wk.ch * T + sb + qrow) * Hq + h) * D, hh);
    } else if (qvalid) {
        __bf16* dqp = dQ + ((size_t)(sb + qrow) * Hq + h) * D;
#pragma unroll
        for (int db = 0; db < D / 32; ++db) store_channels<32>(dqp + 32 * db, dqacc[db], scale, hh);
        if constexpr (D % 32 != 0) store_channels<16>(dqp + D - 16, dqacc[C::DB - 1], scale, hh);
    }
    wg_clock.end(clock_probe);
}

template <int D, bool CAUSAL>
static hipError_t launch_dq_dc(const BwdArgs& a, hipStream_t stream) {
    auto q = (const __bf16*)a.q; auto k = (const __bf16*)a.k; auto v = (const __bf16*)a.v;
    auto dO = (const __bf16*)a.dout;
    auto o = (const __bf16*)a.o;
    auto st = (float2*)a.stats;
    DqSmall sm = {};
    if (a.small) {
        sm = DqSmall{a.cu_seqlens, a.num_seqs, a.plan_q, a.part_dq,
                     sched_job(BWD_TILE_KV, BWD_STEP_Q, CAUSAL ? COST_CAUSAL_KEY : COST_FULL, a.ws_kv, a.lay_kv),
                     sched_job(BWD_TILE_Q, BWD_STEP_KV, CAUSAL ? COST_CAUSAL_QUERY : COST_FULL, a.ws_q, a.lay_q)};
    }
    dim3 grid((unsigned)(a.max_items_q * a.num_q_heads * a.plan_q.max_chunks + (a.small ? 2 : 0))), block(256);
    if (a.small)
        hipLaunchKernelGGL((dq_kernel<D, CAUSAL, true>), grid, block, 0, stream, q, k, v, dO, o, a.lse, st, (__bf16*)a.dq,
                           a.sched_hdr_q, a.items_q, (int)a.max_items_q, a.total_tokens, a.num_q_heads, a.num_kv_heads,
                           a.scale, sm, a.clock_probe_dq);
    else
        hipLaunchKernelGGL((dq_kernel<D, CAUSAL, false>), grid, block, 0, stream, q, k, v, dO, o, a.lse, st, (__bf16*)a.dq,
                           a.sched_hdr_q, a.items_q, (int)a.max_items_q, a.total_tokens, a.num_q_heads, a.num_kv_heads,
                           a.scale, sm, a.clock_probe_dq);
    return hipGetLastError();
}
template <int D>
static hipError_t launch_dq_d(const BwdArgs& a, hipStream_t stream) {
    return a.causal ? launch_dq_dc<D, true>(a, stream) : launch_dq_dc<D, false>(a, stream);
}

#if VA_BWD_PART == 2
hipError_t launch_bwd_dq(const BwdArgs& a, hipStream_t stream) {
    switch (a.head_dim) {
        case 64: return launch_dq_d<64>(a, stream);
        case 80: return launch_dq_d<80>(a, stream);
        case 96: return launch_dq_d<96>(a, stream);
        case 128: return launch_dq_d<128>(a, stream);
        default: return hipErrorInvalidValue;
    }
}
#elif VA_BWD_PART == 0
int bwd_dq_slots(int head_dim) { return 256 * (head_dim == 64 ? kDqWgsPerCu<64> : kDqWgsPerCu<128>); }

// Sum of the chunks the small-launch backward left (fp32, in chunk order): one workgroup per (tile, `rows` of its
// rows, head), the query tiles' dQ first, then the key tiles' dK and dV; tiles that were not split are already done.
template <int D, bool CAUSAL>
__global__ void __launch_bounds__(256)
bwd_sum_small(const float* __restrict__ part_dq, const float* __restrict__ part_dk, const float* __restrict__ part_dv,
              __bf16* __restrict__ dQ, __bf16* __restrict__ dK, __bf16* __restrict__ dV, const int32_t* __restrict__ cu,
              int num_seqs, int wgs_q, int rows, int T, int Hq, int Hkv, float scale, SmallPlan plan_q, SmallPlan plan_kv) {
    constexpr int CPR = D / 8;  // 16-byte output pieces per row
    static_assert(BWD_TILE_Q == BWD_TILE_KV, "the same shares of both");
    const int shares = BWD_TILE_Q / rows, pieces = rows * CPR;
    const bool is_q = (int)blockIdx.x < wgs_q;
    const unsigned bid = is_q ? blockIdx.x : blockIdx.x - wgs_q;
    const int H = is_q ? Hq : Hkv;
    const int h = __builtin_amdgcn_readfirstlane((int)(bid % (unsigned)H));
    const int share = __builtin_amdgcn_readfirstlane((int)(bid / (unsigned)H % (unsigned)shares));
    // (one workgroup per tile, not per chunk: only the chunk-0 entries, which come first, are asked for)
    SmallTile tl;
    if (!small_tile(cu, num_seqs, T, is_q ? dq_small_shape<CAUSAL>(Hq, plan_q) : dkdv_small_shape<CAUSAL>(Hq, Hkv, plan_kv),
                    __builtin_amdgcn_readfirstlane((int)(bid / (unsigned)(shares * H))), tl) ||
        tl.ch > 0 || tl.nch == 1)
        return;
    const int L = tl.len, r0 = tl.tile * BWD_TILE_Q, nch = tl.nch;
    const size_t stride = (size_t)T * H * D;
    for (int u = threadIdx.x; u < pieces * (is_q ? 1 : 2); u += 256) {
        const bool second = u >= pieces;  // dV
        const int x = second ? u - pieces : u;
        const int row = r0 + share * rows + x / CPR;
        if (row >= L) continue;
        const size_t off = ((size_t)(tl.begin + row) * H + h) * D + 8 * (x % CPR);
        const float* p = (is_q ? part_dq : second ? part_dv : part_dk) + off;
        float4 v[VA_SMALL_CHUNKS][2];
#pragma unroll
        for (int i = 0; i < VA_SMALL_CHUNKS; ++i)  // (all loads in flight together)
            if (i < nch) { v[i][0] = *(const float4*)(p + i * stride); v[i][1] = *(const float4*)(p + i * stride + 4); }
        float acc[8] = {v[0][0].x, v[0][0].y, v[0][0].z, v[0][0].w, v[0][1].x, v[0][1].y, v[0][1].z, v[0][1].w};
#pragma unroll
        for (int i = 1; i < VA_SMALL_CHUNKS; ++i)
            if (i < nch) {
                acc[0] += v[i][0].x; acc[1] += v[i][0].y; acc[2] += v[i][0].z; acc[3] += v[i][0].w;
                acc[4] += v[i][1].x; acc[5] += v[i][1].y; acc[6] += v[i][1].z; acc[7] += v[i][1].w;
            }
        const float f = second ? 1.f : scale;
        bf16x8 out;
#pragma unroll
        for (int e = 0; e < 8; ++e) out[e] = (__bf16)(acc[e] * f);
        *(bf16x8*)((is_q ? dQ : second ? dV : dK) + off) = out;
    }
}

template <int D>
static hipError_t launch_sum_d(const BwdArgs& a, hipStream_t stream) {
    const int tiles_q = a.plan_q.max_chunks > 1 ? (int)(a.max_items_q * a.num_q_heads) : 0;
    const int tiles_kv = a.plan_kv.max_chunks > 1 ? (int)(a.max_items_kv * a.num_kv_heads) : 0;
    // Rows per workgroup: every thread sums two or four pieces one after the other at 32, a memory round trip each, which is most
    // of the kernel while there are no more than four such workgroups to a CU; beyond, fewer workgroups find their tile faster.
    // Measured at 16 / 32, us (70 random cut backwards): workgroups of 32 up to 500 6.1 / 6.5 to 11.8 / 12.5, 5 to 27 % for 16; from
    // there to 1008 even, 7.2 / 7.4, 14.2 / 14.9, 12.1 / 11.7; 1032 to 1600 11.8 / 11.7, 17.3 / 17.3, 14.2 / 13.8; beyond, one sample
    // 16.5 / 15.7, 18.0 / 16.9, with short samples among them 11.7 / 9.4, 20.0 / 15.4, 17.7 / 12.7.
    const int rows = 4 * (tiles_q + tiles_kv) <= 1024 ? 16 : 32;
    const int wgs_q = tiles_q * (BWD_TILE_Q / rows), wgs_kv = tiles_kv * (BWD_TILE_KV / rows);
    auto dq = (__bf16*)a.dq; auto dk = (__bf16*)a.dk; auto dv = (__bf16*)a.dv;
    if (a.causal)
        hipLaunchKernelGGL((bwd_sum_small<D, true>), dim3(wgs_q + wgs_kv), dim3(256), 0, stream, a.part_dq, a.part_dk,
                           a.part_dv, dq, dk, dv, a.cu_seqlens, a.num_seqs, wgs_q, rows, a.total_tokens,
                           a.num_q_heads, a.num_kv_heads, a.scale, a.plan_q, a.plan_kv);
    else
        hipLaunchKernelGGL((bwd_sum_small<D, false>), dim3(wgs_q + wgs_kv), dim3(256), 0, stream, a.part_dq, a.part_dk,
                           a.part_dv, dq, dk, dv, a.cu_seqlens, a.num_seqs, wgs_q, rows, a.total_tokens,
                           a.num_q_heads, a.num_kv_heads, a.scale, a.plan_q, a.plan_kv);
    return hipGetLastError();
}
hipError_t launch_bwd_sum_small(const BwdArgs& a, hipStream_t stream) {
    switch (a.head_dim) {
        case 64: return launch_sum_d<64>(a, stream);
        case 80: return launch_sum_d<80>(a, stream);
        case 96: return launch_sum_d<96>(a, stream);
        case 128: return launch_sum_d<128>(a, stream);
        default: return hipErrorInvalidValue;
    }
}
#endif

}  // namespace va
