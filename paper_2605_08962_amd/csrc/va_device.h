// Device-side helpers for the gfx950 kernels: vector types, MFMA, LDS transposing reads,
// cross-half exchange.  Lane layouts used throughout (wave64, v_mfma_f32_32x32x16_bf16):
//   A operand: lane l holds A[m = l % 32][k = 8*(l/32) .. 8*(l/32)+7]
//   B operand: lane l holds B[k = 8*(l/32) .. +7][n = l % 32]
//   C/D      : lane l, register r holds C[m = 8*(r/4) + 4*(l/32) + r%4][n = l % 32]
// A C tile X[m][n] therefore already is the B operand of a product that contracts over m,
// provided the A operand enumerates k in the order  k(l/32, e) = 8*(e/4) + 4*(l/32) + e%4
// per 16-wide step (registers 0..7 = step 0, 8..15 = step 1).
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

#include <type_traits>

namespace va {

typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef __bf16 bf16x4 __attribute__((ext_vector_type(4)));
typedef __bf16 bf16x2 __attribute__((ext_vector_type(2)));
typedef short s16x4 __attribute__((ext_vector_type(4)));
typedef float f32x16 __attribute__((ext_vector_type(16)));
typedef float f32x2 __attribute__((ext_vector_type(2)));
typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));
typedef uint32_t u32x2 __attribute__((ext_vector_type(2)));

#define VA_LDS __attribute__((address_space(3)))

__device__ __forceinline__ f32x16 mfma32(bf16x8 a, bf16x8 b, f32x16 c) {
    return __builtin_amdgcn_mfma_f32_32x32x16_bf16(a, b, c, 0, 0, 0);
}

// max / sum of x between lane l and lane l ^ 32 (v_permlane32_swap exchanges the upper half of
// its first operand with the lower half of its second).
__device__ __forceinline__ float xhalf_max(float x) {
    auto r = __builtin_amdgcn_permlane32_swap(__float_as_uint(x), __float_as_uint(x), false, false);
    return fmaxf(__uint_as_float(r[0]), __uint_as_float(r[1]));
}
__device__ __forceinline__ float xhalf_sum(float x) {
    auto r = __builtin_amdgcn_permlane32_swap(__float_as_uint(x), __float_as_uint(x), false, false);
    return __uint_as_float(r[0]) + __uint_as_float(r[1]);
}

// ds_read_b64_tr_b16: inside each group of 16 lanes, lane 4*k + j supplies the LDS address of
// elements [row k][cols 4j .. 4j+3] of a 4 x 16 block of 16-bit values; lane i receives
// [rows 0..3][col i].  Two of them give one 8-deep MFMA A operand of a row-major tile read
// "down the columns".
__device__ __forceinline__ bf16x4 lds_read_tr(const unsigned char* p) {
    s16x4 r = __builtin_amdgcn_ds_read_tr16_b64_v4i16((s16x4 VA_LDS*)(p));
    return __builtin_bit_cast(bf16x4, r);
}
__device__ __forceinline__ bf16x8 cat4(bf16x4 a, bf16x4 b) {
    return __builtin_shufflevector(a, b, 0, 1, 2, 3, 4, 5, 6, 7);
}
// Per-lane byte offset, inside a row-major LDS tile with `stride` bytes per row, of the address
// this lane supplies to lds_read_tr for the block whose origin is (row 0, col 0) for lanes 0..15,
// col 16 for lanes 16..31, and 4 rows further down for lanes 32..63.
__device__ __forceinline__ int tr_lane_offset(int lane, int stride) {
    return (4 * (lane >> 5) + ((lane & 15) >> 2)) * stride + (16 * ((lane >> 4) & 1) + 4 * (lane & 3)) * 2;
}

// ------------------------------------------------------------------------------------------------
// LDS tiles filled by direct-to-LDS loads (global_load_lds_dwordx4).
// (The layout functions are host-callable as well: a CPU test checks their bank properties.)
//
// Such a load writes the 64 lanes' 16-byte chunks to 1024 CONTIGUOUS LDS bytes, so rows cannot be
// padded against bank conflicts.  Instead the 16-byte chunks of a row are permuted: logical chunk c
// of row r lives in slot c ^ swz(r).  swz is chosen so that (a) 16 consecutive rows read at one
// logical chunk (MFMA A operand read along the row) and (b) 4 consecutive rows read over one
// 64-byte span (transposing read down the columns) both cover all 64 banks exactly once.
// Rows are 128 bytes for head_dim 64 and 256 bytes for 128; head_dim 80 and 96 have a packed layout of
// their own (PackedLdsTile).
// ------------------------------------------------------------------------------------------------
#define VA_GLOBAL __attribute__((address_space(1)))

template <int D>
struct LdsTile {
    static constexpr int ROWB = D <= 64 ? 128 : 256;  // bytes per row
    static constexpr int SLOTS = ROWB / 16;
    static constexpr int CHUNKS = SLOTS;
    static constexpr int BLOCK_POS = 16 * SLOTS;      // 16-byte positions in a block of 16 rows
    __host__ __device__ __forceinline__ static constexpr int swz(int r) {
        if (ROWB == 256) return ((r & 3) << 2) | ((r >> 2) & 3);
        const int x = (r >> 1) & 7;
        return ((x & 1) << 2) | (x >> 1);
    }
    __host__ __device__ __forceinline__ static constexpr int off(int r, int c) { return r * ROWB + ((c ^ swz(r)) << 4); }
    // Byte offset this lane passes to lds_read_tr for the 4 x 16 block at rows row0.., columns
    // 32*db + (0 or 16).. of the tile; row0 must be a multiple of 8 (see tr_lane_offset).
    __host__ __device__ __forceinline__ static int tr_off(int lane, int row0, int db) {
        const int r = row0 + 4 * (lane >> 5) + ((lane & 15) >> 2);
        const int c = 4 * db + 2 * ((lane >> 4) & 1) + ((lane & 3) >> 1);
        return off(r, c) + 8 * (lane & 1);
    }
    // Which (row of the block, logical chunk) lives at 16-byte position p of a 16-row block (true: every position
    // holds data).  The inverse of off(), used to aim the direct-to-LDS loads.
    __host__ __device__ __forceinline__ static constexpr bool locate(int p, int& r, int& c) {
        r = p / SLOTS;
        c = (p % SLOTS) ^ swz(r);
        return true;
    }
};

// head_dim 80 and 96: rows of 160 and 192 bytes, stored without padding: a 64-row tile takes 10 or 12 KB instead of 16 KB
// (more workgroups per CU), and every lane of the loads that fill it has data to fetch (10 or 12 loads instead of 16).
// Such a row rules out an XOR swizzle, so each block of 16 rows (10 or 12 segments of 256 bytes = 16 positions) is laid out
// by hand.  With a = r / 4 and b = r % 4 inside the block, chunk c of row r sits in
//     segment FULL * a + c/4  (c < 4 * FULL)   or   segment c  (the two chunks 8 and 9 that head_dim 80 has beyond its two
//     groups of four),     position 4b + (c + a) % 4.
// (a) For one c the 16 rows occupy 16 different positions, so a row-wise 16-byte read of 16 rows covers
// all 64 banks once.  (b) For one a (4 rows) and one group of 4 chunks the 16 (row, chunk) pairs do too,
// which is the footprint of half a transposing read.  (c) The four chunks of a group of a row are adjacent in
// LDS (rotated), so four lanes of a load still fetch 64 contiguous bytes from memory.
template <int D>
struct PackedLdsTile {
    static constexpr int ROWB = 2 * D;  // nominal: a block of 16 rows is 16 * ROWB bytes
    static constexpr int CHUNKS = D / 8;
    static constexpr int FULL = CHUNKS / 4;  // groups of four chunks
    static constexpr int BLOCK_POS = 16 * CHUNKS;
    __host__ __device__ __forceinline__ static constexpr int pos(int r, int c) {  // r in [0, 16)
        const int a = r >> 2, b = r & 3;
        const int seg = c < 4 * FULL ? FULL * a + (c >> 2) : c;
        return 16 * seg + 4 * b + ((c + a) & 3);
    }
    __host__ __device__ __forceinline__ static constexpr int off(int r, int c) { return (r >> 4) * (16 * ROWB) + 16 * pos(r & 15, c); }
    // Columns 80..95 of head_dim 80's third 32-column block do not exist: the lanes that would address them
    // re-read chunks 8 and 9 (same addresses as their partner lanes; the results are never used).
    __host__ __device__ __forceinline__ static int tr_off(int lane, int row0, int db) {
        const int r = row0 + 4 * (lane >> 5) + ((lane & 15) >> 2);
        int c = 4 * db + 2 * ((lane >> 4) & 1) + ((lane & 3) >> 1);
        if (c >= CHUNKS) c -= 2;
        return off(r, c) + 8 * (lane & 1);
    }
    __host__ __device__ __forceinline__ static constexpr bool locate(int p, int& r, int& c) {
        const int seg = p >> 4, b = (p >> 2) & 3, e = p & 3;
        int a = 0;
        if (CHUNKS % 4 == 0) {
            a = seg / FULL; c = 4 * (seg % FULL) + ((e - a) & 3);
        } else {
            // Unsigned and by selects: 30 to 100 instructions less at the start of every workgroup than with branches.  Few-token
            // samples at head_dim 80 are little else, us: 200 of 5..25 tokens, 16 heads, causal, forward 23.5 -> 22.8, dQ 29.0 ->
            // 28.6, dK/dV 36.1 -> 35.6; 28 of them, 32/16 heads, 11.2 -> 10.9, 11.6 -> 11.4, 10.4 -> 10.3.
            const unsigned s = (unsigned)p >> 4;
            a = s >= 4 * FULL ? (e - seg) & 3 : (int)(s / FULL);
            c = s >= 4 * FULL ? seg : (int)(4 * (s % FULL)) + ((e - a) & 3);
        }
        r = 4 * a + b;
        return true;
    }
};
template <> struct LdsTile<80> : PackedLdsTile<80> {};
template <> struct LdsTile<96> : PackedLdsTile<96> {};

// One direct-to-LDS load: every active lane fetches 16 bytes from base + its own byte offset; lane
// i's data lands at lds_addr + 16 * i (lds_addr is a wave-uniform LDS byte address and goes through
// M0; base is wave-uniform and stays in scalar registers).  Written as inline assembly on purpose: the compiler
// then does not see an LDS write in flight and so does not put a wait for ALL outstanding loads in
// front of every LDS read (which is what it does for the equivalent builtin, and which would
// serialise the prefetch with the compute).  The price is that completion must be waited for by
// hand (wait_vmcnt) before the barrier that publishes the tile.
// (readfirstlane of a value the compiler already knows to be uniform folds away; it is there for the
// cases it cannot prove, because an "s" operand must never be handed a vector register.  The statements
// name M0 as clobbered: they overwrite it, and the compiler may keep a value of its own there.)
__device__ __forceinline__ uint64_t uniform_u64(const void* p) {
    const uint64_t b = (uint64_t)(uintptr_t)p;
    const uint32_t lo = __builtin_amdgcn_readfirstlane((uint32_t)b);
    const uint32_t hi = __builtin_amdgcn_readfirstlane((uint32_t)(b >> 32));
    return ((uint64_t)hi << 32) | lo;
}
__device__ __forceinline__ void dma16(const void* base, uint32_t byte_off, uint32_t lds_addr) {
    asm volatile("s_mov_b32 m0, %0\n\tglobal_load_lds_dwordx4 %1, %2"
                 : : "s"(__builtin_amdgcn_readfirstlane(lds_addr)), "v"(byte_off), "s"(uniform_u64(base)) : "memory", "m0");
}
// Same with 4 bytes per lane: lane i's dword lands at lds_addr + 4 * i.
__device__ __forceinline__ void dma4(const void* base, uint32_t byte_off, uint32_t lds_addr) {
    asm volatile("s_mov_b32 m0, %0\n\tglobal_load_lds_dword %1, %2"
                 : : "s"(__builtin_amdgcn_readfirstlane(lds_addr)), "v"(byte_off), "s"(uniform_u64(base)) : "memory", "m0");
}
// LDS byte address (what M0 and ds instructions use) of a pointer into a __shared__ array.
__device__ __forceinline__ uint32_t lds_address(const void* p) {
    return (uint32_t)(uintptr_t)(VA_LDS const unsigned char*)p;
}
// Gives the waves that share a SIMD different, fixed issue priorities (by the parity of their
// hardware wave slot).  Workgroups of equal work start together and, with equal priority, stay in
// lock-step: both waves of a SIMD want the matrix pipe at the same time, then the vector ALU at the
// same time, and each pipe idles while the other is fought over (measured: MFMA-busy + VALU-busy
// = 100 %, co-execution < 20 %).  With unequal priorities one wave runs unhindered and the other
// fills the gaps, so its MFMAs run under the first one's vector work and vice versa.
__device__ __forceinline__ void stagger_wave_priority() {
    const unsigned slot = __builtin_amdgcn_s_getreg((3 << 11) | (0 << 6) | 4);  // HW_ID[3:0]: wave slot in the SIMD
    if (slot & 1) __builtin_amdgcn_s_setprio(2); else __builtin_amdgcn_s_setprio(0);
}

// Optional clock probe of a compute kernel: when `probe` is not null, every workgroup adds the time
// it was resident in ticks of the 100 MHz real-time counter to probe[0] and in shader cycles to
// probe[1].  Their ratio is the shader clock the kernel actually ran at (the chip lowers it under
// load).  Two scalar clock reads and, for one lane, two atomics per workgroup.
struct ClockProbe {
    unsigned long long rt0 = 0, cc0 = 0;
    __device__ __forceinline__ void begin(const unsigned long long* probe) {
        if (probe) { rt0 = __builtin_amdgcn_s_memrealtime(); cc0 = __builtin_readcyclecounter(); }
    }
    __device__ __forceinline__ void end(unsigned long long* probe) const {
        if (probe && threadIdx.x == 0) {
            atomicAdd(&probe[0], (unsigned long long)(__builtin_amdgcn_s_memrealtime() - rt0));
            atomicAdd(&probe[1], (unsigned long long)(__builtin_readcyclecounter() - cc0));
        }
    }
};

// Workgroup id -> (work item, head slot) for a launch of n_items x heads workgroups; head slot hp stands
// for kv head hp % kv_heads and member hp / kv_heads of its group of query heads.  Workgroup ids are
// dealt round-robin to the 8 XCDs, each with an L2 of its own.  With kv_heads a multiple of 8, XCD x
// gets the kv heads x, x + 8, ... and all their query heads.  It walks the (cost-sorted) work list in
// chunks of `chunk` items and finishes a chunk for one kv head (all query heads of the group side by
// side: they read the same K/V) before it takes the chunk for its next kv head.
//   chunk = kXcdChunk (long samples): the workgroups running together on an XCD stream the K/V (or
//     Q/dO) of ONE kv head where an item-major order interleaves all of the XCD's heads; the same bytes
//     serve more workgroups and stay in L2 for longer (HBM-side traffic of a 65536-token sample halved).
//   chunk = 1 (short samples only; item-major): the workgroups of all heads of an item run together and
//     read whole token rows of Q/K/V at once.  Nothing is re-read in this regime, and visiting every
//     DRAM row once instead of once per head of the XCD is worth 10 % at 128-token samples.  The head
//     slots are rotated by the item index there, so that an XCD reads every head in turn: with a fixed
//     pair of heads per XCD all its requests have the same two byte offsets inside the token rows, and the
//     memory side serves them 5-25 % slower (measured: 64-token samples at head_dim 64, forward 193 -> 155 us,
//     dQ 311 -> 237 us, dK/dV 339 -> 289 us; no difference in the chunked order, where L2 serves the reads).
// The scheduler kernel picks the chunk from the longest sample and leaves it in its header; the compute kernels go
// through short_item_head / short_rotated_head in the second case.
constexpr int kXcdChunk = 128;
constexpr int kXcdChunkMinLen = 1024;  // longest sample from which the chunked order is used
__host__ __device__ __forceinline__ void xcd_item_head(unsigned bid, int n_items, int heads, int kv_heads, int chunk,
                                                       int& item, int& hp) {
    if (kv_heads % 8 != 0) {
        item = (int)(bid / (unsigned)heads);
        hp = (int)(bid % (unsigned)heads);
        if (chunk == 1) hp = (int)((unsigned)(hp + item) % (unsigned)heads);  // (see chunk = 1 above)
        return;
    }
    const unsigned C = (unsigned)chunk;
    const unsigned g = (unsigned)(heads / kv_heads), kx = (unsigned)kv_heads / 8;
    const unsigned x = bid % 8, k = bid / 8;        // k-th workgroup of XCD x
    const unsigned full = (unsigned)n_items / C * C;  // items in whole chunks
    const unsigned per_chunk = C * g;                 // workgroups of one (chunk, kv head)
    unsigned kvslot, i, gq;
    if (k < full * g * kx) {
        const unsigned c = k / (per_chunk * kx), rem = k % (per_chunk * kx);
        kvslot = rem / per_chunk;
        i = c * C + (rem % per_chunk) / g;
        gq = rem % g;
    } else {
        const unsigned kk = k - full * g * kx, r = (unsigned)n_items - full;
        kvslot = kk / (r * g);
        i = full + (kk % (r * g)) / g;
        gq = kk % g;
    }
    item = (int)i;
    hp = (int)(x + 8 * kvslot + (unsigned)kv_heads * gq);
    if (C == 1) hp = (int)(((unsigned)hp + i) % (unsigned)heads);
}

// The order of a batch of short samples (header: chunk = 1).  What counts there is which L2 the tiles of one sample
// meet in: the 2..8 tiles of a sample stand next to each other in the work list and read the same K/V (dK/dV: the same
// Q/dO), which in the order above, rotated by the item, came from another XCD's L2 each time.
//   Rows of whole 128-byte lines (head_dim 64, 128) and kv_heads a multiple of 8: the order above, but rotated by a
//     hash of the sample's first row, which all tiles of a sample share, instead of by the item: short_rotated_head,
//     once the item is loaded.
//   Otherwise: XCD x takes kShortRun items in turn with all their heads.  At head_dim 80 and 96 a head's 160 or 192
//     bytes of a token share lines with its neighbours', which the order above fetches into two L2s; and with
//     another number of kv heads it gives a head no XCD of its own anyway.
// Measured, forward / dQ / dK/dV, 83k..130k tokens, 16 heads, order above -> this one, and the choice not taken:
//   head_dim 64, 64..384 tokens    212/331/438 -> 204/316/433 us (whole items 212/328/424)
//   head_dim 128, 64..1000 tokens  583/844/1395 -> 528/795/1344 us (whole items 543/812/1356)
//   head_dim 80, 64..384 tokens    323/567/648 -> 296/507/596 us (rotated by sample 310/554/631)
//   head_dim 96, 64..1000 tokens   524/716/1234 -> 489/674/1166 us (rotated by sample 491/673/1183)
//   12 heads of 80, 64..1000 tokens  303/449/536 -> 263/411/501 us
//   64-token samples, head_dim 64  154/245/296 -> 148/229/280 us (whole items 163/262/314)
// Runs of 1, 4 or 8 items instead of 2: 0..5 % slower at head_dim 80.
constexpr unsigned kShortRun = 2;
__host__ __device__ __forceinline__ bool short_whole_items(int head_dim, int kv_heads) {
    return head_dim * 2 % 128 != 0 || kv_heads % 8 != 0;
}
__host__ __device__ __forceinline__ void short_item_head(unsigned bid, int n_items, int heads, int kv_heads, int head_dim,
                                                         int& item, int& hp) {
    if (!short_whole_items(head_dim, kv_heads)) return xcd_item_head(bid, n_items, heads, kv_heads, 1, item, hp);
    const unsigned H = (unsigned)heads, full = (unsigned)n_items / (8 * kShortRun) * (8 * kShortRun);  // items in whole rounds
    if (bid < full * H) {
        const unsigned x = bid % 8, k = bid / 8, rem = k % (kShortRun * H);
        item = (int)((k / (kShortRun * H) * 8 + x) * kShortRun + rem / H);
        hp = (int)(rem % H);
    } else {
        item = (int)(bid / H);
        hp = (int)(bid % H);
    }
}
// sample: the packed row the item's sample starts at.
__host__ __device__ __forceinline__ int short_rotated_head(int hp, int item, int sample, int heads, int kv_heads, int head_dim) {
    if (short_whole_items(head_dim, kv_heads)) return hp;
    const unsigned H = (unsigned)heads;  // (takes the rotation by the item off again)
    return (int)(((unsigned)hp + ((unsigned)sample * 2654435761u >> 16) % H + H - (unsigned)item % H) % H);
}

// Index of this wave inside its workgroup, as a value the compiler knows to be wave-uniform.
__device__ __forceinline__ int uniform_wave_id() { return __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6)); }

// Per-lane source offsets of the direct-to-LDS loads that fill one LdsTile of ROWS rows of a
// [rows, heads, D] tensor, split over the four waves of the workgroup.  The offsets are relative to
// the tile's first row; they are computed once per kernel, so that issuing a tile costs no vector
// ALU work.  `last` holds the offsets for the sample's ragged last tile, where rows past the sample
// end re-read its last row (finite data that the caller masks).
// A tile is PIECES loads of 64 x 16 contiguous LDS bytes, whatever rows those hold.  Every wave takes NI of them; two
// may be left (10 pieces at head_dim 80 over 4 waves).  Tiles come in pairs (K and V, Q and dO) of one shape: the left
// pieces of the first tensor go to waves 0 and 1, those of the second to waves 2 and 3, so that every wave issues
// 2 NI + EXTRA loads for the pair.  (A load costs the SIMD about 26 cycles of issue however many of its lanes fetch
// something.  One block of 16 rows per wave took six loads for the pair instead of five at head_dim 80, the third of each
// half empty, and at 96, in rows padded to 256 bytes, eight instead of six.  64 ViT samples, 16 heads of 96: forward 4548 ->
// 4238 us, dQ 6215 -> 5858, dK/dV 10129 -> 9725; at head_dim 80, 256 samples of 64..1024 tokens, dQ 632 -> 615, the others 0.6 %.)
template <int D, int ROWS>
struct TileDma {
    using T = LdsTile<D>;
    static constexpr int WAVES = 4;
    static constexpr int PIECES = ROWS / 16 * T::BLOCK_POS / 64;
    static constexpr int NI = PIECES / WAVES;                  // loads per wave per tile, without
    static constexpr int EXTRA = PIECES % WAVES ? 1 : 0;       // the one per pair of tiles
    static_assert(ROWS % 16 == 0 && ROWS / 16 * T::BLOCK_POS % 64 == 0 && PIECES % WAVES % 2 == 0, "pieces of a tile");
    uint32_t full[NI + EXTRA], last[NI + EXTRA];
    // Piece that load i of a wave fills (i == NI: the extra one).
    __device__ __forceinline__ static int piece(int wave, int i) { return i < NI ? wave * NI + i : WAVES * NI + (wave & 1); }
    // row_bytes: bytes between consecutive rows of the tensor; L: rows in the sample
    __device__ __forceinline__ void init(uint32_t row_bytes, int L, int wave, int lane) {
        const int last_r0 = (L - 1) / ROWS * ROWS;
#pragma unroll
        for (int i = 0; i < NI + EXTRA; ++i) {
            int r = 0, c = 0, row = 0;
            if constexpr (EXTRA == 0 && 64 * NI % T::BLOCK_POS == 0) {  // whole blocks of 16 rows per wave
                const int p = 64 * i + lane;
                T::locate(p % T::BLOCK_POS, r, c);
                row = 16 * (wave * (64 * NI / T::BLOCK_POS) + p / T::BLOCK_POS) + r;
            } else {
                const unsigned p = 64 * piece(wave, i) + lane;  // 16-byte position inside the tile
                T::locate((int)(p % T::BLOCK_POS), r, c);
                row = (int)(16 * (p / T::BLOCK_POS)) + r;
            }
            full[i] = (uint32_t)row * row_bytes + c * 16;
            last[i] = (uint32_t)min(row, L - 1 - last_r0) * row_bytes + c * 16;
        }
    }
    // Load i of a tile (known after unrolling): src = first byte of the tile's first row at this head, tile = LDS byte
    // address of the tile, wave = uniform_wave_id().  Lets a caller spread a tile's loads over its compute phases: a wave
    // that issues them back to back right after a barrier queues up behind every other wave doing the same and sits in the
    // issue stage for hundreds of cycles.
    __device__ __forceinline__ void issue_one(int i, const unsigned char* src, bool ragged, uint32_t tile, int wave) const {
        const uint32_t off = ragged ? last[i] : full[i];
        dma16(src, off, tile + piece(wave, i) * 1024);
    }
    // Whether this wave's extra load belongs to the second tensor of a pair.
    __device__ __forceinline__ static bool extra_is_second(int wave) { return wave >= 2; }
    // All of this wave's loads of one tile of the first or second tensor.
    __device__ __forceinline__ void issue_tile(const unsigned char* src, bool ragged, uint32_t tile, int wave, bool second) const {
#pragma unroll
        for (int i = 0; i < NI; ++i) issue_one(i, src, ragged, tile, wave);
        if (EXTRA && extra_is_second(wave) == second) issue_one(NI, src, ragged, tile, wave);
    }
    // The extra load of a pair of tiles, without a branch.
    __device__ __forceinline__ void issue_extra(const unsigned char* first, const unsigned char* second, bool first_ragged,
                                                bool second_ragged, uint32_t first_tile, uint32_t second_tile, int wave) const {
        const bool s = extra_is_second(wave);
        if (EXTRA) issue_one(NI, s ? second : first, s ? second_ragged : first_ragged, s ? second_tile : first_tile, wave);
    }
};

// Wait until at most N of this wave's vector-memory loads (direct-to-LDS ones included) are still
// outstanding; LDS and scalar counters are left alone.
template <int N>
__device__ __forceinline__ void wait_vmcnt() {
    static_assert(N >= 0 && N < 64, "vmcnt is 6 bits");
    __builtin_amdgcn_s_waitcnt(0x0F70 | (N & 15) | ((N >> 4) << 14));
}
// Workgroup barrier without the memory fence of __syncthreads (which would wait for every
// outstanding load, including the prefetches that are meant to stay in flight).
__device__ __forceinline__ void wg_barrier() {
    asm volatile("" ::: "memory");
    // this wave's own LDS reads must have returned before another wave may refill the tile
    __builtin_amdgcn_s_waitcnt(0xC07F);  // lgkmcnt(0), vmcnt and expcnt untouched
    __builtin_amdgcn_s_barrier();
    asm volatile("" ::: "memory");
}

// Moves a loop-invariant MFMA operand into the accumulation half of the register file.  A kernel that
// runs one wave per SIMD has 512 registers, but the vector ALU only reaches the 256 "architectural"
// ones; when those run short the compiler parks MFMA RESULTS in the other half and pays one copy
// instruction per register every time the vector ALU needs them (64 per step for S and dP).  The
// matrix instructions read their A/B operands from either half, so operands that only they touch
// are the right thing to keep there.
__device__ __forceinline__ void park_in_acc_registers(bf16x8& x) { asm volatile("" : "+a"(x)); }

__device__ __forceinline__ bf16x8 pack8(float a0, float a1, float a2, float a3, float a4, float a5, float a6, float a7) {
    bf16x8 r;
    r[0] = (__bf16)a0; r[1] = (__bf16)a1; r[2] = (__bf16)a2; r[3] = (__bf16)a3;
    r[4] = (__bf16)a4; r[5] = (__bf16)a5; r[6] = (__bf16)a6; r[7] = (__bf16)a7;
    return r;
}

// Element e of x as a float, from its bits: written as a conversion the compiler rounds the value that went into x once more,
// 32 instructions per 16 scores (not used in the forward: at head_dim 64 and 128 it costs registers the kernel does not have).
__device__ __forceinline__ float bf16_as_float(bf16x8 x, int e) {
    const u32x4 w = __builtin_bit_cast(u32x4, x);
    return __uint_as_float(e & 1 ? w[e >> 1] & 0xffff0000u : w[e >> 1] << 16);
}

// Rounds a 32-channel block of a result to bf16 and stores it: x is an MFMA result with channels down and rows across, lane l
// holds channels 8 i + 4 (l / 32) .. + 3 (i = 0..3) of row l % 32.  The halves of the wave trade, so that a lane stores 16 bytes
// where it has 8: half as many stores, each of which reaches 32 rows.  What a workgroup of a few steps spends at its end is these
// stores.  Measured, 8 bytes -> 16, forward / dK/dV / dQ, us: 64..384 tokens, 16 heads of 64, 191.6/385.8/288.9 ->
// 180.9/356.2/278.4; 64..1024 tokens, of 80 384/717/567 -> 369/684/552, of 96 436/922/594 -> 418/878/577, of 128 causal 483/908/676 ->
// 474/840/666; ViT batch 2853/5089/3767 -> 2832/5042/3743; long walks even.  CHANNELS: 32, or 16 where the row ends there; dst: the
// row's first channel of the block.  Must be reached by lanes l and l ^ 32 together (they share the row).
template <int CHANNELS>
__device__ __forceinline__ void store_channels(__bf16* dst, const f32x16& x, float f, int half) {
#pragma unroll
    for (int i = 0; i < CHANNELS / 16; ++i) {
        bf16x8 v;
#pragma unroll
        for (int e = 0; e < 8; ++e) v[e] = (__bf16)(x[8 * i + e] * f);
        const u32x4 w = __builtin_bit_cast(u32x4, v);
        const auto a = __builtin_amdgcn_permlane32_swap(w[0], w[2], false, false);
        const auto b = __builtin_amdgcn_permlane32_swap(w[1], w[3], false, false);
        const u32x4 out = {a[0], b[0], a[1], b[1]};
        *(u32x4*)(dst + 16 * i + 8 * half) = out;
    }
}

__device__ __forceinline__ float fast_exp2(float x) { return __builtin_amdgcn_exp2f(x); }

constexpr float kLog2e = 1.4426950408889634f;
constexpr float kLn2 = 0.6931471805599453f;
constexpr float kMaskedScore = -1.0e30f;  // finite stand-in for -inf: keeps 0 * score finite

}  // namespace va
