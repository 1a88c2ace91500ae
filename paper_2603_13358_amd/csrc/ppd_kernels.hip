// gfx950 kernels of libppd: paged KV append, the one-launch mixed attention kernel (narrow tiles for
// decode-like rows, MFMA row-block tiles for append-prefill / full prefill) and the log-sum-exp merge of
// split partials.
//
// Operation (paper section 4.1, "Full Prefill vs. Append Prefill"; L = cached, n = new): new row j of a
// sequence attends to keys 0 .. L + j, all read from the page pool.  Both tile kinds compute the
// transposed products  S^T = K Q^T  and  O^T = V^T P^T  so that the accumulator layout of the first
// product is already the operand layout of the second, and every per-row softmax quantity lives in the
// lane that owns the row's column.
#include <hip/hip_runtime.h>

#include <type_traits>

#include "ppd_internal.h"

#ifndef PPD_PINGPONG
#define PPD_PINGPONG 1  // 0: all waves take the loop barrier at the end of the iteration; 1: waves 4..7 mid-iteration
#endif

namespace ppd {

typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef __bf16 bf16x2 __attribute__((ext_vector_type(2)));
typedef float f32x2 __attribute__((ext_vector_type(2)));
typedef float f32x4 __attribute__((ext_vector_type(4)));
typedef float f32x16 __attribute__((ext_vector_type(16)));
typedef uint32_t u32x2 __attribute__((ext_vector_type(2)));
typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));
typedef short s16x4 __attribute__((ext_vector_type(4)));

#define NEG_INF (-__builtin_inff())

__device__ __forceinline__ uint32_t pack_bf16(float a, float b) {
    f32x2 f = {a, b};
    bf16x2 r = __builtin_convertvector(f, bf16x2);  // round to nearest even
    return __builtin_bit_cast(uint32_t, r);
}

__device__ __forceinline__ bf16x8 as_bf16x8(u32x4 v) { return __builtin_bit_cast(bf16x8, v); }

__device__ __forceinline__ float fast_exp2(float x) { return __builtin_amdgcn_exp2f(x); }
// Query row of a column of a row block (columns are row-major over the G query heads of the group): col / G
// with inv = 65536 / G + 1, exact for col < 4096 and G <= 16.
__device__ __forceinline__ int col_row(int col, int inv) { return (int)(((unsigned)col * (unsigned)inv) >> 16); }

__device__ __forceinline__ float xor_shuffle(float v, int mask) { return __shfl_xor(v, mask, 64); }

// max / sum of v over lanes l and l^32 (v_permlane32_swap: no LDS round trip).  The instruction exchanges
// the upper half of its first register with the lower half of its second.  It is written as inline asm on
// two copies of v (the builtin's second result was folded into the first by the compiler when both inputs
// hold the same value); the s_nop cover the VALU-write -> permlane-read wait states on both sides.
__device__ __forceinline__ void swap_halves(float v, float* lo, float* hi) {
    float a = v, b = v;
    asm volatile("s_nop 1\n\tv_permlane32_swap_b32 %0, %1\n\ts_nop 1" : "+v"(a), "+v"(b));
    *lo = a;  // {v[0..31], v[0..31]}
    *hi = b;  // {v[32..63], v[32..63]}
}
__device__ __forceinline__ float max_halves(float v) {
    float lo, hi;
    swap_halves(v, &lo, &hi);
    return fmaxf(lo, hi);
}
__device__ __forceinline__ float sum_halves(float v) {
    float lo, hi;
    swap_halves(v, &lo, &hi);
    return lo + hi;
}

// The running maximum is only raised (and the accumulators rescaled) when it would grow by more than this many
// powers of two; until then probabilities may exceed 1, by at most 2^kLazyRescale.  The final o / l is unchanged.
// (Row-block tiles do not look for the maximum: there the bound is on the sum of a lane's 32 probabilities.)
#ifndef kLazyRescale
#define kLazyRescale 8.0f
#endif
constexpr float power_of_two(float e) { return e >= 1.0f ? 2.0f * power_of_two(e - 1.0f) : 1.0f; }
constexpr float kMaxLazyP = power_of_two(kLazyRescale);
static_assert((int)kLazyRescale == kLazyRescale, "a whole number of powers of two");

// Raw page-table entry of logical page `pi` of a sequence; pi is clamped so that no access leaves the page
// table row.  The value is NOT inspected here: a caller that prefetches it must not wait for the load.
__device__ __forceinline__ int load_page_id(const int32_t* pt_row, int pi, int last_page) {
    pi = pi < last_page ? pi : last_page;
    return pt_row[pi];
}

// Checks a page id at the point of use: an id outside the pool raises the sticky flag and is replaced by
// page 0, so that no access leaves the pool.
__device__ __forceinline__ int64_t checked_page(const KParams& P, int page) {
    if (page < 0 || page >= P.num_pages) {
        atomicOr(&P.counters[9], 2u);
        page = 0;
    }
    return page;
}

// FP8 pages hold OCP FP8 E4M3 codes (1 sign, 4 exponent bits of bias 7, 3 mantissa bits).  Every code's value is a
// bf16 number, so the tiles turn codes into bf16 MFMA operands exactly; the tensor's scale is applied once, to the
// scores (K) and to the final output (V).
// Four codes of a dword -> four bf16, in order (the conversion instruction takes the two codes of one 16-bit half).
__device__ __forceinline__ u32x2 fp8x4_to_bf16x4(uint32_t w) {
    const bf16x2 lo = __builtin_amdgcn_cvt_scalef32_pk_bf16_fp8(w, 1.0f, false);
    const bf16x2 hi = __builtin_amdgcn_cvt_scalef32_pk_bf16_fp8(w, 1.0f, true);
    return u32x2{__builtin_bit_cast(uint32_t, lo), __builtin_bit_cast(uint32_t, hi)};
}
__device__ __forceinline__ u32x4 fp8x8_to_bf16x8(u32x2 w) {
    const u32x2 a = fp8x4_to_bf16x4(w[0]), b = fp8x4_to_bf16x4(w[1]);
    return u32x4{a[0], a[1], b[0], b[1]};
}

// Clamp to the code's range with the NaN-propagating minimum and maximum: magnitudes from 448 on (infinities included)
// become 448, a NaN stays one.
__device__ __forceinline__ float e4m3_clamp(float y) {
    return __builtin_elementwise_minimum(__builtin_elementwise_maximum(y, -448.0f), 448.0f);
}
__device__ __forceinline__ float bf16_bits_to_f32(uint32_t bits) { return __builtin_bit_cast(float, bits << 16); }

// Codes of x * inv for the four bf16 of two dwords, in order: one binary32 product each, clamped, then the conversion
// instruction (two values each; nearest, ties to the even code; a clamped value cannot overflow).  Its treatment of
// ties and subnormals is what the definition asks for -- the tests compare every bf16 bit pattern with the oracle.
// 5 vector instructions per element; the same decision in integer arithmetic on the bits took ~25 and bound the
// append of FP8 pages (landing of 5589 tokens x 32 layers: 314 us, now 255).
__device__ __forceinline__ uint32_t e4m3_codes(uint32_t lo, uint32_t hi, float inv) {
    int w = __builtin_amdgcn_cvt_pk_fp8_f32(e4m3_clamp(bf16_bits_to_f32(lo & 0xFFFFu) * inv),
                                            e4m3_clamp(__builtin_bit_cast(float, lo & 0xFFFF0000u) * inv), 0, false);
    w = __builtin_amdgcn_cvt_pk_fp8_f32(e4m3_clamp(bf16_bits_to_f32(hi & 0xFFFFu) * inv),
                                        e4m3_clamp(__builtin_bit_cast(float, hi & 0xFFFF0000u) * inv), w, true);
    // the instruction gives every NaN the same sign: the codes take theirs from the inputs (inv > 0)
    const uint32_t signs = __builtin_amdgcn_perm(hi, lo, 0x07050301u);  // the upper byte of each bf16
    return ((uint32_t)w & 0x7F7F7F7Fu) | (signs & 0x80808080u);
}

// Zeroes the bf16 elements e of a granule of 8 tokens whose position first + e is >= kv_total (never written).
__device__ __forceinline__ u32x4 zero_unwritten(u32x4 v, int first, int kv_total) {
#pragma unroll
    for (int e = 0; e < 8; ++e)
        if (first + e >= kv_total) v[e >> 1] &= (e & 1) ? 0x0000FFFFu : 0xFFFF0000u;
    return v;
}

// ---------------------------------------------------------------------------------------------------
// MFMA row-block tile: up to kMfmaCols query columns (rows x G heads of one KV head) against keys
// [kv_begin, kv_end).  kWaves waves x 32 columns; key tiles of 64 tokens (4 pages); v_mfma_f32_32x32x16_bf16 for
// both products.  K and V tiles go from the pool straight into LDS (global_load_lds, 16 bytes per lane, no
// staging registers), each in a ring.  With NS = kStages tiles of prefetch distance and rings of NS + 1 stages:
//   iteration i:  loads K(i+NS) -> Kring[(i+NS) % (NS+1)], V(i+NS-1) -> Vring[(i+NS-1) % (NS+1)]
//                 vector phase on S^T(i); matrix phase reads V(i) and K(i+1)
//   one barrier per iteration, after K(i+2) and V(i+1) have landed (loads issued in the last NS-2 iterations may
//   still be in flight); half of the waves take it between their two phases (see the loop).
// ---------------------------------------------------------------------------------------------------
// 16 bytes per lane from global memory straight into LDS: lane i of the wave writes lds_base + 16*i
// (lds_base is wave-uniform and travels in M0).  Written as inline asm so that the compiler's wait-count pass
// does not see an LDS write it would have to order every later LDS read behind (it would drain the memory
// counter before the first operand read of each tile); completion is awaited explicitly with s_waitcnt vmcnt.
// The global address is a wave-uniform base (scalar register pair) plus a 32-bit byte offset per lane.
__device__ __forceinline__ void lds_direct_load16(const void* gbase, uint32_t lane_off, const char* lds_base) {
    const uint32_t lds_off = (uint32_t)(uintptr_t)(__attribute__((address_space(3))) const char*)lds_base;
    asm volatile("s_mov_b32 m0, %2\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %0, %1"
                 :
                 : "v"(lane_off), "s"(gbase), "s"(__builtin_amdgcn_readfirstlane(lds_off))
                 : "memory", "m0");
}

// HALF = false: the vector phase covers the 64 keys of a tile, then the matrix phase (the loop described above).
// HALF = true: the same tile is worked in two halves of 32 keys -- vector phase, matrix phase, vector phase, matrix
// phase -- with S^T of 32 keys and half of the packed probabilities live at a time: 24 registers less per lane,
// which is what lets two such waves and a stream wave share a SIMD (three waves of 168 registers).  The late waves
// then take the loop barrier between the second vector phase and the second matrix phase.
// LDS byte address of p as an opaque 32-bit register value: operand reads then address LDS as this register plus a
// compile-time offset below 64 KiB, which fits the instruction's offset field (left to itself the compiler folds
// ring and stage offsets into constants beyond that field and spends one vector add per read).
// (x + k) mod N for 0 <= x, k < N
template <int N>
__device__ __forceinline__ int ring_add(int x, int k) {
    if constexpr ((N & (N - 1)) == 0) return (x + k) & (N - 1);
    const int y = x + k;
    return y >= N ? y - N : y;
}
// The same with the LDS byte address given as a wave-uniform integer (no pointer cast per load).
__device__ __forceinline__ void lds_direct_load16_at(const void* gbase, uint32_t lane_off, uint32_t lds_addr) {
    asm volatile("s_mov_b32 m0, %2\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %0, %1"
                 :
                 : "v"(lane_off), "s"(gbase), "s"(lds_addr)
                 : "memory", "m0");
}
__device__ __forceinline__ uint32_t lds_base(const char* p) {
    uint32_t a = (uint32_t)(uintptr_t)(__attribute__((address_space(3))) const char*)p;
    asm volatile("" : "+v"(a));
    return a;
}
__device__ __forceinline__ u32x4 lds_read16(uint32_t base, int offset) {
    return *reinterpret_cast<const __attribute__((address_space(3))) u32x4*>(base + (uint32_t)offset);
}

// FP8 (pages of one-byte codes): the loads land the tile's codes in a staging ring of their own (half the bytes, NS - 1
// stages of K and of V), and at the end of the iteration before a tile is first read every thread turns the 16 codes it
// loaded itself into bf16 in the operand rings -- once per workgroup, not once per wave and operand read -- so the
// loop's matrix and vector phases are the ones of bf16 pages.  The operand rings then need three stages each (the tile
// being written, the one the early waves read and the one the late waves read), which with the staging ring is the same
// LDS as the four-stage rings of bf16 pages.
template <int HD, bool HALF, bool FP8 = false>
__device__ __forceinline__ void mfma_item(const KParams& P, const ppd_work_item& it, char* smem) {
    static_assert(!(FP8 && HALF), "FP8 pages are read by the full-tile loop only");
    static_assert(!FP8 || kStages == 3, "the staging of FP8 tiles is written for a prefetch distance of 3");
    constexpr int EB = FP8 ? 1 : 2;            // bytes per pool element
    constexpr int PB = kPage * HD * 2;         // bytes of one (page, head) block of K or of V as bf16 operands in LDS
    constexpr int GPP = PB / 16;               // 16-byte granules per such block
    constexpr int KBYTES = 4 * PB;             // one stage: 4 pages of K (or of V)
    constexpr int NS = kStages;
    constexpr int NSV = FP8 ? 3 : kStages + (PPD_PINGPONG ? 1 : 0);  // the late half of the waves reads V one barrier later
    constexpr int NSK = FP8 ? 3 : kStages + (PPD_PINGPONG ? 1 : 0);  // ... and K as well
    constexpr int VRING = NSK * KBYTES;        // LDS: K ring at 0, V ring behind it
    constexpr int LPB = PB / 2 * EB;           // bytes of a block as the loads move it
    constexpr int LGPP = LPB / 16;             // 16-byte granules per loaded block
    constexpr int LBYTES = 4 * LPB;            // one loaded tile of K (or of V)
    constexpr int LOADERS = 4 * LGPP < kThreads ? 4 * LGPP : kThreads;  // threads that load (all, or the first waves)
    constexpr int ROUNDS = 4 * LGPP / LOADERS; // granules of K (and of V) each loading thread moves per tile
    constexpr int NST = NS - 1;                // FP8: stages of the staging ring of K, and of V
    constexpr int STAGE_K = (NSK + NSV) * KBYTES, STAGE_V = STAGE_K + NST * LBYTES;
    constexpr int IDS_AT = (NSK + NSV) * KBYTES + (FP8 ? 2 * NST * LBYTES : 0);
    static_assert(IDS_AT <= (2 * kStages + 2 * (PPD_PINGPONG ? 1 : 0)) * KBYTES, "the kernel's LDS is sized for the bf16 rings");
    constexpr int KS = HD / 16;                // k-steps of S^T = K Q^T
    constexpr int DB = HD / 32;                // 32-row d blocks of O^T

    const int tid = threadIdx.x;
    const int lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int h = lane >> 5;
    const int l32 = lane & 31;
    const int G = P.G;
    const int ncols = it.nrows * G;
    const int col = wave * 32 + l32;
    const int colc = col < ncols ? col : ncols - 1;
    const int jrow = col_row(colc, P.invG);
    const int head = it.kvh * G + (colc - jrow * G);
    const int limit = it.L + it.row0 + jrow;  // last key position this column may see
    const bool wave_active = wave * 32 < ncols;
    const int wmin_limit = it.L + it.row0 + col_row((wave * 32) < ncols ? wave * 32 : ncols - 1, P.invG);

    // Q^T operand: column = lane % 32, d = ks*16 + (lane/32)*8 .. +8
    bf16x8 qreg[KS];
    {
        const uint16_t* qp = P.q + ((int64_t)(it.grow0 + jrow) * P.Hq + head) * HD + h * 8;
#pragma unroll
        for (int ks = 0; ks < KS; ++ks) qreg[ks] = as_bf16x8(*reinterpret_cast<const u32x4*>(qp + ks * 16));
    }

    const int32_t* pt_row = P.page_tables + (int64_t)it.seq * P.max_pages;
    const int last_page = (it.kv_total - 1) >> 4;
    const int first_page = it.kv_begin >> 4;
    const int ntiles = (it.kv_end - it.kv_begin + kTileTokens - 1) / kTileTokens;
    const int64_t head_off = (int64_t)it.kvh * (kPage * HD);
    const int64_t v_off = (int64_t)P.Hkv * (kPage * HD);

    // Page ids of the whole key range go to LDS once, checked, before the loop (at most 2048: the planner
    // caps a row-block tile at kMaxMfmaChunk keys); a tile reads its four ids with one broadcast LDS read.  Nothing in
    // the loop then depends on a page-table load, so no wait on the memory counter is needed there.
    // Granule gid = r*256 + tid ... of the tile's 4 page blocks goes to LDS byte gid*16 of the stage: a wave writes
    // 1 KiB contiguous per round, which is what a wave-wide LDS-direct load does.  The page a wave reads in
    // round r is wave-uniform, s = r * (kThreads / GPP) + (wave * 64) / GPP, and the lane's offset inside the
    // page block is the same in every round: the load's address is a scalar base plus a per-lane constant.
    constexpr int PAGES_PER_ROUND = LOADERS / LGPP;
    static_assert(LOADERS % 64 == 0 && LOADERS % LGPP == 0 && ROUNDS * PAGES_PER_ROUND == 4, "one round covers whole page blocks");
    static_assert(!FP8 || ROUNDS == 1, "a thread stages one granule of codes per tile");
    const bool loader = LOADERS == kThreads || tid < LOADERS;  // wave-uniform
    const int page_sel = loader ? (wave * 64) / LGPP : 0;
    const uint32_t lane_off = (uint32_t)(tid % LGPP) * 16u;
    // The pages this wave loads from, one per round, as byte offsets of the page in the pool: the id read from LDS
    // becomes a scalar and the 64-bit product is made once per tile on the scalar unit (a page is at most 8 MiB, so
    // its size fits 32 bits); a load then costs two scalar additions for its global address and two for its LDS
    // address.
    struct TilePages { uint32_t lo[ROUNDS], hi[ROUNDS]; };
    int* lds_ids = reinterpret_cast<int*>(smem + IDS_AT);
    for (int i = tid; i < ntiles * 4; i += kThreads)
        lds_ids[i] = (int)checked_page(P, load_page_id(pt_row, first_page + i, last_page));
    struct RawPages { int p[ROUNDS]; };  // the ids as they come from LDS (vector registers)
    const uint32_t page_bytes = (uint32_t)P.page_stride * EB;
    auto tile_pages_raw = [&](int ti) {
        RawPages t;
#pragma unroll
        for (int r = 0; r < ROUNDS; ++r) t.p[r] = lds_ids[ti * 4 + r * PAGES_PER_ROUND + page_sel];
        return t;
    };
    auto to_scalar = [&](const RawPages& v) {
        TilePages t;
#pragma unroll
        for (int r = 0; r < ROUNDS; ++r) {
            const uint32_t id = (uint32_t)__builtin_amdgcn_readfirstlane(v.p[r]);
            if constexpr (FP8) {  // this kernel has no scalar registers to spare for the pair: the product is made at the load
                t.lo[r] = id;
                t.hi[r] = 0;
            } else {
                const uint64_t off = (uint64_t)id * page_bytes;
                t.lo[r] = (uint32_t)off;
                t.hi[r] = (uint32_t)(off >> 32);
            }
        }
        return t;
    };
    auto tile_pages = [&](int ti) { return to_scalar(tile_pages_raw(ti)); };
    // Workgroup barrier for LDS traffic only: unlike __syncthreads() it does not drain the memory counter, so
    // LDS-direct loads of later tiles stay in flight across it.
    auto lds_barrier = [&]() { asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory"); };
    const char* const pool_k = reinterpret_cast<const char*>(P.pool) + head_off * EB;  // this KV head's K block of page 0
    const char* const pool_v = pool_k + v_off * EB;                                    // ... and its V block
    const uint32_t smem_addr = __builtin_amdgcn_readfirstlane((uint32_t)(uintptr_t)(__attribute__((address_space(3))) const char*)smem) + (uint32_t)wave * 1024u;
    auto load_round = [&](const TilePages& t, int r, int lds_byte, bool is_v) {
        if (!loader) return;
        const uint64_t off = FP8 ? (uint64_t)t.lo[r] * page_bytes : (((uint64_t)t.hi[r] << 32) | t.lo[r]);
        const char* base = (is_v ? pool_v : pool_k) + off;
        lds_direct_load16_at(base, lane_off, smem_addr + (uint32_t)(lds_byte + r * (kThreads * 16)));
    };
    auto load_block = [&](const TilePages& t, int lds_byte, bool is_v) {
#pragma unroll
        for (int r = 0; r < ROUNDS; ++r) load_round(t, r, lds_byte, is_v);
    };
    // FP8: the 16 codes this thread staged at src_byte become two bf16 granules of the operand tile at dst_byte (the
    // element order of a tile is the same in both); V rows of positions >= kv_total were never written and become 0.
    auto convert_staged = [&](int src_byte, int dst_byte, bool is_v, int tile) {
        if (!loader) return;
        const u32x4 raw = *reinterpret_cast<const u32x4*>(smem + src_byte + tid * 16);
        u32x4 lo = fp8x8_to_bf16x8(u32x2{raw[0], raw[1]}), hi = fp8x8_to_bf16x8(u32x2{raw[2], raw[3]});
        if (is_v) {
            const int tile_base = it.kv_begin + tile * kTileTokens;
            if (tile_base + kTileTokens > it.kv_total) {
                const int g0 = 2 * tid, g1 = 2 * tid + 1;  // bf16 granules of the tile: page g / GPP, (octet, d) = g % GPP
                lo = zero_unwritten(lo, tile_base + (g0 / GPP) * 16 + ((g0 % GPP) / HD) * 8, it.kv_total);
                hi = zero_unwritten(hi, tile_base + (g1 / GPP) * 16 + ((g1 % GPP) / HD) * 8, it.kv_total);
            }
        }
        u32x4* dst = reinterpret_cast<u32x4*>(smem + dst_byte + tid * 32);
        dst[0] = lo;
        dst[1] = hi;
    };
    // V rows of positions >= kv_total were never written: zero them in LDS (each thread fixes the granules it
    // loaded itself, after its own loads have landed).  Only the sequence's last tile needs it.
    auto fix_v_tail = [&](int ti, int lds_byte) {
        const int tile_base = it.kv_begin + ti * kTileTokens;
        if (tile_base + kTileTokens > it.kv_total) {
#pragma unroll
            for (int r = 0; r < ROUNDS; ++r) {
                const int gid = r * kThreads + tid;
                const int s = gid / GPP, within = gid % GPP;
                u32x4* cell = reinterpret_cast<u32x4*>(smem + lds_byte + gid * 16);
                *cell = zero_unwritten(*cell, tile_base + s * 16 + (within / HD) * 8, it.kv_total);
            }
        }
    };
    // Loads retire in order: waiting until at most `newer` are outstanding guarantees everything issued
    // before those has landed in LDS.
    auto wait_all_loads = [&]() { asm volatile("s_waitcnt vmcnt(0)" ::: "memory"); };
    // all but the loads of the last NS - 2 iterations (2*ROUNDS each): K(ti+2) and V(ti+1) were issued before those
    auto wait_older_loads = [&]() {
        constexpr int kKeep = (NS - 2) * 2 * ROUNDS;
        static_assert(kKeep < 64, "the memory counter has six bits");
        // s_waitcnt immediate on gfx9: vmcnt in bits 3:0 and 15:14, expcnt (7 = no wait) in 6:4, lgkmcnt (15) in 11:8
        __builtin_amdgcn_s_waitcnt((kKeep & 15) | ((kKeep >> 4) << 14) | (7 << 4) | (15 << 8));
        asm volatile("" ::: "memory");
    };

    f32x16 oacc[DB];
#pragma unroll
    for (int db = 0; db < DB; ++db)
#pragma unroll
        for (int i = 0; i < 16; ++i) oacc[db][i] = 0.f;
    float m_run = NEG_INF, l_run = 0.f;
    const float c = P.scale_log2e;

    // K operand row of this lane inside a 32-token block: MFMA row r holds token
    //   page = bit4(r), token-in-page = 8*bit2(r) + 4*bit3(r) + (r & 3)
    // so that accumulator registers 8*s2 .. 8*s2+7 of a lane are 8 consecutive tokens of one page.
    const int k_tok = ((l32 >> 2) & 1) * 8 + ((l32 >> 3) & 1) * 4 + (l32 & 3);
    const int k_lane_off = (l32 >> 4) * PB + k_tok * 16 + h * 256;  // + stage + tb*2*PB + ks*512
    const int v_lane_off = VRING + (h * HD + l32) * 16;             // + stage + s*PB + db*512

    auto qk_tile = [&](int stage, f32x16 (&sacc)[2]) {
        const uint32_t kb = lds_base(smem + stage * KBYTES + k_lane_off);
#pragma unroll
        for (int tb = 0; tb < 2; ++tb)
#pragma unroll
            for (int i = 0; i < 16; ++i) sacc[tb][i] = 0.f;
#pragma unroll
        for (int ks = 0; ks < KS; ++ks)
#pragma unroll
            for (int tb = 0; tb < 2; ++tb) {
                bf16x8 a = as_bf16x8(lds_read16(kb, tb * 2 * PB + ks * 512));
                sacc[tb] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a, qreg[ks], sacc[tb], 0, 0, 0);
            }
    };

    // prologue: K(0..NS-1) and V(0..NS-2) are issued, K(0), K(1), V(0) must land; S^T of tile 0
    __syncthreads();  // page ids are in LDS
    if constexpr (FP8) {
        // K(0), K(1) and V(0) are staged and converted; K(2) and V(1) are then issued into the slots of K(0) and beside V(0)
        const TilePages tp0 = tile_pages(0), tp1 = tile_pages(1 < ntiles ? 1 : 0);
        load_block(tp0, STAGE_K, false);
        load_block(tp0, STAGE_V, true);
        if (1 < ntiles) load_block(tp1, STAGE_K + LBYTES, false);
        wait_all_loads();
#pragma unroll
        for (int ks = 0; ks < KS; ++ks) asm volatile("" ::"v"(qreg[ks]));
        convert_staged(STAGE_K, 0, false, 0);
        if (1 < ntiles) convert_staged(STAGE_K + LBYTES, KBYTES, false, 1);
        convert_staged(STAGE_V, VRING, true, 0);
        if (2 < ntiles) load_block(tile_pages(2), STAGE_K, false);
        if (1 < ntiles) load_block(tp1, STAGE_V + LBYTES, true);
    } else {
#pragma unroll
        for (int t = 0; t < NS; ++t) {
            if (t < ntiles) {
                const TilePages tp = tile_pages(t);
                load_block(tp, t * KBYTES, false);
                if (t < NS - 1) load_block(tp, VRING + t * KBYTES, true);
            }
        }
        wait_all_loads();
        // The compiler does not count the asm loads; make it settle its own pending loads (the Q operand) here, or
        // it would place ever-decreasing memory-counter waits at their first use inside the loop and drain the
        // LDS-direct loads in flight there.
#pragma unroll
        for (int ks = 0; ks < KS; ++ks) asm volatile("" ::"v"(qreg[ks]));
#pragma unroll
        for (int t = 0; t < NS - 1; ++t)
            if (t < ntiles) fix_v_tail(t, VRING + t * KBYTES);
    }
    lds_barrier();
    if constexpr (!HALF) {
    f32x16 s_cur[2];
    if (wave_active) qk_tile(0, s_cur);
    lds_barrier();  // with rings of NS stages the first iteration's loads overwrite K stage 0
    int st_cur = 0;   // ti % NS
    int sv_cur = 0;   // ti % NSV: V stage of tile ti
    // Two waves share a SIMD, and a wave issues in order.  An iteration is a vector phase (mask, max, rescale, the
    // tile's exponentials, packed to bf16) followed by a matrix phase (O^T += V^T P^T of this tile, then S^T of the
    // next tile into the registers the probabilities have left), each pure, so that one wave's matrix phase can
    // run under the other's vector phase.  Left alone the two waves would run the same phase at the same time
    // (the loop barrier aligns them); the "late" half of the waves therefore takes the barrier between its two
    // phases instead of at the end of the iteration, which locks it half an iteration behind the other half.
    // A late wave reads V(ti) and K(ti+1) after the barrier at which the early waves start loading V(ti+NS) and
    // K(ti+1+NS): one more stage in each ring (measured: +4.5 % with the shift, -9 % with pure phases alone).
#if PPD_PINGPONG
    const bool late = wave >= kWaves / 2;  // waves w and w + 4 share a SIMD
#else
    const bool late = false;
#endif

    u32x4 pw[4];  // the tile's probabilities as bf16, B operand of the four 16-key steps of the PV product
    TilePages tp_v = tile_pages(NS - 1 < ntiles ? NS - 1 : ntiles - 1);  // pages of the loads the first iteration issues
    TilePages tp_k = tile_pages(NS < ntiles ? NS : ntiles - 1);
    for (int ti = 0; ti < ntiles; ++ti) {
        const int st_nxt = st_cur + 1 == NSK ? 0 : st_cur + 1;           // (ti + 1) % NSK
        const int st_far = ring_add<NSK>(st_cur, NS % NSK);                           // (ti + NS) % NSK
        const int sv_nxt = sv_cur + 1 == NSV ? 0 : sv_cur + 1;           // (ti + 1) % NSV
        const int sv_far = ring_add<NSV>(sv_cur, (NS - 1) % NSV);                       // (ti + NS - 1) % NSV
        const bool full_issue = ti + NS < ntiles;
        const bool v_issue = ti + NS - 1 < ntiles;
        // the iteration's loads, one round of K or of V at a time
        auto issue_round = [&](int j) {
            const bool is_v = j < ROUNDS;
            const int r = is_v ? j : j - ROUNDS;
            if (is_v ? v_issue : full_issue) {
                const int at = is_v ? (FP8 ? STAGE_V + (ti & 1) * LBYTES : VRING + sv_far * KBYTES)
                                    : (FP8 ? STAGE_K + ((ti + 1) & 1) * LBYTES : st_far * KBYTES);  // FP8: tile t is staged in slot t % 2
                load_round(is_v ? tp_v : tp_k, r, at, is_v);
            }
        };
        // The V tile of the next iteration is this iteration's K tile; the ids of its K tile are read from LDS
        // now and turned into scalars at the end of the iteration: under the other waves' operand reads that
        // small LDS read takes hundreds of cycles, which nothing waits for this way.
        const RawPages tp_raw = tile_pages_raw(ti + 1 + NS < ntiles ? ti + 1 + NS : ntiles - 1);
        // K(ti+2) and V(ti+1) must have landed before the barrier; with NS = 3 the loads issued in this iteration
        // may stay in flight
        auto close_iteration = [&]() {
            if (full_issue)  // then the last NS - 2 iterations all issued their full share
                wait_older_loads();
            else
                wait_all_loads();
            if constexpr (FP8) {
                if (ti + 2 < ntiles) convert_staged(STAGE_K + (ti & 1) * LBYTES, ring_add<NSK>(st_cur, 2 % NSK) * KBYTES, false, ti + 2);
                if (ti + 1 < ntiles) convert_staged(STAGE_V + ((ti + 1) & 1) * LBYTES, VRING + sv_nxt * KBYTES, true, ti + 1);
            } else {
                if (ti + 1 < ntiles) fix_v_tail(ti + 1, VRING + sv_nxt * KBYTES);
            }
            lds_barrier();
        };
        if (wave_active) {
            const int tile_base = it.kv_begin + ti * kTileTokens;
            if (tile_base + kTileTokens - 1 > wmin_limit) {  // causal boundary crosses this tile
#pragma unroll
                for (int tb = 0; tb < 2; ++tb)
#pragma unroll
                    for (int i = 0; i < 16; ++i) {
                        const int pos = tile_base + (tb * 2 + (i >> 3)) * 16 + h * 8 + (i & 7);
                        if (pos > limit) s_cur[tb][i] = NEG_INF;
                    }
            }
            // Vector phase: all exponentials of this tile, packed to bf16 at once.  Nothing for the matrix pipe in
            // it, and nothing for the vector pipe in the matrix phase below, so that the late waves (half an
            // iteration behind) run their matrix phase under this vector phase and the other way round.
            float psum = 0.f;
            auto exponentials = [&](int s, float mc) {
#pragma unroll
                for (int e = 0; e < 4; ++e) {
                    const int i0 = (s & 1) * 8 + 2 * e;
                    const float p0 = fast_exp2(__builtin_fmaf(s_cur[s >> 1][i0], c, -mc));
                    const float p1 = fast_exp2(__builtin_fmaf(s_cur[s >> 1][i0 + 1], c, -mc));
                    psum += p0 + p1;
                    pw[s][e] = pack_bf16(p0, p1);
                }
            };
#pragma unroll
            for (int s = 0; s < 4; ++s) {
#pragma unroll
                for (int j = s * 2 * ROUNDS / 4; j < (s + 1) * 2 * ROUNDS / 4; ++j) issue_round(j);
                exponentials(s, m_run * c);
                __builtin_amdgcn_sched_barrier(0);
            }
            // The tile's maximum (17 dependent instructions and a half-wave exchange) is not looked for: the exponentials
            // are taken against the running reference as it is, and only if a lane's sum of 32 of them is above
            // 2^kLazyRescale (or not a number: no reference yet, m_run = -inf) is the maximum found, the accumulators
            // rescaled and the exponentials taken again.  A single probability is then never above 2^kLazyRescale.
            if (__any(!(psum <= kMaxLazyP))) {
                float mx = s_cur[0][0];
#pragma unroll
                for (int tb = 0; tb < 2; ++tb)
#pragma unroll
                    for (int i = 0; i < 16; ++i) mx = fmaxf(mx, s_cur[tb][i]);
                mx = max_halves(mx);
                const float m_new = fmaxf(m_run, mx);
                const float m_use = m_new == NEG_INF ? 0.f : m_new;
                const float alpha = fast_exp2(m_run * c - m_use * c);  // m_run = -inf gives 0
                l_run *= alpha;
#pragma unroll
                for (int db = 0; db < DB; ++db)
#pragma unroll
                    for (int i = 0; i < 16; ++i) oacc[db][i] *= alpha;
                m_run = m_new;
                psum = 0.f;
#pragma unroll
                for (int s = 0; s < 4; ++s) exponentials(s, m_use * c);
            }
            l_run += psum;
        } else {
#pragma unroll
            for (int j = 0; j < 2 * ROUNDS; ++j) issue_round(j);
        }
        // The V tile of the next iteration is this iteration's K tile
        tp_v = tp_k;
        __builtin_amdgcn_sched_barrier(0);
        if (late) close_iteration();
        if (wave_active) {
            // Matrix phase: O^T += V^T P^T of this tile, then S^T of the next one, as one straight run of products whose
            // operands are read AHEAD of them (after the last tile the S^T of whatever the ring holds, not used).
            // Clocks per 64-key tile of one unit at full clock: 3515 with a branch between the two products, one
            // operand pair read at a time and the maximum looked for; 3200 with this run; 3050 without the maximum as well.
            // The whole chip runs the loop at its power limit (2.0 -> 1.8 GHz), so two full prefills of 8192 went from 1077 to 1014 us.
            const uint32_t vb = lds_base(smem + sv_cur * KBYTES + v_lane_off);
            const uint32_t kb = lds_base(smem + st_nxt * KBYTES + k_lane_off);
            constexpr int NPV = 4 * DB, NQK = 2 * KS, NOP = NPV + NQK;
            constexpr int AHEAD = 4;  // operands read ahead of their product
            auto operand = [&](int j) {
                if (j < NPV) return lds_read16(vb, (j / DB) * PB + (j % DB) * 512);
                return lds_read16(kb, ((j - NPV) % 2) * 2 * PB + ((j - NPV) / 2) * 512);
            };
            u32x4 abuf[AHEAD];
#pragma unroll
            for (int j = 0; j < AHEAD; ++j) abuf[j] = operand(j);
#pragma unroll
            for (int tb = 0; tb < 2; ++tb)
#pragma unroll
                for (int i = 0; i < 16; ++i) s_cur[tb][i] = 0.f;
#pragma unroll
            for (int j = 0; j < NOP; ++j) {
                const bf16x8 a = as_bf16x8(abuf[j % AHEAD]);
                if (j < NPV)
                    oacc[j % DB] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a, as_bf16x8(pw[j / DB]), oacc[j % DB], 0, 0, 0);
                else
                    s_cur[(j - NPV) % 2] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a, qreg[(j - NPV) / 2], s_cur[(j - NPV) % 2], 0, 0, 0);
                if (j + AHEAD < NOP) abuf[j % AHEAD] = operand(j + AHEAD);
            }
            __builtin_amdgcn_sched_group_barrier(0x100, AHEAD, 0);
#pragma unroll
            for (int j = 0; j < NOP - AHEAD; ++j) {
                __builtin_amdgcn_sched_group_barrier(0x008, 1, 0);
                __builtin_amdgcn_sched_group_barrier(0x100, 1, 0);
            }
            __builtin_amdgcn_sched_group_barrier(0x008, AHEAD, 0);
        }
        __builtin_amdgcn_sched_barrier(0);
        if (!late) close_iteration();
        tp_k = to_scalar(tp_raw);
        st_cur = st_nxt;
        sv_cur = sv_nxt;
    }

    } else {
    // S^T of 32 keys: the tb-th pair of pages of a K stage
    auto qk_half = [&](int stage, int tb, f32x16& sacc) {
        const uint32_t kb = lds_base(smem + stage * KBYTES + k_lane_off + tb * 2 * PB);
#pragma unroll
        for (int i = 0; i < 16; ++i) sacc[i] = 0.f;
#pragma unroll
        for (int ks = 0; ks < KS; ++ks) {
            bf16x8 a = as_bf16x8(lds_read16(kb, ks * 512));
            sacc = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a, qreg[ks], sacc, 0, 0, 0);
        }
    };
    f32x16 s_half;
    if (wave_active) qk_half(0, 0, s_half);
    lds_barrier();  // with rings of NS stages the first iteration's loads overwrite K stage 0
    int st_cur = 0;   // ti % NSK
    int sv_cur = 0;   // ti % NSV: V stage of tile ti
#if PPD_PINGPONG
    const bool late = wave >= kWaves / 2;  // waves w and w + 4 share a SIMD
#else
    const bool late = false;
#endif
    TilePages tp_v = tile_pages(NS - 1 < ntiles ? NS - 1 : ntiles - 1);  // pages of the loads the first iteration issues
    TilePages tp_k = tile_pages(NS < ntiles ? NS : ntiles - 1);
    for (int ti = 0; ti < ntiles; ++ti) {
        const int st_nxt = st_cur + 1 == NSK ? 0 : st_cur + 1;           // (ti + 1) % NSK
        const int st_far = ring_add<NSK>(st_cur, NS % NSK);                           // (ti + NS) % NSK
        const int sv_nxt = sv_cur + 1 == NSV ? 0 : sv_cur + 1;           // (ti + 1) % NSV
        const int sv_far = ring_add<NSV>(sv_cur, (NS - 1) % NSV);                       // (ti + NS - 1) % NSV
        const bool full_issue = ti + NS < ntiles;
        if (ti + NS - 1 < ntiles) load_block(tp_v, VRING + sv_far * KBYTES, true);
        if (full_issue) load_block(tp_k, st_far * KBYTES, false);
        tp_v = tp_k;
        const RawPages tp_raw = tile_pages_raw(ti + 1 + NS < ntiles ? ti + 1 + NS : ntiles - 1);
        auto close_iteration = [&]() {
            if (full_issue)  // then the last NS - 2 iterations all issued their full share
                wait_older_loads();
            else
                wait_all_loads();
            if (ti + 1 < ntiles) fix_v_tail(ti + 1, VRING + sv_nxt * KBYTES);
            lds_barrier();
        };
#pragma unroll
        for (int hb = 0; hb < 2; ++hb) {
            u32x4 pw[2];  // the half's probabilities as bf16, B operand of its two 16-key steps of the PV product
            if (wave_active) {
                const int half_base = it.kv_begin + ti * kTileTokens + hb * 32;
                if (half_base + 31 > wmin_limit) {  // causal boundary crosses this half
#pragma unroll
                    for (int i = 0; i < 16; ++i) {
                        const int pos = half_base + (i >> 3) * 16 + h * 8 + (i & 7);
                        if (pos > limit) s_half[i] = NEG_INF;
                    }
                }
                float mx = s_half[0];
#pragma unroll
                for (int i = 1; i < 16; ++i) mx = fmaxf(mx, s_half[i]);
                mx = max_halves(mx);
                const float m_new = fmaxf(m_run, mx);
                if (__any((m_new - m_run) * c > kLazyRescale)) {  // -inf -> finite counts; -inf -> -inf does not
                    const float m_use = m_new == NEG_INF ? 0.f : m_new;
                    const float alpha = fast_exp2(m_run * c - m_use * c);  // m_run = -inf gives 0
                    l_run *= alpha;
#pragma unroll
                    for (int db = 0; db < DB; ++db)
#pragma unroll
                        for (int i = 0; i < 16; ++i) oacc[db][i] *= alpha;
                    m_run = m_new;
                }
                const float mc = m_run == NEG_INF ? 0.f : m_run * c;
                float psum = 0.f;
#pragma unroll
                for (int s2 = 0; s2 < 2; ++s2)
#pragma unroll
                    for (int e = 0; e < 4; ++e) {
                        const int i0 = s2 * 8 + 2 * e;
                        const float p0 = fast_exp2(__builtin_fmaf(s_half[i0], c, -mc));
                        const float p1 = fast_exp2(__builtin_fmaf(s_half[i0 + 1], c, -mc));
                        psum += p0 + p1;
                        pw[s2][e] = pack_bf16(p0, p1);
                    }
                l_run += psum;
            }
            __builtin_amdgcn_sched_barrier(0);
            if (hb == 1 && late) close_iteration();
            if (wave_active) {
                // O^T += V^T P^T of this half, then S^T of the next half into the registers the probabilities left
                const uint32_t vb = lds_base(smem + sv_cur * KBYTES + v_lane_off + hb * 2 * PB);
#pragma unroll
                for (int s2 = 0; s2 < 2; ++s2) {
                    const bf16x8 pb = as_bf16x8(pw[s2]);
#pragma unroll
                    for (int db = 0; db < DB; ++db) {
                        bf16x8 a = as_bf16x8(lds_read16(vb, s2 * PB + db * 512));
                        oacc[db] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a, pb, oacc[db], 0, 0, 0);
                    }
                }
                if (hb == 0)
                    qk_half(st_cur, 1, s_half);
                else if (ti + 1 < ntiles)
                    qk_half(st_nxt, 0, s_half);
            }
            __builtin_amdgcn_sched_barrier(0);
        }
        if (!late) close_iteration();
        tp_k = to_scalar(tp_raw);
        st_cur = st_nxt;
        sv_cur = sv_nxt;
    }

    }
    // epilogue: O^T register i of block db is d = db*32 + (i/4)*8 + h*4 + i%4 of column `col`
    const float l_tot = sum_halves(l_run);
    if (it.part_off < 0) {
        // A lane holds 8-byte pieces of 32 different result rows: stored from here, every instruction would touch 32
        // lines.  Each wave turns its 32 columns round in LDS of its own, half a row at a time, and writes
        // whole lines.  The space is the K ring's: no load is in flight, and what the late waves may still read there
        // (the S^T after the last tile) is not used.  2048 row blocks of one 64-key tile (8 to a workgroup, a block is 64
        // KiB of results): 111 -> 90 us.
        constexpr int RS = HD + 16;       // bytes of a staged half row: 16 of padding spread the columns over the banks
        constexpr int LPR = HD / 16;      // lanes that store a half row, 16 bytes each
        static_assert(kWaves * 32 * RS <= NSK * KBYTES, "the staged columns fit the K ring");
        char* const stage = smem + wave * (32 * RS);
        char* const out0 = reinterpret_cast<char*>(P.out) + ((int64_t)it.grow0 * P.Hq + it.kvh * G) * (HD * 2);
        const float inv = P.v_scale / l_tot;
        if (wave_active) {
#pragma unroll
            for (int half = 0; half < 2; ++half) {
#pragma unroll
                for (int db = half * (DB / 2); db < (half + 1) * (DB / 2); ++db)
#pragma unroll
                    for (int i4 = 0; i4 < 4; ++i4) {
                        u32x2 w;
                        w[0] = pack_bf16(oacc[db][i4 * 4 + 0] * inv, oacc[db][i4 * 4 + 1] * inv);
                        w[1] = pack_bf16(oacc[db][i4 * 4 + 2] * inv, oacc[db][i4 * 4 + 3] * inv);
                        *reinterpret_cast<u32x2*>(stage + l32 * RS + ((db - half * (DB / 2)) * 32 + i4 * 8 + h * 4) * 2) = w;
                    }
                asm volatile("" ::: "memory");  // a wave's LDS operations run in order
#pragma unroll
                for (int r = 0; r < 32 * LPR / 64; ++r) {
                    const int c32 = r * (64 / LPR) + lane / LPR, ocol = wave * 32 + c32;
                    const u32x4 w = *reinterpret_cast<const u32x4*>(stage + c32 * RS + (lane % LPR) * 16);
                    const int orow = col_row(ocol, P.invG);
                    const uint32_t off = (uint32_t)(orow * (P.Hq - G) + ocol) * (HD * 2) + (lane % LPR) * 16;  // a block's rows span at most 2 GiB
                    if (ocol < ncols) *reinterpret_cast<u32x4*>(out0 + half * HD + off) = w;
                }
                asm volatile("" ::: "memory");
            }
        }
    } else {
        if (col < ncols) {
            float* pp = P.partials + it.part_off;
            float* po = pp + (int64_t)col * HD + h * 4;
#pragma unroll
            for (int db = 0; db < DB; ++db)
#pragma unroll
                for (int i4 = 0; i4 < 4; ++i4) {
                    f32x4 w = {oacc[db][i4 * 4 + 0], oacc[db][i4 * 4 + 1], oacc[db][i4 * 4 + 2], oacc[db][i4 * 4 + 3]};
                    *reinterpret_cast<f32x4*>(po + db * 32 + i4 * 8) = w;
                }
            if (h == 0) {
                float* ml = pp + (int64_t)ncols * HD + col * 2;
                ml[0] = m_run;
                ml[1] = l_tot;
            }
        }
    }
}

// ---------------------------------------------------------------------------------------------------
// Narrow tile: rows*G <= 16 query columns (decode: 1 row x G heads).  HBM-bound: each of the NW waves
// streams its own share of the key range straight from the pool into MFMA operand registers
// (v_mfma_f32_16x16x32_bf16 for S^T, v_mfma_f32_16x16x16_bf16 for O^T; one page per step; NK register sets for
// K and NV <= NK for V rotate, so that K of NK - 1 and V of NV - 1 pages per wave are in flight while one page is
// computed), then the waves' (o, m, l) are combined through LDS, CB columns per pass.
// ---------------------------------------------------------------------------------------------------
// How a narrow tile's partial leaves.  Where the launch merges split ranges itself, another workgroup of the launch reads it
// (merge_last): it goes past the caches of this XCD, which the other XCDs do not see.  Where a launch behind it merges, the L2
// holds a few of them for it (64 sequences of 3500 keys log-normal, 0.6 MB of partials, past the L2 65.1 -> 68.4 us, 40 of 2900, 0.8
// MB, 89.9 -> 92.6), but many cost the streams of a decode-only launch (181 of 8500 keys, 12 MB, 522 -> 513 us past the L2, 236 of
// 15500, 20 MB, 1166 -> 1143; even at 2-3 MB): the launch says which.
enum Partials { kToL2, kPastL2, kAsLaunched };
template <Partials WAY>
__device__ __forceinline__ void store_partial(const KParams& P, float* p, float v) {
    if (WAY == kPastL2 || (WAY == kAsLaunched && P.partials_past_l2)) __hip_atomic_store(p, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    else *p = v;
}
__device__ __forceinline__ f32x2 load_partial2(const float* p) {
    return __builtin_bit_cast(f32x2, __hip_atomic_load(reinterpret_cast<const uint64_t*>(p), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT));
}

template <int NW>
struct NarrowCombine {
    static constexpr int CB = NW >= 8 ? kNarrowCols : 8;  // columns per combine pass
    static constexpr size_t bytes(int head_dim) { return (size_t)NW * CB * (head_dim + 2) * sizeof(float); }
};

// Two probabilities as two bf16 numbers each (see SPLIT_P): the largest one below it, and the rounding of what that left out.
__device__ __forceinline__ u32x2 split_bf16(float p0, float p1) {
    const uint32_t b0 = __builtin_elementwise_sub_sat(__builtin_bit_cast(uint32_t, p0), 1u) & 0xFFFF0000u;
    const uint32_t b1 = __builtin_elementwise_sub_sat(__builtin_bit_cast(uint32_t, p1), 1u) & 0xFFFF0000u;
    return u32x2{b0 >> 16 | b1, pack_bf16(p0 - __builtin_bit_cast(float, b0), p1 - __builtin_bit_cast(float, b1))};
}

// The waves' (o, m, l) of up to CB columns from c0 on, which each wave has left in `all`, become results or a partial.
template <int HD, int NW, Partials WAY>
__device__ __forceinline__ void narrow_combine(const KParams& P, const ppd_work_item& it, const float* all, int c0) {
    constexpr int CB = NarrowCombine<NW>::CB, WSTRIDE = CB * (HD + 2), NT = NW * 64;
    const int tid = threadIdx.x, G = P.G, ncols = it.nrows * G;
    const float c = P.scale_log2e;
    const int nc = ncols - c0 < CB ? ncols - c0 : CB;
    for (int idx = tid; idx < nc * HD; idx += NT) {
        const int cl = idx / HD, d = idx % HD;
        const int col = c0 + cl;
        float mw[NW], mm = NEG_INF;
#pragma unroll
        for (int w = 0; w < NW; ++w) {
            mw[w] = all[w * WSTRIDE + CB * HD + cl * 2];
            mm = fmaxf(mm, mw[w]);
        }
        float o = 0.f, l = 0.f;
#pragma unroll
        for (int w = 0; w < NW; ++w) {
            const float f = mw[w] == NEG_INF ? 0.f : fast_exp2((mw[w] - mm) * c);
            o += f * all[w * WSTRIDE + cl * HD + d];
            l += f * all[w * WSTRIDE + CB * HD + cl * 2 + 1];
        }
        if (it.part_off < 0) {
            const int crow = col_row(col, P.invG);
            const int64_t orow = (int64_t)(it.grow0 + crow) * P.Hq + it.kvh * G + (col - crow * G);
            const float val = (o / l) * P.v_scale;
            const float other = __shfl_xor(val, 1, 64);  // d and d^1 sit in neighbouring lanes
            if ((d & 1) == 0) *reinterpret_cast<uint32_t*>(P.out + orow * HD + d) = pack_bf16(val, other);
        } else {
            float* pp = P.partials + it.part_off;
            store_partial<WAY>(P, pp + (int64_t)col * HD + d, o);
            if (d == 0) {
                store_partial<WAY>(P, pp + (int64_t)ncols * HD + col * 2, mm);
                store_partial<WAY>(P, pp + (int64_t)ncols * HD + col * 2 + 1, l);
            }
        }
    }
}

// One page of a narrow tile: tokens t0 .. t0 + 15 of the sequence, whose K and V operands are in rs and rw.
template <int HD>
struct NarrowK { u32x4 k[HD / 32]; };  // K operand of the page: 16 tokens x 32 d per k-step
template <int HD>
struct NarrowV { u32x2 v[HD / 16]; };  // V^T operand: 4 tokens of one d, one per 16-row d block
// SPLIT_P: a probability enters the second product as two bf16 numbers, the largest one below it and the rounding of what that
// left out.  The probabilities of a wave are rounded relative to the wave's own running reference, and fewer waves have fewer
// of them: four waves without it would have more rounding error than eight.  Below it, not nearest to it: both numbers of a
// probability are then positive, and the products of an infinite V with them are infinite and of one sign, where a second
// number that is zero or negative would make them NaN.  Relative error of 64 sequences of 3100-4400 keys against 64 bits
// 1.65655e-3, of which the rounding of the result to bf16 alone is 1.65654e-3 (1.65654e-3 with the nearest number first).
// Sums of their own for the second numbers keep infinities as well and are 0.5 % slower (decode steps of 64 sequences
// of 1K-8K keys 810.7 -> 814.9 us over four calls with their appends, and 813.4 -> 813.6 this way).
template <int HD, bool SPLIT_P>
__device__ __forceinline__ void narrow_step(const ppd_work_item& it, int t0, int limit, float c, const bf16x8 (&qreg)[HD / 32], const NarrowK<HD>& rs,
                                            NarrowV<HD>& rw, f32x4 (&oacc)[HD / 16], float& m_run, float& l_run) {
    constexpr int KS = HD / 32, DBN = HD / 16;
    const int g4 = (threadIdx.x & 63) >> 4;
    const int min_limit = it.L + it.row0;
    f32x4 sa = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int ks = 0; ks < KS; ++ks)
        sa = __builtin_amdgcn_mfma_f32_16x16x32_bf16(as_bf16x8(rs.k[ks]), qreg[ks], sa, 0, 0, 0);
    // sa[i]: token 4*g4 + i of the page
    const bool masked = t0 + kPage - 1 > min_limit || t0 + kPage > it.kv_end;
    if (masked) {
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            const int pa = t0 + 4 * g4 + i;
            if (pa > limit || pa >= it.kv_end) sa[i] = NEG_INF;
        }
        if (t0 + kPage > it.kv_total) {  // rows of the last page that were never written
#pragma unroll
            for (int db = 0; db < DBN; ++db) {
#pragma unroll
                for (int e = 0; e < 4; ++e) {
                    const int pos = t0 + 4 * g4 + e;
                    if (pos >= it.kv_total) rw.v[db][e >> 1] &= (e & 1) ? 0x0000FFFFu : 0xFFFF0000u;
                }
            }
        }
    }
    float mx = fmaxf(fmaxf(sa[0], sa[1]), fmaxf(sa[2], sa[3]));
    mx = fmaxf(mx, xor_shuffle(mx, 16));
    mx = max_halves(mx);
    const float m_new = fmaxf(m_run, mx);
    if (__any((m_new - m_run) * c > kLazyRescale)) {
        const float m_use = m_new == NEG_INF ? 0.f : m_new;
        const float alpha = fast_exp2(m_run * c - m_use * c);
        l_run *= alpha;
#pragma unroll
        for (int db = 0; db < DBN; ++db) oacc[db] *= alpha;
        m_run = m_new;
    }
    const float mc = m_run == NEG_INF ? 0.f : m_run * c;
    float p[4];
#pragma unroll
    for (int i = 0; i < 4; ++i) p[i] = fast_exp2(__builtin_fmaf(sa[i], c, -mc));
    l_run += (p[0] + p[1]) + (p[2] + p[3]);
    u32x2 pw, rp;
    if constexpr (SPLIT_P) {
        const u32x2 a = split_bf16(p[0], p[1]), b = split_bf16(p[2], p[3]);
        pw = u32x2{a[0], b[0]};
        rp = u32x2{a[1], b[1]};
    } else {
        pw = u32x2{pack_bf16(p[0], p[1]), pack_bf16(p[2], p[3])};
    }
    const s16x4 pb4 = __builtin_bit_cast(s16x4, pw);
#pragma unroll
    for (int db = 0; db < DBN; ++db)
        oacc[db] = __builtin_amdgcn_mfma_f32_16x16x16bf16_1k(__builtin_bit_cast(s16x4, rw.v[db]), pb4, oacc[db], 0, 0, 0);
    if constexpr (SPLIT_P) {
        const s16x4 rb4 = __builtin_bit_cast(s16x4, rp);
#pragma unroll
        for (int db = 0; db < DBN; ++db)
            oacc[db] = __builtin_amdgcn_mfma_f32_16x16x16bf16_1k(__builtin_bit_cast(s16x4, rw.v[db]), rb4, oacc[db], 0, 0, 0);
    }
}

// SOLO: the calling wave runs the whole tile on its own (NW = 1): no LDS, no barrier, the result is written from the
// accumulator registers; the other waves of the workgroup run other tiles at the same time.
// (bf16 pages; FP8 pages are read by narrow_item_wide.)
template <int HD, int NW, int NK, int NV, bool SOLO = false, bool SPLIT_P = false, Partials WAY = kToL2>
__device__ __forceinline__ void narrow_item(const KParams& P, const ppd_work_item& it, char* smem) {
    static_assert(!SOLO || NW == 1, "a solo tile is one wave");
    constexpr int EB = 2;  // bytes per pool element
    using KVec = u32x4;    // 8 elements
    using VVec = u32x2;    // 4 elements
    constexpr int KS = HD / 32;   // k-steps of S^T
    constexpr int DBN = HD / 16;  // 16-row d blocks of O^T
    constexpr int CB = NarrowCombine<NW>::CB;
    constexpr int WSTRIDE = CB * (HD + 2);  // floats per wave in the combine buffer
    constexpr int NT = NW * 64;

    const int tid = threadIdx.x;
    const int lane = tid & 63;
    const int wave = SOLO ? 0 : __builtin_amdgcn_readfirstlane(tid >> 6);
    const int c16 = lane & 15;
    const int g4 = lane >> 4;
    const int G = P.G;
    const int ncols = it.nrows * G;
    const int colc = c16 < ncols ? c16 : ncols - 1;
    const int jrow = col_row(colc, P.invG);
    const int head = it.kvh * G + (colc - jrow * G);
    const int limit = it.L + it.row0 + jrow;
    const int min_limit = it.L + it.row0;

    bf16x8 qreg[KS];
    {
        const uint16_t* qp = P.q + ((int64_t)(it.grow0 + jrow) * P.Hq + head) * HD + g4 * 8;
#pragma unroll
        for (int ks = 0; ks < KS; ++ks) {
            u32x4 w = *reinterpret_cast<const u32x4*>(qp + ks * 32);
            if (c16 >= ncols) w = u32x4{0, 0, 0, 0};
            qreg[ks] = as_bf16x8(w);
        }
    }

    const int32_t* pt_row = P.page_tables + (int64_t)it.seq * P.max_pages;
    const int last_page = (it.kv_total - 1) >> 4;
    const int nsteps = (it.kv_end - it.kv_begin + kPage - 1) >> 4;  // one page per step
    const int s_lo = wave * nsteps / NW, s_hi = (wave + 1) * nsteps / NW;
    const int wave_first_page = (it.kv_begin >> 4) + s_lo;
    const int64_t head_off = (int64_t)it.kvh * (kPage * HD);
    const int64_t v_off = (int64_t)P.Hkv * (kPage * HD);

    f32x4 oacc[DBN];
#pragma unroll
    for (int db = 0; db < DBN; ++db) oacc[db] = f32x4{0.f, 0.f, 0.f, 0.f};
    float m_run = NEG_INF, l_run = 0.f;
    const float c = P.scale_log2e;

    // lane i of `ids_*` holds the page of logical page (batch*64 + i) of this wave's range.  K loads run NK - 1 steps
    // ahead of the computation and drive the rotation of the id batches; V loads run NV - 1 <= NK - 1 steps ahead
    // and may still be in the batch before (ids_old).
    int ids_old = 0, ids_cur = 0, ids_nxt = 0, k_batch = 0;
    auto load_ids = [&](int batch) { return load_page_id(pt_row, wave_first_page + batch * 64 + lane, last_page); };
    using KRegs = NarrowK<HD>;
    using VRegs = NarrowV<HD>;
    KRegs rk[NK];
    VRegs rv[NV];
    const int my_steps = s_hi - s_lo;
    const uint32_t k_lane_bytes = (uint32_t)(g4 * 128 + c16 * 8) * EB;                          // + ks * 512 elements
    const uint32_t v_lane_bytes = (uint32_t)(((g4 >> 1) * HD + c16) * 8 + (g4 & 1) * 4) * EB;  // + db * 128 elements
    // K and V are read once: non-temporal loads (no reuse to keep in the caches) stream ~12 % faster than plain
    // ones on this pattern.  Address = wave-uniform base of the (page, head) block + one 32-bit byte offset per lane.
    auto issue_k = [&](int k, KRegs& r) {  // k = step index relative to s_lo
        if ((k & 63) == 0 && k > 0) {
            ids_old = ids_cur;
            ids_cur = ids_nxt;
            k_batch = k >> 6;
            if (k + 64 < my_steps) ids_nxt = load_ids(k_batch + 1);
        }
        const int64_t pa = checked_page(P, __builtin_amdgcn_readlane(ids_cur, k & 63));
        const char* kb = reinterpret_cast<const char*>(P.pool) + (pa * P.page_stride + head_off) * EB;
#pragma unroll
        for (int ks = 0; ks < KS; ++ks)
            r.k[ks] = __builtin_nontemporal_load(reinterpret_cast<const KVec*>(kb + k_lane_bytes + ks * (512 * EB)));
    };
    auto issue_v = [&](int k, VRegs& r) {
        const int ids = (k >> 6) == k_batch ? ids_cur : ids_old;
        const int64_t pa = checked_page(P, __builtin_amdgcn_readlane(ids, k & 63));
        const char* vb = reinterpret_cast<const char*>(P.pool) + (pa * P.page_stride + head_off + v_off) * EB;
#pragma unroll
        for (int db = 0; db < DBN; ++db)
            r.v[db] = __builtin_nontemporal_load(reinterpret_cast<const VVec*>(vb + v_lane_bytes + db * (128 * EB)));
    };
    auto compute_step = [&](int k, KRegs& rs, VRegs& rw) { narrow_step<HD, SPLIT_P>(it, it.kv_begin + (s_lo + k) * kPage, limit, c, qreg, rs, rw, oacc, m_run, l_run); };

    // K of NK - 1 pages and V of NV - 1 pages (4 KiB each at D = 128) are in flight per wave while one page is being
    // computed; the register sets rotate (period = NK steps if NK = NV, else NK * NV, unrolled).  The loads sit under conditions, so at
    // the points where paths meet the compiler's waits on the memory counter assume the path with the fewest loads
    // issued and mostly drain what was just issued.  That costs nothing here: a loop without any conditional load
    // (waits of 36..47 outstanding loads in its steady state) was built and measured the same -- a compute unit
    // pulls at most ~58 GB/s from HBM however much it keeps in flight (a load-only kernel with 4 KiB or 28 KiB in
    // flight per wave, 8 or 16 waves: 54..60 GB/s per unit), and eight waves with one page each are already there.
    if (my_steps > 0) {
        ids_cur = load_ids(0);
        if (my_steps > 64) ids_nxt = load_ids(1);
#pragma unroll
        for (int j = 0; j < NK - 1; ++j)
            if (j < my_steps) issue_k(j, rk[j]);
#pragma unroll
        for (int j = 0; j < NV - 1; ++j)
            if (j < my_steps) issue_v(j, rv[j]);
    }
    constexpr int PERIOD = NK == NV ? NK : NK * NV;
    for (int k = 0; k < my_steps; k += PERIOD) {
#pragma unroll
        for (int j = 0; j < PERIOD; ++j) {
            if (k + j < my_steps) {
                if (k + j + NK - 1 < my_steps) issue_k(k + j + NK - 1, rk[(j + NK - 1) % NK]);
                if (k + j + NV - 1 < my_steps) issue_v(k + j + NV - 1, rv[(j + NV - 1) % NV]);
                compute_step(k + j, rk[j % NK], rv[j % NV]);
            }
        }
    }
    l_run += xor_shuffle(l_run, 16);
    l_run = sum_halves(l_run);

    if constexpr (SOLO) {
        // O^T register i of block db is d = db*16 + 4*g4 + i of column c16; m and l are the column's in every lane
        if (c16 < ncols) {
            if (it.part_off < 0) {
                const float inv = P.v_scale / l_run;
                uint16_t* op = P.out + ((int64_t)(it.grow0 + jrow) * P.Hq + head) * HD + 4 * g4;
#pragma unroll
                for (int db = 0; db < DBN; ++db) {
                    u32x2 w;
                    w[0] = pack_bf16(oacc[db][0] * inv, oacc[db][1] * inv);
                    w[1] = pack_bf16(oacc[db][2] * inv, oacc[db][3] * inv);
                    *reinterpret_cast<u32x2*>(op + db * 16) = w;
                }
            } else {
                float* pp = P.partials + it.part_off;
#pragma unroll
                for (int db = 0; db < DBN; ++db)
                    *reinterpret_cast<f32x4*>(pp + (int64_t)c16 * HD + db * 16 + 4 * g4) = oacc[db];
                if (g4 == 0) {
                    pp[(int64_t)ncols * HD + c16 * 2] = m_run;
                    pp[(int64_t)ncols * HD + c16 * 2 + 1] = l_run;
                }
            }
        }
        return;
    }
    // combine the waves, CB columns per pass: O^T register i of block db is d = db*16 + 4*g4 + i of column c16
    float* wbuf = reinterpret_cast<float*>(smem) + wave * WSTRIDE;
    const float* all = reinterpret_cast<const float*>(smem);
    for (int c0 = 0; c0 < ncols; c0 += CB) {
        if (c0 > 0) __syncthreads();  // the previous pass has been read
        if (c16 >= c0 && c16 < c0 + CB) {
#pragma unroll
            for (int db = 0; db < DBN; ++db)
                *reinterpret_cast<f32x4*>(wbuf + (c16 - c0) * HD + db * 16 + 4 * g4) = oacc[db];
            if (g4 == 0) {
                wbuf[CB * HD + (c16 - c0) * 2] = m_run;
                wbuf[CB * HD + (c16 - c0) * 2 + 1] = l_run;
            }
        }
        __syncthreads();
        narrow_combine<HD, NW, WAY>(P, it, all, c0);
    }
}

// ---------------------------------------------------------------------------------------------------
// Narrow tile on the operand shapes of the row-block tile: v_mfma_f32_32x32x16_bf16 for both products, two pages (32
// keys) per step, operands loaded from the pool straight into registers.  A lane then loads whole granules -- 8 d of one
// key for K, 8 tokens of one d for V -- in runs of 256 and 512 contiguous bytes per half-wave, where the 16x16 shapes of
// narrow_item make a lane own 4 tokens of a d (half a granule).  For FP8 pages that is 8 bytes per lane instead of 4 in
// V, and a compute unit streams a third more (measured with loads alone: 45 against 33 GB/s; bf16 pages 53 against 48).
// Half of the 32 columns of every product are unused (a narrow tile has at most 16), which costs matrix time the
// memory-bound tile has to spare.  Used for FP8 pages.
//   S^T rows: MFMA row r is key (page r >> 4 of the pair, token 8*bit2(r) + 4*bit3(r) + (r & 3)), so that accumulator
//   registers 0..7 of a lane are tokens 8h..8h+7 of the first page and 8..15 those of the second (h = lane / 32):
//   the octet the lane's V granules hold.
// NS register sets of one page pair each rotate: NS - 1 pairs are in flight per wave besides the one being computed.
// ---------------------------------------------------------------------------------------------------
template <int HD, int NW, int NS, bool SOLO, bool FP8, bool SPLIT_P = false, Partials WAY = kToL2>
__device__ __forceinline__ void narrow_item_wide(const KParams& P, const ppd_work_item& it, char* smem) {
    static_assert(!SOLO || NW == 1, "a solo tile is one wave");
    constexpr int EB = FP8 ? 1 : 2;                       // bytes per pool element
    using Vec = std::conditional_t<FP8, u32x2, u32x4>;    // a granule: 8 elements
    constexpr int KS = HD / 16;   // k-steps of S^T
    constexpr int DB = HD / 32;   // 32-row d blocks of O^T
    constexpr int CB = NarrowCombine<NW>::CB;
    constexpr int WSTRIDE = CB * (HD + 2);
    constexpr int NT = NW * 64;

    const int tid = threadIdx.x;
    const int lane = tid & 63;
    const int wave = SOLO ? 0 : __builtin_amdgcn_readfirstlane(tid >> 6);
    const int r = lane & 31;   // column of the products' B operands and results; key row / d row of the A operands
    const int h = lane >> 5;
    const int G = P.G;
    const int ncols = it.nrows * G;
    const int colc = r < ncols ? r : ncols - 1;
    const int jrow = col_row(colc, P.invG);
    const int head = it.kvh * G + (colc - jrow * G);
    const int limit = it.L + it.row0 + jrow;
    const int min_limit = it.L + it.row0;

    bf16x8 qreg[KS];  // Q^T operand: column r, d = ks*16 + h*8 .. +8; zero for the unused columns
    {
        const uint16_t* qp = P.q + ((int64_t)(it.grow0 + jrow) * P.Hq + head) * HD + h * 8;
#pragma unroll
        for (int ks = 0; ks < KS; ++ks) {
            u32x4 w = *reinterpret_cast<const u32x4*>(qp + ks * 16);
            if (r >= ncols) w = u32x4{0, 0, 0, 0};
            qreg[ks] = as_bf16x8(w);
        }
    }

    const int32_t* pt_row = P.page_tables + (int64_t)it.seq * P.max_pages;
    const int last_page = (it.kv_total - 1) >> 4;
    const int npages = (it.kv_end - it.kv_begin + kPage - 1) >> 4;
    const int s_lo = wave * npages / NW, s_hi = (wave + 1) * npages / NW;
    const int my_pages = s_hi - s_lo;
    const int my_steps = (my_pages + 1) >> 1;  // page pairs; the last may lack its second page
    const int wave_first_page = (it.kv_begin >> 4) + s_lo;
    const int64_t head_off = (int64_t)it.kvh * (kPage * HD);
    const int64_t v_off = (int64_t)P.Hkv * (kPage * HD);

    f32x16 oacc[DB];
#pragma unroll
    for (int db = 0; db < DB; ++db)
#pragma unroll
        for (int i = 0; i < 16; ++i) oacc[db][i] = 0.f;
    float m_run = NEG_INF, l_run = 0.f;
    const float c = P.scale_log2e;

    // lane i of ids_cur holds the page of logical page (batch*64 + i) of this wave's range; a pair never straddles batches
    int ids_cur = 0, ids_nxt = 0;
    auto load_ids = [&](int batch) { return load_page_id(pt_row, wave_first_page + batch * 64 + lane, last_page); };
    struct Set {
        Vec k[KS];      // K operand of the pair: 32 keys x 16 d per k-step
        Vec v[2][DB];   // V^T operand of each page: 32 d x 8 tokens (the lane's octet) per d block
    };
    Set rs[NS];
    const int k_tok = ((r >> 2) & 1) * 8 + ((r >> 3) & 1) * 4 + (r & 3);
    const uint32_t k_lane_bytes = (uint32_t)(h * 128 + k_tok * 8) * EB;   // + ks * 256 elements
    const uint32_t v_lane_bytes = (uint32_t)((h * HD + r) * 8) * EB;      // + db * 256 elements
    auto issue = [&](int j, Set& s) {  // j = pair index relative to s_lo
        const int pg0 = 2 * j;
        if ((pg0 & 63) == 0 && pg0 > 0) {
            ids_cur = ids_nxt;
            if (pg0 + 64 < my_pages) ids_nxt = load_ids((pg0 >> 6) + 1);
        }
        const int id_a = __builtin_amdgcn_readlane(ids_cur, pg0 & 63);
        const int id_b = pg0 + 1 < my_pages ? __builtin_amdgcn_readlane(ids_cur, (pg0 + 1) & 63) : id_a;  // absent: re-read the first
        const char* base_a = reinterpret_cast<const char*>(P.pool) + (checked_page(P, id_a) * P.page_stride + head_off) * EB;
        const char* base_b = reinterpret_cast<const char*>(P.pool) + (checked_page(P, id_b) * P.page_stride + head_off) * EB;
        const char* kb = ((r & 16) ? base_b : base_a) + k_lane_bytes;
#pragma unroll
        for (int ks = 0; ks < KS; ++ks) s.k[ks] = __builtin_nontemporal_load(reinterpret_cast<const Vec*>(kb + ks * (256 * EB)));
        const char* va = base_a + v_off * EB + v_lane_bytes;
        const char* vb = base_b + v_off * EB + v_lane_bytes;
#pragma unroll
        for (int db = 0; db < DB; ++db) s.v[0][db] = __builtin_nontemporal_load(reinterpret_cast<const Vec*>(va + db * (256 * EB)));
#pragma unroll
        for (int db = 0; db < DB; ++db) s.v[1][db] = __builtin_nontemporal_load(reinterpret_cast<const Vec*>(vb + db * (256 * EB)));
    };
    auto operand = [&](Vec v) {
        if constexpr (FP8) return as_bf16x8(fp8x8_to_bf16x8(v)); else return as_bf16x8(v);
    };
    auto compute_step = [&](int j, Set& s) {
        f32x16 sa;
#pragma unroll
        for (int i = 0; i < 16; ++i) sa[i] = 0.f;
#pragma unroll
        for (int ks = 0; ks < KS; ++ks) sa = __builtin_amdgcn_mfma_f32_32x32x16_bf16(operand(s.k[ks]), qreg[ks], sa, 0, 0, 0);
        // sa[i]: token 8*h + (i & 7) of page i >> 3 of the pair
        const int t0 = it.kv_begin + (s_lo + 2 * j) * kPage;
        const bool has_b = 2 * j + 1 < my_pages;
        if (t0 + 2 * kPage - 1 > min_limit || t0 + 2 * kPage > it.kv_end || !has_b) {
#pragma unroll
            for (int i = 0; i < 16; ++i) {
                const int pos = t0 + (i >> 3) * kPage + h * 8 + (i & 7);
                if (pos > limit || pos >= it.kv_end || ((i >> 3) && !has_b)) sa[i] = NEG_INF;
            }
            if (t0 + 2 * kPage > it.kv_total || !has_b) {  // rows never written, or the page that is not there
#pragma unroll
                for (int pg = 0; pg < 2; ++pg)
#pragma unroll
                    for (int db = 0; db < DB; ++db)
#pragma unroll
                        for (int e = 0; e < 8; ++e) {
                            const int pos = t0 + pg * kPage + h * 8 + e;
                            if (pos >= it.kv_total || (pg && !has_b)) {
                                if constexpr (FP8) s.v[pg][db][e >> 2] &= ~(0xFFu << (8 * (e & 3)));  // code 0 is 0.0
                                else s.v[pg][db][e >> 1] &= (e & 1) ? 0x0000FFFFu : 0xFFFF0000u;
                            }
                        }
            }
        }
        float mx = sa[0];
#pragma unroll
        for (int i = 1; i < 16; ++i) mx = fmaxf(mx, sa[i]);
        mx = max_halves(mx);
        const float m_new = fmaxf(m_run, mx);
        if (__any((m_new - m_run) * c > kLazyRescale)) {
            const float m_use = m_new == NEG_INF ? 0.f : m_new;
            const float alpha = fast_exp2(m_run * c - m_use * c);
            l_run *= alpha;
#pragma unroll
            for (int db = 0; db < DB; ++db)
#pragma unroll
                for (int i = 0; i < 16; ++i) oacc[db][i] *= alpha;
            m_run = m_new;
        }
        const float mc = m_run == NEG_INF ? 0.f : m_run * c;
        u32x4 pw[2], rest[2];
        float psum = 0.f;
#pragma unroll
        for (int pg = 0; pg < 2; ++pg)
#pragma unroll
            for (int e = 0; e < 4; ++e) {
                const float p0 = fast_exp2(__builtin_fmaf(sa[pg * 8 + 2 * e], c, -mc));
                const float p1 = fast_exp2(__builtin_fmaf(sa[pg * 8 + 2 * e + 1], c, -mc));
                psum += p0 + p1;
                if constexpr (SPLIT_P) {
                    const u32x2 two = split_bf16(p0, p1);
                    pw[pg][e] = two[0];
                    rest[pg][e] = two[1];
                } else {
                    pw[pg][e] = pack_bf16(p0, p1);
                }
            }
        l_run += psum;
#pragma unroll
        for (int pg = 0; pg < 2; ++pg)
#pragma unroll
            for (int db = 0; db < DB; ++db) {
                const bf16x8 v = operand(s.v[pg][db]);
                oacc[db] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(v, as_bf16x8(pw[pg]), oacc[db], 0, 0, 0);
                if constexpr (SPLIT_P) oacc[db] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(v, as_bf16x8(rest[pg]), oacc[db], 0, 0, 0);
            }
    };

    if (my_steps > 0) {
        ids_cur = load_ids(0);
        if (my_pages > 64) ids_nxt = load_ids(1);
#pragma unroll
        for (int j = 0; j < NS - 1; ++j)
            if (j < my_steps) issue(j, rs[j]);
    }
    for (int k = 0; k < my_steps; k += NS) {
#pragma unroll
        for (int j = 0; j < NS; ++j) {
            if (k + j < my_steps) {
                if (k + j + NS - 1 < my_steps) issue(k + j + NS - 1, rs[(j + NS - 1) % NS]);
                compute_step(k + j, rs[j]);
            }
        }
    }
    const float l_tot = sum_halves(l_run);

    // O^T register i of block db is d = db*32 + (i/4)*8 + h*4 + i%4 of column r; m and l_tot are the column's in both halves
    if constexpr (SOLO) {
        if (r < ncols) {
            if (it.part_off < 0) {
                const float inv = P.v_scale / l_tot;
                uint16_t* op = P.out + ((int64_t)(it.grow0 + jrow) * P.Hq + head) * HD + h * 4;
#pragma unroll
                for (int db = 0; db < DB; ++db)
#pragma unroll
                    for (int i4 = 0; i4 < 4; ++i4) {
                        u32x2 w;
                        w[0] = pack_bf16(oacc[db][i4 * 4 + 0] * inv, oacc[db][i4 * 4 + 1] * inv);
                        w[1] = pack_bf16(oacc[db][i4 * 4 + 2] * inv, oacc[db][i4 * 4 + 3] * inv);
                        *reinterpret_cast<u32x2*>(op + db * 32 + i4 * 8) = w;
                    }
            } else {
                float* pp = P.partials + it.part_off;
                float* po = pp + (int64_t)r * HD + h * 4;
#pragma unroll
                for (int db = 0; db < DB; ++db)
#pragma unroll
                    for (int i4 = 0; i4 < 4; ++i4) {
                        const f32x4 w = {oacc[db][i4 * 4 + 0], oacc[db][i4 * 4 + 1], oacc[db][i4 * 4 + 2], oacc[db][i4 * 4 + 3]};
                        *reinterpret_cast<f32x4*>(po + db * 32 + i4 * 8) = w;
                    }
                if (h == 0) {
                    pp[(int64_t)ncols * HD + r * 2] = m_run;
                    pp[(int64_t)ncols * HD + r * 2 + 1] = l_tot;
                }
            }
        }
        return;
    }
    // combine the waves through LDS, CB columns per pass (the buffer and the second half are those of narrow_item)
    float* wbuf = reinterpret_cast<float*>(smem) + wave * WSTRIDE;
    const float* all = reinterpret_cast<const float*>(smem);
    for (int c0 = 0; c0 < ncols; c0 += CB) {
        if (c0 > 0) __syncthreads();  // the previous pass has been read
        if (r >= c0 && r < c0 + CB && r < ncols) {
#pragma unroll
            for (int db = 0; db < DB; ++db)
#pragma unroll
                for (int i4 = 0; i4 < 4; ++i4) {
                    const f32x4 w = {oacc[db][i4 * 4 + 0], oacc[db][i4 * 4 + 1], oacc[db][i4 * 4 + 2], oacc[db][i4 * 4 + 3]};
                    *reinterpret_cast<f32x4*>(wbuf + (r - c0) * HD + db * 32 + i4 * 8 + h * 4) = w;
                }
            if (h == 0) {
                wbuf[CB * HD + (r - c0) * 2] = m_run;
                wbuf[CB * HD + (r - c0) * 2 + 1] = l_tot;
            }
        }
        __syncthreads();
        narrow_combine<HD, NW, WAY>(P, it, all, c0);
    }
}

// Claims the next tile of queue q: its index in the work list, or -1 when the queue is exhausted.  A claim on the
// wave-tile queue covers kWaves consecutive tiles and returns the index of the first.
__device__ __forceinline__ int claim_from(const KParams& P, int q) {
    const int got = (int)atomicAdd(&P.counters[kCursorBase + q * kCursorStride], 1u) * (q == kWaveQueue ? kWaves : 1);
    return got < P.queue_begin[q + 1] - P.queue_begin[q] ? P.queue_begin[q] + got : -1;
}

// The last workgroup of a kernel to run out of work re-arms the cursors of queues [q0, q1) and the kernel's own
// count of finished workgroups (word `done_word`) for the next launch.
__device__ __forceinline__ void rearm_cursors(const KParams& P, int q0, int q1, int done_word) {
    const unsigned done = atomicAdd(&P.counters[done_word], 1u);
    if (done == gridDim.x - 1) {
        for (int q = q0; q < q1; ++q)
            __hip_atomic_store(&P.counters[kCursorBase + q * kCursorStride], 0u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        __hip_atomic_store(&P.counters[done_word], 0u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    }
}

// The tile of the mixed kernels that stands at `idx` of the list; one-wave tiles, which are those from n_wg to `end`, kWaves at a time.
template <int HD, bool FP8>
__device__ __forceinline__ void mixed_tile(const KParams& P, int idx, int n_wg, int end, char* smem) {
    if (idx >= n_wg) {
        // wave w runs tile idx + w on its own
        const int mine = idx + __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
        if (mine < end) {
            const ppd_work_item it = P.items[mine];
            if constexpr (FP8) narrow_item_wide<HD, 1, fp8_sets(HD), true, true>(P, it, smem);
            else narrow_item<HD, 1, mixed_sets(HD), mixed_sets(HD), true>(P, it, smem);
        }
        return;
    }
    const ppd_work_item it = P.items[idx];
    if (it.kind == 0) {
        if constexpr (FP8) narrow_item_wide<HD, kWaves, fp8_sets(HD), false, true>(P, it, smem);
        else narrow_item<HD, kWaves, mixed_sets(HD), mixed_sets(HD), false>(P, it, smem);
    } else {
        mfma_item<HD, false, FP8>(P, it, smem);
    }
}

template <int HD, bool FP8>
__global__ __launch_bounds__(kThreads, 2) void ppd_mixed_kernel(const KParams P) {
    // Dynamic LDS: rings of kStages + 1 stages of 4 pages of K and as many of V, then the page ids of a tile's key
    // range, for the MFMA path (136 KiB at HD = 128); the narrow path's combine buffer (kWaves * 16 * (HD+2)
    // floats) uses the front of it.
    extern __shared__ __attribute__((aligned(16))) char smem[];
    __shared__ int s_next_slot;
    volatile int* s_next = &s_next_slot;
    const int tid = threadIdx.x;
    // Ten queues in one list: MFMA row-block tiles in eight queues, one per XCD (tiles that read the same K/V
    // sit in the same queue, next to each other, so the workgroups of one XCD find them in their L2), and one
    // queue of narrow tiles run by the whole workgroup and one of short narrow tiles run one per wave; each longest tile
    // first.  A workgroup prefers one kind, chosen by the compute
    // unit it runs on (narrow_cus of the 32 units of every XCD take narrow tiles, spread evenly over the shader
    // engines; the planner sizes the split so that both kinds finish together): workgroups that share a unit
    // then run the same kind, and HBM-bound and MFMA-bound tiles run side by side on different units.
    // It takes MFMA tiles from its own XCD's queue first, and steals from the other queues when its own run dry.
    int pref;
    switch (P.pref_mode) {
        case 1: pref = (blockIdx.x >> 3) & 1; break;
        case 2: {
            // HW_REG_HW_ID: cu_id in bits 11:8, se_id in bits 15:13 (eight active units per shader engine, ids
            // 0..8 with one gap, so the low three bits tell them apart)
            const unsigned hw = __builtin_amdgcn_s_getreg((15 << 11) | (0 << 6) | 4);
            const int unit = (int)(((hw >> 8) & 7) << 2 | ((hw >> 13) & 3));
            pref = unit < P.narrow_cus ? 1 : 0;
            break;
        }
        case 3: pref = 1; break;
        default: pref = 0; break;
    }
    const int xcd = (int)(__builtin_amdgcn_s_getreg((3 << 11) | (0 << 6) | 20) & (kXcds - 1));  // HW_REG_XCC_ID
    // bit q: queue q is exhausted (only thread 0 uses it).  Queues that are empty by construction never cost an
    // atomic; when a claim finds a queue exhausted, one batch of plain loads of all nine cursors tells which
    // others are, instead of one failing atomic (a round trip to the L2 each, one after the other) per queue --
    // that chain used to be the last ~10 us of every workgroup, and so of every launch.
    unsigned dry = 0;
#pragma unroll
    for (int q = 0; q < kQueues; ++q)
        if (P.queue_begin[q + 1] == P.queue_begin[q]) dry |= 1u << q;
    constexpr unsigned kAllDry = (1u << kQueues) - 1;
    auto look_at_cursors = [&]() {
        unsigned cur[kQueues];
#pragma unroll
        for (int q = 0; q < kQueues; ++q)
            cur[q] = __hip_atomic_load(&P.counters[kCursorBase + q * kCursorStride], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
#pragma unroll
        for (int q = 0; q < kQueues; ++q)
            if ((int)(cur[q] * (q == kWaveQueue ? kWaves : 1)) >= P.queue_begin[q + 1] - P.queue_begin[q]) dry |= 1u << q;
    };
    for (;;) {
        if (tid == 0) {
            int idx = -1;
#pragma unroll
            for (int attempt = 0; attempt < 2 && idx < 0; ++attempt) {
                const bool want_narrow = (attempt == 0) == (pref == 1);
                if (want_narrow) {
                    // whole-workgroup tiles first (the long ones), then the very short ones, eight to a claim
                    for (int q = kNarrowQueue; q <= kWaveQueue && idx < 0; ++q) {
                        if (dry & (1u << q)) continue;
                        idx = claim_from(P, q);
                        if (idx < 0) {
                            dry |= 1u << q;
                            if (dry != kAllDry) look_at_cursors();
                        }
                    }
                } else {
                    for (int a = 0; a < kXcds && idx < 0; ++a) {
                        const int q = (xcd + a) & (kXcds - 1);
                        if (dry & (1u << q)) continue;
                        idx = claim_from(P, q);
                        if (idx < 0) {
                            dry |= 1u << q;
                            if (dry != kAllDry) look_at_cursors();
                        }
                    }
                }
            }
            *s_next = idx;
        }
        __syncthreads();
        const int idx = __builtin_amdgcn_readfirstlane(*s_next);
        __syncthreads();  // everyone has read s_next, and the previous tile's LDS use is over
        if (idx < 0) break;
        mixed_tile<HD, FP8>(P, idx, P.queue_begin[kWaveQueue], P.queue_begin[kQueues], smem);
    }
    if (tid == 0) rearm_cursors(P, 0, kCursors, 10);
}

// A launch of the mixed kernel with a workgroup for every entry (a tile, or kWaves one-wave tiles) claims nothing: its list is in the order
// of the workgroups, the one-wave tiles behind the others.  A claim costs such a launch ~4 us of ~13: the first one, the one that finds the
// queues empty, and the re-arming of the cursors (small steps of 4 layers 233 -> 218, 59.3 -> 55.3 us); and with the order in the list
// the first read from memory is the work item, where the queues' bounds and a search in them came before it (steps of 8, 80 and 48 tiles 9.14 -> 8.57, 25.2 -> 23.4 and 12.1 -> 11.5 us).
// A kernel of its own: with both in one, what this one knows (its tile, the list's bounds) was kept over the other's loop, 91 spilled scalars
// on FP8 pages against 83 and 22 against 11 on bf16 pages.  66 decodes and turns of FP8 pages by 8 heads, 2176 tiles, 889 us in one kernel, 863 in
// two; 110 drawn launches with claims of FP8 pages 0.98 of the time, 190 of bf16 pages equal; 600 drawn launches without 0.97.
template <int HD, bool FP8>
__global__ __launch_bounds__(kThreads, 2) void ppd_mixed_by_block_kernel(const KParams P) {
    extern __shared__ __attribute__((aligned(16))) char smem[];
    const int block = (int)blockIdx.x;
    mixed_tile<HD, FP8>(P, block < P.n_wg ? block : P.n_wg + (block - P.n_wg) * kWaves, P.n_wg, P.n_items, smem);
}

// Merge of a split range by the last of its tiles, in the launch that made them: every tile of the group has counted itself in
// once its partial had reached the memory side, and the one that finds all others there does what ppd_merge_kernel does, splits
// in index order (bit for bit the same results).  Bound by latency: the count (one trip) and the partials (one trip for up to
// eight splits: the (m, l) pairs of all splits go to LDS while the first values are on their way).  A second launch costs
// 5.5 us for 4 splits and 10 for 12, this about 3.
// An arriving partial is ordered before its count by the wait below and needs no cache-wide write-back, because its stores go
// past the L2 (store_partial); the reads do so as well.
template <int HD, int NW>
__device__ __forceinline__ void merge_last(const KParams& P, const ppd_work_item* item, char* smem, volatile int* s_arrived) {
    constexpr int NT = NW * 64, LANES = HD / 2;  // lanes of a column, two d each
    constexpr int kStagedPairs = 4096;           // (m, l) pairs that fit the combine buffer
    static_assert(kStagedPairs * sizeof(f32x2) <= (size_t)NW * NarrowCombine<NW>::CB * (HD + 2) * sizeof(float), "staged in the combine buffer");
    const int tid = threadIdx.x;
    asm volatile("s_waitcnt vmcnt(0)" : "+s"(item) : : "memory");  // this wave's part of the partial has arrived
    const ppd_work_item it = *item;                   // read again: kept over the tile's loop it would cost that scalar registers
    __syncthreads();                                  // every wave's part has arrived; the combine buffer is free
    MergeGroup* const g = P.merge_groups + it.group;
    const int nsplit = g->nsplit;
    const int64_t stride = g->part_stride;
    const float* const base = P.partials + g->part_off;
    if (tid == 0) *s_arrived = (int)atomicAdd(&g->arrived, 1u);
    __syncthreads();
    if (__builtin_amdgcn_readfirstlane(*s_arrived) != nsplit - 1) return;
    if (tid == 0) __hip_atomic_store(&g->arrived, 0u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);  // for the next launch
    const int ncols = it.nrows * P.G;
    const float c = P.scale_log2e;
    f32x2* const ml = reinterpret_cast<f32x2*>(smem);  // [split][column]
    const bool staged = nsplit * ncols <= kStagedPairs;
    constexpr int AT_ONCE = 8;
    auto load_values = [&](int idx, int j0, f32x2 (&v)[AT_ONCE]) {
        const float* p = base + (int64_t)(idx / LANES) * HD + (idx % LANES) * 2;
#pragma unroll
        for (int t = 0; t < AT_ONCE; ++t) v[t] = load_partial2(p + stride * (j0 + t < nsplit ? j0 + t : j0));
    };
    auto pair = [&](int j, int col) { return staged ? ml[j * ncols + col] : load_partial2(base + stride * j + (int64_t)ncols * HD + col * 2); };
    f32x2 v[AT_ONCE];
    if (tid < ncols * LANES) load_values(tid, 0, v);
    if (staged) {
        const int col = tid & (kNarrowCols - 1);
        for (int j = tid / kNarrowCols; j < nsplit; j += NT / kNarrowCols)
            if (col < ncols) ml[j * ncols + col] = load_partial2(base + stride * j + (int64_t)ncols * HD + col * 2);
    }
    __syncthreads();
    for (int idx = tid; idx < ncols * LANES; idx += NT) {
        const int col = idx / LANES, d = (idx % LANES) * 2;
        float mm = NEG_INF;
        for (int j = 0; j < nsplit; ++j) mm = fmaxf(mm, pair(j, col)[0]);
        float o0 = 0.f, o1 = 0.f, l = 0.f;
        for (int j0 = 0; j0 < nsplit; j0 += AT_ONCE) {
            if (idx != tid || j0 > 0) load_values(idx, j0, v);
#pragma unroll
            for (int t = 0; t < AT_ONCE; ++t) {
                if (j0 + t < nsplit) {
                    const f32x2 w = pair(j0 + t, col);
                    const float f = w[0] == NEG_INF ? 0.f : fast_exp2((w[0] - mm) * c);
                    l += f * w[1];
                    o0 += f * v[t][0];
                    o1 += f * v[t][1];
                }
            }
        }
        const int crow = col_row(col, P.invG);
        const int64_t orow = (int64_t)(it.grow0 + crow) * P.Hq + it.kvh * P.G + (col - crow * P.G);
        *reinterpret_cast<uint32_t*>(P.out + orow * HD + d) = pack_bf16((o0 / l) * P.v_scale, (o1 / l) * P.v_scale);
    }
}

// ---------------------------------------------------------------------------------------------------
// A launch that holds narrow tiles only (a decode-only step).  Same tile code as in ppd_mixed_kernel, handed out
// differently: a small launch of the mixed kernel spends 1.7 us on its first claim and ~5 us finding out, claim by
// failing claim, that nothing is left, which is a quarter of a 25 us decode step.  Here the whole-workgroup tiles
// (longest first) and then the one-wave tiles, NW to a slot, form one row of slots; workgroup b takes slot b
// without asking, and only a launch with more slots than workgroups claims further ones (from gridDim.x on) with the
// cursor of the narrow queue, which the last workgroup to finish re-arms.  The host launches no more workgroups than
// there are slots.  Where two rounds are enough and the tiles are short, the second is handed out by index as well, from the
// end of the list: the claims (a trip to the memory side for every slot, and one more for each workgroup to learn that nothing is
// left) take as long as a fifth of such a launch.  us of 64 sequences with the append, claimed and by index: D = 128, 64-380 keys
// 19.9 and 18.6, 400-800 33.0 and 31.9, FP8 pages 25.3 and 23.8; D = 64, 64-380 16.0 and 13.1, 400-800 21.6 and 18.9.  The launch
// alone, 64 of equal length: 800 keys 38.6 and 37.1, 1500 64.5 and 63.1, FP8 pages 1600 42.4 and 40.6, 3000 67.5 and 65.9, D = 64
// 1500 36.3 and 34.5 (second_round_by_index has the exact rule and its figures; those of bf16 pages below 640 keys, 1280 at D = 64, are
// from before such tiles ran in ppd_pipelined_kernel).  Longer tiles
// and more rounds are claimed, because they do not take the time that their length says (48 of 2000-6000 keys 129.8 and 133.7, 100
// of 800-1600 88.0 and 90.8, 400 of 800-1600 314 and 327).  Measured and not kept: claiming the next slot before running the
// current one (hides the round trip but holds a slot that an idle workgroup could have run: cfg2 186 -> 206 us).
// The list and its bounds (n_wg whole-workgroup tiles, `end` tiles in all) are arguments of their own, which arrive in scalar registers:
// a workgroup's first read is its work item, where it used to be the arguments, then the bounds, then the item (6 decodes of
// 1K-3K keys 20.0 -> 19.7 us a layer, 11 of 300-6500 33.4 -> 33.1).
// NSETS: rotating register sets of a streaming wave of a whole-workgroup tile, of one page each on bf16 pages (kLongSets where
// the tiles are long and kShortSets where they are short) and of a page pair on FP8 pages (one, or fp8_sets).  NW: eight
// waves, or four of twice the registers where the tiles are long and there are many (long_tiles_on_four_waves); narrow_form has the
// figures of the former.  MERGES: a launch with a workgroup for every tile, none of
// them on a single wave, that merges split ranges itself.  A form of its own: beside the loop over slots the merge costs every
// tile of the other launches registers and spilled scalars, and the loop the merging ones (drawn decode steps, 150 on each format,
// 5 % less time on FP8 pages and 1 % on bf16 pages; of up to 12 long sequences, 120 each, 6 % and 2 %).
// ---------------------------------------------------------------------------------------------------
template <int HD, bool FP8, int NW, int NSETS, bool MERGES = false>
__global__ __launch_bounds__(64 * NW, NW / 4) void ppd_narrow_kernel(const ppd_work_item* items, int n_wg, int end, const KParams P) {
    extern __shared__ __attribute__((aligned(16))) char smem[];  // the combine buffer
    __shared__ int s_shared;
    volatile int* s_next = &s_shared;
    if constexpr (MERGES) {
        const int slot = blockIdx.x;
        if (slot >= n_wg) return;
        const ppd_work_item it = items[slot];
        if constexpr (FP8) narrow_item_wide<HD, NW, NSETS, false, true, false, kPastL2>(P, it, smem);
        else narrow_item<HD, NW, NSETS, NSETS, false, false, kPastL2>(P, it, smem);
        if (it.part_off >= 0) merge_last<HD, NW>(P, items + slot, smem, s_next);
        return;
    }
    const int tid = threadIdx.x;
    const int slots = n_wg + (end - n_wg + NW - 1) / NW;
    const bool claims = slots > (int)gridDim.x && !P.by_index;  // the same for every workgroup of the launch
    int slot = blockIdx.x;
    while (slot < slots) {
        if (slot < n_wg) {
            const ppd_work_item it = items[slot];
            if constexpr (FP8) narrow_item_wide<HD, NW, NSETS, false, true, false, kAsLaunched>(P, it, smem);
            else narrow_item<HD, NW, NSETS, NSETS, false, NW != kWaves, kAsLaunched>(P, it, smem);
        } else if constexpr (NW == kWaves) {
            const int mine = n_wg + (slot - n_wg) * NW + __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
            if (mine < end) {
                const ppd_work_item it = items[mine];
                if constexpr (FP8) narrow_item_wide<HD, 1, fp8_sets(HD), true, true>(P, it, smem);
                else narrow_item<HD, 1, NSETS, NSETS, true>(P, it, smem);
            }
        }
        if (!claims) {
            // by index: a second slot from the end of the list, so that the longest and the shortest tiles meet
            slot = slot < (int)gridDim.x ? 2 * (int)gridDim.x - 1 - slot : slots;
            if (slot < slots) __syncthreads();  // the tile's combine is over
            continue;
        }
        if (tid == 0) *s_next = (int)gridDim.x + (int)atomicAdd(&P.counters[kCursorBase + kNarrowQueue * kCursorStride], 1u);
        __syncthreads();
        slot = __builtin_amdgcn_readfirstlane(*s_next);
        __syncthreads();  // everyone has read s_next, and the previous tile's combine is over
    }
    if (claims && tid == 0) rearm_cursors(P, kNarrowQueue, kNarrowQueue + 1, 10);
}

// ---------------------------------------------------------------------------------------------------
// Decode-only launches of several rounds of short tiles (bf16 pages; whole-workgroup tiles).  A short tile streams for a few
// microseconds, and the same again went by between its last load and the first one of the next tile: the combine, the claim, and
// three reads that wait for one another (work item, page ids, K and V).  Here all of that happens ahead.  While a tile runs, the
// workgroup holds the work item of the next two, page ids and queries of the next one, and a claim under way; the first kPipelinedSets
// pages of the next tile are asked for as soon as a wave is through with its share of this one, before the waves' results meet in
// LDS (two buffers, so that a tile needs one barrier, which leaves the loads in flight).
// The first three slots of a workgroup go by index, up, down and up the list, longest tiles first; the others are claimed.  Bit for bit
// the results of ppd_narrow_kernel.  A launch of 8 tiles of 100 keys to a workgroup 47.0 -> 37.5 us, of 8 of 382 79.3 -> 74.3 (both run on
// single waves now), of 3 of 800-1600 79.1 -> 75.5 (6.2 TB/s); 90 decodes of 420-600 keys by 8 heads, 720 tiles, 33 us, 5.8 TB/s, and HBM reads 1.02 times
// K, V and queries (64 of 100-300 keys 1.05); two, three and four register sets, and the heads of a page on one XCD or on eight, are within 1 %.  What is left of a
// tile of 100 keys is 4 us: one trip of its loads, and its pages worked.
// ---------------------------------------------------------------------------------------------------
constexpr int kPipelinedSets = 3, kByIndexSlots = 3;
template <int HD>
constexpr size_t pipelined_lds_bytes() { return 2 * NarrowCombine<kWaves>::bytes(HD); }

template <int HD>
__global__ __launch_bounds__(kThreads, 2) void ppd_pipelined_kernel(const ppd_work_item* items, int slots, const KParams P) {
    constexpr int NW = kWaves, NS = kPipelinedSets, KS = HD / 32, DBN = HD / 16, CB = NarrowCombine<NW>::CB, WSTRIDE = CB * (HD + 2);
    static_assert(CB == kNarrowCols, "one pass of the combine takes all columns");
    extern __shared__ __attribute__((aligned(16))) char smem[];  // two combine buffers
    __shared__ int s_claimed[2];
    const int tid = threadIdx.x, lane = tid & 63, c16 = lane & 15, g4 = lane >> 4;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int grid = (int)gridDim.x, block = (int)blockIdx.x, G = P.G;
    if (block >= slots) return;
    const float c = P.scale_log2e;
    const bool claims = slots > kByIndexSlots * grid;
    typedef const __attribute__((address_space(4))) ppd_work_item* ItemPtr;  // read through the scalar cache: work items are written by the upload, an earlier launch on this stream, only
    // a tile as the workgroup holds it; one of no steps where the slot does not exist
    struct Tile {
        ppd_work_item it;
        int slot, first_page, steps;  // of this wave: its share of the pages
    };
    auto tile_of = [&](int slot) {
        Tile t;
        t.slot = slot;
        const ItemPtr p = (ItemPtr)(uintptr_t)(items + (slot < slots ? slot : slots - 1));
        t.it.seq = p->seq; t.it.kvh = p->kvh; t.it.row0 = p->row0; t.it.nrows = p->nrows; t.it.grow0 = p->grow0; t.it.L = p->L;
        t.it.kv_total = p->kv_total; t.it.kv_begin = p->kv_begin; t.it.kv_end = p->kv_end; t.it.part_off = p->part_off;
        const int npages = (t.it.kv_end - t.it.kv_begin + kPage - 1) >> 4;
        t.first_page = wave * npages / NW;
        t.steps = slot < slots ? (wave + 1) * npages / NW - t.first_page : 0;
        t.first_page += t.it.kv_begin >> 4;
        return t;
    };
    // lane i: the page of the share's logical page i (a share is at most 64 pages)
    auto ids_of = [&](const Tile& t) {
        return load_page_id(P.page_tables + (int64_t)t.it.seq * P.max_pages, t.first_page + lane, (t.it.kv_total - 1) >> 4);
    };
    struct Column { int jrow, head; };
    auto column = [&](const Tile& t) {
        const int ncols = t.it.nrows * G, colc = c16 < ncols ? c16 : ncols - 1, jrow = col_row(colc, P.invG);
        return Column{jrow, t.it.kvh * G + (colc - jrow * G)};
    };
    struct Queries { u32x4 w[KS]; };
    auto queries_of = [&](const Tile& t) {
        const Column col = column(t);
        const uint16_t* qp = P.q + ((int64_t)(t.it.grow0 + col.jrow) * P.Hq + col.head) * HD + g4 * 8;
        Queries q;
#pragma unroll
        for (int ks = 0; ks < KS; ++ks) q.w[ks] = *reinterpret_cast<const u32x4*>(qp + ks * 32);
        return q;
    };
    NarrowK<HD> rk[NS];
    NarrowV<HD> rv[NS];
    const uint32_t k_lane_bytes = (uint32_t)(g4 * 128 + c16 * 8) * 2;                          // + ks * 512 elements
    const uint32_t v_lane_bytes = (uint32_t)(((g4 >> 1) * HD + c16) * 8 + (g4 & 1) * 4) * 2;  // + db * 128 elements
    const int64_t v_off = (int64_t)P.Hkv * (kPage * HD);
    auto issue = [&](const Tile& t, int ids, int k, NarrowK<HD>& r, NarrowV<HD>& w) {
        const int64_t pa = checked_page(P, __builtin_amdgcn_readlane(ids, k));
        const char* kb = reinterpret_cast<const char*>(P.pool) + (pa * P.page_stride + (int64_t)t.it.kvh * (kPage * HD)) * 2;
#pragma unroll
        for (int ks = 0; ks < KS; ++ks) r.k[ks] = __builtin_nontemporal_load(reinterpret_cast<const u32x4*>(kb + k_lane_bytes + ks * 1024));
        const char* vb = kb + v_off * 2;
#pragma unroll
        for (int db = 0; db < DBN; ++db) w.v[db] = __builtin_nontemporal_load(reinterpret_cast<const u32x2*>(vb + v_lane_bytes + db * 256));
    };
    auto begin = [&](const Tile& t, int ids) {
#pragma unroll
        for (int j = 0; j < NS; ++j)
            if (j < t.steps) issue(t, ids, j, rk[j], rv[j]);
    };
    unsigned claim = 0;
    auto draw = [&]() {  // only thread 0's is used
        if (claims && tid == 0) claim = atomicAdd(&P.counters[kCursorBase + kNarrowQueue * kCursorStride], 1u);
    };

    // The first tile's pages before anything of the tiles behind it.  With the reads of those in front, a launch whose longest tiles have a
    // workgroup to themselves took longer than one tile after the other does: 280 tiles of 37-485 keys 10.6 us against 10.2, 10.05 this way.
    Tile cur = tile_of(block);
    int ids_cur = ids_of(cur);
    Queries q_cur = queries_of(cur);
    begin(cur, ids_cur);
    Tile nxt = tile_of(2 * grid - 1 - block), far = tile_of(2 * grid + block);
    int ids_nxt = ids_of(nxt);
    Queries q_nxt = queries_of(nxt);
    draw();
    for (int parity = 0;; parity ^= 1) {
        const int ncols = cur.it.nrows * G, limit = cur.it.L + cur.it.row0 + column(cur).jrow;
        bf16x8 qreg[KS];
#pragma unroll
        for (int ks = 0; ks < KS; ++ks) qreg[ks] = as_bf16x8(c16 < ncols ? q_cur.w[ks] : u32x4{0, 0, 0, 0});
        f32x4 oacc[DBN];
#pragma unroll
        for (int db = 0; db < DBN; ++db) oacc[db] = f32x4{0.f, 0.f, 0.f, 0.f};
        float m_run = NEG_INF, l_run = 0.f;
        for (int k = 0; k < cur.steps; k += NS) {
#pragma unroll
            for (int j = 0; j < NS; ++j) {
                if (k + j < cur.steps) {
                    narrow_step<HD, false>(cur.it, (cur.first_page + k + j) * kPage, limit, c, qreg, rk[j], rv[j], oacc, m_run, l_run);
                    if (k + j + NS < cur.steps) issue(cur, ids_cur, k + j + NS, rk[j], rv[j]);
                }
            }
        }
        // the next tile's pages, and what the one behind it needs
        begin(nxt, ids_nxt);
        ids_cur = ids_nxt;
        q_cur = q_nxt;
        ids_nxt = ids_of(far);
        q_nxt = queries_of(far);
        const int drawn = (int)claim;
        if (grid * kByIndexSlots + drawn < slots) draw();
        l_run += xor_shuffle(l_run, 16);
        l_run = sum_halves(l_run);
        float* const all = reinterpret_cast<float*>(smem) + parity * (NW * WSTRIDE);
        float* const wbuf = all + wave * WSTRIDE;
        if (c16 < ncols) {
#pragma unroll
            for (int db = 0; db < DBN; ++db) *reinterpret_cast<f32x4*>(wbuf + c16 * HD + db * 16 + 4 * g4) = oacc[db];
            if (g4 == 0) {
                wbuf[CB * HD + c16 * 2] = m_run;
                wbuf[CB * HD + c16 * 2 + 1] = l_run;
            }
        }
        if (tid == 0) s_claimed[parity] = drawn;
        asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory");  // for LDS only: the loads stay in flight
        const int slot = claims ? kByIndexSlots * grid + __builtin_amdgcn_readfirstlane(*(volatile int*)&s_claimed[parity]) : slots;
        const Tile got = tile_of(slot);
        narrow_combine<HD, NW, kAsLaunched>(P, cur.it, all, 0);
        cur = nxt;
        nxt = far;
        far = got;
        if (cur.slot >= slots) break;
    }
    // this workgroup's last claim has to have reached its cursor before the cursor is re-armed
    asm volatile("" : : "v"(claim));
    if (claims && tid == 0) rearm_cursors(P, kNarrowQueue, kNarrowQueue + 1, 10);
}

// ---------------------------------------------------------------------------------------------------
// Decode-only launches of many tiles, each on one wave (tiles_on_waves decides, and says what it measured).  A wave goes from
// tile to tile on its own -- no LDS, no barrier, no claim -- so that what a tile costs before and after its stream of loads passes
// under the streams of the unit's other waves.  Tiles come longest first and are taken in units of neighbours, which read the heads'
// pieces of the same pages: units go to the workgroups up, down, up the list (of 256, the first workgroup takes units 0, 511
// and 512), so that every compute unit has as many bytes to read, and to the 8 / unit groups of a workgroup's waves in turn.
// A wave has one running reference for a whole tile where eight have eight, hence SPLIT_P.  256 sequences of
// 64-700 keys by 8 heads, 405 MB, 81 us on whole workgroups (5.0 TB/s), 75 with a tile to a wave in the list's order (the first units
// have the longest tiles only and cannot stream faster than 55 GB/s), 67.5 this way: 6.0 TB/s, where a plain read loop reaches 7.2.  HBM reads
// 1.02 times K, V and queries.  What is missing are both ends: of 2048 tiles every wave has one, so nothing passes under the 4 us before its first loads,
// nor under the last waves' tails.  FP8 pages 39 us (5.3 TB/s), D = 64 39 (5.2), both 26 (4.0: 4 KiB a wave in flight; the FP8 forms spill 54 scalars).  Two register sets, on FP8 pages two page
// pairs: three and four of bf16 pages are 7 and 5 % slower on average over 260 drawn launches and one FP8 pair 8 %, single wave or full chip.
// ---------------------------------------------------------------------------------------------------
template <int HD, bool FP8>
__global__ __launch_bounds__(kThreads, 2) void ppd_wave_kernel(const ppd_work_item* items, int n_items, int unit, const KParams P) {
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int grid = (int)gridDim.x, block = (int)blockIdx.x, groups = kWaves / unit;
    for (int round = wave / unit;; round += groups) {
        const int64_t mine = (int64_t)(round & 1 ? (round + 1) * grid - 1 - block : round * grid + block) * unit + wave % unit;
        if (mine >= n_items) break;  // later rounds are further down the list
        const ppd_work_item it = items[mine];
        if constexpr (FP8) narrow_item_wide<HD, 1, kSoloSets, true, true, true>(P, it, nullptr);
        else narrow_item<HD, 1, kSoloSets, kSoloSets, true, true>(P, it, nullptr);
    }
}

// ---------------------------------------------------------------------------------------------------
// The co-resident pair.  A step that holds both kinds of tiles is launched as two kernels on two streams, sized so
// that one workgroup of each fits on every compute unit at the same time: the row-block kernel (8 waves, two per
// SIMD, 168 registers each, the K/V rings in LDS) keeps the matrix cores busy while the stream kernel (4 waves, one
// per SIMD, 168 registers, a small combine buffer) keeps HBM busy from the same unit -- a compute unit streams
// about 50 GB/s at most, whatever is in flight, so memory-bound tiles need most of the chip's units and so do the
// matrix-bound ones.  Each kernel has its own queues, cursors and count of finished workgroups.
// ---------------------------------------------------------------------------------------------------
template <int HD>
__global__ __launch_bounds__(kThreads) __attribute__((amdgpu_waves_per_eu(3, 3))) void ppd_mfma_kernel(const KParams P) {
    extern __shared__ __attribute__((aligned(16))) char smem[];
    __shared__ int s_next_slot;
    volatile int* s_next = &s_next_slot;
    const int tid = threadIdx.x;
    const int xcd = (int)(__builtin_amdgcn_s_getreg((3 << 11) | (0 << 6) | 20) & (kXcds - 1));  // HW_REG_XCC_ID
    unsigned dry = 0;  // bit q: queue q is exhausted (only thread 0 uses it)
#pragma unroll
    for (int q = 0; q < kXcds; ++q)
        if (P.queue_begin[q + 1] == P.queue_begin[q]) dry |= 1u << q;
    for (;;) {
        if (tid == 0) {
            int idx = -1;
            for (int a = 0; a < kXcds && idx < 0; ++a) {
                const int q = (xcd + a) & (kXcds - 1);
                if (dry & (1u << q)) continue;
                idx = claim_from(P, q);
                if (idx < 0) {
                    dry |= 1u << q;
                    if (dry != (1u << kXcds) - 1) {  // one batch of plain loads tells which other queues are exhausted
                        unsigned cur[kXcds];
#pragma unroll
                        for (int j = 0; j < kXcds; ++j)
                            cur[j] = __hip_atomic_load(&P.counters[kCursorBase + j * kCursorStride], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
#pragma unroll
                        for (int j = 0; j < kXcds; ++j)
                            if ((int)cur[j] >= P.queue_begin[j + 1] - P.queue_begin[j]) dry |= 1u << j;
                    }
                }
            }
            *s_next = idx;
        }
        __syncthreads();
        const int idx = __builtin_amdgcn_readfirstlane(*s_next);
        __syncthreads();
        if (idx < 0) break;
        const ppd_work_item it = P.items[idx];
        mfma_item<HD, true>(P, it, smem);
    }
    if (tid == 0) rearm_cursors(P, 0, kXcds, 10);
}

template <int HD>
__global__ __launch_bounds__(kStreamThreads) __attribute__((amdgpu_waves_per_eu(3, 3))) void ppd_stream_kernel(const KParams P) {
    extern __shared__ __attribute__((aligned(16))) char smem[];
    __shared__ int s_next_slot;
    volatile int* s_next = &s_next_slot;
    const int tid = threadIdx.x;
    for (;;) {
        if (tid == 0) *s_next = claim_from(P, kNarrowQueue);
        __syncthreads();
        const int idx = __builtin_amdgcn_readfirstlane(*s_next);
        __syncthreads();  // everyone has read s_next, and the previous tile's combine is over
        if (idx < 0) break;
        const ppd_work_item it = P.items[idx];
        narrow_item<HD, kStreamWaves, kStreamKSets, kStreamVSets>(P, it, smem);
    }
    if (tid == 0) rearm_cursors(P, kNarrowQueue, kNarrowQueue + 1, 11);
}

// ---------------------------------------------------------------------------------------------------
// Log-sum-exp merge of split partials: out = sum_j o_j 2^{(m_j - m*) c} / sum_j l_j 2^{(m_j - m*) c},
// splits taken in index order (deterministic).  Block b takes the kMergeCols columns starting at units[b].col0 of
// group units[b].group, each wave kMergeCols / 4 of them.  A wave moves little data, so its time is its chain of
// dependent loads: the loads of all its columns (four splits at a time) are issued before the first use.
// ---------------------------------------------------------------------------------------------------
__global__ __launch_bounds__(kSmallThreads) void ppd_merge_kernel(const MergeParams M) {
    constexpr int CPW = kMergeCols / (kSmallThreads / 64);  // columns per wave
    const MergeUnit u = M.units[blockIdx.x];
    const MergeGroup g = M.groups[u.group];
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const int ncols = g.nrows * M.G;
    const int D = M.D;
    const int d = lane * 2;
    const bool live = d < D;
    const float* base = M.partials + g.part_off;
    float o0[CPW], o1[CPW], l[CPW];
#pragma unroll
    for (int c = 0; c < CPW; ++c) {
        const int colr = u.col0 + wave * CPW + c;
        const int col = colr < ncols ? colr : ncols - 1;  // columns past the end redo the last one and store nothing
        const int64_t ml_off = (int64_t)ncols * D + col * 2;
        const int64_t v_off = (int64_t)col * D + (live ? d : 0);
        float mm = NEG_INF;
        o0[c] = o1[c] = l[c] = 0.f;
        if (g.nsplit <= 4) {
            float m4[4], l4[4];
            f32x2 v4[4];
#pragma unroll
            for (int t = 0; t < 4; ++t) {
                const float* pp = base + g.part_stride * (t < g.nsplit ? t : 0);
                m4[t] = pp[ml_off];
                l4[t] = pp[ml_off + 1];
                v4[t] = *reinterpret_cast<const f32x2*>(pp + v_off);
            }
#pragma unroll
            for (int t = 0; t < 4; ++t)
                if (t < g.nsplit) mm = fmaxf(mm, m4[t]);
#pragma unroll
            for (int t = 0; t < 4; ++t) {
                if (t < g.nsplit) {
                    const float f = m4[t] == NEG_INF ? 0.f : fast_exp2((m4[t] - mm) * M.scale_log2e);
                    l[c] += f * l4[t];
                    o0[c] += f * v4[t][0];
                    o1[c] += f * v4[t][1];
                }
            }
        } else {
            for (int j0 = 0; j0 < g.nsplit; j0 += 4) {
                float m4[4];
#pragma unroll
                for (int t = 0; t < 4; ++t) m4[t] = base[g.part_stride * (j0 + t < g.nsplit ? j0 + t : j0) + ml_off];
#pragma unroll
                for (int t = 0; t < 4; ++t) mm = fmaxf(mm, m4[t]);
            }
            for (int j0 = 0; j0 < g.nsplit; j0 += 4) {
                float m4[4], l4[4];
                f32x2 v4[4];
#pragma unroll
                for (int t = 0; t < 4; ++t) {
                    const float* pp = base + g.part_stride * (j0 + t < g.nsplit ? j0 + t : j0);
                    m4[t] = pp[ml_off];
                    l4[t] = pp[ml_off + 1];
                    v4[t] = *reinterpret_cast<const f32x2*>(pp + v_off);
                }
#pragma unroll
                for (int t = 0; t < 4; ++t) {
                    if (j0 + t < g.nsplit) {
                        const float f = m4[t] == NEG_INF ? 0.f : fast_exp2((m4[t] - mm) * M.scale_log2e);
                        l[c] += f * l4[t];
                        o0[c] += f * v4[t][0];
                        o1[c] += f * v4[t][1];
                    }
                }
            }
        }
    }
#pragma unroll
    for (int c = 0; c < CPW; ++c) {
        const int col = u.col0 + wave * CPW + c;
        if (live && col < ncols) {
            const int crow = col_row(col, M.invG);
            const int64_t orow = (int64_t)(g.grow0 + crow) * M.Hq + g.kvh * M.G + (col - crow * M.G);
            *reinterpret_cast<uint32_t*>(M.out + orow * D + d) = pack_bf16((o0[c] / l[c]) * M.v_scale, (o1[c] / l[c]) * M.v_scale);
        }
    }
}

// ---------------------------------------------------------------------------------------------------
// Paged KV append (and, with several layers in one launch, the landing of transferred KV).  One workgroup
// moves TOK consecutive tokens of the batch for one KV head of one layer.
// Bound by memory for the landing of requests, by latency for the few tokens of a decode step: the source rows and
// the slots are therefore loaded side by side (whole rows of D elements, 16 bytes per lane), staged in LDS, and what
// goes where is decided while they are on their way.
// K: 16-byte granules (8 d of one token) leave LDS token-minor, so that tokens in consecutive slots write one run.
// V: a granule is 8 tokens of one d, i.e. 8 consecutive slots starting at a multiple of 8.  The new tokens of a
//    sequence sit in consecutive slots but start anywhere (at its cached length), so the workgroup's own
//    tokens rarely fill whole granules; runs of 8 batch tokens that do ("octets") are found in a window of slots
//    around the workgroup's tokens instead: the workgroup writes, as whole 16-byte granules, the octets that
//    START at one of its tokens (the last one's tokens may reach into the next workgroup's range,
//    which only reads them), and element by element those of its tokens that belong to no octet (heads and tails
//    of runs, skipped neighbours).  Every token is written exactly once.
// Measured, against 8 tokens per workgroup with a request for the slots first and V read 2 bytes per lane: 5115 tokens x
// 32 layers 260 -> 232 us (5.8 TB/s read + write; a plain copy of the same bytes 4.9-5.2), FP8 pages 301 -> 180 us (5.6 TB/s),
// 11188 tokens of first prompts 32 -> 26 us, 3900 of append-prefills 13.8 -> 10.8 us, 256 decodes 8.8 -> 7.0 us.
// ---------------------------------------------------------------------------------------------------
// source and pool are each touched once: non-temporal loads and stores (the landing of a whole request runs 7 %
// faster with them)
#define APPEND_LOAD(p) __builtin_nontemporal_load(p)
#define APPEND_STORE(v, p) __builtin_nontemporal_store(v, p)
// FP8: the pool's elements are bytes; element x of K is stored as the code of x * inv_k (of V: x * inv_v), one
// binary32 product each.
template <int D, int TOK, bool FP8>
__global__ __launch_bounds__(kSmallThreads) void ppd_kv_append_kernel(const uint16_t* __restrict__ k,
                                                                 const uint16_t* __restrict__ v,
                                                                 std::conditional_t<FP8, uint8_t, uint16_t>* __restrict__ pool,
                                                                 const int64_t* __restrict__ slots, int64_t T,
                                                                 int Hkv, int64_t num_pages,
                                                                 int64_t pool_layer_stride, uint32_t* err_flags,
                                                                 float inv_k, float inv_v) {
    static_assert(TOK == 8 || TOK == 16, "the window of slots fits a wave");
    constexpr int GR = D / 8;              // granules of a source row
    constexpr int UNITS = TOK * GR;        // granules of the workgroup's K rows (and of its V rows)
    constexpr int ROW = D + 8;             // elements of a staged row: 16 bytes of padding spread the rows over the banks
    constexpr int LOADS = (2 * UNITS + kSmallThreads - 1) / kSmallThreads;
    static_assert(UNITS % 64 == 0, "a wave loads granules of one kind");
    __shared__ __attribute__((aligned(16))) uint16_t sk[TOK * ROW];
    __shared__ __attribute__((aligned(16))) uint16_t sv[(TOK + 7) * ROW];
    // blockIdx.z = layer: source layers are contiguous [layer][T][Hkv][D], pools pool_layer_stride apart
    const int64_t HD = (int64_t)Hkv * D;
    k += (int64_t)blockIdx.z * T * HD + blockIdx.y * D;
    v += (int64_t)blockIdx.z * T * HD + blockIdx.y * D;
    pool += (int64_t)blockIdx.z * pool_layer_stride;
    const int tid = threadIdx.x;
    const int lane = tid & 63;
    const int64_t t0 = (int64_t)blockIdx.x * TOK;
    u32x4 val[LOADS];
#pragma unroll
    for (int p = 0; p < LOADS; ++p) {
        const int u = tid + p * kSmallThreads, row = (u % UNITS) / GR;
        val[p] = u32x4{0, 0, 0, 0};
        if (u < 2 * UNITS && t0 + row < T)
            val[p] = APPEND_LOAD(reinterpret_cast<const u32x4*>((u < UNITS ? k : v) + (t0 + row) * HD + (u % GR) * 8));
    }
    // Window of slots: batch tokens t0-7 .. t0+TOK+6, one per lane (lane 7 holds token t0), in every wave; tokens
    // outside the batch and slots outside the pool count as skipped.  What follows is a handful of wave-wide
    // votes: the per-workgroup bookkeeping has to stay far below the cost of moving the tokens.
    constexpr int kWin = TOK + 14;
    constexpr uint32_t kOwn = (1u << TOK) - 1;
    const int64_t tw = t0 - 7 + lane;
    int64_t ws = -1;
    if (lane < kWin && tw >= 0 && tw < T) ws = slots[tw];
    const bool outside = ws >= num_pages * kPage;
    if (__ballot(outside && lane >= 7 && lane < 7 + TOK) != 0 && tid == 0 && blockIdx.y == 0 && blockIdx.z == 0)
        atomicOr(err_flags, 1u);
    if (outside) ws = -1;
    // bit i of `runs`: entry i+1 holds the slot after entry i's; bit c of `octets`: the 8 tokens from entry c on
    // sit in the 8 slots of one V granule, in order
    const int64_t ws_next = __shfl_down(ws, 1);
    const uint64_t runs = __ballot(lane < kWin - 1 && ws_next == ws + 1);
    const uint64_t starts = __ballot(ws >= 0 && (ws & 7) == 0);
    const uint32_t octets = (uint32_t)(starts & runs & (runs >> 1) & (runs >> 2) & (runs >> 3) & (runs >> 4) &
                                       (runs >> 5) & (runs >> 6)) & ((1u << (TOK + 7)) - 1);
    // own tokens: which of them no octet covers (a token with slot s would be entry s % 8 of one), and the
    // octets that start at one of them
    const int my_start = (ws >= 0 && lane >= 7) ? lane - (int)(ws & 7) : 0;
    const uint32_t single =
        (uint32_t)(__ballot(lane >= 7 && lane < 7 + TOK && ws >= 0 && !((octets >> my_start) & 1u)) >> 7) & kOwn;
    const uint32_t own_octets = (octets >> 7) & kOwn;  // at most TOK / 8
    // rows beyond the own ones that the last octet reaches into
    const int last_oct = own_octets ? 31 - __builtin_clz(own_octets) : 0;
    const int extra = own_octets && last_oct + 8 > TOK ? last_oct + 8 - TOK : 0;
    if (tid < extra * GR)
        *reinterpret_cast<u32x4*>(sv + (TOK + tid / GR) * ROW + (tid % GR) * 8) =
            APPEND_LOAD(reinterpret_cast<const u32x4*>(v + (t0 + TOK + tid / GR) * HD + (tid % GR) * 8));
#pragma unroll
    for (int p = 0; p < LOADS; ++p) {
        const int u = tid + p * kSmallThreads;
        if (u < 2 * UNITS)
            *reinterpret_cast<u32x4*>((u < UNITS ? sk : sv) + ((u % UNITS) / GR) * ROW + (u % GR) * 8) = val[p];
    }
    __syncthreads();
    const int64_t S = 2LL * Hkv * kPage * D;
    const int64_t koff = (int64_t)blockIdx.y * kPage * D;
    const int64_t voff = (int64_t)Hkv * kPage * D + koff;
    // K: work unit = (granule c, token), token fastest; whole waves take part
#pragma unroll
    for (int p = 0; p < (UNITS + kSmallThreads - 1) / kSmallThreads; ++p) {
        const int u = tid + p * kSmallThreads;
        if (u >= UNITS) break;
        const int tok = u % TOK, c = u / TOK;
        const int64_t s = __shfl(ws, 7 + tok);
        if (s < 0) continue;
        const u32x4 g = *reinterpret_cast<const u32x4*>(sk + tok * ROW + c * 8);
        auto* dst = pool + (s >> 4) * S + koff + c * (kPage * 8) + (int)(s & 15) * 8;
        if constexpr (FP8) {
            const u32x2 codes = {e4m3_codes(g[0], g[1], inv_k), e4m3_codes(g[2], g[3], inv_k)};
            APPEND_STORE(codes, reinterpret_cast<u32x2*>(dst));
        } else {
            APPEND_STORE(g, reinterpret_cast<u32x4*>(dst));
        }
    }
    // V, whole granules: work unit = (octet, d)
    uint32_t left = own_octets;
#pragma unroll
    for (int o = 0; o < TOK / 8; ++o) {
        if (!left) break;
        const int tok = __builtin_ctz(left);
        left &= left - 1;
        const int64_t s = __shfl(ws, 7 + tok);
        // the octets take turns at starting with the first thread, so that at D < 256 each has threads of its own
        const int d = (tid + o * D) % kSmallThreads;
        if (d < D) {
            uint32_t g[4];
#pragma unroll
            for (int e = 0; e < 4; ++e)
                g[e] = (uint32_t)sv[(tok + 2 * e) * ROW + d] | ((uint32_t)sv[(tok + 2 * e + 1) * ROW + d] << 16);
            auto* dst = pool + (s >> 4) * S + voff + (int)((s & 15) >> 3) * (D * 8) + d * 8;
            if constexpr (FP8) {
                const u32x2 codes = {e4m3_codes(g[0], g[1], inv_v), e4m3_codes(g[2], g[3], inv_v)};
                APPEND_STORE(codes, reinterpret_cast<u32x2*>(dst));
            } else {
                APPEND_STORE((u32x4{g[0], g[1], g[2], g[3]}), reinterpret_cast<u32x4*>(dst));
            }
        }
    }
    // V, element by element: work unit = (token, d)
    if (single) {
        for (int u = tid; u < D * TOK; u += kSmallThreads) {
            const int tok = u / D, d = u % D;
            const int64_t s = __shfl(ws, 7 + tok);  // before any lane drops out
            if (!((single >> tok) & 1u)) continue;
            const int off = (int)(s & 15);
            const uint16_t x = sv[tok * ROW + d];
            auto* dst = pool + (s >> 4) * S + voff + (off >> 3) * (D * 8) + d * 8 + (off & 7);
            if constexpr (FP8) *dst = (uint8_t)e4m3_codes(x, 0u, inv_v); else *dst = x;
        }
    }
}

// ---------------------------------------------------------------------------------------------------
static size_t ring_lds_bytes(int head_dim) {
    return (size_t)(2 * kStages + (PPD_PINGPONG ? 1 : 0) + (PPD_PINGPONG ? 1 : 0)) * 4 * kPage * head_dim * 2 +
           (kMaxMfmaChunk / kPage) * 4;  // + page ids of one row-block tile
}
static size_t mixed_lds_bytes(int head_dim) {
    const size_t rings = ring_lds_bytes(head_dim), combine = NarrowCombine<kWaves>::bytes(head_dim);
    return rings > combine ? rings : combine;
}

// The forms of the decode-only kernel.
struct NarrowForm {
    void (*kernel)(const ppd_work_item*, int, int, const KParams);
    int waves;
    size_t lds;
};
template <int HD, bool FP8, int NSETS>
static NarrowForm narrow_form_of(bool merges) {
    constexpr int NW = kNarrowKernelWaves;
    return {merges ? &ppd_narrow_kernel<HD, FP8, NW, NSETS, true> : &ppd_narrow_kernel<HD, FP8, NW, NSETS, false>, NW, NarrowCombine<NW>::bytes(HD)};
}
static NarrowForm narrow_form(int head_dim, bool fp8_pages, bool four_waves, int64_t mean_tile_keys, int64_t pace_keys, bool merges) {
    // Register sets on bf16 pages.  Two make a loop of half the instructions, which short tiles never get to stream from a warm
    // instruction cache; long tiles want K and V of two pages in flight.  Two and three sets, us a layer with its append: 64
    // decodes of 200-400 keys 22.8 and 24.0, of 400-800 33.2 and 34.1, of 800-1600 (8 KV heads, tiles of 1200 on average) 54.7
    // and 55.2; 64 of 1600-3200 99.9 and 98.8, of 6400-9000 306 and 303; 8 of 6400-9000 (tiles of 2000) 59.3 and 58.3.  The four
    // sets that all tiles had were behind both at every length but 200-400 (200-400 23.6, 400-800 34.0, 6400-9000 308).  At
    // D = 64 a page is half the bytes and two sets are ahead at every length (32 of 6400-9000 keys 37.1 and 42.2).
    const bool long_tiles = mean_tile_keys >= 1536;
    // FP8 pages at D = 64: eight waves by two pairs are 512 keys.  Shorter tiles do not fill two sets, and what counts is the tiles
    // that make the time: all of them in many rounds, the longest in one.  Two sets against one, 300 drawn decode steps: one round
    // with a longest tile below 200 keys -8 %, of 200-500 -3, 500-700 +1, 700-1500 +6, more +16; several rounds of tiles of
    // up to 200 keys on average -9, 200-500 -2, 500-700 +3, 700-1500 +9, more +16; split and merged in the launch, at 512 and 768
    // keys -3, 1024 +1, 1536 and more +3.
    if (four_waves)
        return {&ppd_narrow_kernel<128, false, kStreamingWaves, kStreamingSets>, kStreamingWaves, NarrowCombine<kStreamingWaves>::bytes(128)};
    if (head_dim == 128 && fp8_pages) return narrow_form_of<128, true, fp8_sets(128)>(merges);
    if (head_dim == 128 && long_tiles) return narrow_form_of<128, false, kLongSets>(merges);
    if (head_dim == 128) return narrow_form_of<128, false, kShortSets>(merges);
    if (fp8_pages && pace_keys < (merges ? 1024 : 512)) return narrow_form_of<64, true, 1>(merges);
    if (fp8_pages) return narrow_form_of<64, true, fp8_sets(64)>(merges);
    return narrow_form_of<64, false, kShortSets>(merges);
}

// More than 64 KiB of dynamic LDS has to be allowed per kernel, on the device that is current (ppd_create calls
// this once per context, with the context's device current).
int prepare_mixed_kernels() {
    hipError_t e = hipSuccess;
    auto allow = [&](const void* fn, size_t bytes) {
        if (e == hipSuccess) e = hipFuncSetAttribute(fn, hipFuncAttributeMaxDynamicSharedMemorySize, (int)bytes);
    };
    allow(reinterpret_cast<const void*>(&ppd_mixed_kernel<128, false>), mixed_lds_bytes(128));
    allow(reinterpret_cast<const void*>(&ppd_mixed_kernel<64, false>), mixed_lds_bytes(64));
    allow(reinterpret_cast<const void*>(&ppd_mixed_kernel<128, true>), mixed_lds_bytes(128));
    allow(reinterpret_cast<const void*>(&ppd_mixed_kernel<64, true>), mixed_lds_bytes(64));
    allow(reinterpret_cast<const void*>(&ppd_mixed_by_block_kernel<128, false>), mixed_lds_bytes(128));
    allow(reinterpret_cast<const void*>(&ppd_mixed_by_block_kernel<64, false>), mixed_lds_bytes(64));
    allow(reinterpret_cast<const void*>(&ppd_mixed_by_block_kernel<128, true>), mixed_lds_bytes(128));
    allow(reinterpret_cast<const void*>(&ppd_mixed_by_block_kernel<64, true>), mixed_lds_bytes(64));
    for (int form = 0; form < 8; ++form) {  // of the decode-only kernel eight waves at D = 128: page format, short and long tiles, merged in the launch or not
        const int64_t keys = form & 2 ? 1 << 20 : 0;
        const NarrowForm f = narrow_form(128, (form & 1) != 0, false, keys, keys, (form & 4) != 0);
        allow(reinterpret_cast<const void*>(f.kernel), f.lds);
    }
    static_assert(NarrowCombine<kNarrowKernelWaves>::bytes(64) < 64 * 1024 - 16 && NarrowCombine<kStreamingWaves>::bytes(128) < 64 * 1024 - 16, "the other forms fit");
    allow(reinterpret_cast<const void*>(&ppd_pipelined_kernel<128>), pipelined_lds_bytes<128>());
    allow(reinterpret_cast<const void*>(&ppd_pipelined_kernel<64>), pipelined_lds_bytes<64>());
    allow(reinterpret_cast<const void*>(&ppd_mfma_kernel<128>), ring_lds_bytes(128));
    allow(reinterpret_cast<const void*>(&ppd_mfma_kernel<64>), ring_lds_bytes(64));
    return (int)e;
}

int launch_mixed(const KParams& p, int head_dim, int grid, void* stream, bool fp8_pages) {
    auto* const kernel = head_dim == 128 ? (fp8_pages ? (p.by_block ? &ppd_mixed_by_block_kernel<128, true> : &ppd_mixed_kernel<128, true>)
                                                      : (p.by_block ? &ppd_mixed_by_block_kernel<128, false> : &ppd_mixed_kernel<128, false>))
                                         : (fp8_pages ? (p.by_block ? &ppd_mixed_by_block_kernel<64, true> : &ppd_mixed_kernel<64, true>)
                                                      : (p.by_block ? &ppd_mixed_by_block_kernel<64, false> : &ppd_mixed_kernel<64, false>));
    hipLaunchKernelGGL(kernel, dim3(grid), dim3(kThreads), mixed_lds_bytes(head_dim), static_cast<hipStream_t>(stream), p);
    return (int)hipGetLastError();
}

int launch_narrow(const KParams& p, int head_dim, int grid, void* stream, bool fp8_pages) {
    if (p.pipelined) {
        if (head_dim == 128)
            hipLaunchKernelGGL(ppd_pipelined_kernel<128>, dim3(grid), dim3(kThreads), pipelined_lds_bytes<128>(), static_cast<hipStream_t>(stream), p.items, p.n_wg, p);
        else
            hipLaunchKernelGGL(ppd_pipelined_kernel<64>, dim3(grid), dim3(kThreads), pipelined_lds_bytes<64>(), static_cast<hipStream_t>(stream), p.items, p.n_wg, p);
        return (int)hipGetLastError();
    }
    if (p.wave_unit > 0) {
        auto* const kernel = head_dim == 128 ? (fp8_pages ? &ppd_wave_kernel<128, true> : &ppd_wave_kernel<128, false>)
                                             : (fp8_pages ? &ppd_wave_kernel<64, true> : &ppd_wave_kernel<64, false>);
        hipLaunchKernelGGL(kernel, dim3(grid), dim3(kThreads), 0, static_cast<hipStream_t>(stream), p.items, p.n_items, p.wave_unit, p);
        return (int)hipGetLastError();
    }
    const NarrowForm f = narrow_form(head_dim, fp8_pages, p.four_waves != 0, p.mean_tile_keys, p.pace_keys, p.merge_groups != nullptr);
    hipLaunchKernelGGL(f.kernel, dim3(grid), dim3(64 * f.waves), f.lds, static_cast<hipStream_t>(stream), p.items, p.n_wg, p.n_items, p);
    return (int)hipGetLastError();
}

int launch_mfma_only(const KParams& p, int head_dim, int grid, void* stream) {
    hipStream_t st = static_cast<hipStream_t>(stream);
    if (head_dim == 128)
        hipLaunchKernelGGL(ppd_mfma_kernel<128>, dim3(grid), dim3(kThreads), ring_lds_bytes(128), st, p);
    else
        hipLaunchKernelGGL(ppd_mfma_kernel<64>, dim3(grid), dim3(kThreads), ring_lds_bytes(64), st, p);
    return (int)hipGetLastError();
}

int launch_stream_only(const KParams& p, int head_dim, int grid, void* stream) {
    hipStream_t st = static_cast<hipStream_t>(stream);
    if (head_dim == 128)
        hipLaunchKernelGGL(ppd_stream_kernel<128>, dim3(grid), dim3(kStreamThreads),
                           NarrowCombine<kStreamWaves>::bytes(128), st, p);
    else
        hipLaunchKernelGGL(ppd_stream_kernel<64>, dim3(grid), dim3(kStreamThreads),
                           NarrowCombine<kStreamWaves>::bytes(64), st, p);
    return (int)hipGetLastError();
}

int launch_merge(const MergeParams& p, void* stream) {
    hipLaunchKernelGGL(ppd_merge_kernel, dim3(p.n_units), dim3(kSmallThreads), 0, static_cast<hipStream_t>(stream), p);
    return (int)hipGetLastError();
}

template <int D, int TOK, bool FP8>
static void append_launch(const uint16_t* k, const uint16_t* v, void* pool, const int64_t* slots, int64_t T, int Hkv,
                          int64_t num_pages, int layers, int64_t pool_layer_stride, uint32_t* err_flags, hipStream_t st,
                          float inv_k, float inv_v) {
    using Elem = std::conditional_t<FP8, uint8_t, uint16_t>;
    hipLaunchKernelGGL((ppd_kv_append_kernel<D, TOK, FP8>), dim3((unsigned)((T + TOK - 1) / TOK), (unsigned)Hkv, (unsigned)layers),
                       dim3(kSmallThreads), 0, st, k, v, static_cast<Elem*>(pool), slots, T, Hkv, num_pages, pool_layer_stride,
                       err_flags, inv_k, inv_v);
}

int launch_kv_append(const uint16_t* k, const uint16_t* v, void* pool, const int64_t* slots, int64_t T, int Hkv,
                     int D, int64_t num_pages, int layers, int64_t pool_layer_stride, uint32_t* err_flags,
                     void* stream, bool fp8_pages, float inv_k_scale, float inv_v_scale) {
    // 16 tokens to a workgroup write whole page blocks of K and fewer half-filled lines (3900 tokens of 8 heads 13.2 us
    // with 8 and 10.8 with 16 tokens, FP8 landing 207 and 180); a decode step has only workgroups to gain from 8 (256
    // tokens of 8 heads 7.6 us with 16 and 7.0 with 8); in between (700 tokens) the two are equal.
    const bool wide = T * Hkv * layers >= 8192;
    auto go = [&](auto fn) {
        fn(k, v, pool, slots, T, Hkv, num_pages, layers, pool_layer_stride, err_flags, static_cast<hipStream_t>(stream), inv_k_scale, inv_v_scale);
    };
    if (D == 128) {
        if (wide) fp8_pages ? go(append_launch<128, 16, true>) : go(append_launch<128, 16, false>);
        else fp8_pages ? go(append_launch<128, 8, true>) : go(append_launch<128, 8, false>);
    } else {
        if (wide) fp8_pages ? go(append_launch<64, 16, true>) : go(append_launch<64, 16, false>);
        else fp8_pages ? go(append_launch<64, 8, true>) : go(append_launch<64, 8, false>);
    }
    return (int)hipGetLastError();
}

}  // namespace ppd
