// Importance scores of the prompt keys under the soft-token queries
// (paper Section 4.3, Eq. 3), as two K-streaming MFMA passes for gfx950.
//
//   pass 1 (stats):  per query row r, an offset m_r and Z_r = sum_j 2^(t_rj - m_r) of its base-2 logits
//                    t_rj = c * q_r.k_j, c = scale * log2(e); one (m, Z) partial per workgroup.
//   merge:           beta_r = m_r + log2 Z_r over a sequence's partials, as -beta_r / c split into three
//                    bf16 terms -- done by every pass-2 workgroup for its own head in its start-up (a
//                    separate small kernel only when a sequence leaves more than 64 partials).
// An eviction whose workgroups all run at once does both passes in one launch, jq_passes_kernel: a workgroup scores the keys it has
// swept as soon as the others that share their sequence have published their statistics.
//   pass 2 (score):  score_j = sum_r 2^(c * (q_r.k_j - beta_r / c)).  The -beta_r/c term enters
//                    through one extra MFMA step whose key-side operand is 1.0, so the epilogue is one
//                    multiply, one exp2 and one add per logit.
// With more than 128 query rows per KV head pass 1 takes a grid slice per 128 rows, the merge is done by the workgroup that completes
// a (layer, sequence), head and group of rows, and pass 2 turns around: jq_score_rows_kernel keeps 128 keys in registers and streams the query rows past them, so that a
// key's score is complete in one launch whatever the number of rows.
// Variants of the same kernels: supplied normalisers (pass 2 alone), the soft tokens' own keys or the prompt's
// own last tokens as causally masked tiles of pass 1, keys read out of a paged pool.
//
// Otherwise a wave has one (layer, sequence, KV head) at a time and a set of that sequence's 32-key tiles (see Share), and
// keeps the head's (up to) 128 query rows in registers as MFMA operands.  The four waves of a workgroup
// work on the same head and fetch its query rows together (one row tile each, whole rows, turned into
// operand order through LDS) -- gathering them one row per lane would cost every wave 32 row-strided
// loads that touch 32 cache lines each.  Key tiles of 32 keys x 128 channels are
// fetched asynchronously, straight from global memory into a private, XOR-swizzled 8 KiB LDS slot
// (buffer loads with the LDS modifier, 16 B per lane, 16 lanes per 256-byte key row, so every 128-byte
// line is requested whole), two slots per wave used alternately, and read back in MFMA operand order without
// bank conflicts.  After the start-up waves never share LDS, so the streaming loop has no workgroup barrier;
// its only synchronisation is the wave's own s_waitcnt on its outstanding loads.
//
// MFMA 32x32x16 bf16 operand layout used here: lane l supplies row/column (l & 31) and the 8
// contraction elements selected by (l >> 5); both operands use the same element order, so any
// fixed channel permutation cancels.  Result: lane l holds column (l & 31), register v holds row
// 8*(v/4) + 4*(l>>5) + (v&3).
#include <atomic>
#include <chrono>
#include <random>
#include <type_traits>

#include "jq_common.h"

namespace jq {

typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef float f32x16 __attribute__((ext_vector_type(16)));
typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));

struct ScoreArgs {
    // What a workgroup needs to find its share and make its first requests comes first, in the few lines of constant memory that
    // argument_lines() has fetched at once: a wave's first reads of its arguments take about 1 us each where they chain.
    int32_t n_layers, n_seq, h_kv;
    uint32_t inv_h_kv;    // for udiv()
    int32_t n_rg, rg0;    // first pass: groups of NQT query-row tiles in this launch (1 unless a head has more than
                          // kMaxRowTiles), and the first of them
    int32_t one_L;        // single-sequence calls: the sequence's length (0 otherwise): no per-sequence table is read then
    int32_t layer_quads;  // groups of four tiles (128 keys) per layer and head, rounded up per sequence
    SplitArgs own;        // how this launch's workgroups share the keys out
    int32_t n_q, h_q, group, rows, RP;
    int32_t group_shift;  // log2(group) when group is a power of two, else -1
    int32_t tiles1;       // two query sets: row tiles of the first (kOneSet: there is one set)
    const uint16_t* Q;
    const uint16_t* K;
    int64_t T;
    const uint16_t* K_tail;  // [n_layers][n_seq][n_q][h_kv][d] keys of the soft tokens themselves, or null
    uint32_t* zero;      // words to clear for the later selection stage (nullable)
    uint64_t zero_words;
    float2* stats;    // [sets][h_kv][RP]: (m, Z) of every share of a (layer, sequence), see Share
    float c;             // scale * log2(e)
    int32_t window;       // 1: the queries are the sequence's own last n_q tokens; query i sees keys 0 .. L - n_q + i
    // flags[h_kv][n_sets], set to `token` when a set of statistics is complete (first pass alone: [h_kv][n_rg][n_sets], with many
    // query rows only); both passes in one launch: how long (ticks of 10 ns) a workgroup waits for others' before it forms them itself
    uint64_t* flags;
    uint64_t token;
    int64_t wait_ticks;
    int32_t n_sets;
    int32_t holds;        // second pass: scores are held back, see score_share
    float* scores;        // [n_layers][h_kv][T]
    const float* lse;     // [n_layers][n_seq][n_q][h_q] caller-supplied natural-log normalisers, or null
    uint2* aug;           // [n_layers][n_seq][h_kv][RP]: bf16 terms of -beta/c
    double inv_scale, inv_c;  // 1 / scale, 1 / c
    SplitArgs part;       // how the workgroups that left the statistics shared the keys out (second pass alone, merge)
    int32_t fuse_combine; // second pass alone: it merges the statistics itself (otherwise jq_combine_kernel has filled `aug`)
    // paged K (PAGED kernels): K is [n_layers][n_pages][1 << page_shift][h_kv][d]; token t of sequence s lives in
    // page block_table[s * max_pages + (t >> page_shift)]
    int32_t page_shift, n_pages, max_pages;
    const int32_t* block_table;
    // Two query sets in one call (training-side forward, Eq. 3-5): row tiles tiles1 .. of a head hold the rows of the second
    // set.  Their launch of jq_score_rows_kernel compares the two maps instead of storing either and leaves one partial sum
    // of squared differences per workgroup.
    const uint16_t* Q2;
    int32_t n_q2, rows2;
    float inv_rows1, inv_rows2;  // 1 / summed probability rows of either map
    double* diff_part;           // [n_layers][layer_quads][h_kv]
    int32_t cu_seq[JQ_MAX_SEQ + 1], cu_quad[JQ_MAX_SEQ + 1];
    int32_t cu_wg[JQ_MAX_SEQ + 1], cu_part[JQ_MAX_SEQ + 1];  // Split::cu of `own` and `part`
};
constexpr int kOneSet = 0x7FFFFFFF;  // tiles1 of a call with one query set

// A kernel's own arguments, which lie in constant memory, reached through a pointer that the compiler knows nothing about: what is
// read through it is read where it is used.  A workgroup with several shares repeats everything below; without this the
// compiler keeps every scalar of every phase in registers across all of them (200 spilled).
typedef const ScoreArgs __attribute__((address_space(4))) KArgs;
__device__ __forceinline__ KArgs& kernel_args() {
    KArgs* p = (KArgs*)__builtin_amdgcn_kernarg_segment_ptr();
    asm volatile("" : "+s"(p));
    return *p;
}
__device__ __forceinline__ int lane_again() {  // the same for what derives from the lane
    int lane = (int)threadIdx.x & 63;
    asm volatile("" : "+v"(lane));
    return lane;
}

constexpr int kSlotBytes = kKeyTile * kHeadDim * 2;  // 8 KiB

__device__ __forceinline__ bf16x8 as_bf16x8(u32x4 v) { return __builtin_bit_cast(bf16x8, v); }

// Key tiles arrive through loads that write LDS directly; the compiler does not track them, so the
// waits are explicit.
// (s_waitcnt immediates: vmcnt in bits 3:0 and 15:14, expcnt 6:4, lgkmcnt 11:8; unused fields = no wait.)
__device__ __forceinline__ void wait_tile_landed() {
    __builtin_amdgcn_s_waitcnt(0x0F70);  // vmcnt(0)
    __builtin_amdgcn_sched_barrier(0);
    asm volatile("" ::: "memory");
}

// The same with one younger request, a store, that may still be on its way (vector memory operations complete in order).
__device__ __forceinline__ void wait_tile_landed_before_store() {
    __builtin_amdgcn_s_waitcnt(0x0F71);  // vmcnt(1)
    __builtin_amdgcn_sched_barrier(0);
    asm volatile("" ::: "memory");
}

// The fragments just read from an LDS slot must be in registers before the slot is refilled.
__device__ __forceinline__ void wait_frags_read() {
    asm volatile("" ::: "memory");
    __builtin_amdgcn_sched_barrier(0);
    __builtin_amdgcn_s_waitcnt(0xC07F);  // lgkmcnt(0)
    __builtin_amdgcn_sched_barrier(0);
    asm volatile("" ::: "memory");
}

// ---- key tiles: global -> LDS (layout and addresses: jq_sweep.h) ----------------------------------
__device__ __forceinline__ void lds_dma16(__amdgpu_buffer_rsrc_t rsrc, char* dst, uint32_t voff, uint32_t soff) {
    __builtin_amdgcn_raw_ptr_buffer_load_lds(rsrc, (__attribute__((address_space(3))) void*)dst, 16, (int)voff,
                                             (int)soff, 0, 0);
}

// `tile_off` = byte offset of the tile's first key row inside the buffer resource (uniform), `tl` = tile_lane(), `last` =
// last_request() of the resource.  What arrives for rows past the end of a sequence is zeros or rows of the sequence -- in a
// paged pool, whatever the rest of the page holds; the first pass masks those keys, the second does not store them, and no
// other key's values meet them.
__device__ __forceinline__ void fetch_tile(__amdgpu_buffer_rsrc_t rsrc, char* slot, uint32_t tile_off, uint32_t row_bytes, uint32_t tl, uint32_t last) {
#pragma unroll
    for (int i = 0; i < 8; ++i) lds_dma16(rsrc, slot + 1024 * i, tl ^ (64u * (i & 3)), request_offset(tile_off, i, row_bytes, last));
}

// MFMA operand fragments of the tile in `slot`: lane l takes key row (l & 31), logical chunks
// 2 ks + (l >> 5), ks = 0..7.  The 16 lanes of a quarter wave hit 16 distinct physical chunks.
// `at` = frag_addr(): the address of ks = 0; the others differ from it by an exclusive or (the swizzle of chunk 2 ks + h is
// (h ^ r) ^ 2 ks, and a row's 256 bytes are aligned), so that one register serves all eight.
__device__ __forceinline__ uint32_t frag_addr(const char* slot, int lane) {
    const uint32_t r = (uint32_t)lane & 31u;
    return (uint32_t)(uintptr_t)(__attribute__((address_space(3))) const char*)slot + r * 256u + ((((uint32_t)lane >> 5) ^ (r & 15u)) << 4);
}
__device__ __forceinline__ bf16x8 lds_get_frag(uint32_t at, int ks) {
    return as_bf16x8(*(const u32x4 __attribute__((address_space(3)))*)(uintptr_t)(at ^ ((uint32_t)ks << 5)));
}
__device__ __forceinline__ void lds_get_frags(const char* slot, bf16x8 (&kf)[8], int lane) {
    const uint32_t at = frag_addr(slot, lane);
#pragma unroll
    for (int ks = 0; ks < 8; ++ks) kf[ks] = lds_get_frag(at, ks);
}

// ---- start-up: the query rows as MFMA operands of every wave, with the first key tile in flight ---------
// Query rows of the workgroup's KV head (row r = i * group + hh  <->  Q[i, g*group + hh]): wave qt fetches row
// tile qt like a key tile -- every load instruction covers four whole 256-byte rows (lane l takes 16 B of row
// 4i + (l >> 4)), so each cache line is requested once -- and writes it, swizzled, into its own second LDS slot;
// after a barrier every wave reads all tiles in operand order; a second barrier frees the slots for key tiles.
// The compiler cannot tell which LDS bytes a direct-to-LDS load writes, so before any LDS access it generates
// it waits for every such load that is outstanding -- here that would be the first key tile, whose flight
// (the first sixteenth of K arriving at the rate of the memory system) is exactly what the start-up should hide
// behind.  The LDS instructions of the start-up are therefore written out, with their own waits: nothing the
// compiler generates touches LDS between the request of the first key tile and the first wait_tile_landed().
// Global loads into registers issued BEFORE the tile's request still get their exact waits from the compiler
// (loads return in issue order, so waiting for one of them never waits for the younger tile).
__device__ __forceinline__ uint32_t lds_addr(const void* p) {
    return (uint32_t)(uintptr_t)(__attribute__((address_space(3))) const char*)p;
}
__device__ __forceinline__ void lds_wait_all() { asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory"); }
__device__ __forceinline__ void lds_put16(uint32_t addr, u32x4 v) { asm volatile("ds_write_b128 %0, %1" ::"v"(addr), "v"(v) : "memory"); }
__device__ __forceinline__ void lds_put8(uint32_t addr, uint2 v) {
    const uint64_t x = (uint64_t)v.x | ((uint64_t)v.y << 32);
    asm volatile("ds_write_b64 %0, %1" ::"v"(addr), "v"(x) : "memory");
}
__device__ __forceinline__ void lds_put4(uint32_t addr, uint32_t v) { asm volatile("ds_write_b32 %0, %1" ::"v"(addr), "v"(v) : "memory"); }
__device__ __forceinline__ uint2 lds_get8_waited(uint32_t addr) {
    uint64_t x;
    asm volatile("ds_read_b64 %0, %1\n\ts_waitcnt lgkmcnt(0)" : "=&v"(x) : "v"(addr) : "memory");
    return make_uint2((uint32_t)x, (uint32_t)(x >> 32));
}
// N of them, `step` bytes apart
template <int N>
__device__ __forceinline__ void lds_get8s_waited(uint32_t addr, uint32_t step, uint2 (&v)[N]) {
    static_assert(N >= 1 && N <= 4, "written out");
    uint64_t x0, x1, x2, x3;
    if constexpr (N == 4)
        asm volatile("ds_read_b64 %0, %4\n\tds_read_b64 %1, %5\n\tds_read_b64 %2, %6\n\tds_read_b64 %3, %7\n\ts_waitcnt lgkmcnt(0)"
                     : "=&v"(x0), "=&v"(x1), "=&v"(x2), "=&v"(x3) : "v"(addr), "v"(addr + step), "v"(addr + 2 * step), "v"(addr + 3 * step) : "memory");
    else if constexpr (N == 3)
        asm volatile("ds_read_b64 %0, %3\n\tds_read_b64 %1, %4\n\tds_read_b64 %2, %5\n\ts_waitcnt lgkmcnt(0)"
                     : "=&v"(x0), "=&v"(x1), "=&v"(x2) : "v"(addr), "v"(addr + step), "v"(addr + 2 * step) : "memory");
    else if constexpr (N == 2)
        asm volatile("ds_read_b64 %0, %2\n\tds_read_b64 %1, %3\n\ts_waitcnt lgkmcnt(0)" : "=&v"(x0), "=&v"(x1) : "v"(addr), "v"(addr + step) : "memory");
    else
        asm volatile("ds_read_b64 %0, %1\n\ts_waitcnt lgkmcnt(0)" : "=&v"(x0) : "v"(addr) : "memory");
    v[0] = make_uint2((uint32_t)x0, (uint32_t)(x0 >> 32));
    if constexpr (N > 1) v[1] = make_uint2((uint32_t)x1, (uint32_t)(x1 >> 32));
    if constexpr (N > 2) v[2] = make_uint2((uint32_t)x2, (uint32_t)(x2 >> 32));
    if constexpr (N > 3) v[3] = make_uint2((uint32_t)x3, (uint32_t)(x3 >> 32));
}
// lds_get_frags with explicit instructions; returns when the fragments are in registers
__device__ __forceinline__ void lds_get_frags_waited(uint32_t slot, bf16x8 (&kf)[8], int lane) {
    const uint32_t r = (uint32_t)lane & 31u, hi = (uint32_t)lane >> 5;
    uint32_t ad[8];
#pragma unroll
    for (int ks = 0; ks < 8; ++ks) ad[ks] = slot + r * 256u + (((2u * ks + hi) ^ (r & 15u)) << 4);
    u32x4 o0, o1, o2, o3, o4, o5, o6, o7;
    asm volatile(
        "ds_read_b128 %0, %8\n\tds_read_b128 %1, %9\n\tds_read_b128 %2, %10\n\tds_read_b128 %3, %11\n\t"
        "ds_read_b128 %4, %12\n\tds_read_b128 %5, %13\n\tds_read_b128 %6, %14\n\tds_read_b128 %7, %15\n\t"
        "s_waitcnt lgkmcnt(0)"
        : "=&v"(o0), "=&v"(o1), "=&v"(o2), "=&v"(o3), "=&v"(o4), "=&v"(o5), "=&v"(o6), "=&v"(o7)
        : "v"(ad[0]), "v"(ad[1]), "v"(ad[2]), "v"(ad[3]), "v"(ad[4]), "v"(ad[5]), "v"(ad[6]), "v"(ad[7])
        : "memory");
    kf[0] = as_bf16x8(o0); kf[1] = as_bf16x8(o1); kf[2] = as_bf16x8(o2); kf[3] = as_bf16x8(o3);
    kf[4] = as_bf16x8(o4); kf[5] = as_bf16x8(o5); kf[6] = as_bf16x8(o6); kf[7] = as_bf16x8(o7);
}
// Barrier between phases that communicate through the LDS instructions above (each of which has waited for its
// own completion): no fence, hence no wait the compiler would add for loads in flight.
__device__ __forceinline__ void bare_barrier() {
    asm volatile("" ::: "memory");
    __builtin_amdgcn_s_barrier();
    asm volatile("" ::: "memory");
}
// The query rows that this wave stages: requested into registers, 16 B per lane, four whole 256-byte rows per instruction.  Every
// wave requests (those beyond the row tiles the last tile's, and they never store them), so that the requests sit in one basic
// block with others.  Rows past the end are zeros, or rows of the same head.  With a power-of-two group of up to 32 heads a
// tile's rows lie where a key tile's would: a lane part that never changes and a uniform part per request (4 i + a, a < 4, splits
// without carry), through a resource that ends with the last token (query_tile()).
template <int NQT>
__device__ __forceinline__ void q_rows_request(KArgs& a, const Share& h, int g, int rg, int lane, u32x4 (&raw)[8]) {
    const int wv = min(__builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6)), NQT - 1);
    const int rt = rg * NQT + wv;  // (uniform)
    const bool second = rt >= a.tiles1;
    const int n_q = second ? a.n_q2 : a.n_q, r0 = (second ? rt - a.tiles1 : rt) * kRowTile;
    const char* qbase = (const char*)(second ? a.Q2 : a.Q) + (((int64_t)(h.layer * a.n_seq + h.seq) * n_q) * a.h_q + g * a.group) * kHeadDim * 2;
    const int64_t tok_bytes = (int64_t)a.h_q * kHeadDim * 2;  // from one query token to the next
    const int gs = a.group_shift;
    const uint32_t rl = (uint32_t)lane >> 4, piece = ((uint32_t)lane & 15u) ^ rl;
    if (gs >= 0 && gs <= 5 && tok_bytes < (1 << 25)) {  // uniform; a tile's bytes fit a 32-bit offset
        const QueryTile qt = query_tile(n_q, r0, gs, (uint32_t)tok_bytes, (uint32_t)a.group);
        const __amdgpu_buffer_rsrc_t rsrc = __builtin_amdgcn_make_buffer_rsrc((void*)(qbase + qt.first * tok_bytes), 0, (int)qt.bytes, 0x00020000);
        const uint32_t tq = (rl >> gs) * (uint32_t)tok_bytes + (rl & ((uint32_t)a.group - 1)) * (kHeadDim * 2) + (piece << 4);
#pragma unroll
        for (int i = 0; i < 8; ++i)
            raw[i] = __builtin_amdgcn_raw_buffer_load_b128(rsrc, (int)(tq ^ (64u * (i & 3))),
                                                           (int)min(query_offset(i, gs, (uint32_t)tok_bytes, (uint32_t)a.group), qt.last), 0);
    } else {
        const int rows = second ? a.rows2 : a.rows;
#pragma unroll
        for (int i = 0; i < 8; ++i) {
            const int r = 4 * i + (lane >> 4), row = r0 + r, rowc = row < rows ? row : 0;
            int it, hh;
            if (gs >= 0) { it = rowc >> gs; hh = rowc & (a.group - 1); }
            else { it = rowc / a.group; hh = rowc % a.group; }
            const u32x4 v = *(const u32x4*)(qbase + it * tok_bytes + (int64_t)hh * (kHeadDim * 2) + (((lane & 15) ^ (r & 15)) << 4));
            raw[i] = row < rows ? v : u32x4{0u, 0u, 0u, 0u};
        }
    }
}
// ... and their way through LDS into operand order, with the first key tile in flight.  Every wave of the
// workgroup must call this (two barriers).
template <int NQT>
__device__ __forceinline__ void q_rows_stage(int lane, char* area, int stride, const u32x4 (&raw)[8], bf16x8 (&qf)[NQT][8]) {
    static_assert(NQT <= kScoreWaves, "one wave per query-row tile");
    const int wv = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
    if (wv < NQT) {
        const uint32_t slot = lds_addr(area + wv * stride);
#pragma unroll
        for (int i = 0; i < 8; ++i) lds_put16(slot + 1024u * i + 16u * lane, raw[i]);
        lds_wait_all();
    }
    bare_barrier();
#pragma unroll
    for (int qt = 0; qt < NQT; ++qt) lds_get_frags_waited(lds_addr(area + qt * stride), qf[qt], lane);
    bare_barrier();
}

// LDS of a pass: every wave's two tile slots; the kernel of both passes keeps more behind them.
constexpr int kSlotsBytes = kScoreWaves * 2 * kSlotBytes;
constexpr int kLdsQ = kSlotsBytes;                                  // query rows of the present (layer, sequence), one slot per row tile
constexpr int kLdsSet = kLdsQ + kMaxRowTiles * kSlotBytes;          // the set of statistics formed last (a float2 per row)
constexpr int kLdsAug = kLdsSet + kMaxRowTiles * kRowTile * 8;     // the rows' normalisers
constexpr int kLdsWord = kLdsAug + kMaxRowTiles * kRowTile * 8;
constexpr int kLdsBoth = kLdsWord + 16;
// Where a second pass holds scores back: per wave the scores of a number of tiles, then the tiles' numbers.  In the kernel of both
// passes they take the place of the query rows, which are in registers by then, a wave's in the slot that it fills itself: it needs no
// more LDS than the one that stores at once.  (With room for 119 tiles a wave it filled a CU's 160 KB, nothing of another stream that uses
// LDS could share a CU with it, and workgroups that so started late had their statistics formed by others: 8 x 65536 tokens beside 64
// workgroups of 32 KB 534 us a call, 404 stored at once, 422 so; 16 ragged sequences 989, 770, 750.  Alone 119 take up to 1.1 % less.)
// jq_score_kernel keeps them behind its slots: as many as two workgroups per CU have room for, also where there is one, so that kernels of
// other streams with up to 80 KB share the CU.  (60 and 119 tiles take 0.5 to 2.5 % less alone, but beside 4096^3 matrix products a call of
// 8 x 65536 530 to 542 us instead of 361, 359 to 390 stored at once, 400000 tokens 373, 305 and 306.)
constexpr int kHeldTile = kKeyTile * 4 + 4;
constexpr int kHeldPasses = 62, kHeldScore = 31;
static_assert(kHeldPasses * kHeldTile <= kSlotBytes, "in place of a wave's query rows");
static_assert(2 * (kSlotsBytes + kScoreWaves * kHeldScore * kHeldTile) <= 160 * 1024, "LDS of a CU");

struct KeyStream {
    __amdgpu_buffer_rsrc_t rsrc;  // this head's rows of the whole sequence (PAGED: of the layer's whole pool)
    uint32_t row_bytes;
    uint32_t last;                // last_request() of the resource; a page has whole tiles, and nothing is clamped there
    const int32_t* pages;         // PAGED: the sequence's row of the block table
    uint32_t page_shift, page_mask, last_page;
};

template <bool PAGED>
__device__ __forceinline__ KeyStream key_stream(KArgs& a, int layer, int seq, int64_t tok0, int L, int g) {
    KeyStream ks;
    ks.row_bytes = (uint32_t)a.h_kv * kHeadDim * 2;
    // the resource covers exactly this head's rows of the sequence, or of the layer's pool (the host checks
    // that this is below 4 GiB); every generated offset stays inside it
    const int64_t first_row = PAGED ? ((int64_t)layer * a.n_pages) << a.page_shift : (int64_t)layer * a.T + tok0;
    const uint32_t n_rows = PAGED ? (uint32_t)a.n_pages << a.page_shift : (uint32_t)L;
    const char* kseq = (const char*)a.K + (first_row * a.h_kv + g) * kHeadDim * 2;
    const uint32_t bytes = (n_rows - 1) * ks.row_bytes + kHeadDim * 2;
    ks.last = PAGED ? 0xFFFFFFFFu : last_request(L, ks.row_bytes);
    ks.rsrc = __builtin_amdgcn_make_buffer_rsrc((void*)kseq, 0, (int)bytes, 0x00020000);
    ks.pages = PAGED ? a.block_table + (int64_t)seq * a.max_pages : nullptr;
    ks.page_shift = (uint32_t)a.page_shift;
    ks.page_mask = (1u << a.page_shift) - 1u;
    ks.last_page = (uint32_t)a.n_pages - 1u;
    return ks;
}

template <bool PAGED>
__device__ __forceinline__ KeyStream key_stream(KArgs& a, const Share& h, int g) {
    return key_stream<PAGED>(a, h.layer, h.seq, h.tok0, h.L, g);
}

// Byte offset of sequence tile t inside the key stream's resource.  A page holds a whole number of 32-key
// tiles, so a tile never straddles pages; `page` is the block-table entry of the tile's page (clamped here,
// so that a corrupt table cannot send a load outside the pool).
template <bool PAGED>
__device__ __forceinline__ uint32_t tile_offset(const KeyStream& ks, int t, int page) {
    const uint32_t tok = (uint32_t)t * kKeyTile;
    if (!PAGED) return tok * ks.row_bytes;
    const uint32_t p = (uint32_t)clamp_page(page, (int32_t)ks.last_page + 1);  // the same clamp as the gather's
    return ((p << ks.page_shift) + (tok & ks.page_mask)) * ks.row_bytes;
}
// One table word per tile, at a wave-uniform address.  The table is read-only for the whole launch, so it is
// read through the constant address space: that makes the load a scalar one with a wait of its own -- a
// vector load would have to be waited for together with every key tile in flight.
template <bool PAGED>
__device__ __forceinline__ int tile_page(const KeyStream& ks, int t) {
    return PAGED ? ((const_i32_ptr)ks.pages)[((uint32_t)t * kKeyTile) >> ks.page_shift] : 0;
}

// x of the lane and of the one 32 further on (or back): of the lower one first
__device__ __forceinline__ float2 both_halves(float x) {
    const auto y = __builtin_amdgcn_permlane32_swap(__float_as_uint(x), __float_as_uint(x), false, false);
    return make_float2(__uint_as_float(y[0]), __uint_as_float(y[1]));
}
__device__ __forceinline__ float add_halves(float x) {
    const float2 y = both_halves(x);
    return y.x + y.y;
}

// One stage of the sweeps' software pipeline: `step(i)`, i = 0 .. NM - 1, issues the i-th matrix instruction of the NEXT
// 32 x 32 block (and whatever goes with it, one LDS read), and the sum of 2^arg(v) over the lane's 16 logits of the
// CURRENT one is formed in between.  A wave issues in order and the matrix core takes 32 cycles per instruction, during
// which about six VALU instructions (two of them v_exp_f32, 8 cycles) fit; spread evenly, 8 MFMA + 48 VALU take 340
// cycles, against 435 with the MFMAs in pairs, 520 with them in front, and 260 + 270 where either half stands alone.
// The order is therefore written out, packet by packet, every value a packet or more ahead of its use, and each value is
// pinned to its place (an empty volatile asm that names it; sched_barrier alone does not hold pure arithmetic).
template <class T>
__device__ __forceinline__ void pin(T& x) { asm volatile("" : "+v"(x)); }
template <int NM, class Step, class Arg>
__device__ __forceinline__ float exp2_sum_stage(Step step, Arg arg) {
    static_assert(NM == 8 || NM == 9, "packets are laid out for 8 or 9 MFMAs");
    float x[16], s[4];
    auto f = [&](int v) __attribute__((always_inline)) { x[v] = arg(v); pin(x[v]); };
    auto e = [&](int v) __attribute__((always_inline)) {
        x[v] = __builtin_amdgcn_exp2f(x[v]);
        pin(x[v]);
        if (v < 4) s[v] = x[v];
    };
    auto a = [&](int v) __attribute__((always_inline)) { s[v & 3] += x[v]; pin(s[v & 3]); };
    auto packet = [&](int i) __attribute__((always_inline)) {
        __builtin_amdgcn_sched_barrier(0);
        step(i);
        __builtin_amdgcn_sched_barrier(0);
    };
    packet(0); f(0); f(1); f(2); f(3); e(0); e(1);
    packet(1); f(4); f(5); f(6); f(7); e(2); e(3);
    packet(2); f(8); f(9); f(10); f(11); e(4); e(5);
    packet(3); f(12); f(13); f(14); f(15); e(6); e(7);
    packet(4); e(8); e(9); a(4); a(5); a(6); a(7);
    if (NM == 8) {
        packet(5); e(10); e(11); e(12); a(8); a(9);
        packet(6); e(13); e(14); a(10); a(11); a(12);
        packet(7); e(15); a(13); a(14);
    } else {
        packet(5); e(10); e(11); a(8); a(9);
        packet(6); e(12); e(13); a(10); a(11);
        packet(7); e(14); e(15); a(12); a(13);
        packet(8); a(14);
    }
    a(15);
    float sum = (s[0] + s[1]) + (s[2] + s[3]);
    pin(sum);
    __builtin_amdgcn_sched_barrier(0);
    return sum;
}

// ------------------------------------------------------------------------------------------------
// pass 1: softmax statistics
// ------------------------------------------------------------------------------------------------
// One 32-key tile against the wave's query rows: rows of the MFMA result are keys, columns are
// query rows, so each lane updates the running (m, Z) of its own query column from its 16 keys.
// Key (row of the tile) number >= valid[qt] does not exist for query tile qt's column of this lane -- the last, partial
// tile of a sequence (one uniform bound) and the tiles of the soft tokens' own keys, where the bound is causal and
// differs per lane.
__device__ __forceinline__ f32x16 mfma_bf16(bf16x8 a, bf16x8 b, f32x16 acc) { return __builtin_amdgcn_mfma_f32_32x32x16_bf16(a, b, acc, 0, 0, 0); }
__device__ __forceinline__ f32x16 zero_acc() { return f32x16{0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f}; }
__device__ __forceinline__ f32x16 stats_chain(const bf16x8 (&kf)[8], const bf16x8 (&q)[8]) {
    f32x16 acc = zero_acc();
#pragma unroll
    for (int k8 = 0; k8 < 8; ++k8) acc = mfma_bf16(kf[k8], q[k8], acc);
    return acc;
}

// The largest Z that a lane hands on with an offset that is not the maximum of its logits.  The merges that follow (two
// lane halves, the waves of a workgroup, a sequence's workgroups) add lanes' Z without looking again, at equal offsets in
// the worst case: a row has at most two lanes per 32-key tile, 2^20 of them (a sequence is below 2^24 tokens: 256 bytes a
// row in a 32-bit buffer offset), and 2^20 * 2^96 is still finite.  With the limit at infinity a group of late keys 111..128
// octaves above every wave's first tile left each lane finite and the merged Z infinite, hence NaN scores.
constexpr float kLargestZ = 0x1p96f;

// The general tile: masked, and `keep` says whether the offsets stay as they are (any offset gives the same (m, Z) pair
// up to rounding as long as no term overflows; terms that underflow are negligible next to the contribution of the
// offset's own key) or follow the running maximum.
template <int NQT>
__device__ __forceinline__ void stats_tile(const bf16x8 (&kf)[8], const bf16x8 (&qf)[NQT][8], float (&m)[NQT],
                                           float (&z)[NQT], float c, const int (&valid)[NQT], int half, bool keep) {
    f32x16 acc = stats_chain(kf, qf[0]);
#pragma unroll
    for (int qt = 0; qt < NQT; ++qt) {
#pragma unroll
        for (int v = 0; v < 16; ++v)
            if (8 * (v >> 2) + 4 * half + (v & 3) >= valid[qt]) acc[v] = -INFINITY;
        float tmax = fmaxf(acc[0], acc[1]);
#pragma unroll
        for (int v = 2; v < 16; ++v) tmax = fmaxf(tmax, acc[v]);
        // a fully masked column keeps m: 2^(-inf - m) = 0 either way
        const float mnew = keep ? m[qt] : fmaxf(m[qt], tmax * c);
        z[qt] *= __builtin_amdgcn_exp2f(m[qt] - mnew);
        m[qt] = mnew;
        f32x16 nxt = zero_acc();
        z[qt] += exp2_sum_stage<8>(
            [&](int i) __attribute__((always_inline)) {
                if (qt + 1 < NQT) { nxt = mfma_bf16(kf[i], qf[(qt + 1) % NQT][i], nxt); pin(nxt); }
            },
            [&](int v) __attribute__((always_inline)) { return fmaf(acc[v], c, -mnew); });
        acc = nxt;
    }
}

// A workgroup's share of one (layer, sequence): its waves sweep their tiles and leave one set of statistics, in a.stats.
// SHARED: the launch does both passes (see jq_passes_kernel): others read the set, the query rows stay in LDS (`q_there`: they are).
template <int NQT, bool PAGED, bool SHARED>
__device__ __forceinline__ void stats_share(KArgs& a, const Share& h, int g, int rg, char* lds, bool q_there = false) {
    const int lane = lane_again(), half = lane >> 5;
    const int wv = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
    char* slots = lds + wv * 2 * kSlotBytes;
    auto tile_of = [&](int k) __attribute__((always_inline)) { return kScoreWaves * h.quad(h.x + k) + wv; };
    const int n_tiles = h.len - (tile_of(h.len - 1) >= h.seq_tiles ? 1 : 0);  // only the sequence's last quad may lack tiles

    const KeyStream ks = key_stream<PAGED>(a, h, g);
    const uint32_t tl = tile_lane(lane, ks.row_bytes);
    // With the soft tokens' own keys in the softmax, the sequence's first wave takes them as further tiles
    // after its prompt tiles (same row stride, n_q rows), masked causally per query row.
    const int n_tail = (a.K_tail && h.rank == 0 && wv == 0) ? (a.n_q + kKeyTile - 1) / kKeyTile : 0;  // wave 0 always has tiles
    const int n_all = n_tiles + n_tail;
    __amdgpu_buffer_rsrc_t tail_rsrc = ks.rsrc;
    if (n_tail) {
        const char* kt = (const char*)a.K_tail + ((int64_t)(h.layer * a.n_seq + h.seq) * a.n_q * a.h_kv + g) * kHeadDim * 2;
        tail_rsrc = __builtin_amdgcn_make_buffer_rsrc((void*)kt, 0, (int)((uint32_t)(a.n_q - 1) * ks.row_bytes + kHeadDim * 2),
                                                      0x00020000);
    }
    // The wave's k-th tile is tile_of(k) of the sequence and uses slot k & 1.  PAGED: tiles are
    // requested in the order k = 0, 1, 2, ...; the table word of the NEXT request is loaded while this one is
    // issued, so its latency never sits in front of a tile's loads (primed where a sweep starts).
    int page_next = 0;
    Walk<false> walk;  // at the next tile to request
    auto fetch = [&](int k) __attribute__((always_inline)) {
        if (k < n_tiles) {
            const int t = walk.t, page = page_next;
            walk.step(h);
            if (PAGED && k + 1 < n_tiles) page_next = tile_page<PAGED>(ks, walk.t);
            fetch_tile(ks.rsrc, slots + (k & 1) * kSlotBytes, tile_offset<PAGED>(ks, t, page), ks.row_bytes, tl, ks.last);
        } else {
            const int t = k - n_tiles;
            fetch_tile(tail_rsrc, slots + (k & 1) * kSlotBytes, (uint32_t)t * kKeyTile * ks.row_bytes, ks.row_bytes, tl, last_request(a.n_q, ks.row_bytes));
        }
    };
    // The first key tile goes to slot 0 at once; the second slots first serve as the staging area that turns
    // the workgroup's query rows into operand order.  From then on the wave's tiles alternate between its two
    // slots, and the next tile is requested as soon as the current one's fragments are in registers.
    // As in the second pass the query rows are requested first, into registers, the key tile after them, and the
    // rows pass through LDS while the tile is in flight (explicit LDS instructions, every request unconditional in
    // one basic block: see lds_addr()).  A wave without tiles requests the sequence's first tile and drops it.
    walk.start(h, h.x, wv);
    const int t_first = n_tiles > 0 ? walk.t : 0;
    const int page_first = PAGED ? tile_page<PAGED>(ks, t_first) : 0;
    walk.step(h);
    if (PAGED && n_tiles > 1) page_next = tile_page<PAGED>(ks, walk.t);
    const uint32_t off_first = tile_offset<PAGED>(ks, t_first, page_first);
    bf16x8 qf[NQT][8];
    if (SHARED && q_there) {
        fetch_tile(ks.rsrc, slots, off_first, ks.row_bytes, tl, ks.last);
#pragma unroll
        for (int qt = 0; qt < NQT; ++qt) lds_get_frags_waited(lds_addr(lds + kLdsQ + qt * kSlotBytes), qf[qt], lane);
    } else {
        u32x4 qraw[8];
        q_rows_request<NQT>(a, h, g, rg, lane, qraw);
        __builtin_amdgcn_sched_barrier(0);
        fetch_tile(ks.rsrc, slots, off_first, ks.row_bytes, tl, ks.last);
        __builtin_amdgcn_sched_barrier(0);
        q_rows_stage<NQT>(lane, SHARED ? lds + kLdsQ : lds + kSlotBytes, SHARED ? kSlotBytes : 2 * kSlotBytes, qraw, qf);
    }
    const float c = a.c;
    float m[NQT], z[NQT];
#pragma unroll
    for (int qt = 0; qt < NQT; ++qt) { m[qt] = -1.0e30f; z[qt] = 0.0f; }
    if (n_all > 0) {  // not a wave without tiles in the sequence's last quad

    // Every load older than the second tile's eight (first tile, query rows) is covered
    // by the first wait of the sweep.  Tiles that lie entirely inside the keys every query row sees (all L
    // prompt keys, or the L - n_q keys in front of the window when the queries are the prompt's own last
    // tokens) need no mask; the others -- the sequence's partial last tile, the window's tiles -- are the
    // last of the tiles of whichever waves own them.
    const int n_common = a.window ? h.L - a.n_q : h.L;
    const int common_tiles = n_common / kKeyTile;  // sequence tiles 0 .. common_tiles - 1 are unmasked
    int n_full = n_tiles;
    while (n_full > 0 && tile_of(n_full - 1) >= common_tiles) --n_full;
    // Besides the hot sweep's body the kernel holds ONE general one, for the few masked tiles (partial last tile, window,
    // soft tokens' own keys) and the rare repeat of a sweep.  (A copy per case made the kernel 45 KB of code, for no
    // gain in time.)
    auto tile_prologue = [&](int k, bf16x8 (&kf)[8]) __attribute__((always_inline)) {
        int l = lane;
        asm volatile("" : "+v"(l));  // as in valid_rows
        wait_tile_landed();
        lds_get_frags(slots + (k & 1) * kSlotBytes, kf, l);
        if (k + 1 < n_all) {
            wait_frags_read();
            fetch(k + 1);
        }
    };
    // rows of tile k that exist for this lane's query row of each query tile (32 or more: all of them)
    auto valid_rows = [&](int k, int (&valid)[NQT]) __attribute__((always_inline)) {
        int l = lane & 31;
        asm volatile("" : "+v"(l));  // rarely taken: keeps what follows out of the hot sweep's registers
#pragma unroll
        for (int qt = 0; qt < NQT; ++qt) {
            // soft token of the lane's row (row r = i * group + hh): it sees soft tokens 0..i
            const int soft_i = a.window || k >= n_tiles ? ((rg * NQT + qt) * kRowTile + l) / a.group : 0;
            if (k < n_tiles) {
                const int t0 = tile_of(k) * kKeyTile;
                valid[qt] = (a.window ? n_common + soft_i + 1 : h.L) - t0;
            } else {  // soft token t * 32 + j is visible to the row of soft token i iff it is <= i
                valid[qt] = soft_i + 1 - (k - n_tiles) * kKeyTile;
            }
        }
    };
    // First sweep: the wave's first tile sets each lane's offset m (to the largest of four of its 16 logits), later tiles
    // keep it -- no maximum to track.  Logits far above that offset overflow Z to infinity, which cannot be repaired
    // afterwards, so a wave with a Z of kLargestZ or more (wave-uniform decision) sweeps again with the running maximum.
    int k = 0;
    if (n_full > 0) {
        // The hot sweep, tiles 0 .. n_full - 1, software-pipelined across tiles: while query tile qt's logits are
        // exponentiated the MFMA chain of the next one runs, and behind the last one the chain of the NEXT tile's first,
        // whose fragments were read during the stage before.  At every iteration's end tile k + 1 sits in registers and
        // tile k + 2 is in flight.  The last iteration's look-ahead reads whatever its slot holds and drops it (a masked
        // tile that follows is read again by its own prologue).
        bf16x8 kf[8];
        wait_tile_landed();
        lds_get_frags(slots, kf, lane);
        wait_frags_read();
        if (n_all > 1) fetch(1);
        f32x16 acc = stats_chain(kf, qf[0]);
        auto hot_tile = [&](bool first) __attribute__((always_inline)) {  // `first` is a constant in either copy
#pragma unroll
            for (int qt = 0; qt < NQT; ++qt) {
                const bool reads = qt == (NQT > 1 ? NQT - 2 : 0);
                const char* next_slot = slots + ((k + 1) & 1) * kSlotBytes;
                const uint32_t next_at = frag_addr(next_slot, lane);
                if (reads) wait_tile_landed();
                if (NQT == 1) lds_get_frags(next_slot, kf, lane);
                if (first) m[qt] = fmaxf(fmaxf(acc[0], acc[5]), fmaxf(acc[10], acc[15])) * c;
                f32x16 nxt = zero_acc();
                z[qt] += exp2_sum_stage<8>(
                    [&](int i) __attribute__((always_inline)) {
                        nxt = mfma_bf16(kf[i], qf[(qt + 1) % NQT][i], nxt);
                        pin(nxt);
                        if (reads && NQT > 1) kf[i] = lds_get_frag(next_at, i);  // its last use was this MFMA
                    },
                    [&](int v) __attribute__((always_inline)) { return fmaf(acc[v], c, -m[qt]); });
                if (reads) {
                    wait_frags_read();
                    if (k + 2 < n_all && k + 2 <= n_full) fetch(k + 2);
                }
                acc = nxt;
            }
            ++k;
        };
        hot_tile(true);
        while (k < n_full) hot_tile(false);
    }
    bool repeat = false;  // uniform
    for (;;) {
        for (; k < n_all; ++k) {
            bf16x8 kf[8];
            tile_prologue(k, kf);
            int valid[NQT];
            valid_rows(k, valid);
            stats_tile<NQT>(kf, qf, m, z, c, valid, half, !repeat && k > 0);
        }
        bool overflow = false;
#pragma unroll
        for (int qt = 0; qt < NQT; ++qt) overflow |= !(z[qt] < kLargestZ);
        if (repeat || !__builtin_expect(__any(overflow), 0)) break;
        repeat = true;
#pragma unroll
        for (int qt = 0; qt < NQT; ++qt) { m[qt] = -1.0e30f; z[qt] = 0.0f; }
        wait_frags_read();
        walk.start(h, h.x, wv);
        if (PAGED && n_tiles > 0) page_next = tile_page<PAGED>(ks, walk.t);
        fetch(0);
        k = 0;
    }

    }  // n_all > 0

    // Lanes l and l+32 hold the same query rows over complementary keys: merge them; then the four waves of
    // the workgroup merge their rows through LDS (every slot is idle by now), in wave order, into the one
    // set the share leaves.
    float2* mine = (float2*)slots;  // [NQT * 32] of this wave
#pragma unroll
    for (int qt = 0; qt < NQT; ++qt) {
        const float2 mh = both_halves(m[qt]), zh = both_halves(z[qt]);
        const float mm = fmaxf(mh.x, mh.y);
        const float zz = zh.x * __builtin_amdgcn_exp2f(mh.x - mm) + zh.y * __builtin_amdgcn_exp2f(mh.y - mm);
        if (half == 0) mine[qt * kRowTile + lane] = make_float2(mm, zz);
    }
    __syncthreads();
    const int row = rg * NQT * kRowTile + (int)threadIdx.x;  // the last group may reach past the head's row tiles
    const int set = h.set0 + h.rank;
    if (threadIdx.x < NQT * kRowTile && row < a.RP) {
        float2 mz[kScoreWaves];
        float M = -1.0e30f, Z = 0.f;
#pragma unroll
        for (int w = 0; w < kScoreWaves; ++w) mz[w] = ((const float2*)(lds + w * 2 * kSlotBytes))[threadIdx.x];
#pragma unroll
        for (int w = 0; w < kScoreWaves; ++w) M = fmaxf(M, mz[w].x);
#pragma unroll
        for (int w = 0; w < kScoreWaves; ++w) Z = fmaf(mz[w].y, __builtin_amdgcn_exp2f(mz[w].x - M), Z);
        float2* to = &a.stats[((int64_t)set * a.h_kv + g) * a.RP + row];
        if (SHARED || a.flags) {
            __hip_atomic_store((uint64_t*)to, (uint64_t)__float_as_uint(M) | (uint64_t)__float_as_uint(Z) << 32, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            if (SHARED) ((float2*)(lds + kLdsSet))[threadIdx.x] = make_float2(M, Z);
        } else {
            *to = make_float2(M, Z);
        }
    }
    if (SHARED) {  // the set has to be where every XCD sees it before its flag is
        asm volatile("s_waitcnt vmcnt(0) lgkmcnt(0)" ::: "memory");
        bare_barrier();
        if (threadIdx.x == 0 && h.n_sets > 1) __hip_atomic_store(&a.flags[(int64_t)g * a.n_sets + set], a.token, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    }
}

// -beta/c as the three bf16 terms (all 24 bits of an fp32 number) that enter the second pass through its extra MFMA step.
// (A fourth term, bits 25..32, is truncated away inside the MFMA's addition: a common factor 1 + 3e-7.)
__device__ __forceinline__ uint2 split_bf16x3(float x) {
    const uint32_t hi = __float_as_uint(x) & 0xFFFF0000u;
    const float r1 = x - __uint_as_float(hi);
    const uint32_t mid = __float_as_uint(r1) & 0xFFFF0000u;
    const float r2 = r1 - __uint_as_float(mid);
    const uint32_t lo = __float_as_uint(r2) & 0xFFFF0000u;
    return make_uint2((hi >> 16) | mid, lo >> 16);
}
// ... of a query row with statistics (m, Z): beta = m + log2 Z.  Every error here is a common factor in all scores of the
// row, so it is formed in fp64 and rounded once.  v_log_f32 rounds towards zero -- at Z in 2^10..2^16 its results are
// 4.7e-7 too small on average, a factor 1 + 3.2e-7 in every score -- so it only sees the mantissa (mean error 1e-8).
// Scores are now 1e-7 from the 64-bit result (2-norm; 3.6e-7 before).
__device__ __forceinline__ uint2 neg_beta_terms(float m, float z, double inv_c) {
    const double beta = (double)m + (double)__builtin_amdgcn_frexp_expf(z) + (double)__builtin_amdgcn_logf(__builtin_amdgcn_frexp_mantf(z));
    return split_bf16x3((float)(-beta * inv_c));
}
constexpr float kPadTerm = -1.0e30f;  // for padded rows: 2^(c * x) = 0

// (m, Z) of a row merged with those of up to N more sets, number from, from + 2, ... of the n there are, which `t` holds
template <int N>
__device__ __forceinline__ void merge_sets(const float2 (&t)[N], int from, int n, float& M, float& Z) {
    float mm = M;
#pragma unroll
    for (int u = 0; u < N; ++u) mm = fmaxf(mm, from + 2 * u < n ? t[u].x : -1.0e30f);
    Z *= __builtin_amdgcn_exp2f(M - mm);
#pragma unroll
    for (int u = 0; u < N; ++u) Z = fmaf(t[u].y, from + 2 * u < n ? __builtin_amdgcn_exp2f(t[u].x - mm) : 0.f, Z);
    M = mm;
}
// a set's pair for one row, formed and stored by another workgroup of this launch: read past the caches that are not shared
__device__ __forceinline__ float2 load_pair(const float2* p) {
    const uint64_t v = __hip_atomic_load((const uint64_t*)p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    return make_float2(__uint_as_float((uint32_t)v), __uint_as_float((uint32_t)(v >> 32)));
}

// Many query rows: the workgroup whose set completes those of a (layer, sequence), head and group of rows merges them, so that no
// launch has to.  Each stores its set where every XCD sees it, then its flag, and then looks at all flags: whoever stored the
// last one finds them all (two may, and write the same bits).  Nobody waits for another workgroup.  The three round trips and the
// merge lengthen the first pass by 2.8 us, the launch took 4.3-6.8 and the gap in front of it 2.2: 16384 keys under 1024 rows 92.0 -> 90.8
// us an evaluation step, training forward of 4 x 6007 keys 84.7 -> 81.7, 2000 keys under 256 rows 41.8 -> 37.4, 1500 keys trained 23.7 -> 20.4.
// (Adding up the training objective's partial sums the same way costs every workgroup of the second pass a round trip with its
// LDS held, several rounds of them: 1 x 16384 keys, 64 response tokens 44.0 -> 47.3 us, 4 x 16384 135.5 -> 141; that stays a launch.)
template <int NQT>
__device__ __forceinline__ void merge_if_last(KArgs& a, const Share& h, int g, int rg, char* lds) {
    static_assert(kScoreWaves * 64 >= 2 * NQT * kRowTile, "two threads a row");
    const int lane = lane_again();
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");  // the set
    __syncthreads();
    if (threadIdx.x < 64) {
        uint64_t* flag = a.flags + ((int64_t)g * a.n_rg + rg) * a.n_sets + h.set0;
        if (lane == 0) __hip_atomic_store(flag + h.rank, a.token, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
        const bool all = __all(__hip_atomic_load(flag + min(lane, h.n_sets - 1), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) == a.token);
        if (lane == 0) *(int*)lds = all;
    }
    __syncthreads();
    if (!*(const int*)lds) return;
    const int p0 = (int)(threadIdx.x & 1), in_group = (int)(threadIdx.x >> 1), row = rg * NQT * kRowTile + in_group;
    if (in_group >= NQT * kRowTile || row >= a.RP) return;  // both threads of a row
    const float2* from = a.stats + ((int64_t)h.set0 * a.h_kv + g) * a.RP + row;
    const int64_t step = (int64_t)a.h_kv * a.RP;
    float M = -1.0e30f, Z = 0.f;
    for (int k = p0; k < h.n_sets; k += 16) {
        float2 t[8];
#pragma unroll
        for (int u = 0; u < 8; ++u) t[u] = load_pair(from + min(k + 2 * u, h.n_sets - 1) * step);
        merge_sets(t, k, h.n_sets, M, Z);
    }
    const float oM = __shfl_xor(M, 1), oZ = __shfl_xor(Z, 1);
    const float mm = fmaxf(M, oM), zz = Z * __builtin_amdgcn_exp2f(M - mm) + oZ * __builtin_amdgcn_exp2f(oM - mm);
    if (p0) return;
    const bool real = row < a.tiles1 * (int64_t)kRowTile ? row < a.rows : row - a.tiles1 * kRowTile < a.rows2;
    a.aug[((int64_t)(h.layer * a.n_seq + h.seq) * a.h_kv + g) * a.RP + row] = real ? neg_beta_terms(mm, zz, a.inv_c) : split_bf16x3(kPadTerm);
}

__device__ __forceinline__ void clear_words(KArgs& a) {  // every workgroup its part
    if (!a.zero) return;
    const uint64_t per = (a.zero_words + gridDim.x - 1) / gridDim.x;
    const uint64_t z0 = per * blockIdx.x, z1 = z0 + per < a.zero_words ? z0 + per : a.zero_words;
    for (uint64_t i = z0 + threadIdx.x; i < z1; i += blockDim.x) a.zero[i] = 0u;
}

template <int NQT, bool PAGED>
__global__ __launch_bounds__(kScoreWaves * 64, 2) void jq_stats_kernel(ScoreArgs) {
    __shared__ __attribute__((aligned(1024))) char lds[kSlotsBytes];
    argument_lines<5>();
    Place at = place_of(kernel_args(), blockIdx.x, false);
    const bool many_rows = kernel_args().flags != nullptr;  // uniform
    for (;;) {
        KArgs& a = kernel_args();
        const Share h = share_of(a, at.c, at.layer, at.seq);
        stats_share<NQT, PAGED, false>(a, h, at.g, at.rg, lds);
        if (many_rows) merge_if_last<NQT>(a, h, at.g, at.rg, lds);
        if (!next_share(a, h, false, at)) break;
        bare_barrier();  // the statistics have left the slots
    }
}

// The instance of the headline shape (128 query rows per KV head, dense cache), emitted here so that it lies next
// to the other kernels of a step in the library's code (see jq_lib.hip).
template __global__ void jq_stats_kernel<4, false>(ScoreArgs);

constexpr int kCombineLanes = 32;  // partial-lanes per query row
__global__ __launch_bounds__(kRowTile * kCombineLanes) void jq_combine_kernel(ScoreArgs) {
    argument_lines<5>();
    KArgs& a = kernel_args();
    // one workgroup per (layer, sequence, head, tile of 32 rows); thread = (row r, partial-lane kl)
    __shared__ float2 part[kCombineLanes][kRowTile];
    const int r = threadIdx.x & (kRowTile - 1), kl = threadIdx.x / kRowTile;
    const int tiles = a.RP / kRowTile;
    if (a.zero) {  // clear the selection histograms and counters while we are here
        const uint64_t per = (a.zero_words + gridDim.x - 1) / gridDim.x;
        const uint64_t z0 = per * blockIdx.x, z1 = z0 + per < a.zero_words ? z0 + per : a.zero_words;
        for (uint64_t i = z0 + threadIdx.x; i < z1; i += blockDim.x) a.zero[i] = 0u;
    }

    const int64_t n_items = (int64_t)a.n_layers * a.n_seq * a.h_kv * tiles;  // every workgroup of a normal call has one
    for (int64_t item = blockIdx.x; item < n_items; item += gridDim.x) {
        const int rt = (int)(item % tiles);
        int64_t rest = item / tiles;
        const int g = (int)(rest % a.h_kv);
        rest /= a.h_kv;
        const int s = (int)(rest % a.n_seq);
        const int layer = (int)(rest / a.n_seq);
        const int row = rt * kRowTile + r;
        if (item != blockIdx.x) __syncthreads();  // `part` is still being read
        int set0, n_sets;
        sets_of(a, a.part, a.cu_part, layer, s, set0, n_sets);
        const float2* p = a.stats + ((int64_t)set0 * a.h_kv + g) * a.RP + row;
        const int64_t step = (int64_t)a.h_kv * a.RP;
        float M = -1.0e30f, Z = 0.f;
        for (int k0 = kl; k0 < n_sets; k0 += 8 * kCombineLanes) {  // 8 independent loads in flight per thread
            float2 mz[8];
#pragma unroll
            for (int u = 0; u < 8; ++u) {
                const int k = k0 + u * kCombineLanes;
                mz[u] = k < n_sets ? p[k * step] : make_float2(-1.0e30f, 0.f);
            }
#pragma unroll
            for (int u = 0; u < 8; ++u) {
                const float mm = fmaxf(M, mz[u].x);
                Z = Z * __builtin_amdgcn_exp2f(M - mm) + mz[u].y * __builtin_amdgcn_exp2f(mz[u].x - mm);
                M = mm;
            }
        }
        part[kl][r] = make_float2(M, Z);
        __syncthreads();
        if (kl == 0) {
            for (int k = 1; k < kCombineLanes; ++k) {  // fixed order: deterministic
                const float2 mz = part[k][r];
                const float mm = fmaxf(M, mz.x);
                Z = Z * __builtin_amdgcn_exp2f(M - mm) + mz.y * __builtin_amdgcn_exp2f(mz.x - mm);
                M = mm;
            }
            const bool real = rt < a.tiles1 ? row < a.rows : row - a.tiles1 * kRowTile < a.rows2;
            a.aug[((int64_t)(layer * a.n_seq + s) * a.h_kv + g) * a.RP + row] = real ? neg_beta_terms(M, Z, a.inv_c) : split_bf16x3(kPadTerm);
        }
    }
}

// ------------------------------------------------------------------------------------------------
// pass 2: normalised probabilities summed over the query rows
// ------------------------------------------------------------------------------------------------
// q.k - beta/c for one tile of 32 query rows against the 32 keys in `kf` (rows = query rows, columns = keys).
__device__ __forceinline__ f32x16 score_chain(const bf16x8 (&q)[8], bf16x8 qaug, const bf16x8 (&kf)[8], bf16x8 ones) {
    f32x16 acc = {0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int k8 = 0; k8 < 8; ++k8) acc = __builtin_amdgcn_mfma_f32_32x32x16_bf16(q[k8], kf[k8], acc, 0, 0, 0);
    return __builtin_amdgcn_mfma_f32_32x32x16_bf16(qaug, ones, acc, 0, 0, 0);  // - beta_r / c
}

// Where a second pass gets its normalisers from.
enum Norms {
    kNormsMerged,  // sets of statistics that an earlier launch has left (or `aug`, if a combine launch has merged them)
    kNormsLse,     // the caller: lse becomes the -beta/c terms on the fly (beta = lse * log2 e, c = scale * log2 e, so
                   // -beta/c = -lse / scale)
    kNormsShared,  // sets of statistics that this launch's workgroups form and publish
};

// A workgroup's share of one (layer, sequence): its waves score their tiles, from the share's last to its first (the first pass went
// the other way, and the caches still hold what it read last: front to back it takes 1.7 us longer on the 128K layer).
// Returns -1, or (kNormsShared) the number of a set that others have not published within `patience` ticks; nothing is scored then.
template <int NQT, Norms NORMS, bool PAGED, bool HOLD>
__device__ __forceinline__ int score_share(KArgs& a, const Share& h, int g, char* lds, char* held_lds, int64_t patience, bool q_there = false) {
    const int lane = lane_again(), half = lane >> 5;
    const int wv = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
    char* slots = lds + wv * 2 * kSlotBytes;
    const int x_last = h.x + h.len - 1;
    const int skip = kScoreWaves * h.quad(x_last) + wv >= h.seq_tiles ? 1 : 0;  // no tile for this wave in the sequence's last quad
    const int n_tiles = h.len - skip;

    const KeyStream ks = key_stream<PAGED>(a, h, g);
    const uint32_t tl = tile_lane(lane, ks.row_bytes);
    // PAGED: as in the first pass, the table word of the next request (k + 1) is loaded one request ahead
    int page_next = 0;  // set by the start-up's first request
    Walk<true> walk;    // at the next tile to request
    auto fetch = [&](int k) __attribute__((always_inline)) {  // returns the tile
        const int t = walk.t, page = page_next;
        walk.step(h);
        if (PAGED && k + 1 < n_tiles) page_next = tile_page<PAGED>(ks, walk.t);
        fetch_tile(ks.rsrc, slots + (k & 1) * kSlotBytes, tile_offset<PAGED>(ks, t, page), ks.row_bytes, tl, ks.last);
        return t;
    };
    bf16x8 qf[NQT][8];
    // Start-up.  Requested first, into registers: the query rows, the first pass's statistics (or the
    // normalisers themselves); then the first key tile, straight into LDS.  Everything up to the sweep works on the
    // former while the latter is in flight (see lds_addr() above for why the LDS instructions here are explicit).
    // The compiler can only count on loads that are certain to have been issued, so every request below is
    // unconditional -- addresses are clamped, values that turn out not to be needed are dropped -- and all of them
    // sit in one basic block: then each wait is exactly "everything older than this value", never the key tile.
    const bool merging = NORMS == kNormsShared || (NORMS == kNormsMerged && a.fuse_combine);  // uniform
    constexpr int kFirstParts = 16;  // sets per thread requested up front: all of them for up to 32 per row
    const int p0 = (int)(threadIdx.x & 1);
    // Unless a combine launch has merged them already, this
    // workgroup merges the sets of its head's rows itself: thread t takes row t / 2 and every second
    // set; pairs meet by shuffle, and the rows' -beta/c terms pass through LDS.
    const int mrow = min((int)(threadIdx.x >> 1), NQT * kRowTile - 1);
    int set0 = h.set0, n_p = h.n_sets;
    if (NORMS == kNormsMerged) {
        set0 = 0; n_p = 1;
        if (merging) sets_of(a, a.part, a.cu_part, h.layer, h.seq, set0, n_p);
    }
    const float2* pp = a.stats + ((int64_t)set0 * a.h_kv + g) * a.RP + mrow;
    const int64_t pstep = (int64_t)a.h_kv * a.RP;
    walk.start(h, x_last - skip, wv);
    const int t_first = n_tiles > 0 ? walk.t : 0;  // a wave without tiles requests the sequence's first tile and drops it
    const int page_first = PAGED ? tile_page<PAGED>(ks, t_first) : 0;
    walk.step(h);
    if (PAGED && n_tiles > 1) page_next = tile_page<PAGED>(ks, walk.t);
    const uint32_t off_first = tile_offset<PAGED>(ks, t_first, page_first);
    float2 mz[kFirstParts];
    uint2 aug_direct[NQT];  // the terms of the lane's rows where no merging is due
    if (NORMS == kNormsShared && q_there) {
        fetch_tile(ks.rsrc, slots, off_first, ks.row_bytes, tl, ks.last);
    } else {
        const float* nsrc[NQT];  // kNormsLse: the lane's rows' normalisers; kNormsMerged: the terms of a combine launch
#pragma unroll
        for (int qt = 0; qt < NQT; ++qt) {
            const int row = min(qt * kRowTile + (lane & 31), a.rows - 1);
            if (NORMS == kNormsLse) {
                const int i = row / a.group, hd = g * a.group + row % a.group;
                nsrc[qt] = a.lse + ((int64_t)(h.layer * a.n_seq + h.seq) * a.n_q + i) * a.h_q + hd;
            } else if (NORMS == kNormsMerged) {
                nsrc[qt] = (const float*)(a.aug + ((int64_t)(h.layer * a.n_seq + h.seq) * a.h_kv + g) * a.RP + qt * kRowTile + (lane & 31));
            }
        }
        u32x4 qraw[8];
        q_rows_request<NQT>(a, h, g, 0, lane, qraw);
        if (NORMS == kNormsMerged) {
#pragma unroll
            for (int u = 0; u < kFirstParts; ++u) mz[u] = pp[min(p0 + 2 * u, n_p - 1) * pstep];
        }
#pragma unroll
        for (int qt = 0; qt < NQT; ++qt) {
            if (NORMS == kNormsLse) aug_direct[qt] = make_uint2(__float_as_uint(*nsrc[qt]), 0u);
            else if (NORMS == kNormsMerged) aug_direct[qt] = *(const uint2*)nsrc[qt];
        }
        __builtin_amdgcn_sched_barrier(0);
        fetch_tile(ks.rsrc, slots, off_first, ks.row_bytes, tl, ks.last);
        __builtin_amdgcn_sched_barrier(0);
        if (NORMS == kNormsLse) {
#pragma unroll
            for (int qt = 0; qt < NQT; ++qt) {
                const int row = qt * kRowTile + (lane & 31);
                aug_direct[qt] = split_bf16x3(row < a.rows ? (float)(-(double)__uint_as_float(aug_direct[qt].x) * a.inv_scale) : kPadTerm);
            }
        }
        q_rows_stage<NQT>(lane, NORMS == kNormsShared ? lds + kLdsQ : lds + kSlotBytes, NORMS == kNormsShared ? kSlotBytes : 2 * kSlotBytes, qraw, qf);
    }
    // the rows' -beta/c terms pass through LDS; in a launch of the second pass alone through wave 0's second slot, free until its second tile
    const uint32_t aug_s = lds_addr(NORMS == kNormsShared ? lds + kLdsAug : lds + kSlotBytes);
    const bool own_set = NORMS == kNormsShared && q_there && n_p == 1;  // nobody else has keys of the sequence, and LDS holds the set
    if (NORMS == kNormsShared && !own_set) {
        if (n_p > 1) {
            // Wave 0 watches the flags of the (layer, sequence), one per lane (at most 64, the host has seen to it); the other
            // waves wait at the barrier, where they take no issue slots.  The wait ends after `patience` ticks whatever happens.
            const uint32_t word = lds_addr(lds + kLdsWord);
            if (wv == 0) {
                const uint64_t* flag = a.flags + (int64_t)g * a.n_sets + set0 + min(lane, n_p - 1);
                const int64_t t0 = wall_clock64();
                uint32_t missing = 0u;  // number of a missing set + 1
                for (;;) {
                    const uint64_t late = __ballot(__hip_atomic_load(flag, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) != a.token);
                    if (late == 0u) break;
                    if (wall_clock64() - t0 >= patience) {  // the missing one that falls to this workgroup
                        uint64_t m = n_p < 64 ? late & ((1ull << n_p) - 1) : late;
                        for (int skip = h.rank % __builtin_popcountll(m); skip > 0; --skip) m &= m - 1;
                        missing = 1u + (uint32_t)__builtin_ctzll(m);
                        break;
                    }
                    __builtin_amdgcn_s_sleep(1);
                }
                if (lane == 0) lds_put8(word, make_uint2(missing, 0u));
                lds_wait_all();
            }
            bare_barrier();
            const uint32_t missing = __builtin_amdgcn_readfirstlane(lds_get8_waited(word).x);
            if (missing) {  // uniform
                wait_tile_landed();  // the request above must not land in a slot that is in use again
                bare_barrier();
                return (int)missing - 1;
            }
        }
#pragma unroll
        for (int u = 0; u < kFirstParts; ++u) mz[u] = load_pair(pp + min(p0 + 2 * u, n_p - 1) * pstep);
    }
    // The query rows out of LDS, half a microsecond of the CU's LDS, while the sets are on their way (in front of the flags: 2048 tokens
    // 14.81 us a call, 14.58 here; 8192 21.2 / 20.8, 16384 27.1 / 26.7, 32768 39.2 / 39.0).
    if (NORMS == kNormsShared && q_there) {
        __builtin_amdgcn_sched_barrier(0);
#pragma unroll
        for (int qt = 0; qt < NQT; ++qt) lds_get_frags_waited(lds_addr(lds + kLdsQ + qt * kSlotBytes), qf[qt], lane);
        __builtin_amdgcn_sched_barrier(0);
    }
    float cM = -1.0e30f, cZ = 0.f;
    if (own_set) {
        const uint2 v = lds_get8_waited(lds_addr(lds + kLdsSet) + 8u * (uint32_t)mrow);
        if (p0 == 0) { cM = __uint_as_float(v.x); cZ = __uint_as_float(v.y); }
    } else if (merging && (threadIdx.x >> 1) < NQT * kRowTile) {  // the same order of additions whatever the number of sets
        merge_sets(mz, p0, n_p, cM, cZ);
        for (int k0 = p0 + 2 * kFirstParts; k0 < n_p; k0 += 16) {  // more than 32 sets
            float2 more[8];
#pragma unroll
            for (int u = 0; u < 8; ++u) {
                const float2* src = pp + min(k0 + 2 * u, n_p - 1) * pstep;
                more[u] = NORMS == kNormsShared ? load_pair(src) : *src;
            }
            merge_sets(more, k0, n_p, cM, cZ);
        }
    }
    bf16x8 qaug[NQT];
    auto set_aug = [&](int qt, uint2 t) {  // the three bf16 terms sit in k-elements 0..2 of the extra MFMA step (lane half 0)
        u32x4 v = {0u, 0u, 0u, 0u};
        if (half == 0) { v[0] = t.x; v[1] = t.y; }
        qaug[qt] = as_bf16x8(v);
    };
    if (merging) {
        const float oM = __shfl_xor(cM, 1), oZ = __shfl_xor(cZ, 1);  // the odd neighbour's half; even threads finish the row
        const float mm = fmaxf(cM, oM);
        const float zz = cZ * __builtin_amdgcn_exp2f(cM - mm) + oZ * __builtin_amdgcn_exp2f(oM - mm);
        const int crow = (int)(threadIdx.x >> 1);
        if (!(threadIdx.x & 1) && crow < NQT * kRowTile) {
            lds_put8(aug_s + 8u * crow, crow < a.rows ? neg_beta_terms(mm, zz, a.inv_c) : split_bf16x3(kPadTerm));
            lds_wait_all();
        }
        bare_barrier();
        uint2 terms[NQT];
        lds_get8s_waited(aug_s + 8u * ((uint32_t)lane & 31u), 8u * kRowTile, terms);
#pragma unroll
        for (int qt = 0; qt < NQT; ++qt) set_aug(qt, terms[qt]);
        if (NORMS != kNormsShared) bare_barrier();  // the slot is refilled with a key tile next
    } else {
#pragma unroll
        for (int qt = 0; qt < NQT; ++qt) set_aug(qt, aug_direct[qt]);
    }
    wait_tile_landed();
    if (n_tiles == 0) return -1;  // a wave without tiles in the sequence's last quad
    u32x4 ones_bits = {0u, 0u, 0u, 0u};
    if (half == 0) { ones_bits[0] = 0x3F803F80u; ones_bits[1] = 0x00003F80u; }  // 1.0 at elements 0..2
    const bf16x8 ones = as_bf16x8(ones_bits);

    const __amdgpu_buffer_rsrc_t out = __builtin_amdgcn_make_buffer_rsrc((void*)(a.scores + ((int64_t)h.layer * a.h_kv + g) * a.T + h.tok0), 0,
                                                                          h.L * 4, 0x00020000);
    const float c = a.c;
    float pending = 0.f;  // previous tile's result, handed out one iteration late
    const int n_scored = a.window ? h.L - a.n_q : h.L;  // the window's own positions report 0
    // Stored at once, a tile is always one store instruction: the upper lane half (which holds the same sums), rows past the end of the
    // sequence's last tile and whatever goes to kNowhere fall behind the end of the resource, where the hardware drops them.
    constexpr int kNowhere = 0x40000000 / (4 * kKeyTile);  // (the resource has at most 2^26 bytes)
    const uint32_t out_lane = half == 0 ? 4u * (uint32_t)lane : 0x40000000u;
    auto store_tile = [&](int t, float v) {
        if (t * kKeyTile + kKeyTile > n_scored && t * kKeyTile + (lane & 31) >= n_scored) v = 0.f;
        __builtin_amdgcn_raw_buffer_store_b32(__float_as_uint(v), out, (int)(out_lane + 4u * (uint32_t)(t * kKeyTile)), 0, 0);
    };
    // HOLD: the scores wait in LDS and leave together, `hold` tiles of every wave at a time -- the whole share's, if they fit.
    // (kNormsShared: where the query rows were; the barrier above is behind every wave's last read of them.)
    int hold = NORMS == kNormsShared ? kHeldPasses : kHeldScore;
    asm("" : "+s"(hold));  // (known to the compiler, it costs 8 to 34 spilled registers)
    const uint32_t held = NORMS == kNormsShared ? lds_addr(lds + kLdsQ + wv * kSlotBytes) : lds_addr(held_lds) + (uint32_t)(wv * hold * kHeldTile);
    const uint32_t held_lane = held + 4u * ((uint32_t)lane & 31u), held_t = held + (uint32_t)hold * (kKeyTile * 4);
    int n_held = 0;
    auto write_out = [&]() __attribute__((always_inline)) {
        lds_wait_all();
        for (int i = 0; i < n_held; i += 8) {  // two tiles per store, one for either lane half (where they are too few, the last one again)
            uint32_t v[4], t[4], at_v[4], at_t[4];
#pragma unroll
            for (int u = 0; u < 4; ++u) {
                const uint32_t j = (uint32_t)min(i + 2 * u + half, n_held - 1);
                at_v[u] = held_lane + j * (kKeyTile * 4);
                at_t[u] = held_t + j * 4u;
            }
            // (explicit, as everything that touches LDS while key tiles are in flight)
            asm volatile("ds_read_b32 %0, %8\n\tds_read_b32 %1, %9\n\tds_read_b32 %2, %10\n\tds_read_b32 %3, %11\n\t"
                         "ds_read_b32 %4, %12\n\tds_read_b32 %5, %13\n\tds_read_b32 %6, %14\n\tds_read_b32 %7, %15\n\t"
                         "s_waitcnt lgkmcnt(0)"
                         : "=&v"(v[0]), "=&v"(v[1]), "=&v"(v[2]), "=&v"(v[3]), "=&v"(t[0]), "=&v"(t[1]), "=&v"(t[2]), "=&v"(t[3])
                         : "v"(at_v[0]), "v"(at_v[1]), "v"(at_v[2]), "v"(at_v[3]), "v"(at_t[0]), "v"(at_t[1]), "v"(at_t[2]), "v"(at_t[3])
                         : "memory");
#pragma unroll
            for (int u = 0; u < 4; ++u) {
                const int key = (int)t[u] * kKeyTile + (lane & 31);  // behind the sequence's end: dropped as above
                __builtin_amdgcn_raw_buffer_store_b32(key < n_scored ? v[u] : 0u, out, 4 * key, 0, 0);
            }
        }
        n_held = 0;
    };
    auto hand_out = [&](int t, float v) __attribute__((always_inline)) {
        if (!HOLD) {
            store_tile(t, v);
        } else if (t != kNowhere) {
            if (n_held == hold) write_out();
            lds_put4(held_lane + (uint32_t)n_held * (kKeyTile * 4), __float_as_uint(v));
            lds_put4(held_t + (uint32_t)n_held * 4u, (uint32_t)t);
            ++n_held;
        }
    };

    // Software pipeline over the query-row tiles and across key tiles, as in the first pass: while one tile's logits are
    // exponentiated the MFMA chain of the next runs, and behind the last one that of the next key tile's first, whose
    // fragments were read a stage earlier.  At an iteration's end tile k + 1 sits in registers and tile k + 2 is in
    // flight; the last iteration's look-ahead reads whatever its slot holds and drops it.
    bf16x8 kf[8];
    lds_get_frags(slots, kf, lane);
    wait_frags_read();
    int t_done = kNowhere, t_here = t_first, t_next = n_tiles > 1 ? fetch(1) : 0;  // the tiles k - 1, k, k + 1
    hand_out(kNowhere, 0.f);  // for the sweep's first wait
    f32x16 acc = score_chain(qf[0], qaug[0], kf, ones);
    for (int k = 0; k < n_tiles; ++k) {
        float sum = 0.f;
#pragma unroll
        for (int qt = 0; qt < NQT; ++qt) {
            const bool reads = qt == (NQT > 1 ? NQT - 2 : 0);
            const char* next_slot = slots + ((k + 1) & 1) * kSlotBytes;
            if (reads) {  // tile k + 1, behind which tile k - 2's scores were stored
                if (!HOLD) wait_tile_landed_before_store();
                else wait_tile_landed();
            }
            const uint32_t next_at = frag_addr(next_slot, lane);
            if (NQT == 1) lds_get_frags(next_slot, kf, lane);
            f32x16 nxt = zero_acc();
            sum += exp2_sum_stage<9>(
                [&](int i) __attribute__((always_inline)) {
                    nxt = i < 8 ? mfma_bf16(qf[(qt + 1) % NQT][i & 7], kf[i & 7], nxt) : mfma_bf16(qaug[(qt + 1) % NQT], ones, nxt);
                    pin(nxt);
                    if (reads && NQT > 1 && i < 8) kf[i & 7] = lds_get_frag(next_at, i);  // its last use was this MFMA
                },
                [&](int v) __attribute__((always_inline)) { return acc[v] * c; });
            if (reads) {
                wait_frags_read();
                const int t_stored = t_done;
                t_done = t_here; t_here = t_next;
                if (k + 2 < n_tiles) t_next = fetch(k + 2);
                hand_out(t_stored, pending);
            }
            acc = nxt;
        }
        pending = add_halves(sum);  // complementary query rows of the same key
    }
    hand_out(t_done, pending);
    if (HOLD) write_out();
    return -1;
}

template <int NQT, bool FROM_LSE, bool PAGED, bool HOLD>
__global__ __launch_bounds__(kScoreWaves * 64, 2) void jq_score_kernel(ScoreArgs) {
    __shared__ __attribute__((aligned(1024))) char lds[kSlotsBytes];
    extern __shared__ char held_lds[];
    argument_lines<5>();
    Place at = place_of(kernel_args(), gridDim.x - 1 - blockIdx.x, true);  // from the end: the keys pass 1 read last are fetched first
    clear_words(kernel_args());
    for (;;) {
        KArgs& a = kernel_args();
        const Share h = share_of(a, at.c, at.layer, at.seq);
        score_share<NQT, FROM_LSE ? kNormsLse : kNormsMerged, PAGED, HOLD>(a, h, at.g, lds, held_lds, 0);
        if (!next_share(a, h, true, at)) break;
    }
}

template __global__ void jq_score_kernel<4, false, false, false>(ScoreArgs);  // placement: see jq_lib.hip

// ------------------------------------------------------------------------------------------------
// both passes in one launch
// ------------------------------------------------------------------------------------------------
// Every workgroup sweeps its shares for their statistics, publishes each set -- the set past its XCD's L2, then a flag -- and scores
// the same shares, last one first, as soon as the other workgroups of the (layer, sequence) have published theirs.  Against a
// launch per pass that saves the boundary between two dependent kernels (2.2 us), the second request for the query rows
// (they wait in LDS) and, where one workgroup has a whole (layer, sequence), the way of the statistics through memory; and no
// workgroup waits for any other sequence's.  Device timestamps, 32768 tokens, 8 heads, from a workgroup's last tile of the
// first pass to its first of the second: waves' statistics merged 0.45 us, set and flag out 0.3, share 0.8, all flags seen 0.4-0.6,
// query rows and sets read and merged 1.25, terms exchanged 0.3.  Whole calls, two launches / one: 2048 tokens and 2 heads 18.7 / 17.0 us, 32768 tokens
// 48.3 / 44.8, 128K layer 114.7 / 113.0, 32 layers of 8192 246 / 240, 8 x 12345 with window queries 97.3 / 92.8; together with the
// even shares a paged batch of 8 196 / 187, 16 ragged sequences 821 / 779.
// No workgroup depends on another one running: it waits for `wait_ticks` (or the time it has run itself, if that is longer), once,
// and from then on it forms what is missing itself, from the same keys in the same order -- the same bits, whoever
// stores them.  Several that miss the same sets begin with different ones.  A launch that gets part of the chip only, beside
// another stream's kernels, so loses a sweep or two over what it has there: 32768 tokens with a quarter of the CUs held by another
// kernel 99 us (two launches 60; 1000 and more while every missing set cost a wait of its own and all workgroups formed the same
// one), 128K layer 506 (420; 2200).  Where the device has fewer CUs than the launch has workgroups both passes go one after the other.
// Two streams with evictions of their own take no longer than one with both.
// The flags need no clearing before the launch: they are compared with a 64-bit token that is the call's
// own.  A captured call has the same token in every replay, so a later kernel of the call clears them.
// One workgroup per CU (99 KB of LDS).
template <int NQT, bool PAGED, bool HOLD>
__global__ __launch_bounds__(kScoreWaves * 64, 1) void jq_passes_kernel(ScoreArgs) {
    __shared__ __attribute__((aligned(1024))) char lds[kLdsBoth];
    argument_lines<5>();
    const int64_t t_entry = wall_clock64();
    Place at = place_of(kernel_args(), blockIdx.x, false);
    clear_words(kernel_args());
    bool scoring = false, q_there = false;  // uniform
    int help = -1;                          // another workgroup, whose set this one forms in its stead
    int64_t patience = kernel_args().wait_ticks;
    for (;;) {
        KArgs& a = kernel_args();
        if (!scoring || help >= 0) {
            const Share h = share_of(a, help < 0 ? at.c : help, at.layer, at.seq);
            stats_share<NQT, PAGED, true>(a, h, at.g, 0, lds, q_there);
            if (scoring) {
                help = -1;
            } else {
                scoring = !next_share(a, h, false, at);
                if (scoring && patience) patience = max(patience, (int64_t)(wall_clock64() - t_entry));
            }
            q_there = scoring;
        } else {
            const Share h = share_of(a, at.c, at.layer, at.seq);
            const int missing = score_share<NQT, kNormsShared, PAGED, HOLD>(a, h, at.g, lds, nullptr, patience, q_there);
            q_there = true;
            if (missing >= 0) {
                help = at.c - h.rank + missing;
                patience = 0;
            } else {
                if (!next_share(a, h, true, at)) break;
                q_there = false;
            }
        }
    }
}

template __global__ void jq_passes_kernel<4, false, false>(ScoreArgs);

// ------------------------------------------------------------------------------------------------
// many query rows (more than kMaxRowTiles tiles per KV head): keys stationary, query rows streamed
// ------------------------------------------------------------------------------------------------
// With n_q * group > 128 (response tokens as queries: the upper bound of Eq. 4, the training objective) a head's rows
// no longer fit a wave's registers.  The first pass then only gets a further grid dimension over groups of row tiles.
// Here the roles swap: a workgroup holds 128 keys (four tiles, every wave all of them, 128 VGPRs) and its four waves
// sweep the head's row tiles, each its own quarter, streaming them through their private LDS slots exactly as the other
// kernels stream key tiles; a key's sum over all rows then forms in registers, is merged over the four waves in wave
// order and stored once.  Before, every 128 rows took a launch of each pass that read K and added to the scores in
// memory: launches of 64..256 keys per wave that were mostly start-up.  The work is a contraction that K does not
// bound (every key is used by all rows): 9 MFMA per 32 x 32 logits against 16 exp2/mul/add per lane.  Measured at 16384
// keys x 8 heads x 1024 rows: eight launches of 12.4 us and eight first passes of 10.9 us before, 39 + 38 us
// now (1.05 PFLOP/s; a plain library product of 8192^3 reaches 1.2 on this card, which lowers its
// clock under matrix work).  Two waves per key group instead of four: 42.9 against 41.5 us there, 5 % better only with
// thousands of workgroups: not kept.
// -beta/c comes from `aug`, which the first pass's last workgroups (or jq_combine_kernel, jq_lse_aug_kernel) have filled.
// DIFF: two query sets, whose row tiles follow each other (tiles1).  A key's two sums form in the same sweep, and instead of
// storing either map the workgroup leaves its sum of (sum1 / rows1 - sum2 / rows2)^2 (Eq. 5 of the paper on the maps of Eq. 3
// and Eq. 4), in fp64 per key, then in a fixed order over lanes and waves.  The first set has four tiles where the second has
// sixteen in the usual sizes, so sweeping them here costs less than the launches of both passes that stored its map before.
template <bool PAGED, bool DIFF>
__global__ __launch_bounds__(kScoreWaves * 64, 2) void jq_score_rows_kernel(ScoreArgs) {
    KArgs& a = kernel_args();
    __shared__ __attribute__((aligned(1024))) char lds[kScoreWaves][2][kSlotBytes];
    __shared__ double diff_s[DIFF ? 2 : 1];
    const int lane = threadIdx.x & 63, half = lane >> 5;
    const int wv = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
    char* slots = &lds[wv][0][0];
    // one workgroup per (layer, group of 128 keys, head), heads fastest: with eight heads an XCD's L2 holds one head's rows
    const int g = (int)(blockIdx.x % (uint32_t)a.h_kv);
    const uint32_t rest = blockIdx.x / (uint32_t)a.h_kv;
    const int quad = (int)(rest % (uint32_t)a.layer_quads), layer = (int)(rest / (uint32_t)a.layer_quads);
    const int seq = a.one_L ? 0 : find_seq(a.cu_quad, a.n_seq, quad);
    const int64_t tok0 = a.cu_seq[seq];
    const int L = a.cu_seq[seq + 1] - a.cu_seq[seq];
    static_assert(kMaxRowTiles == kScoreWaves, "the keys of a workgroup are a quad");
    const int tile0 = (quad - a.cu_quad[seq]) * kMaxRowTiles;  // first key tile of the group

    // ---- query-row tiles: global -> LDS, laid out as key tiles are (see fetch_tile) ----
    const int64_t head0 = (int64_t)g * a.group * kHeadDim * 2, prob = layer * a.n_seq + seq;
    const char* qbase1 = (const char*)a.Q + prob * a.n_q * a.h_q * kHeadDim * 2 + head0;
    const char* qbase2 = (const char*)a.Q2 + prob * a.n_q2 * a.h_q * kHeadDim * 2 + head0;  // DIFF only
    const int n_rt = a.RP / kRowTile;
    const int n_mine = (n_rt - wv + kScoreWaves - 1) / kScoreWaves;  // this wave sweeps row tiles wv, wv + 4, ...; none of few
    const int n_first = DIFF ? min(n_mine, (a.tiles1 - wv + kScoreWaves - 1) / kScoreWaves) : 0;  // ... of them of the first set
    const uint2* aug = a.aug + prob * a.h_kv * a.RP + (int64_t)g * a.RP + (lane & 31);
    const int64_t tok_bytes = (int64_t)a.h_q * kHeadDim * 2;  // from one query token to the next
    // With a power-of-two group of up to 32 heads a tile's rows lie where a key tile's would: a lane part that never changes
    // and a uniform part per load (4 i + a, a < 4, splits without carry), so a request costs no vector arithmetic -- the
    // general addresses below cost 400 of a tile's 1800 cycles (training forward 101 -> 97.5 us, response tokens 104.5 -> 101).
    const int gs = a.group_shift;
    const bool regular = gs >= 0 && gs <= 5 && tok_bytes < (1 << 25);  // uniform; a tile's bytes fit a 32-bit offset
    const uint32_t rl = (uint32_t)lane >> 4, tok32 = (uint32_t)tok_bytes;
    const uint32_t tq = (rl >> (gs & 31)) * tok32 + (rl & (uint32_t)(a.group - 1)) * (kHeadDim * 2) + ((((uint32_t)lane & 15u) ^ rl) << 4);
    auto fetch_rows = [&](int k) __attribute__((always_inline)) {
        const int rt = wv + k * kScoreWaves;
        const bool second = DIFF && rt >= a.tiles1;  // uniform
        const char* qbase = second ? qbase2 : qbase1;
        const int rows = second ? a.rows2 : a.rows, r0 = (second ? rt - a.tiles1 : rt) * kRowTile;
        char* slot = slots + (k & 1) * kSlotBytes;
        if (regular && r0 + kRowTile <= rows) {
            const __amdgpu_buffer_rsrc_t rsrc = __builtin_amdgcn_make_buffer_rsrc(
                (void*)(qbase + (int64_t)(r0 >> gs) * tok_bytes), 0,
                (int)((uint32_t)((kRowTile - 1) >> gs) * tok32 + (uint32_t)min(a.group, kRowTile) * (kHeadDim * 2)), 0x00020000);
#pragma unroll
            for (int i = 0; i < 8; ++i)
                lds_dma16(rsrc, slot + 1024 * i, tq ^ (64u * (i & 3)), ((uint32_t)(4 * i) >> gs) * tok32 + ((uint32_t)(4 * i) & (uint32_t)(a.group - 1)) * (kHeadDim * 2));
            return;
        }
#pragma unroll
        for (int i = 0; i < 8; ++i) {
            const int r = 4 * i + (lane >> 4);
            const int row = min(r0 + r, rows - 1);  // rows past the end re-read the last one: their aug makes every term 0
            int it, hh;
            if (a.group_shift >= 0) { it = row >> a.group_shift; hh = row & (a.group - 1); }
            else { it = row / a.group; hh = row % a.group; }
            const char* src = qbase + it * tok_bytes + (int64_t)hh * (kHeadDim * 2) + (((lane & 15) ^ (r & 15)) << 4);
            __builtin_amdgcn_global_load_lds((const __attribute__((address_space(1))) void*)src,
                                             (__attribute__((address_space(3))) void*)(slot + 1024 * i), 16, 0, 0);
        }
    };

    // ---- start-up: wave wv fetches key tile wv into its second slot, its first row tile into its first ----
    const KeyStream ks = key_stream<PAGED>(a, layer, seq, tok0, L, g);
    const int last_tile = (L - 1) / kKeyTile;
    {
        const int t = min(tile0 + wv, last_tile);  // tiles past the sequence's end repeat its last one and are not stored
        const uint32_t off = tile_offset<PAGED>(ks, t, tile_page<PAGED>(ks, t));
        fetch_tile(ks.rsrc, slots + kSlotBytes, off, ks.row_bytes, tile_lane(lane, ks.row_bytes), ks.last);
    }
    fetch_rows(0);
    uint2 aug_next = aug[min(wv, n_rt - 1) * kRowTile];
    wait_tile_landed();
    bare_barrier();
    bf16x8 kf[kMaxRowTiles][8];
#pragma unroll
    for (int kt = 0; kt < kMaxRowTiles; ++kt) lds_get_frags_waited(lds_addr(&lds[kt][1][0]), kf[kt], lane);
    bare_barrier();

    u32x4 ones_bits = {0u, 0u, 0u, 0u};
    if (half == 0) { ones_bits[0] = 0x3F803F80u; ones_bits[1] = 0x00003F80u; }  // 1.0 at elements 0..2
    const bf16x8 ones = as_bf16x8(ones_bits);
    const float c = a.c;
    float sum[kMaxRowTiles], sum1[kMaxRowTiles];  // sum1: DIFF, the first set's
#pragma unroll
    for (int kt = 0; kt < kMaxRowTiles; ++kt) sum[kt] = sum1[kt] = 0.f;
    auto next_set = [&]() __attribute__((always_inline)) {
#pragma unroll
        for (int kt = 0; kt < kMaxRowTiles; ++kt) { sum1[kt] = sum[kt]; sum[kt] = 0.f; }
    };
    // as in the other sweeps: the next key tile's MFMA chain runs between the exp2 work of this one, and behind the last
    // one the first chain of the next row tile, read a stage earlier
    auto aug_of = [&](uint2 t) __attribute__((always_inline)) {
        u32x4 av = {0u, 0u, 0u, 0u};
        if (half == 0) { av[0] = t.x; av[1] = t.y; }
        return as_bf16x8(av);
    };
    bf16x8 qf[8];
    lds_get_frags(slots, qf, lane);
    bf16x8 qaug = aug_of(aug_next);
    wait_frags_read();
    if (n_mine > 1) {
        fetch_rows(1);
        aug_next = aug[(wv + kScoreWaves) * kRowTile];
    }
    f32x16 acc = score_chain(qf, qaug, kf[0], ones);
    for (int k = 0; k < n_mine; ++k) {
        if (DIFF && k == n_first) next_set();
#pragma unroll
        for (int kt = 0; kt < kMaxRowTiles; ++kt) {
            const bool reads = kt == kMaxRowTiles - 2;
            const char* next_slot = slots + ((k + 1) & 1) * kSlotBytes;
            if (reads) wait_tile_landed();
            const uint32_t next_at = frag_addr(next_slot, lane);
            f32x16 nxt = zero_acc();
            sum[kt] += exp2_sum_stage<9>(
                [&](int i) __attribute__((always_inline)) {
                    nxt = i < 8 ? mfma_bf16(qf[i & 7], kf[(kt + 1) % kMaxRowTiles][i & 7], nxt) : mfma_bf16(qaug, ones, nxt);
                    pin(nxt);
                    if (reads && i < 8) qf[i & 7] = lds_get_frag(next_at, i);  // its last use was this MFMA
                },
                [&](int v) __attribute__((always_inline)) { return acc[v] * c; });
            if (reads) {
                wait_frags_read();
                qaug = aug_of(aug_next);
                if (k + 2 < n_mine) {
                    fetch_rows(k + 2);
                    aug_next = aug[(wv + (k + 2) * kScoreWaves) * kRowTile];
                }
            }
            acc = nxt;
        }
    }
    if (DIFF && n_first == n_mine) next_set();  // a wave with tiles of the first set alone
    clear_words(a);
    constexpr int kKeys = kMaxRowTiles * kKeyTile;
#pragma unroll
    for (int kt = 0; kt < kMaxRowTiles; ++kt) {
        sum[kt] += __shfl_xor(sum[kt], 32);  // the two lane halves hold complementary query rows of the same key
        if (DIFF) sum1[kt] += __shfl_xor(sum1[kt], 32);
        if (half == 0) {  // the wave's slots are idle by now
            ((float*)slots)[kt * kKeyTile + lane] = sum[kt];
            if (DIFF) ((float*)slots)[kKeys + kt * kKeyTile + lane] = sum1[kt];
        }
    }
    __syncthreads();
    const int key = tile0 * kKeyTile + (int)threadIdx.x;  // threads 0..127: one key each
    double dacc = 0.0;
    if (threadIdx.x < kKeys && key < L) {
        float v = 0.f, v1 = 0.f;
#pragma unroll
        for (int i = 0; i < kScoreWaves; ++i) {
            v += ((const float*)&lds[i][0][0])[threadIdx.x];
            if (DIFF) v1 += ((const float*)&lds[i][0][0])[kKeys + threadIdx.x];
        }
        if (DIFF) {
            const double d = (double)v1 * (double)a.inv_rows1 - (double)v * (double)a.inv_rows2;
            dacc = d * d;
        } else {
            if (a.window && key >= L - a.n_q) v = 0.f;  // the window's own positions report 0
            a.scores[((int64_t)layer * a.h_kv + g) * a.T + tok0 + key] = v;
        }
    }
    if constexpr (DIFF) {  // butterfly within waves 0 and 1, then their two sums: a fixed order
#pragma unroll
        for (int off = 32; off >= 1; off >>= 1) dacc += __shfl_xor(dacc, off);
        if (lane == 0 && wv < 2) diff_s[wv] = dacc;
        __syncthreads();
        if (threadIdx.x == 0) a.diff_part[((int64_t)layer * a.layer_quads + quad) * a.h_kv + g] = diff_s[0] + diff_s[1];
    }
}

// Supplied normalisers with many query rows: lse -> the bf16 terms of -beta/c (as jq_score_kernel<FROM_LSE>
// does it per wave), one thread per row, and the words that the selection needs cleared.
__global__ __launch_bounds__(256) void jq_lse_aug_kernel(ScoreArgs a, int64_t n) {
    const int64_t stride = (int64_t)gridDim.x * blockDim.x;
    for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < n; i += stride) {
        const int row = (int)(i % a.RP);
        const int64_t rest = i / a.RP;
        const int g = (int)(rest % a.h_kv);
        const int64_t ls = rest / a.h_kv;  // layer * n_seq + sequence
        const int rowc = min(row, a.rows - 1);
        const float x = a.lse[(ls * a.n_q + rowc / a.group) * a.h_q + (int64_t)g * a.group + rowc % a.group];
        a.aug[i] = split_bf16x3(row < a.rows ? (float)(-(double)x * a.inv_scale) : kPadTerm);
    }
    if (a.zero)
        for (uint64_t i = (uint64_t)blockIdx.x * blockDim.x + threadIdx.x; i < a.zero_words; i += (uint64_t)stride) a.zero[i] = 0u;
}

// ------------------------------------------------------------------------------------------------
// host side
// ------------------------------------------------------------------------------------------------
template <bool PAGED>
static hipError_t launch_stats_n(int nqt, const ScoreArgs& a, dim3 grid, hipStream_t st, void* const* marks) {
    dim3 block(kScoreWaves * 64);
    switch (nqt) {
        case 1: return launch_kernel(jq_stats_kernel<1, PAGED>, grid, block, 0, st, marks, kTrStats, a);
        case 2: return launch_kernel(jq_stats_kernel<2, PAGED>, grid, block, 0, st, marks, kTrStats, a);
        case 3: return launch_kernel(jq_stats_kernel<3, PAGED>, grid, block, 0, st, marks, kTrStats, a);
        default: return launch_kernel(jq_stats_kernel<4, PAGED>, grid, block, 0, st, marks, kTrStats, a);
    }
}

// The kernel that holds scores back where the call wants it and the device grants the LDS they take, else the other one.
template <int NQT, bool FROM_LSE, bool PAGED>
static hipError_t launch_score_k(const ScoreArgs& a, dim3 grid, hipStream_t st, void* const* marks) {
    static std::atomic<uint64_t> allowed;
    const dim3 block(kScoreWaves * 64);
    const auto holding = jq_score_kernel<NQT, FROM_LSE, PAGED, true>;
    constexpr int lds_bytes = kScoreWaves * kHeldScore * kHeldTile;
    if (a.holds && allow_dynamic_lds((const void*)holding, lds_bytes, allowed) == hipSuccess)
        return launch_kernel(holding, grid, block, (size_t)lds_bytes, st, marks, kTrScore, a);
    return launch_kernel(jq_score_kernel<NQT, FROM_LSE, PAGED, false>, grid, block, 0, st, marks, kTrScore, a);
}
template <bool FROM_LSE, bool PAGED>
static hipError_t launch_score_n(int nqt, const ScoreArgs& a, dim3 grid, hipStream_t st, void* const* marks) {
    switch (nqt) {
        case 1: return launch_score_k<1, FROM_LSE, PAGED>(a, grid, st, marks);
        case 2: return launch_score_k<2, FROM_LSE, PAGED>(a, grid, st, marks);
        case 3: return launch_score_k<3, FROM_LSE, PAGED>(a, grid, st, marks);
        default: return launch_score_k<4, FROM_LSE, PAGED>(a, grid, st, marks);
    }
}

template <int NQT, bool PAGED>
static hipError_t launch_passes_k(const ScoreArgs& a, dim3 grid, hipStream_t st) {
    const dim3 block(kScoreWaves * 64);
    if (a.holds) return launch_kernel(jq_passes_kernel<NQT, PAGED, true>, grid, block, 0, st, nullptr, -1, a);
    return launch_kernel(jq_passes_kernel<NQT, PAGED, false>, grid, block, 0, st, nullptr, -1, a);
}
template <bool PAGED>
static hipError_t launch_passes_n(int nqt, const ScoreArgs& a, dim3 grid, hipStream_t st) {
    switch (nqt) {
        case 1: return launch_passes_k<1, PAGED>(a, grid, st);
        case 2: return launch_passes_k<2, PAGED>(a, grid, st);
        case 3: return launch_passes_k<3, PAGED>(a, grid, st);
        default: return launch_passes_k<4, PAGED>(a, grid, st);
    }
}

// Workgroups of jq_passes_kernel that run at the same time on the present device: one per CU.
static int resident_passes() {
    constexpr int kDevices = 64;
    static std::atomic<int> cus[kDevices];
    int dev = 0;
    if (hipGetDevice(&dev) != hipSuccess || dev < 0 || dev >= kDevices) return 0;
    int n = cus[dev].load(std::memory_order_relaxed);
    if (n == 0) {
        if (hipDeviceGetAttribute(&n, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess) return 0;
        cus[dev].store(n, std::memory_order_relaxed);
    }
    return n;
}

// A value that no flag holds by chance (2^-64): every call's is another one.
static uint64_t next_token() {
    static std::atomic<uint64_t> count{[]() -> uint64_t {
        try {
            std::random_device rd;
            return ((uint64_t)rd() << 32) ^ (uint64_t)rd();
        } catch (...) {  // no source of random numbers: the time, in nanoseconds, which no earlier process had either
            return (uint64_t)std::chrono::system_clock::now().time_since_epoch().count();
        }
    }()};
    uint64_t x = count.fetch_add(0x9E3779B97F4A7C15ull, std::memory_order_relaxed);  // splitmix64 (Steele, Lea, Flood 2014): a bijection of the count
    x = (x ^ (x >> 30)) * 0xBF58476D1CE4E5B9ull;
    x = (x ^ (x >> 27)) * 0x94D049BB133111EBull;
    return x ^ (x >> 31);
}

hipError_t launch_score(const Plan& p, const void* Q, const void* K, float* scores, char* ws, hipStream_t st,
                        uint32_t* zero, size_t zero_words, const float* lse, const void* k_tail, const void* Q2, double* diff_part,
                        bool flags_cleared_later) {
    void* const* marks = p.marks;
    ScoreArgs a;
    a.Q = (const uint16_t*)Q;
    a.K = (const uint16_t*)K;
    a.K_tail = (const uint16_t*)k_tail;
    a.stats = (float2*)(ws + p.off_stats);
    a.aug = (uint2*)(ws + p.off_aug);
    a.scores = scores;
    a.n_layers = p.n_layers; a.n_seq = p.n_seq; a.n_q = p.n_q; a.h_q = p.h_q; a.h_kv = p.h_kv;
    a.group = p.group; a.rows = p.rows; a.RP = p.row_tiles * kRowTile;
    a.window = p.window;
    a.group_shift = -1;
    for (int sh = 0; sh < 16; ++sh)
        if (p.group == (1 << sh)) a.group_shift = sh;
    a.n_rg = 1; a.rg0 = 0;
    a.c = (float)(p.scale * 1.4426950408889634074);
    a.inv_scale = 1.0 / p.scale;
    a.inv_c = 1.0 / (double)a.c;
    a.T = p.T;
    a.zero = zero; a.zero_words = zero_words;
    a.block_table = p.block_table; a.page_shift = p.page_shift; a.n_pages = p.n_pages; a.max_pages = p.max_pages;
    a.Q2 = (const uint16_t*)Q2; a.diff_part = diff_part;
    a.n_q2 = p.n_q2; a.rows2 = p.rows2; a.tiles1 = p.n_q2 ? p.row_tiles1 : kOneSet;
    a.inv_rows1 = 1.0f / (float)p.rows; a.inv_rows2 = p.n_q2 ? 1.0f / (float)p.rows2 : 0.0f;
    const bool paged = p.block_table != nullptr;
    if ((diff_part != nullptr) != (p.n_q2 != 0) || (diff_part && (paged || lse))) return hipErrorInvalidValue;  // two sets: dense two-pass calls
    a.one_L = p.n_seq == 1 ? p.tab.cu_seq[1] : 0;
    a.layer_quads = p.cu_quad[p.n_seq];
    for (int s = 0; s <= p.n_seq; ++s) { a.cu_seq[s] = p.tab.cu_seq[s]; a.cu_quad[s] = p.cu_quad[s]; }
    auto share_out = [&](const Split& from, SplitArgs& to, int32_t* cu) {
        to = from.args;
        for (int s = 0; s <= p.n_seq; ++s) cu[s] = from.cu[s];
    };
    share_out(p.split, a.own, a.cu_wg);
    a.inv_h_kv = inverse(p.h_kv);
    a.lse = lse;
    a.part = a.own; a.fuse_combine = 0;
    a.flags = nullptr; a.token = 0; a.wait_ticks = 0; a.n_sets = p.split.n_sets;
    a.holds = 0;
    // Scores are held back where the pass that makes them reads much of K from memory: 1.6 % of its bytes, they cost a tenth of its
    // time when they are written between the reads (a build that stored none took 44.2 us for the pass of 4 x 32768, 51.2 with stores after
    // every tile, 45.4 held back), and next to nothing while the Infinity Cache (256 MB) delivers K.  Written at the end they take
    // 0.5 us of a short call.  Whole calls, stored at once / held back, 8 KV heads, us:
    //   one pass (normalisers supplied) alone or with the one-kernel tail: 30000 tokens 27.7 / 28.0, 2 x 32768 42.6 / 41.1, 4 x 25000 59.9 / 57.2,
    //     4 x 32768 71.5 / 66.9, 16 x 16384 137.4 / 128.0, 8 x 32768 131.2 / 119.5;
    //   one pass and a tail of two kernels (`zero`: the second one's histograms): 80000 tokens 48.4 / 45.9, 120000 64.4 / 62.0, 131072 69.0 / 64.5,
    //     250000 124.8 / 116.9, 400000 201.4 / 184.6, 8 x 65536 244 / 223 -- but up to some 400 MB that depends on the card: on 4 of 21 cards calls
    //     one after the other lose instead, on the worst 80000 53.9 / 56.8, 120000 68.4 / 78.6, 131072 73.5 / 78.4, 2 x 60000 70.0 / 78.9,
    //     200000 109.3 / 114.4, 250000 131.3 / 131.5, 400000 210.5 / 206.8, 8 x 65536 244 / 227; on 4 more nothing is gained up to 131072.
    //     The number of tiles held, the kind of stores and the shader clock make no difference.  No such call holds back below;
    //   the first group on such a card, two runs: alone 2 x 32768 34.4 / 34.8 and 34.7 / 35.3, 4 x 25000 43.1 / 41.1 and 42.9 / 40.8, 4 x 32768 54.4 / 51.2
    //     and 54.1 / 51.5; with the one-kernel tail 2 x 32768 44.7 / 43.4 and 46.2 / 45.4, 4 x 25000 59.3 / 59.8 and 60.5 / 61.6, 4 x 32768 73.8 / 70.5 and
    //     75.1 / 74.9, 8 x 16384 74.1 / 73.5 and 75.1 / 78.8, 16 x 16384 137.4 / 131.5 and 137.7 / 131.6, 8 x 32768 131.6 / 120.1 and 132.3 / 125.3: 3 %
    //     less on average there too, 5 % more at worst;
    //   two passes: 131072 110.2 / 110.9, 28 x 8192 219.6 / 221.1, 4 x 50000 164.7 / 165.4, 250000 203.2 / 197.7, 4 x 60000 paged 209 / 206, 32 x 8192
    //     233.8 / 230.4, 8 x 65536 402 / 387, 16 ragged sequences of 981293 together 751 / 735.
    const int64_t k_bytes = (int64_t)p.n_layers * p.T * p.h_kv * kHeadDim * 2;
    const bool holds = k_bytes >= (knobs().hold_bytes >= 0 ? knobs().hold_bytes : lse && !zero ? (int64_t)110000000 : (int64_t)480000000);
    const dim3 block(kScoreWaves * 64);
    const unsigned wgs = (unsigned)(p.split.n_wg * p.h_kv);
    hipError_t e;
    if (!lse && p.one_launch && flags_cleared_later && !marks && wgs <= (unsigned)resident_passes()) {
        a.flags = (uint64_t*)(ws + p.off_flags);
        a.token = next_token();
        a.wait_ticks = (int64_t)knobs().wait_us * 100;
        a.holds = holds;
        const int nqt = p.row_tiles;
        return paged ? launch_passes_n<true>(nqt, a, dim3(wgs), st) : launch_passes_n<false>(nqt, a, dim3(wgs), st);
    }
    if (!lse) {
        const int nqt = min(p.row_tiles, kMaxRowTiles);
        // all row groups in one launch (in several where the grid would get too large for one)
        const int per_launch = (int)max((int64_t)1, min((int64_t)p.row_groups, ((int64_t)1 << 23) / wgs));
        // Many query rows: the sets are merged by the workgroup that completes them.  Its flags lie in the selection's histograms, which
        // the next launch clears.
        const size_t n_flags = (size_t)p.split.n_sets * p.h_kv * p.row_groups;
        const bool last_merges = p.by_rows && per_launch >= p.row_groups && p.split.max_sets <= kMergedSets &&
                                 n_flags * sizeof(uint64_t) <= p.off_scores - p.off_hist && (!zero || (char*)zero == ws + p.off_hist);
        if (last_merges) {
            a.flags = (uint64_t*)(ws + p.off_hist);
            a.token = next_token();
        }
        for (a.rg0 = 0; a.rg0 < p.row_groups; a.rg0 += per_launch) {
            a.n_rg = min(per_launch, p.row_groups - a.rg0);
            const dim3 g1(wgs * a.n_rg);
            e = paged ? launch_stats_n<true>(nqt, a, g1, st, marks) : launch_stats_n<false>(nqt, a, g1, st, marks);
            if (e != hipSuccess) return e;
        }
        a.n_rg = 1; a.rg0 = 0;
        // Pass 1 leaves one set of statistics per share.  With few of them per sequence every pass-2 workgroup merges
        // its head's sets itself; a very long sequence has hundreds, and then one small launch merges them
        // once (and clears the selection's words on the way).
        share_out(p.split, a.part, a.cu_part);
        a.fuse_combine = p.split.max_sets <= kMergedSets && !p.by_rows;
        if (last_merges) {
            a.flags = nullptr;
            a.zero = (uint32_t*)(ws + p.off_hist);
            a.zero_words = std::max<uint64_t>(zero ? zero_words : 0, 2 * n_flags);
        } else if (!a.fuse_combine) {
            const int64_t n_row_tiles = (int64_t)p.n_layers * p.n_seq * p.h_kv * p.row_tiles;
            e = launch_kernel(jq_combine_kernel, dim3((unsigned)min(n_row_tiles, (int64_t)1 << 20)), dim3(kRowTile * kCombineLanes), 0, st, nullptr, -1, a);
            if (e != hipSuccess) return e;
            a.zero = nullptr;  // done by the combine launch
        }
    }
    if (p.by_rows) {  // more query rows per KV head than a wave holds, or two sets of them
        if (lse) {  // the -beta/c terms, which a combine launch provides otherwise
            const int64_t n = (int64_t)p.n_layers * p.n_seq * p.h_kv * a.RP;
            e = launch_kernel(jq_lse_aug_kernel, dim3((unsigned)min((n + 255) / 256, (int64_t)2048)), dim3(256), 0, st, nullptr, -1, a, n);
            if (e != hipSuccess) return e;
            a.zero = nullptr;  // done by that launch
        }
        const dim3 grid((unsigned)((int64_t)p.n_layers * a.layer_quads * p.h_kv));
        if (diff_part) return launch_kernel(jq_score_rows_kernel<false, true>, grid, block, 0, st, nullptr, -1, a);
        if (paged) return launch_kernel(jq_score_rows_kernel<true, false>, grid, block, 0, st, marks, kTrScore, a);
        return launch_kernel(jq_score_rows_kernel<false, false>, grid, block, 0, st, marks, kTrScore, a);
    }
    // The second pass may share the keys out in its own way; alone, it has no statistics that would have to be merged.
    const bool wider = lse && p.split.fewer;
    Split alone;
    if (wider) {
        int32_t max_quads = 0;
        for (int s = 0; s < p.n_seq; ++s) max_quads = std::max(max_quads, p.cu_quad[s + 1] - p.cu_quad[s]);
        alone = make_split(p, 0, max_quads, false, false);
    }
    const Split& own = wider ? alone : lse ? p.split : p.split2;
    share_out(own, a.own, a.cu_wg);
    const dim3 grid((unsigned)(own.n_wg * p.h_kv));
    a.holds = holds;
    if (paged) return lse ? launch_score_n<true, true>(p.row_tiles, a, grid, st, marks) : launch_score_n<false, true>(p.row_tiles, a, grid, st, marks);
    return lse ? launch_score_n<true, false>(p.row_tiles, a, grid, st, marks) : launch_score_n<false, false>(p.row_tiles, a, grid, st, marks);
}

}  // namespace jq
