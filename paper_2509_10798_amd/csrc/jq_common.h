// Internal declarations shared by the HIP sources of libjq (gfx950 only).
#pragma once

#include <hip/hip_runtime.h>
#include <hip/hip_ext.h>
#include <stddef.h>
#include <stdint.h>

#include <atomic>

#include "jq_sweep.h"

namespace jq {

constexpr int kMaxRowTiles = 4;     // query-row tiles one wave keeps in registers (128 rows)
constexpr int kHistBins = 2048;     // level-1 radix bins (top 11 bits of the sortable key)
constexpr int kHistStride = kHistBins + 16;  // per problem: the bins, then [0] #sure and [1] #candidate counters
constexpr int kSelectThreads = 1024;
constexpr int kSegLen = 1024;       // positions per pooling workgroup = entries per segment of the selection's sorted lists

// Per-call sequence table, passed to kernels by value (about 1 KiB of kernarg).
struct SeqTab {
    int32_t n_seq;
    int32_t cu_seq[JQ_MAX_SEQ + 1];    // token offsets
    int32_t cu_bud[JQ_MAX_SEQ + 1];    // kept-row offsets
};

// Where a layer's K / V rows live: dense [T] rows per layer (block_table null), or a pool of n_pages pages of
// 1 << page_shift rows per layer with a per-sequence block table.
struct PageMap {
    const int32_t* block_table;  // DEVICE [n_seq][max_pages], or null
    int32_t page_shift, n_pages, max_pages;
};

// Everything the host derives from a jq_shape.
struct Plan {
    int32_t n_layers, n_seq, n_q, h_q, h_kv, d, group, pool_k;
    int32_t keep_first, keep_last;  // positions at either end of a sequence that the selection always keeps
    int32_t window;                 // 1: the queries are the last n_q tokens of every sequence (causal inside them)
    const int32_t* layer_budgets;   // DEVICE [n_layers][n_seq] or null: per-layer budgets (tab.cu_bud then holds the largest)
    int32_t rows;         // n_q * group: query rows that share one KV head
    int32_t n_q2, rows2;  // second query set of the call (jq_map_mse_fused): its tokens and rows, 0 elsewhere
    int32_t row_tiles1;   // ceil(rows / 32)
    int32_t row_tiles;    // ... and those of the second set, which follow
    int32_t row_groups;   // ceil(row_tiles / 4): 1, or the groups of rows that the first pass handles side by side
    bool by_rows;         // the second pass streams query rows past keys held in registers (jq_score_rows_kernel)
    Split split, split2;  // the first pass over K (or the only one), and a second launch's
    bool one_launch;      // both passes may go in one launch (jq_passes_kernel): a workgroup per CU at most, room for the flags
    int32_t cu_quad[JQ_MAX_SEQ + 1];  // groups of 128 keys per sequence
    double scale;         // logit scale actually used
    // paged cache (block_table null: dense K, V): page = 1 << page_shift tokens, n_pages per layer's pool
    const int32_t* block_table;  // DEVICE [n_seq][max_pages]
    int32_t page_shift, n_pages, max_pages;
    int64_t T, TB;
    SeqTab tab;
    // pooling workgroups ("segments") per layer and head: ceil(L_s / kSegLen) per sequence, never across sequences
    int32_t n_seg;
    int32_t cu_seg[JQ_MAX_SEQ + 1];
    int32_t seg_head;  // room per segment in the selection's lists: the most entries that a sequence's segments keep (seg_head_of)
    PageMap page_map() const { return PageMap{block_table, page_shift, n_pages, max_pages}; }
    PageMap out_map;      // where the pruned cache goes (block_table null: dense [n_layers][TB] rows)
    void* const* marks;   // host only: nullptr, or 2 * kTraceKernels events (start, stop) for jq_evict_traced
    // workspace layout (byte offsets, 256-aligned)
    size_t off_stats, off_flags, off_aug, off_hist, off_scores, off_pooled, off_idx, off_seg, off_seghdr, ws_bytes;
};

// Entries that a segment of the selection's lists keeps: eight times what a block of kSegLen scores contributes to its sequence's
// kept set on average, as a power of two in 128..kSegLen; blocks that hold more are re-read from the scores by the selection.
__host__ __device__ inline int32_t seg_head_of(int32_t B, int32_t L) {
    int32_t head = 128;
    while (head < kSegLen && (int64_t)head * L < (int64_t)8 * kSegLen * B) head *= 2;
    return head;
}

// Order-preserving map from fp32 to uint32 (larger float <=> larger key); -0 is folded onto +0.
__device__ inline uint32_t sortable_key(float x) {
    uint32_t b = __float_as_uint(x + 0.0f);
    return (b & 0x80000000u) ? ~b : (b | 0x80000000u);
}

// A block-table entry as every kernel uses it: entries outside the pool (a corrupt table, the -1 of an unused slot)
// are clamped into it, so that the scored keys and the gathered rows always come from the same page.
__host__ __device__ inline int32_t clamp_page(int32_t entry, int32_t n_pages) {
    return entry < 0 ? 0 : (entry > n_pages - 1 ? n_pages - 1 : entry);
}

// Row (in units of token rows, over all layers) of token `pos` of sequence `s`; `cu` holds the sequences' dense
// offsets (token offsets for the cache, kept-row offsets for the pruned cache) and T their total.
__device__ inline int64_t kv_row(const PageMap& pm, const int32_t* cu, int64_t T, int layer, int s, int pos) {
    if (!pm.block_table) return (int64_t)layer * T + cu[s] + pos;
    const int32_t e = pm.block_table[(int64_t)s * pm.max_pages + (pos >> pm.page_shift)];
    const int64_t page = (int64_t)layer * pm.n_pages + clamp_page(e, pm.n_pages);
    return (page << pm.page_shift) + (pos & ((1 << pm.page_shift) - 1));
}

// In-place eviction: is the row that holds token `pos` of sequence `s` (row `src_row` of its layer when dense)
// among the rows the call overwrites?  Dense: the front TB rows of the layer.  Paged into the input's own pool:
// any row of a page that the output table names (`dest_bits`: one bit per page of the pool).
__device__ inline bool row_is_overwritten(const PageMap& pm, const uint32_t* dest_bits, int64_t src_row_dense, int64_t TB, int s,
                                          int pos) {
    if (!pm.block_table) return src_row_dense < TB;
    const int32_t e = clamp_page(pm.block_table[(int64_t)s * pm.max_pages + (pos >> pm.page_shift)], pm.n_pages);
    return (dest_bits[e >> 5] >> (e & 31)) & 1u;
}

// The same with the sequence's first dense row (`cu[s]` of kv_row) already looked up.
__device__ inline int64_t kv_row_from(const PageMap& pm, int64_t seq_row0, int64_t T, int layer, int s, int pos) {
    if (!pm.block_table) return (int64_t)layer * T + seq_row0 + pos;
    const int32_t e = pm.block_table[(int64_t)s * pm.max_pages + (pos >> pm.page_shift)];
    const int64_t page = (int64_t)layer * pm.n_pages + clamp_page(e, pm.n_pages);
    return (page << pm.page_shift) + (pos & ((1 << pm.page_shift) - 1));
}

// Budget of (layer, sequence): the table's segment length, or the caller's per-layer value clamped into
// max(1, forced) .. that, where `forced` = keep_first + keep_last is the number of positions that are kept whatever
// they score (the host has checked forced <= segment length; it cannot see the per-layer values).
__device__ inline uint32_t budget_of(const int32_t* layer_budgets, const SeqTab& tab, int layer, int s, int forced) {
    const int32_t cap = tab.cu_bud[s + 1] - tab.cu_bud[s];
    if (!layer_budgets) return (uint32_t)cap;
    return (uint32_t)min(max(layer_budgets[(int64_t)layer * tab.n_seq + s], max(forced, 1)), cap);
}

// Key the top-B selection ranks position j of an L-token sequence by: always-kept positions outrank
// every score.
__device__ inline uint32_t select_key(float x, int j, int L, int keep_first, int keep_last) {
    return (j < keep_first || j >= L - keep_last) ? 0xFFFFFFFFu : sortable_key(x);
}

// Ablation and diagnosis knobs, read from the environment ONCE per process (first use) -- no entry point touches the
// environment on its hot path.  jq_reload_knobs() reads them again (tests use it to force rarely taken paths).
struct Knobs {
    int32_t chunk_keys;   // JQ_CHUNK_KEYS: keys per wave in the pass that reads K cold, in whole workgroups per sequence (0: planned)
    int32_t chunk_keys2;  // JQ_CHUNK_KEYS_2: the same for the second pass (0: JQ_CHUNK_KEYS if set, else planned)
    int32_t wait_us;      // JQ_WAIT_US: how long a workgroup waits, once, for others' statistics before it forms them itself (microseconds)
    int64_t hold_bytes;   // JQ_HOLD_BYTES: bytes of K from which on the second pass holds its scores back (-1: as measured, see launch_score)
    int32_t log;          // JQ_LOG: print the HIP error string when a launch is refused
};
const Knobs& knobs();

// Stores of a kernel's bulk OUTPUT (pooled scores, block heads, kept positions and rows): nothing in the same
// kernel reads them back, the next kernel does.  Left in L2 as dirty lines they are written back when the kernel
// ends, and the next kernel cannot start before that: the gap between two dependent kernels grows with what the
// first one wrote (2.45 / 2.98 / 3.32 us after 4 / 16 / 64 MB, whatever the second kernel's shape).  Stored
// non-temporally they are on their way out while the kernel still runs.  Measured with the builds side by side in
// one process: kept rows -1.1 us per step (the next step's first kernel starts sooner), pooling's outputs -0.4 us
// more; for the second pass's scores it makes no difference, so they stay plain stores.  Agent-scope stores (sc1)
// did the same for pooling and nothing for the kept rows.
typedef uint32_t jq_u32x4 __attribute__((ext_vector_type(4)));
template <class T>
__device__ __forceinline__ void store_stream(T* p, T v) {  // T: float or int32_t
    __builtin_nontemporal_store(v, p);
}
__device__ __forceinline__ void store_stream16(void* p, uint4 v) {
    const jq_u32x4 x = {v.x, v.y, v.z, v.w};
    __builtin_nontemporal_store(x, (jq_u32x4*)p);
}
// Sixteen bytes at an address that is a multiple of four only: rows of odd lengths.  One store all the same; four of four bytes each
// touched every line of the wave's kilobyte four times (see the callers for what that cost).
typedef float any_f32x4 __attribute__((ext_vector_type(4), aligned(4)));
template <bool STREAM>
__device__ __forceinline__ void store16_any(float* p, const float* v) {
    const any_f32x4 x = {v[0], v[1], v[2], v[3]};
    if (STREAM) __builtin_nontemporal_store(x, (any_f32x4*)p);
    else *(any_f32x4*)p = x;
}

typedef const int32_t __attribute__((address_space(4))) * const_i32_ptr;
// The first lines of a kernel's arguments, which lie in memory, requested together: read where they are used, they arrive one
// after the other, up to 1 us each.
template <int LINES>
__device__ __forceinline__ void argument_lines() {
    const_i32_ptr p = (const_i32_ptr)__builtin_amdgcn_kernarg_segment_ptr();
    int32_t x[LINES];
#pragma unroll
    for (int i = 0; i < LINES; ++i) x[i] = p[16 * i];
#pragma unroll
    for (int i = 0; i < LINES; ++i) asm volatile("" ::"s"(x[i]));
}

// Workgroup barrier that orders LDS traffic only: global loads and stores that are still outstanding stay in
// flight across it (a plain __syncthreads() waits for all of them first).  For workgroups that communicate
// through LDS alone.
__device__ __forceinline__ void lds_barrier() {
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup", "local");
    __builtin_amdgcn_s_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "workgroup", "local");
}

// Wave-wide scans and reductions in the vector ALU (DPP): lane i takes the value of lane i - 1, - 2, - 4, - 8 of its row of 16,
// then whole rows take the last lane of the row, of the half before them.  Through LDS (shuffles) each of the six steps was a
// round trip of some 120 cycles in kernels that are chains of such steps.
template <int CTRL, int ROWS>
__device__ __forceinline__ uint32_t dpp_or(uint32_t otherwise, uint32_t x) {
    return (uint32_t)__builtin_amdgcn_update_dpp((int)otherwise, (int)x, CTRL, ROWS, 0xF, false);
}
template <class Op>  // lane 63 (and in ROW every lane of it) ends with everything up to it: an inclusive scan
__device__ __forceinline__ uint32_t row_scan(uint32_t x, uint32_t identity, Op op) {
    x = op(x, dpp_or<0x111, 0xF>(identity, x));
    x = op(x, dpp_or<0x112, 0xF>(identity, x));
    x = op(x, dpp_or<0x114, 0xF>(identity, x));
    return op(x, dpp_or<0x118, 0xF>(identity, x));
}
template <class Op>
__device__ __forceinline__ uint32_t wave_scan(uint32_t x, uint32_t identity, Op op) {
    x = row_scan(x, identity, op);
    x = op(x, dpp_or<0x142, 0xA>(identity, x));  // the last lane of rows 0 and 2 for rows 1 and 3
    return op(x, dpp_or<0x143, 0xC>(identity, x));  // the last lane of the lower half for the upper
}
__device__ __forceinline__ uint32_t wave_min(uint32_t x) {
    return (uint32_t)__builtin_amdgcn_readlane((int)wave_scan(x, 0xFFFFFFFFu, [](uint32_t a, uint32_t b) { return a < b ? a : b; }), 63);
}
__device__ __forceinline__ uint32_t wave_max(uint32_t x) {
    return (uint32_t)__builtin_amdgcn_readlane((int)wave_scan(x, 0u, [](uint32_t a, uint32_t b) { return a > b ? a : b; }), 63);
}

// Inclusive prefix sum over a block of THREADS threads (thread order); `tmp` (LDS) holds THREADS/64 words.  Every wave scans the
// waves' totals itself.
template <int THREADS>
__device__ __forceinline__ uint32_t block_scan_incl(uint32_t v, uint32_t* tmp, uint32_t* total) {
    constexpr int kW = THREADS / 64;
    static_assert(kW <= 16, "the totals fill a row at most");
    auto add = [](uint32_t a, uint32_t b) { return a + b; };
    const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
    const uint32_t x = wave_scan(v, 0u, add);
    lds_barrier();  // tmp may still be read from a previous call
    if (lane == 63) tmp[wave] = x;
    lds_barrier();
    const uint32_t w = row_scan(lane < kW ? tmp[lane] : 0u, 0u, add);
    *total = (uint32_t)__builtin_amdgcn_readlane((int)w, kW - 1);
    const uint32_t before = (uint32_t)__builtin_amdgcn_readlane((int)w, wave > 0 ? wave - 1 : 0);
    return x + (wave > 0 ? before : 0u);
}

// Kernels whose start/stop timestamps jq_evict_traced reports, in launch order.
enum TraceKernel { kTrStats = 0, kTrScore, kTrPool, kTrFinalize, kTraceKernels };

// Launch through hipLaunchKernel so that the status belongs to this launch alone (the sticky
// "last error" of the runtime may hold an unrelated, earlier code from the host application).
// With `marks` set, the launch carries the (start, stop) events of slot `tr`, which receive the
// dispatch's own begin/end timestamps.
template <typename Kernel, typename... Args>
inline hipError_t launch_kernel(Kernel kernel, dim3 grid, dim3 block, size_t lds_bytes, hipStream_t st,
                                void* const* marks, int tr, Args... args) {
    void* ptrs[] = {(void*)&args...};
    if (marks && tr >= 0)
        return hipExtLaunchKernel((const void*)kernel, grid, block, ptrs, lds_bytes, st, (hipEvent_t)marks[2 * tr],
                                  (hipEvent_t)marks[2 * tr + 1], 0);
    return hipLaunchKernel((const void*)kernel, grid, block, ptrs, lds_bytes, st);
}

// Launches with more than 64 KiB of dynamic LDS need the function's limit raised.  That
// is done once per device, to the fixed maximum any call can ask for (never to a call's own size: the attribute is
// process-wide, and two host threads with different sequence lengths must not undo each other's setting).
inline hipError_t allow_dynamic_lds(const void* kernel, int most, std::atomic<uint64_t>& done) {  // done, bit d: device d has the limit raised
    int dev = 0;
    hipError_t e = hipGetDevice(&dev);
    if (e != hipSuccess) return e;
    const uint64_t bit = dev < 64 ? (uint64_t)1 << dev : 0;
    if (bit && (done.load(std::memory_order_acquire) & bit)) return hipSuccess;
    e = hipFuncSetAttribute(kernel, hipFuncAttributeMaxDynamicSharedMemorySize, most);
    if (e == hipSuccess && bit) done.fetch_or(bit, std::memory_order_release);
    return e;
}

// Stage launchers (enqueue only).  Each returns a hipError_t from the launch.
// `zero_words` words at `zero` (nullable) are cleared on the way (between the two K passes).
// With `lse` (nullable, [n_layers, n_seq, n_q, h_q] natural-log normalisers) the statistics pass is skipped.
// With `k_tail` (nullable, [n_layers, n_seq, n_q, h_kv, d] bf16) the normalisers also cover those keys, causally.
// With two query sets in the plan, Q2 and `diff_part` ([n_layers][workgroups of the second pass per layer and head][h_kv]) the
// last launch stores no scores: it leaves one partial sum per workgroup of the squared differences of the sets' maps (Eq. 5
// forward, see launch_mse_reduce).
// `flags_cleared_later`: the caller launches a kernel behind this that clears the plan's flags (split.n_sets * h_kv 64-bit words at off_flags),
// so that both passes may go in one launch.
hipError_t launch_score(const Plan& p, const void* Q, const void* K, float* scores, char* ws, hipStream_t st,
                        uint32_t* zero = nullptr, size_t zero_words = 0, const float* lse = nullptr,
                        const void* k_tail = nullptr, const void* Q2 = nullptr, double* diff_part = nullptr,
                        bool flags_cleared_later = false);
// Sums the per-workgroup partials of a fused launch in workgroup order and divides by the sequence length.
hipError_t launch_mse_reduce(const Plan& p, const double* part, float* mse, hipStream_t st);
// With `hist` the pooling kernel also builds the selection's level-1 histograms, and with `ws` on top of that
// the per-workgroup sorted lists (segments) that the selection's fast path reads.
hipError_t launch_pool(const Plan& p, const float* scores, float* pooled, uint32_t* hist_or_null, char* ws_or_null,
                       hipStream_t st);
hipError_t launch_map_mse(const Plan& p, const float* scores_a, float rows_a, const float* scores_b, float rows_b,
                          float* mse, hipStream_t st);
hipError_t launch_fill_u32(uint32_t* dst, size_t n, uint32_t v, hipStream_t st);
hipError_t launch_hist(const Plan& p, const float* pooled, uint32_t* hist, char* ws_or_null, hipStream_t st);
// Whether every sequence of the plan fits the selection's fast path (LDS bitmaps); otherwise it streams.
bool select_fast_path(const Plan& p);
// Calls whose sequences all have at most kSmallMax positions: pooling (unless `pool` is false: `in` then holds the values
// to select by), selection and gather in ONE kernel, which needs no histogram and no lists.  `out` (nullable) takes the
// pooled scores; the other arguments as launch_select.  The scores of a longer sequence do not fit a workgroup's LDS.
// A selection alone always takes it (32768 values, 512 kept: 14.9 us against 35.6 for the three launches of the other way).
// An eviction weighs it against the pooling kernel followed by the selection's (evict_tail_small): every slice of a problem
// repeats pooling and selection in its one workgroup, which costs more the longer the sequence, while the lists of the other
// way cost more the more is kept.  Whole calls of one layer with 8 KV heads, keys drawn so that the kept ones stand out, one kernel / two, in us:
//   kept:          256          512          1024         2048         3072
//    2048     15.4 / 24.6
//   12000     25.2 / 28.0               25.4 / 30.7
//   16384     27.5 / 30.4               27.1 / 32.7  27.0 / 35.3
//   20000     33.6 / 32.6               33.3 / 34.5  34.3 / 36.6
//   24576     35.5 / 35.1               35.4 / 37.1  36.9 / 39.2
//   28000     38.5 / 37.2  37.8 / 37.5               39.4 / 42.6  39.9 / 45.2
//   32768     40.8 / 40.1  39.7 / 40.2  39.7 / 41.1  42.7 / 45.5  42.8 / 47.4
// and on flat scores, of which the lists of the two kernels hold many more than are kept: 16384, 512 kept 28.5 / 45.1, 32768 42.4 / 92.3, 4 layers of
// 32768 with 1024 113.5 / 160.5 -- far more than the 1 us by which two kernels are ahead where few are kept and stand out.
// 4 layers: 20000, 256 kept 73.9 / 74.3; 32768 105.0 / 106.4, 3072 kept 120.2 / 126.8; 30 layers of 32768 790 / 778.  Above 16384 positions one workgroup
// fills a CU's LDS, and more than 256 problems take turns: 32768 + 63 x 300 (512 problems) 95.8 / 91.5, 36 x 18000 586 / 575, 32 x 32768 856 / 831,
// 20000 + 35 x 500 71.3 / 67.1 -- two kernels then, except without pooling.  Up to 16384 it wins there too (48 x 9000 417 / 428, 40 x 16000 570 / 572).
// Widths 1, 5 and 7 are compiled in; any other is summed tap by tap out of LDS, for 4 to 32 positions per thread (256 kept):
//   width:        3            9            13           31           63
//    2048                               18.0 / 26.1  21.4 / 27.0  28.7 / 30.9
//    4096                               21.7 / 25.6  28.6 / 27.1  41.7 / 30.7
//    8192                  27.8 / 26.9  31.1 / 27.8  44.5 / 28.5
//   16384     29.6 / 31.0  34.5 / 31.2  37.8 / 31.6
// (Flat scores: width 31, 4096 tokens 29.6 / 32.9, 2100 tokens 29.5 / 36.4, 8 layers of 4096 46.8 / 51.2 -- one kernel up to width 31 there, and up to 9
// at 8192.)
constexpr int kSmallMax = 32768;
bool select_small(const Plan& p);
bool evict_tail_small(const Plan& p);
hipError_t launch_pool_select(const Plan& p, const float* in, float* out, bool pool, char* ws, int32_t* idx, hipStream_t st,
                              const void* K = nullptr, const void* V = nullptr, void* K_out = nullptr, void* V_out = nullptr,
                              void* stage = nullptr, const int32_t* pos_in = nullptr, int32_t* pos_out = nullptr,
                              const uint32_t* dest_bits = nullptr);
// With K, V, K_out, V_out (all or none) the selection also gathers the kept rows when its fast path runs;
// `*gathered` tells whether it did (otherwise launch_compact is still due).  With K, V and `stage` (in-place
// eviction, dense layouts, no K_out / V_out) it copies the kept rows whose sources are about to be overwritten to
// `stage` instead; launch_compact_inplace_write then finishes the job (`*gathered` false: the full
// launch_compact_inplace is due).  With pos_in / pos_out (streaming eviction: [n_layers][h_kv][T] and
// [n_layers][h_kv][TB]) every kept row's entry of pos_in is written next to its position.
hipError_t launch_select(const Plan& p, const float* pooled, uint32_t* hist, char* ws, int32_t* idx, hipStream_t st,
                         const void* K = nullptr, const void* V = nullptr, void* K_out = nullptr, void* V_out = nullptr,
                         bool* gathered = nullptr, void* stage = nullptr, const int32_t* pos_in = nullptr,
                         int32_t* pos_out = nullptr, const uint32_t* dest_bits = nullptr);
hipError_t launch_compact(const Plan& p, const void* K, const void* V, const int32_t* idx, void* K_out, void* V_out,
                          hipStream_t st);
// In place: kept rows land at the front of K / V themselves; `stage` holds 2 * n_layers * TB * h_kv rows.
hipError_t launch_compact_inplace(const Plan& p, void* K, void* V, const int32_t* idx, void* stage, hipStream_t st,
                                  const uint32_t* dest_bits = nullptr);
// Only its second launch: every kept row written, from `stage` (rows staged earlier) or from its untouched source.
// With paged K / V (p.block_table) the kept rows go where p.out_map says, inside the same pools; `dest_bits` then
// marks the pages that receive rows (one bit per page; null for the dense layout).
hipError_t launch_compact_inplace_write(const Plan& p, void* K, void* V, const int32_t* idx, void* stage, hipStream_t st,
                                        const uint32_t* dest_bits = nullptr);
// Bitmap of the pages that p.out_map's table names for kept rows (one launch; ceil(n_pages / 32) words).
hipError_t launch_mark_dest_pages(const Plan& p, uint32_t* dest_bits, hipStream_t st);

// `cu_ref_budgets`: n_seq + 1 prefix sums of the reference list lengths, `tb_ref` their total.
hipError_t launch_hit_rate(const Plan& p, const int32_t* cu_ref_budgets, int64_t tb_ref, const int32_t* cur,
                           const int32_t* ref, float* rate, hipStream_t st);
hipError_t launch_copy_probe(const void* src, void* dst, size_t bytes, hipStream_t st);

}  // namespace jq
