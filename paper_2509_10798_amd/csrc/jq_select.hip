// Top-B retention per (layer, sequence, KV head): the B best-scored key-value pairs stay, the rest is
// dropped (paper Section 4.3) -- as an exact radix select on the order-preserving 32-bit key of the
// pooled fp32 score.  Ties go to the lower position; output is ascending.
//
//   level 1: bits 31..21, histogram supplied by the pooling kernel                    -> bin b1
//   level 2: bits 20..10 of the elements in b1                                         -> bin b2
//   level 3: bits  9..0  of the elements in (b1, b2)                                   -> threshold key tau
//   result : every key > tau, plus the first (B - #greater) positions with key == tau
//
// Fast path (every sequence of the call fits the LDS bitmaps): ONE kernel after the pooling kernel, which
// has left the best elements of every 1024-position block of the scores as a "segment" of (key, position)
// pairs ordered by level-1 bin, highest first.  A workgroup picks b1 from the histogram, reads each segment
// of its problem until the bins fall below b1 (a few dozen entries per segment; a block with more qualifying
// elements than its segment holds is classified from its pooled scores instead), marks positions above b1 in
// an L-bit LDS bitmap and resolves levels 2 and 3 on the pairs inside b1 (all of them sit in one LDS list),
// marks the chosen positions, trims the tie group to its lowest positions and emits set bits in ascending
// order.  Several workgroups ("slices") work on one problem: each repeats the (cheap, cache-resident)
// resolution and emits its own range of output slots; in the fused eviction call it also gathers the K/V
// rows of those slots, so the pruned cache needs no further kernel.
// Short sequences (up to kSmallMax tokens; evict_tail_small says which calls): pooling, selection and gather in one kernel.
// General path (very long sequences): one workgroup per problem streams the row three times.
#include <atomic>

#include "jq_common.h"

namespace jq {

struct SelectArgs {
    const float* pooled;  // [n_layers][h_kv][T]
    uint32_t* hist;       // [n_layers][n_seq][h_kv][kHistStride]: level-1 bins
    const uint2* seg;     // [n_layers][h_kv][n_seg][head]  (key, position) by level-1 bin, highest first
    const uint4* seg_hdr; // [n_layers][h_kv][n_seg]  (lowest bin of the block's window, elements inside it, last slot's key, -)
    int32_t head;         // entries kept per segment (a multiple of 64)
    int32_t* idx;         // [n_layers][h_kv][TB]
    // streaming eviction: the cache rows' original positions [n_layers][h_kv][T] and where those of the kept rows
    // go [n_layers][h_kv][TB] (both null otherwise)
    const int32_t* pos_in; int32_t* pos_out;
    int32_t n_layers, h_kv;
    int32_t keep_first, keep_last;  // always-kept positions at either end of every sequence
    int32_t one_L, one_B;           // single-sequence calls: the sequence's length and budget (0 otherwise), next to
                                    // the other scalars, so that a workgroup's first kernel-argument reads do not
                                    // chain through the per-sequence tables further down
    int64_t T, TB;
    // fused gather (all four null when the kept rows are not wanted): K,V [n_layers][T][h_kv][d] bf16,
    // K_out,V_out [n_layers][TB][h_kv][d]
    const char* K; const char* V;
    char* K_out; char* V_out;
    // in-place eviction (dense layouts; K_out, V_out null): kept rows whose source lies inside the front that a later
    // kernel overwrites are copied to `stage` [2][n_layers][TB][h_kv][d] here; that kernel then writes every kept row
    char* stage;
    const uint32_t* dest_bits;  // in-place eviction inside a paged pool: the pages that receive kept rows (else null)
    PageMap pm;      // where the rows of K and V live (dense or paged)
    PageMap pm_out;  // where the kept rows go
    const int32_t* layer_budgets;  // DEVICE [n_layers][n_seq] or null
    int32_t n_seg;                   // segments per layer and head
    int32_t cu_seg[JQ_MAX_SEQ + 1];  // ... per sequence
    SeqTab tab;
};

// The thread's PER counts (c[e] = count of bin n_bins - 1 - (PER * thread + e)) in one load; `bins` is aligned to it, n_bins = PER * THREADS.
// (Word by word they were 2- to 4-way bank conflicts each: 2048 tokens 14.94 -> 14.76 us a call, 32768 41.35 -> 40.7, 8192 21.6 -> 21.3.)
template <int PER, typename BinPtr>
__device__ __forceinline__ void counts_down(BinPtr bins, int n_bins, uint32_t (&c)[PER]) {
    static_assert(PER == 1 || PER == 2 || PER == 4, "one load");
    const auto* from = bins + (n_bins - PER - PER * (int)threadIdx.x);
    if constexpr (PER == 4) {
        const uint4 v = *(const uint4*)from;
        c[0] = v.w; c[1] = v.z; c[2] = v.y; c[3] = v.x;
    } else if constexpr (PER == 2) {
        const uint2 v = *(const uint2*)from;
        c[0] = v.y; c[1] = v.x;
    } else {
        c[0] = *from;
    }
}

// bins[0..n_bins): find the bin b with (#elements in bins > b) < need <= (#elements in bins >= b).
// Thread t owns PER consecutive bins, highest bins first.  result[0] = b, result[1] = #elements above,
// result[2] = #elements inside b.  pick_bin_counts takes the thread's counts as counts_down has loaded them.
template <int THREADS, int PER>
__device__ __forceinline__ void pick_bin_counts(const uint32_t (&c)[PER], int n_bins, uint32_t need, uint32_t* tmp,
                                                uint32_t* result) {
    uint32_t sum = 0;
#pragma unroll
    for (int e = 0; e < PER; ++e) sum += c[e];
    uint32_t total;
    const uint32_t incl = block_scan_incl<THREADS>(sum, tmp, &total);
    uint32_t before = incl - sum;
#pragma unroll
    for (int e = 0; e < PER; ++e) {
        if (before < need && need <= before + c[e]) {
            result[0] = (uint32_t)(n_bins - 1 - (PER * (int)threadIdx.x + e));
            result[1] = before;
            result[2] = c[e];
        }
        before += c[e];
    }
    lds_barrier();
}

template <int THREADS, int PER, typename BinPtr>
__device__ __forceinline__ void pick_bin(BinPtr bins, int n_bins, uint32_t need, uint32_t* tmp, uint32_t* result) {
    uint32_t c[PER];
    counts_down<PER>(bins, n_bins, c);
    pick_bin_counts<THREADS, PER>(c, n_bins, need, tmp, result);
}

struct Problem {
    int layer, s, g, L;
    int tok0, bud0;  // first token row / first kept row of the sequence (dense layouts)
    uint32_t B;
    const float* x;
    int32_t* out;
    uint32_t* hist;
    const int32_t* pos_in; int32_t* pos_out;  // this problem's slices of the position tables, or null
    __device__ void emit(uint32_t slot, int row) const {
        store_stream(&out[slot], (int32_t)row);
        if (pos_out) store_stream(&pos_out[slot], pos_in[row]);
    }
};

__device__ __forceinline__ Problem problem_of(const SelectArgs& a, int prob) {
    Problem p;
    if (a.one_L) {  // one sequence: nothing to look up
        p.g = prob % a.h_kv;
        p.s = 0;
        p.layer = prob / a.h_kv;
        p.L = a.one_L;
        p.tok0 = 0; p.bud0 = 0;
        p.B = a.layer_budgets ? budget_of(a.layer_budgets, a.tab, p.layer, 0, a.keep_first + a.keep_last) : (uint32_t)a.one_B;
        p.x = a.pooled ? a.pooled + ((int64_t)p.layer * a.h_kv + p.g) * a.T : nullptr;
        p.out = a.idx + ((int64_t)p.layer * a.h_kv + p.g) * a.TB;
        p.hist = a.hist + ((int64_t)p.layer * a.h_kv + p.g) * kHistStride;
        p.pos_in = a.pos_out ? a.pos_in + ((int64_t)p.layer * a.h_kv + p.g) * a.T : nullptr;
        p.pos_out = a.pos_out ? a.pos_out + ((int64_t)p.layer * a.h_kv + p.g) * a.TB : nullptr;
        return p;
    }
    p.g = prob % a.h_kv;
    p.s = (prob / a.h_kv) % a.tab.n_seq;
    p.layer = prob / (a.h_kv * a.tab.n_seq);
    p.L = a.tab.cu_seq[p.s + 1] - a.tab.cu_seq[p.s];
    p.tok0 = a.tab.cu_seq[p.s]; p.bud0 = a.tab.cu_bud[p.s];
    p.B = budget_of(a.layer_budgets, a.tab, p.layer, p.s, a.keep_first + a.keep_last);
    p.x = a.pooled ? a.pooled + ((int64_t)p.layer * a.h_kv + p.g) * a.T + a.tab.cu_seq[p.s] : nullptr;
    p.out = a.idx + ((int64_t)p.layer * a.h_kv + p.g) * a.TB + a.tab.cu_bud[p.s];
    p.hist = a.hist + (((int64_t)p.layer * a.tab.n_seq + p.s) * a.h_kv + p.g) * kHistStride;
    p.pos_in = a.pos_out ? a.pos_in + ((int64_t)p.layer * a.h_kv + p.g) * a.T + a.tab.cu_seq[p.s] : nullptr;
    p.pos_out = a.pos_out ? a.pos_out + ((int64_t)p.layer * a.h_kv + p.g) * a.TB + a.tab.cu_bud[p.s] : nullptr;
    return p;
}

// ------------------------------------------------------------------------------------------------
// general path: one workgroup streams its row three times
// ------------------------------------------------------------------------------------------------
__global__ __launch_bounds__(kSelectThreads) void jq_select_stream_kernel(SelectArgs a) {
    __shared__ __attribute__((aligned(16))) uint32_t bins[kHistBins];
    __shared__ uint32_t tmp[kSelectThreads / 64 + 1];
    __shared__ uint32_t res[4];
    const Problem p = problem_of(a, blockIdx.x);
    const float* x = p.x;
    const int L = p.L;

    uint32_t need = p.B;
    pick_bin<kSelectThreads, 2>(p.hist, kHistBins, need, tmp, res);
    const uint32_t b1 = res[0];
    need -= res[1];
    __syncthreads();

    for (int b = threadIdx.x; b < kHistBins; b += kSelectThreads) bins[b] = 0;
    __syncthreads();
    for (int j = threadIdx.x; j < L; j += kSelectThreads) {
        const uint32_t k = select_key(x[j], j, L, a.keep_first, a.keep_last);
        if ((k >> 21) == b1) atomicAdd(&bins[(k >> 10) & 2047u], 1u);
    }
    __syncthreads();
    pick_bin<kSelectThreads, 2>(bins, 2048, need, tmp, res);
    const uint32_t prefix22 = (b1 << 11) | res[0];
    need -= res[1];
    __syncthreads();

    for (int b = threadIdx.x; b < 1024; b += kSelectThreads) bins[b] = 0;
    __syncthreads();
    for (int j = threadIdx.x; j < L; j += kSelectThreads) {
        const uint32_t k = select_key(x[j], j, L, a.keep_first, a.keep_last);
        if ((k >> 10) == prefix22) atomicAdd(&bins[k & 1023u], 1u);
    }
    __syncthreads();
    pick_bin<kSelectThreads, 1>(bins, 1024, need, tmp, res);
    const uint32_t tau = (prefix22 << 10) | res[0];
    need -= res[1];  // how many elements equal to tau are kept
    __syncthreads();

    // ordered compaction: each thread takes 4 consecutive positions per round
    uint32_t gt_done = 0, eq_done = 0;
    for (int base = 0; base < L; base += kSelectThreads * 4) {
        const int j0 = base + threadIdx.x * 4;
        uint32_t kk[4];
        uint32_t n_gt = 0, n_eq = 0;
#pragma unroll
        for (int e = 0; e < 4; ++e) {
            kk[e] = (j0 + e < L) ? select_key(x[j0 + e], j0 + e, L, a.keep_first, a.keep_last) : 0u;
            n_gt += (j0 + e < L) && kk[e] > tau;
            n_eq += (j0 + e < L) && kk[e] == tau;
        }
        uint32_t total;
        const uint32_t packed = n_gt | (n_eq << 16);  // at most 4096 per field and round
        const uint32_t incl = block_scan_incl<kSelectThreads>(packed, tmp, &total);
        uint32_t gt_before = gt_done + ((incl - packed) & 0xFFFFu);
        uint32_t eq_before = eq_done + ((incl - packed) >> 16);
#pragma unroll
        for (int e = 0; e < 4; ++e) {
            if (j0 + e >= L) break;
            const bool is_gt = kk[e] > tau, is_eq = kk[e] == tau;
            if (is_gt || (is_eq && eq_before < need)) {
                const uint32_t slot = gt_before + min(eq_before, need);
                if (slot < p.B) p.emit(slot, j0 + e);  // always true for consistent histograms
            }
            gt_before += is_gt;
            eq_before += is_eq;
        }
        gt_done += total & 0xFFFFu;
        eq_done += total >> 16;
        if (gt_done + min(eq_done, need) >= p.B) break;  // uniform: everything kept already
    }
}

// Pruned cache (paper Section 4.3): the kept rows of output slots o0 .. o0 + n_rows - 1 of a problem, whose positions are
// in slot_pos[0 .. n_rows - 1] (LDS); 16 lanes x 16 B per 256-byte head row.  Every thread takes kGatherRows rows at a time,
// so that that many K and V loads are in flight together: one pair per thread left a workgroup with 1024 rows to gather
// waiting for 32 round trips to memory.
constexpr int kGatherRows = 4;
template <int THREADS>
__device__ __forceinline__ void gather_slots(const SelectArgs& a, const Problem& p, const uint32_t* slot_pos, uint32_t o0, uint32_t n_rows) {
    const int part = threadIdx.x & 15;
    constexpr uint32_t kStep = THREADS / 16;
    if (a.stage) {  // uniform
        const int64_t v_stage = (int64_t)a.n_layers * a.TB * a.h_kv * (kHeadDim * 2);
        for (uint32_t rr = threadIdx.x >> 4; rr < n_rows; rr += kStep) {
            const int64_t src_row = (int64_t)p.tok0 + slot_pos[rr];  // within the layer (dense layout)
            if (!row_is_overwritten(a.pm, a.dest_bits, src_row, a.TB, p.s, (int)slot_pos[rr])) continue;  // read in place later
            const int64_t src = ((kv_row_from(a.pm, p.tok0, a.T, p.layer, p.s, (int)slot_pos[rr]) * a.h_kv + p.g) * kHeadDim) * 2 + part * 16;
            const int64_t stg = ((((int64_t)p.layer * a.TB + p.bud0 + o0 + rr) * a.h_kv + p.g) * kHeadDim) * 2 + part * 16;
            *(uint4*)(a.stage + stg) = *(const uint4*)(a.K + src);
            *(uint4*)(a.stage + v_stage + stg) = *(const uint4*)(a.V + src);
        }
        return;
    }
    for (uint32_t r0 = threadIdx.x >> 4; r0 < n_rows; r0 += kGatherRows * kStep) {
        uint4 kv[kGatherRows], vv[kGatherRows];
#pragma unroll
        for (int u = 0; u < kGatherRows; ++u) {
            const uint32_t rr = min(r0 + u * kStep, n_rows - 1);  // past the end: the last row again, not stored
            const int64_t src = ((kv_row_from(a.pm, p.tok0, a.T, p.layer, p.s, (int)slot_pos[rr]) * a.h_kv + p.g) * kHeadDim) * 2 + part * 16;
            kv[u] = *(const uint4*)(a.K + src);
            vv[u] = *(const uint4*)(a.V + src);
        }
#pragma unroll
        for (int u = 0; u < kGatherRows; ++u) {
            const uint32_t rr = r0 + u * kStep;
            if (rr >= n_rows) continue;
            const int64_t dst = ((kv_row_from(a.pm_out, p.bud0, a.TB, p.layer, p.s, (int)(o0 + rr)) * a.h_kv + p.g) * kHeadDim) * 2 + part * 16;
            store_stream16(a.K_out + dst, kv[u]);
            store_stream16(a.V_out + dst, vv[u]);
        }
    }
}

// ------------------------------------------------------------------------------------------------
// short sequences: pooling, selection and gather in one kernel
// ------------------------------------------------------------------------------------------------
// A problem of up to THREADS * VPT positions fits one workgroup: its scores are staged in LDS, thread t pools the run of
// VPT consecutive positions t * VPT .. and keeps their keys in registers.  The threshold is found by a radix descent over
// the range that the problem's own keys span -- 2048 bins over [lowest, highest], then over the bin that holds the B-th
// largest -- so that crowded scores spread over many bins, and runs in thread order are runs in position order, so one
// block-wide scan of the threads' kept counts gives every kept position its slot: no histogram or lists in memory and no
// kernel (and no boundary between kernels) of its own for the pooling.  The slices of a problem repeat the selection and
// share the output (pooled scores by thread, kept rows by slot).  Latency-bound: a chain of about ten barriers.
struct PoolSelectArgs {
    const float* in;   // [n_layers][h_kv][T]: unpooled scores, or (K == 1) the values to select by
    float* out;        // pooled scores, or null
    int32_t pool_k;
    float inv_k;
    uint64_t* flags;   // words to clear: the flags of a launch that did both passes over K (or null)
    int32_t n_flags;
    SelectArgs sel;
};
constexpr int kSmallBins = 2048;
constexpr int kSmallFixedWords = kSmallBins + 32 + 32 + 64;  // bins, scan scratch, pick results, per-wave extremes
// Runs are VPT words apart from thread to thread: four words of padding per 32 spread the 16-byte reads of eight
// neighbouring threads over all banks.
__host__ __device__ constexpr int small_pad(int i) { return i + ((i >> 5) << 2); }

// K: pooling width 5 or 7 with unrolled taps, 1 for no pooling, 0 for any width
template <int THREADS, int VPT, int K>
__global__ __launch_bounds__(THREADS) void jq_pool_select_kernel(PoolSelectArgs pa) {
    extern __shared__ __attribute__((aligned(16))) uint32_t lds[];
    uint32_t* bins = lds;
    uint32_t* tmp = bins + kSmallBins;
    uint32_t* res = tmp + 32;
    uint32_t* ext = res + 32;                          // per wave: lowest, highest free key
    float* tile = (float*)(ext + 64);                  // staged scores; later the kept positions of the slice's slots
    uint32_t* slot_pos = ext + 64;
    argument_lines<5>();
    const SelectArgs& a = pa.sel;
    const Problem p = problem_of(a, blockIdx.x);
    const int L = p.L, tid = (int)threadIdx.x;
    const int64_t row = ((int64_t)p.layer * a.h_kv + p.g) * a.T + p.tok0;
    const float* in_row = pa.in + row;
    constexpr int kHalo = K > 1 ? 4 : 0;               // staged in front of and behind the sequence, zeros
    float raw[VPT];
#pragma unroll
    for (int u = 0; u < VPT; ++u) {
        raw[u] = in_row[min((uint32_t)(u * THREADS + tid), (uint32_t)L - 1u)];
    }
    for (int b = tid; b < kSmallBins; b += THREADS) bins[b] = 0u;
    if (pa.flags && blockIdx.y == 0)
        for (int i = (int)blockIdx.x * THREADS + tid; i < pa.n_flags; i += (int)gridDim.x * THREADS) pa.flags[i] = 0;
#pragma unroll
    for (int u = 0; u < VPT; ++u) {
        const int j = u * THREADS + tid;
        tile[small_pad(tid + kHalo) + u * small_pad(THREADS)] = j < L ? raw[u] : 0.f;  // THREADS is a multiple of 32
    }
    if (kHalo && tid < 2 * kHalo) tile[small_pad(tid < kHalo ? tid : THREADS * VPT + tid)] = 0.f;
    lds_barrier();

    const int j0 = tid * VPT;  // this thread's run of positions
    float v[VPT];
    if constexpr (K > 1) {
        float x[VPT + 2 * kHalo];
#pragma unroll
        for (int q = 0; q < VPT + 2 * kHalo; q += 4) {
            const float4 f = *(const float4*)&tile[small_pad(j0 + q)];
            x[q] = f.x; x[q + 1] = f.y; x[q + 2] = f.z; x[q + 3] = f.w;
        }
#pragma unroll
        for (int u = 0; u < VPT; ++u) {
            float acc = 0.f;
#pragma unroll
            for (int k = 0; k < K; ++k) acc += x[u + kHalo - K / 2 + k];  // ascending position order, as jq_pool_kernel
            v[u] = acc * pa.inv_k;
        }
    } else if (K == 1) {
#pragma unroll
        for (int q = 0; q < VPT; q += 4) {
            const float4 f = *(const float4*)&tile[small_pad(j0 + q)];
            v[q] = f.x; v[q + 1] = f.y; v[q + 2] = f.z; v[q + 3] = f.w;
        }
    } else {
        const int r = (pa.pool_k - 1) / 2;
#pragma unroll
        for (int u = 0; u < VPT; ++u) {
            const int q0 = max(0, j0 + u - r), q1 = min(L - 1, j0 + u + r);
            float acc = 0.f;
            for (int q = q0; q <= q1 && j0 + u < L; ++q) acc += tile[small_pad(q)];
            v[u] = acc * pa.inv_k;
        }
    }
    // This slice's share of the pooled scores, stored non-temporally like the pooling kernel's (see store_stream): as plain
    // stores they were 4 MB of dirty lines at the end of a call over 4 x 32768 tokens, 79.3 us against 78.4, 32 x 8192 251.8
    // against 246.4, 7 x 28000 + 28000 190.6 against 187.6.  Rows that are not 16-byte aligned (odd lengths) get 16-byte stores too,
    // where four of 4 bytes each had cost 8 x 12345 tokens 89.4 us a call (87.7 through the caches, 86.9 streamed), 12 ragged sequences of
    // 3001 to 15001 105.2 (103.2, 101.5), 16 x 3001 53.0 (52.7, 51.9); with 32 positions per thread, whose stores lie 128 bytes apart,
    // the caches are better (8 x 30001 189.2 / 188.3 / 190.3), and so they are for a few problems (5001 tokens 21.8 / 21.7 / 22.0).
    if (pa.out && (uint32_t)tid * gridDim.y / THREADS == blockIdx.y && j0 < L) {  // this slice's share of the pooled scores
        float* o = pa.out + row + j0;
        const bool streams = VPT <= 16 && gridDim.x > 32;  // uniform
        if (j0 + VPT <= L && (((uintptr_t)o) & 15u) == 0) {
#pragma unroll
            for (int q = 0; q < VPT; q += 4)  // streamed, as the pooling kernel's
                store_stream16(o + q, make_uint4(__float_as_uint(v[q]), __float_as_uint(v[q + 1]), __float_as_uint(v[q + 2]), __float_as_uint(v[q + 3])));
        } else if (j0 + VPT <= L && streams) {
#pragma unroll
            for (int q = 0; q < VPT; q += 4) store16_any<true>(o + q, v + q);
            asm volatile("" ::: "memory");  // or the compiler makes one loop of both, with plain stores
        } else if (j0 + VPT <= L) {
#pragma unroll
            for (int q = 0; q < VPT; q += 4) store16_any<false>(o + q, v + q);
        } else {
#pragma unroll
            for (int u = 0; u < VPT; ++u)
                if (j0 + u < L) o[u] = v[u];
        }
    }

    // Keys.  Always-kept positions get the largest key and positions past the end key 0; all others keep to 1 .. 2^32 - 2,
    // so that every later test of a position is one comparison.
    const int f0 = a.keep_first, f1 = L - a.keep_last;  // free positions: [f0, f1)
    uint32_t key[VPT];
    uint32_t lo = 0xFFFFFFFFu, hi = 0u;                 // lowest free key - 1, highest free key + 1
    // Scores are sums of probabilities: where a wave finds no sign bit, a key is the value's bits and one more instruction instead
    // of six (32 positions per thread on one CU: 2.4 us of the kernel's 15.7 went into keys and extremes, 1.5 now).
    uint32_t signs = 0u;
#pragma unroll
    for (int u = 0; u < VPT; ++u) signs |= __float_as_uint(v[u]);
    if (__any((int)signs < 0)) {
#pragma unroll
        for (int u = 0; u < VPT; ++u) key[u] = min(max(sortable_key(v[u]), 1u), 0xFFFFFFFEu);
    } else {
#pragma unroll
        for (int u = 0; u < VPT; ++u) key[u] = __float_as_uint(v[u]) | 0x80000000u;
    }
    if (j0 < f0 || j0 + VPT > f1) {  // runs that are not all free
#pragma unroll
        for (int u = 0; u < VPT; ++u) {
            const int j = j0 + u;
            key[u] = j < f0 || j >= f1 ? (j < L ? 0xFFFFFFFFu : 0u) : min(key[u], 0xFFFFFFFEu);
            lo = min(lo, j < f0 || j >= f1 ? 0xFFFFFFFFu : key[u] - 1u);
            hi = max(hi, key[u] + 1u);  // the largest key wraps to 0
        }
    } else {
#pragma unroll
        for (int u = 0; u < VPT; ++u) { lo = min(lo, key[u]); hi = max(hi, key[u]); }
        if (__any(hi == 0xFFFFFFFFu)) {  // a NaN of all ones, whose bits make the key of the positions that are always kept
#pragma unroll
            for (int u = 0; u < VPT; ++u) key[u] = min(key[u], 0xFFFFFFFEu);
            lo = min(lo, 0xFFFFFFFEu); hi = min(hi, 0xFFFFFFFEu);
        }
        lo -= 1u; hi += 1u;
    }
    lo = wave_min(lo);
    hi = wave_max(hi);
    if ((tid & 63) == 0) { ext[tid >> 6] = lo; ext[32 + (tid >> 6)] = hi; }
    lds_barrier();
#pragma unroll
    for (int w = 0; w < THREADS / 64; ++w) { lo = min(lo, ext[w]); hi = max(hi, ext[32 + w]); }
    const uint32_t n_forced = (uint32_t)(a.keep_first + a.keep_last);
    uint32_t need = p.B - min(p.B, n_forced);  // places for free positions
    uint32_t tau = 0xFFFFFFFEu;                // kept: key > tau, and the first `need` positions with key == tau
    if (need > 0) {                            // uniform; there are free positions then
        lo += 1u; hi -= 1u;
        uint32_t base = lo, span = hi - lo;    // the need-th largest free key lies in [base, base + span]
        // Long runs: a lower bound first.  The largest key of every group of kGroup positions goes into the histogram; the
        // bin of the need-th largest of THEM has at least `need` keys at or above its lowest key, so only those few enter
        // the descent -- counting all 32 keys of every thread took longer than everything else here, LDS atomics of a wave
        // being served a few lanes at a time.
        constexpr int kGroup = 8;
        if (VPT >= 2 * kGroup && need <= (uint32_t)(THREADS * VPT / kGroup / 2)) {  // uniform
            const int shift = max(0, 32 - __clz((int)(span | 1u)) - 11);
#pragma unroll
            for (int u = 0; u < VPT; u += kGroup) {
                uint32_t top = 0u;
#pragma unroll
                for (int e = 0; e < kGroup; ++e) top = max(top, key[u + e] + 1u);  // + 1: see hi
                if (top > base) atomicAdd(&bins[(top - 1u - base) >> shift], 1u);  // a group without free positions has 0 or 1
            }
            if (tid == 0) res[8] = 0u;  // stays 0 when there are fewer groups than `need`
            lds_barrier();
            uint32_t* found = res + 8;
            pick_bin<THREADS, kSmallBins / THREADS>(bins, kSmallBins, need, tmp, found);
            base += found[0] << shift;
            span = hi - base;
            for (int b = tid; b < kSmallBins; b += THREADS) bins[b] = 0u;
            lds_barrier();
        }
        for (;;) {
            const int shift = max(0, 32 - __clz((int)(span | 1u)) - 11);
#pragma unroll
            for (int u = 0; u < VPT; ++u) {
                const uint32_t d = key[u] - base;
                if (d <= span) atomicAdd(&bins[d >> shift], 1u);  // (a key below base wraps above span; so do 0 and 2^32 - 1)
            }
            lds_barrier();
            pick_bin<THREADS, kSmallBins / THREADS>(bins, kSmallBins, need, tmp, res);
            base += res[0] << shift;
            need -= res[1];
            tau = base;
            if (shift == 0) break;
            if (res[2] == need) {  // the whole bin is kept: everything from its lowest key (>= 1) on, no tie to trim
                tau = base - 1u;
                need = 0u;
                break;
            }
            span = min((1u << shift) - 1u, hi - base);
            for (int b = tid; b < kSmallBins; b += THREADS) bins[b] = 0u;
            lds_barrier();
        }
    }

    uint32_t m_gt = 0, m_eq = 0;  // bit u: position j0 + u
#pragma unroll
    for (int u = 0; u < VPT; ++u) m_gt |= key[u] > tau ? 1u << u : 0u;
    if (need > 0) {  // uniform; otherwise no position with key == tau is kept
#pragma unroll
        for (int u = 0; u < VPT; ++u) m_eq |= key[u] == tau ? 1u << u : 0u;
    }
    const uint32_t n_gt = __popc(m_gt), n_eq = __popc(m_eq);
    uint32_t total;
    const uint32_t packed = n_gt | (n_eq << 16);  // at most 32768 per field
    const uint32_t incl = block_scan_incl<THREADS>(packed, tmp, &total);
    uint32_t gt = (incl - packed) & 0xFFFFu, eq = (incl - packed) >> 16;  // before this thread's run
    const uint32_t per_slice = (p.B + gridDim.y - 1) / gridDim.y;
    const uint32_t o_begin = min(p.B, blockIdx.y * per_slice), n_rows = min(p.B, o_begin + per_slice) - o_begin;
    // (Slots rise with the positions: most threads' kept positions belong to other slices, and whole waves have nothing to
    // list.  The others test a bit per position: going from set bit to set bit, a wave went through its fullest thread's, 2 us
    // with 32 positions per thread.)
    uint32_t kept = m_gt, slot = gt + min(eq, need) - o_begin;
    if (eq < need) {
        uint32_t ties = m_eq;
        for (uint32_t room = need - eq, n = n_eq; n > room; --n) ties &= ~(0x80000000u >> __builtin_clz(ties));  // the highest ones go
        kept |= ties;
    }
    if (kept != 0u && (int)slot < (int)n_rows && (int)(slot + __popc(kept)) > 0) {
#pragma unroll
        for (int u = 0; u < VPT; ++u) {
            if (((kept >> u) & 1u) && slot < n_rows) slot_pos[slot] = (uint32_t)(j0 + u);  // the staged scores are dead
            slot += (kept >> u) & 1u;
        }
    }
    lds_barrier();
    for (uint32_t o = threadIdx.x; o < n_rows; o += THREADS) p.emit(o_begin + o, (int)slot_pos[o]);
    if (a.K_out != nullptr || a.stage != nullptr) gather_slots<THREADS>(a, p, slot_pos, o_begin, n_rows);
}

// ------------------------------------------------------------------------------------------------
// fast path: resolve the threshold from the sorted segments and emit ascending positions
// ------------------------------------------------------------------------------------------------
constexpr int kFinThreads = 512;
constexpr int kFinWaves = kFinThreads / 64;
constexpr int kSegBatch = 16;  // segments whose first entries a wave requests before it knows the threshold bin

__global__ __launch_bounds__(kFinThreads) void jq_select_finalize_kernel(SelectArgs a, int words_cap, int qual_cap) {
    argument_lines<5>();
    extern __shared__ __attribute__((aligned(16))) uint32_t lds[];
    uint32_t* bins2 = lds;                        // 2048: level-2 histogram
    uint32_t* bins3 = bins2 + 2048;               // 1024: level-3 histogram
    uint32_t* tmp = bins3 + 1024;                 // scan scratch (padded to 32)
    uint32_t* res = tmp + 32;                     // pick results (padded to 32)
    uint32_t* cnt = res + 32;                     // [0] elements with bin >= b1 (padded to 32)
    uint32_t* keep = cnt + 32;                    // words_cap: bitmap of kept positions
    uint32_t* ties = keep + words_cap;            // words_cap: bitmap of positions with key == tau
    uint2* qual = (uint2*)(ties + words_cap);     // qual_cap: (key, position) of the elements with bin >= b1
    int32_t* seg_n = (int32_t*)(qual + qual_cap); // segs_cap: usable entries of each segment of the problem (-1: none)

    const Problem p = problem_of(a, blockIdx.x);  // blockIdx.y: which slice of the problem's output slots
    const int words = (p.L + 31) >> 5;
    const int lane = threadIdx.x & 63;
    const int wave = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
    const int n_seg = a.one_L ? a.n_seg : a.cu_seg[p.s + 1] - a.cu_seg[p.s];
    const int64_t seg0 = ((int64_t)p.layer * a.h_kv + p.g) * a.n_seg + (a.one_L ? 0 : a.cu_seg[p.s]);
    const int head = a.one_L ? a.head : seg_head_of(a.tab.cu_bud[p.s + 1] - a.tab.cu_bud[p.s], p.L);  // as the pooling kernel has it
    const uint2* segs = a.seg + seg0 * a.head;
    const uint4* seg_hdr = a.seg_hdr + seg0;

    // Requested first: this thread's four level-1 bins, the header of "its" segment (thread t looks after segment
    // t), and the first entries of the wave's first segments; all of that arrives while the
    // threshold bin is being picked (the CU's load path is what bounds this phase, and it counts instructions and bytes: a load covers
    // 64 entries of two segments, two per lane; where a block keeps more than 32 positions on average -- `dense` -- the next 64
    // are requested as well (from 16 on: 65536 tokens with 2048 kept 68.3 us a call, 67.3 so, 50000 with 1536 56.7 / 55.7).  With 128
    // entries of one segment per load, whatever the density, the list was complete 10.0 us after entry on the 128K layer, 6.2 so, the
    // call 110.5 -> 106.4; 65536 tokens 65.3 -> 62.7, 100000 with 3072 kept 93.9 -> 92.9).  The entry loads are unconditional, from clamped
    // and therefore always valid addresses -- a segment's storage holds `head` entries whatever its element count -- so that all of
    // them are in flight together; what lies outside is masked afterwards.
    uint32_t c1[kHistBins / kFinThreads];
    counts_down<kHistBins / kFinThreads>(p.hist, kHistBins, c1);
    const uint4 my_hdr = seg_hdr[min((int)threadIdx.x, n_seg - 1)];
    // (Or the compiler requests the bins behind the entries, and the scan of the bins waits for all of them: 131072 tokens 107.5 us a call,
    // 106.9 so, a paged batch of 8 175.2 / 174.7, 4 x 38189 with 1433 kept 127.4 / 127.0; where every block is scanned it costs 1 %.)
    __builtin_amdgcn_sched_barrier(0);
    constexpr int kPairs = kSegBatch / 2;
    const bool dense = head > 256;  // uniform
    const int half = lane >> 5, l32 = lane & 31;
    const char* entries = (const char*)segs;
    uint32_t ent_at[kPairs];  // bytes from there to the lane's part of its segment of the i-th pair (at most 2^14 segments of 2^13 bytes)
    uint4 ent[kPairs], ent2[kPairs];  // its entries 2 * l32 and 2 * l32 + 1, and 64 further on: (key, position) twice
#pragma unroll
    for (int i = 0; i < kPairs; ++i) {
        ent_at[i] = (uint32_t)min(wave + (2 * i + half) * kFinWaves, n_seg - 1) * (uint32_t)(a.head * 8) + 16u * (uint32_t)l32;
        ent[i] = *(const uint4*)(entries + ent_at[i]);
    }
    if (dense) {
#pragma unroll
        for (int i = 0; i < kPairs; ++i) ent2[i] = *(const uint4*)(entries + ent_at[i] + 512);
    }
    for (int w = 4 * threadIdx.x; w < 2 * words_cap; w += 4 * kFinThreads) *(uint4*)&keep[w] = make_uint4(0u, 0u, 0u, 0u);  // keep, ties
    for (int b = 4 * threadIdx.x; b < 3072 + 96; b += 4 * kFinThreads) *(uint4*)&bins2[b] = make_uint4(0u, 0u, 0u, 0u);  // histograms, tmp, res, cnt
    lds_barrier();
    pick_bin_counts<kFinThreads, kHistBins / kFinThreads>(c1, kHistBins, p.B, tmp, res);
    const uint32_t b1 = res[0];
    const uint32_t n_above = res[1];  // positions above bin b1 (all of them are kept); < B

    // header = (lowest bin of the block's window, elements inside the window, key of the segment's last slot);
    // usable entries of a segment, or -1 when the segment cannot answer -- more qualifying elements than it holds,
    // or a window that ends above b1 -- and the block is classified from its pooled scores instead
    auto usable = [&](uint4 hdr) {
        const bool answers = b1 >= hdr.x && !((int)hdr.y > head && (hdr.z >> 21) >= b1);
        return answers ? min(head, (int)hdr.y) : -1;
    };
    for (int t = threadIdx.x; t < n_seg; t += kFinThreads) seg_n[t] = usable(t == (int)threadIdx.x ? my_hdr : seg_hdr[t]);
    lds_barrier();

    // Every entry with bin >= b1 goes into one flat LDS list `qual` (as far as it reaches; cnt[0] counts them all),
    // which the passes below work through evenly, a few entries per thread.  The entries of a wave's first segments
    // are counted with ballots first, so that the whole batch needs ONE reservation: atomics of many lanes on one
    // LDS word are served one at a time.
    auto put = [&](uint32_t key, uint32_t pos) __attribute__((always_inline)) {  // rare paths: one reservation per entry
        const uint32_t to = atomicAdd(&cnt[0], 1u);
        if (to < (uint32_t)qual_cap) qual[to] = make_uint2(key, pos);
    };
    auto scan_block = [&](int sg, auto f) __attribute__((always_inline)) {
        const int j0 = sg * kSegLen, j1 = min(p.L, j0 + kSegLen);
        for (int j = j0 + lane; j < j1; j += 64) {
            const uint32_t key = select_key(p.x[j], j, p.L, a.keep_first, a.keep_last);
            if ((key >> 21) >= b1) f(key, (uint32_t)j);
        }
    };
    const int my_seg = wave + (lane & (kSegBatch - 1)) * kFinWaves, my_n = my_seg < n_seg ? seg_n[my_seg] : 0;  // lane i < 16: the wave's i-th segment
    uint32_t again = 0;  // bit i: the last entry looked at of the i-th segment still qualified
    auto list_entries = [&](const uint4 (&e)[kPairs], int first) __attribute__((always_inline)) {
        uint64_t ge_even[kPairs], ge_odd[kPairs];  // wave-uniform: lanes whose even / odd entry qualifies
        uint32_t n_mine = 0;
#pragma unroll
        for (int i = 0; i < kPairs; ++i) {
            const int na = __builtin_amdgcn_readlane(my_n, 2 * i), nb = __builtin_amdgcn_readlane(my_n, 2 * i + 1), n = half ? nb : na;  // -1: not from its entries
            ge_even[i] = __ballot(first + 2 * l32 < n && (e[i].x >> 21) >= b1);
            ge_odd[i] = __ballot(first + 2 * l32 + 1 < n && (e[i].z >> 21) >= b1);
            n_mine += (uint32_t)(__popcll(ge_even[i]) + __popcll(ge_odd[i]));
            again |= (uint32_t)((ge_odd[i] >> 31) & 1) << (2 * i) | (uint32_t)(ge_odd[i] >> 63) << (2 * i + 1);
        }
        if (n_mine) {  // wave-uniform
            uint32_t to = 0;
            if (lane == 0) to = atomicAdd(&cnt[0], n_mine);
            to = __builtin_amdgcn_readfirstlane(to);
#pragma unroll
            for (int i = 0; i < kPairs; ++i) {
                const uint64_t me = ge_even[i], mo = ge_odd[i];
                const uint32_t se = to + __builtin_amdgcn_mbcnt_hi((uint32_t)(me >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)me, 0u));
                if (((me >> lane) & 1) && se < (uint32_t)qual_cap) qual[se] = make_uint2(e[i].x, e[i].y);
                to += (uint32_t)__popcll(me);
                const uint32_t so = to + __builtin_amdgcn_mbcnt_hi((uint32_t)(mo >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)mo, 0u));
                if (((mo >> lane) & 1) && so < (uint32_t)qual_cap) qual[so] = make_uint2(e[i].z, e[i].w);
                to += (uint32_t)__popcll(mo);
            }
        }
    };
    // Where the last of the 64 still qualified in more than two of the wave's segments, the next 64 of all of them are read together: one
    // round trip, where one after the other 2048 kept of 131072 flat scores (threshold bins that reach far down) lost the call 2.5 us
    // against 128 entries read at once (107.1 / 109.8; 106.7 so).  One or two are visited below, which costs a wave less than
    // this turn: pooling left out, 131072 scores, together from one / two / three segments on and never: 4 blocks with 100 kept
    // each 19.2 / 18.7 / 18.5 / 18.6 us, 8 with 90 19.7 / 19.5 / 19.3 / 19.5, 26 with 80 20.7 / 20.5 / 20.4 / 22.1.
    // One copy of the code, gone through twice: two are 2.5 KB more, which every wave fetches from cold (4 x 38189 tokens with 1433 kept
    // 127.7 us a call, 126.7 so; 5 ragged sequences of 145197 together with 1634 kept each 130.9 / 130.3).
    int listed_to = 64;
#pragma nounroll
    for (int first = 0;; first = 64) {
        list_entries(ent, first);
        if (first || !(dense || __popc(again) > 2)) break;  // wave-uniform
        listed_to = 128;
        again = 0;
        if (dense) {
#pragma unroll
            for (int i = 0; i < kPairs; ++i) ent[i] = ent2[i];
        } else {
#pragma unroll
            for (int i = 0; i < kPairs; ++i) ent[i] = *(const uint4*)(entries + ent_at[i] + 512);
        }
    }
    // Second visits (a segment whose last entry looked at still qualified, a block that is classified from its scores), and
    // the segments beyond the first batch: rare, so the common case only tests one mask.
    again |= (uint32_t)__ballot(lane < kSegBatch && wave + lane * kFinWaves < n_seg && my_n < 0);
    for (int beyond = wave + kSegBatch * kFinWaves;;) {  // wave-uniform
        int sg, off;
        if (again) {
            sg = wave + __builtin_ctz(again) * kFinWaves;
            off = listed_to;
            again &= again - 1;
        } else {
            if (beyond >= n_seg) break;
            sg = beyond;
            off = 0;
            beyond += kFinWaves;
        }
        const int n = seg_n[sg];
        if (n < 0) {  // four requests at a time: one after the other they were 16 memory latencies a block (16 blocks with 128 kept each
                      // out of 131072: 150.4 us a call, 118.0 so; written out at every call of scan_block it is 3 KB more code, for
                      // which calls that never come here lost 1 us)
            const int j0 = sg * kSegLen + lane, j1 = min(p.L, (sg + 1) * kSegLen);
            for (int j = j0; j < j1; j += 4 * 64) {
                float x[4];
#pragma unroll
                for (int u = 0; u < 4; ++u) x[u] = p.x[min(j + 64 * u, j1 - 1)];
#pragma unroll
                for (int u = 0; u < 4; ++u) {
                    const int at = j + 64 * u;
                    const uint32_t key = select_key(x[u], at, p.L, a.keep_first, a.keep_last);
                    if (at < j1 && (key >> 21) >= b1) put(key, (uint32_t)at);
                }
            }
            continue;
        }
        // chunks of 64 entries while the previous chunk's last entry still qualified
        bool last_in = true;
        for (; off < n && last_in; off += 64) {
            const uint2 e = segs[(int64_t)sg * a.head + min(off + lane, head - 1)];
            const bool ge = off + lane < n && (e.x >> 21) >= b1;
            if (ge) put(e.x, e.y);
            last_in = (__ballot(ge) >> 63) != 0;
        }
    }
    lds_barrier();
    const uint32_t n_qual = cnt[0];
    const bool listed = n_qual <= (uint32_t)qual_cap;  // uniform; otherwise every pass re-reads the scores
    uint32_t need = p.B - min(n_above, p.B - 1);       // >= 1: the threshold bin always contributes

    // f(key, position) for every element with bin >= b1
    auto for_each_qual = [&](auto f) __attribute__((always_inline)) {
        if (listed) {
            for (uint32_t i = threadIdx.x; i < n_qual; i += kFinThreads) f(qual[i].x, qual[i].y);
        } else {
            for (int sg = wave; sg < n_seg; sg += kFinWaves) scan_block(sg, f);
        }
    };
    // positions above b1 are kept; level 2 on the pairs inside b1
    for_each_qual([&](uint32_t key, uint32_t pos) {
        if (pos >= (uint32_t)p.L) return;
        if ((key >> 21) > b1) atomicOr(&keep[pos >> 5], 1u << (pos & 31));
        else atomicAdd(&bins2[(key >> 10) & 2047u], 1u);
    });
    lds_barrier();
    pick_bin<kFinThreads, 2048 / kFinThreads>(bins2, 2048, need, tmp, res);
    const uint32_t b2 = res[0];
    need -= res[1];
    uint32_t tau = ((b1 << 11) | b2) << 10;
    bool all_ties = res[2] == need;  // uniform: the whole bin is kept, from its lowest key on (the usual case: 22 bits tell most
    // scores apart; without the last level and its scan the 128K layer takes 116.0 us instead of 118.6, 65536 tokens 68.0 instead of 68.7)
    if (!all_ties) {                 // level 3
        for_each_qual([&](uint32_t key, uint32_t pos) {
            if (pos < (uint32_t)p.L && (key >> 10) == ((b1 << 11) | b2)) atomicAdd(&bins3[key & 1023u], 1u);
        });
        lds_barrier();
        pick_bin<kFinThreads, 1024 / kFinThreads>(bins3, 1024, need, tmp, res + 4);
        tau |= res[4];
        need -= res[5];              // how many positions with key == tau are kept
        all_ties = need == res[6];   // the whole tie group is
    }
    for_each_qual([&](uint32_t key, uint32_t pos) {
        if (pos >= (uint32_t)p.L || (key >> 21) != b1) return;
        if (key > tau || (all_ties && key == tau)) atomicOr(&keep[pos >> 5], 1u << (pos & 31));
        else if (key == tau) atomicOr(&ties[pos >> 5], 1u << (pos & 31));
    });
    lds_barrier();

    // Thread t owns a contiguous run of `wpt` words (a multiple of four, read as 16-byte vectors; the bitmaps are
    // padded with zero words up to kFinThreads * wpt), so thread order is position order.
    const int wpt = words_cap / kFinThreads;
    const int w0 = threadIdx.x * wpt;
    uint32_t total;
    if (!all_ties) {  // the lowest `need` tie positions join the kept set
        uint32_t n_t = 0;
        for (int w = w0; w < w0 + wpt; ++w) n_t += __popc(ties[w]);
        uint32_t before = block_scan_incl<kFinThreads>(n_t, tmp, &total) - n_t;
        for (int w = w0; w < w0 + wpt && before < need; ++w) {
            uint32_t t = ties[w];
            const uint32_t cnt_w = __popc(t);
            uint32_t take = min(cnt_w, need - before);
            before += cnt_w;
            uint32_t add = 0;
            while (take--) { const uint32_t low = t & (0u - t); add |= low; t ^= low; }
            keep[w] |= add;  // only this thread touches word w here
        }
        lds_barrier();
    }
    // Exclusive prefix of the kept count per 32-position word.
    uint32_t n_k = 0;
    for (int w = w0; w < w0 + wpt; w += 4) {
        const uint4 k4 = *(const uint4*)&keep[w];
        n_k += __popc(k4.x) + __popc(k4.y) + __popc(k4.z) + __popc(k4.w);
    }
    uint32_t run = block_scan_incl<kFinThreads>(n_k, tmp, &total) - n_k;
    uint32_t* wpre = ties;  // the tie bitmap is dead by now
    for (int w = w0; w < w0 + wpt; w += 4) {
        const uint4 k4 = *(const uint4*)&keep[w];
        uint4 pre;
        pre.x = run; run += __popc(k4.x);
        pre.y = run; run += __popc(k4.y);
        pre.z = run; run += __popc(k4.z);
        pre.w = run; run += __popc(k4.w);
        *(uint4*)&wpre[w] = pre;
    }
    lds_barrier();
    const uint32_t per_slice = (p.B + gridDim.y - 1) / gridDim.y;
    const uint32_t o_begin = min(p.B, blockIdx.y * per_slice), o_end = min(p.B, o_begin + per_slice);
    uint32_t* slot_pos = bins2;  // the histograms are dead: kept positions of (a batch of) the slice's output slots
    auto gather_rows = [&](uint32_t o0, uint32_t n_rows) __attribute__((always_inline)) { gather_slots<kFinThreads>(a, p, slot_pos, o0, n_rows); };
    const bool want_rows = a.K_out != nullptr || a.stage != nullptr;  // uniform
    if (listed && o_end - o_begin <= 3072u) {
        // Every kept element sits in the flat list, and its output slot is its rank among the kept positions:
        // the words before its own (prefix array) plus the set bits below it in its word.
        for (uint32_t i = threadIdx.x; i < n_qual; i += kFinThreads) {
            const uint32_t pos = qual[i].y;
            if (pos >= (uint32_t)p.L) continue;
            const uint32_t word = keep[pos >> 5], bit = pos & 31;
            if (!((word >> bit) & 1u)) continue;
            const uint32_t o = wpre[pos >> 5] + __popc(word & ((1u << bit) - 1u));
            if (o >= o_begin && o < o_end) {
                p.emit(o, (int)pos);
                slot_pos[o - o_begin] = pos;
            }
        }
        if (!want_rows) return;  // uniform
        lds_barrier();
        gather_rows(o_begin, o_end - o_begin);
        return;
    }
    // Otherwise emission is parallel over OUTPUT slots: slot o lives in the last word w with wpre[w] <= o (binary
    // search in LDS, same trip count for every thread); inside the word, the (o - wpre[w])-th set bit is found by
    // five popcount halvings.  Consecutive threads write consecutive slots.
    for (uint32_t o0 = o_begin; o0 < o_end; o0 += kFinThreads) {  // uniform trip count
        const uint32_t o = o0 + threadIdx.x;
        if (o < o_end) {
            int lo = 0, hi = words;  // invariant: wpre[lo] <= o, and hi == words or wpre[hi] > o
            while (hi - lo > 1) {
                const int mid = (lo + hi) >> 1;
                if (wpre[mid] <= o) lo = mid; else hi = mid;
            }
            uint32_t r = o - wpre[lo];
            const uint32_t k = keep[lo];
            uint32_t pos = 0;
#pragma unroll
            for (int sft = 16; sft >= 1; sft >>= 1) {
                const uint32_t c = __popc((k >> pos) & ((1u << sft) - 1u));
                if (r >= c) { r -= c; pos += sft; }
            }
            // (with consistent counts this is a kept position; the clamp keeps the gather inside the sequence whatever
            // the lists hold)
            const uint32_t at = min((uint32_t)(lo << 5) + pos, (uint32_t)p.L - 1u);
            p.emit(o, (int)at);
            slot_pos[threadIdx.x] = at;
        }
        if (!want_rows) continue;  // uniform
        lds_barrier();
        gather_rows(o0, min((uint32_t)kFinThreads, o_end - o0));
        lds_barrier();  // slot_pos is rewritten by the next batch
    }
}

constexpr int kFinalizeFixedWords = 2048 + 1024 + 32 + 32 + 32;
constexpr size_t kMaxLds = 160 * 1024;
constexpr int kQualCap = 8192;     // elements at or above the threshold bin that the LDS list holds when there is room
constexpr int kQualCapMin = 1024;

// LDS of the finalize kernel for the plan's longest sequence: the two bitmaps, one word per segment, then as much
// list as fits.
static size_t finalize_lds(const Plan& p, int* words_cap, int* qual_cap) {
    int max_len = 0;
    for (int s = 0; s < p.n_seq; ++s) max_len = max(max_len, p.tab.cu_seq[s + 1] - p.tab.cu_seq[s]);
    *words_cap = ((max_len + 31) / 32 + 4 * kFinThreads - 1) / (4 * kFinThreads) * (4 * kFinThreads);  // whole 16-byte vectors per thread
    const size_t segs_cap = ((size_t)max_len + kSegLen - 1) / kSegLen;
    const size_t fixed = ((size_t)kFinalizeFixedWords + 2 * (size_t)*words_cap + segs_cap) * sizeof(uint32_t);
    const size_t room = kMaxLds - 1024 > fixed ? (kMaxLds - 1024 - fixed) / sizeof(uint2) : 0;
    *qual_cap = (int)(room < (size_t)kQualCap ? room : (size_t)kQualCap);
    return fixed + (size_t)*qual_cap * sizeof(uint2);
}

bool select_fast_path(const Plan& p) {
    int words_cap, qual_cap;
    finalize_lds(p, &words_cap, &qual_cap);
    return qual_cap >= kQualCapMin;  // otherwise the bitmaps (nearly) fill LDS: stream instead
}

static SelectArgs select_args(const Plan& p, const float* pooled, uint32_t* hist, char* ws, int32_t* idx, const void* K, const void* V,
                              void* K_out, void* V_out, void* stage, const int32_t* pos_in, int32_t* pos_out, const uint32_t* dest_bits) {
    SelectArgs a;
    a.dest_bits = dest_bits;
    a.pooled = pooled; a.hist = hist; a.idx = idx;
    a.pos_in = pos_in; a.pos_out = pos_out;
    a.K = (const char*)K; a.V = (const char*)V; a.K_out = (char*)K_out; a.V_out = (char*)V_out;
    a.stage = (char*)stage;
    a.seg = (const uint2*)(ws + p.off_seg);
    a.seg_hdr = (const uint4*)(ws + p.off_seghdr);
    a.head = p.seg_head;
    a.n_layers = p.n_layers; a.h_kv = p.h_kv; a.T = p.T; a.TB = p.TB;
    a.keep_first = p.keep_first; a.keep_last = p.keep_last;
    a.one_L = p.n_seq == 1 ? p.tab.cu_seq[1] : 0;
    a.one_B = p.n_seq == 1 ? p.tab.cu_bud[1] : 0;
    a.pm = p.page_map();
    a.pm_out = p.out_map;
    a.layer_budgets = p.layer_budgets;
    a.n_seg = p.n_seg;
    for (int s = 0; s <= p.n_seq; ++s) a.cu_seg[s] = p.cu_seg[s];
    a.tab = p.tab;
    return a;
}

// Slices per problem: enough workgroups to spread the emission (and the gather) over the chip's 256 CUs, each with at least
// 64 output slots.  Where only one workgroup fits a CU (`alone`), some more than 256 of them are a second round of the whole
// selection: then as many as fit in one, unless that leaves a slice more than 1000 rows to gather -- whole calls, rounded up /
// down: 30000 + 8 x 9000 tokens, 256 kept 124.5 / 108.1 us, 3000 kept 135.9 / 129.3; 3 x 20000, 2048 kept 96.2 / 79.3; but
// 6 x 24000 + 6 x 3000 (96 problems), 1024 kept 161.2 / 154.4, 2048 kept 163.4 / 169.8.
static unsigned slices_of(const Plan& p, bool alone) {
    const int64_t n_prob = (int64_t)p.n_layers * p.n_seq * p.h_kv;
    int64_t min_budget = INT32_MAX, max_budget = 0;
    for (int s = 0; s < p.n_seq; ++s) {
        min_budget = min(min_budget, (int64_t)(p.tab.cu_bud[s + 1] - p.tab.cu_bud[s]));
        max_budget = max(max_budget, (int64_t)(p.tab.cu_bud[s + 1] - p.tab.cu_bud[s]));
    }
    int64_t slices = (256 + n_prob - 1) / n_prob;
    if (alone && max_budget <= 1000 * (256 / n_prob)) slices = 256 / n_prob;
    slices = min(slices, (min_budget + 63) / 64);
    return (unsigned)max((int64_t)1, min(slices, (int64_t)64));
}

static int longest_sequence(const Plan& p) {
    int max_len = 0;
    for (int s = 0; s < p.n_seq; ++s) max_len = max(max_len, p.tab.cu_seq[s + 1] - p.tab.cu_seq[s]);
    return max_len;
}

bool select_small(const Plan& p) { return longest_sequence(p) <= kSmallMax; }

bool evict_tail_small(const Plan& p) {
    const int L = longest_sequence(p);
    if (L > kSmallMax) return false;
    if (p.pool_k != 1 && p.pool_k != 5 && p.pool_k != 7)
        return L <= 2048 || p.pool_k <= (L <= 4096 ? 31 : L <= 8192 ? 9 : L <= 16384 ? 3 : 0);
    return p.pool_k == 1 || L <= 16384 || (int64_t)p.n_layers * p.n_seq * p.h_kv <= 256;
}

template <int THREADS, int VPT, int K>
static hipError_t launch_small_k(const Plan& p, const PoolSelectArgs& a, hipStream_t st) {
    static std::atomic<uint64_t> done{0};
    const int words = kSmallFixedWords + small_pad(THREADS * VPT + 8) + 4;
    const size_t lds_bytes = (size_t)words * sizeof(uint32_t);
    if (lds_bytes > 64 * 1024) {
        const hipError_t e = allow_dynamic_lds((const void*)jq_pool_select_kernel<THREADS, VPT, K>, (int)(kMaxLds - 1024), done);
        if (e != hipSuccess) return e;
    }
    const unsigned n_prob = (unsigned)((int64_t)p.n_layers * p.n_seq * p.h_kv);
    return launch_kernel(jq_pool_select_kernel<THREADS, VPT, K>, dim3(n_prob, slices_of(p, lds_bytes > kMaxLds / 2)), dim3(THREADS), lds_bytes, st, p.marks, kTrFinalize, a);
}
template <int K>
static hipError_t launch_small(const Plan& p, const PoolSelectArgs& a, hipStream_t st) {
    const int L = longest_sequence(p);
    if (L <= 512 * 4) return launch_small_k<512, 4, K>(p, a, st);
    if (L <= 512 * 8) return launch_small_k<512, 8, K>(p, a, st);
    if (L <= 512 * 16) return launch_small_k<512, 16, K>(p, a, st);
    if (L <= 1024 * 16) return launch_small_k<1024, 16, K>(p, a, st);
    if constexpr (K == 0) return hipErrorInvalidValue;  // no caller pools so long a sequence here
    else return launch_small_k<1024, 32, K>(p, a, st);
}

hipError_t launch_pool_select(const Plan& p, const float* in, float* out, bool pool, char* ws, int32_t* idx, hipStream_t st, const void* K,
                              const void* V, void* K_out, void* V_out, void* stage, const int32_t* pos_in, int32_t* pos_out,
                              const uint32_t* dest_bits) {
    PoolSelectArgs a;
    a.in = in; a.out = out;
    a.pool_k = p.pool_k; a.inv_k = 1.0f / (float)p.pool_k;
    a.flags = p.one_launch && pool ? (uint64_t*)(ws + p.off_flags) : nullptr;  // an eviction's
    a.n_flags = p.split.n_sets * p.h_kv;
    if (p.marks)  // no pooling kernel of its own: an interval with nothing in it
        for (int i = 0; i < 2; ++i) {
            const hipError_t e = hipEventRecord((hipEvent_t)p.marks[2 * kTrPool + i], st);
            if (e != hipSuccess) return e;
        }
    a.sel = select_args(p, nullptr, (uint32_t*)(ws + p.off_hist), ws, idx, K, V, K_out, V_out, stage, pos_in, pos_out, dest_bits);
    if (!pool || p.pool_k == 1) return launch_small<1>(p, a, st);
    if (p.pool_k == 7) return launch_small<7>(p, a, st);
    if (p.pool_k == 5) return launch_small<5>(p, a, st);
    return launch_small<0>(p, a, st);
}

hipError_t launch_select(const Plan& p, const float* pooled, uint32_t* hist, char* ws, int32_t* idx, hipStream_t st,
                         const void* K, const void* V, void* K_out, void* V_out, bool* gathered, void* stage,
                         const int32_t* pos_in, int32_t* pos_out, const uint32_t* dest_bits) {
    const SelectArgs a = select_args(p, pooled, hist, ws, idx, K, V, K_out, V_out, stage, pos_in, pos_out, dest_bits);
    if (gathered) *gathered = false;
    const unsigned n_prob = (unsigned)((int64_t)p.n_layers * p.n_seq * p.h_kv);

    if (!select_fast_path(p))  // bitmaps do not fit: stream instead
        return launch_kernel(jq_select_stream_kernel, dim3(n_prob), dim3(kSelectThreads), 0, st, p.marks, kTrFinalize, a);

    int words_cap, qual_cap;
    const size_t lds_bytes = finalize_lds(p, &words_cap, &qual_cap);
    if (lds_bytes > 64 * 1024) {
        static std::atomic<uint64_t> done{0};
        const hipError_t e = allow_dynamic_lds((const void*)jq_select_finalize_kernel, (int)(kMaxLds - 1024), done);
        if (e != hipSuccess) return e;
    }
    const unsigned slices = slices_of(p, false);
    if (gathered) *gathered = K_out != nullptr || stage != nullptr;
    return launch_kernel(jq_select_finalize_kernel, dim3(n_prob, slices), dim3(kFinThreads), lds_bytes, st, p.marks,
                         kTrFinalize, a, words_cap, qual_cap);
}

}  // namespace jq
