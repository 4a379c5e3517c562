// Which keys the workgroups of a pass over K sweep, in which order, and where their requests lie: the index arithmetic of the
// passes.  Plain integer code without any HIP call, so that a host compiler takes it too and a test can walk every share of any
// call on the CPU.
#pragma once

#include <stdint.h>

#include <algorithm>
#include <cmath>

#include "jq.h"

#ifdef __HIPCC__
#define JQ_HD __host__ __device__ __forceinline__
#else
#define JQ_HD inline
#endif

namespace jq {

constexpr int kKeyTile = 32;        // keys per MFMA tile (one 32x32 block column)
constexpr int kRowTile = 32;        // query rows per MFMA tile
constexpr int kHeadDim = 128;
constexpr int kMergedSets = 64;     // sets of statistics of a (layer, sequence) that the second pass merges itself
constexpr int kScoreWaves = 4;      // waves per workgroup in the score kernels

JQ_HD int lesser(int a, int b) { return a < b ? a : b; }
JQ_HD int greater(int a, int b) { return a > b ? a : b; }

// Largest s with cu[s] <= v (cu[0] = 0, strictly increasing, v < cu[n]).
template <class Table>  // a pointer to int32_t, in whatever memory
JQ_HD int find_seq(Table cu, int n, int64_t v) {
    int lo = 0, hi = n;  // answer in [lo, hi)
    while (hi - lo > 1) {
        int mid = (lo + hi) >> 1;
        if ((int64_t)cu[mid] <= v) lo = mid; else hi = mid;
    }
    return lo;
}

// x / d for the d that `inv` was made of (ceil(2^32 / d), 0 for 1): the product is at most one too large
JQ_HD uint32_t udiv(uint32_t x, uint32_t d, uint32_t inv) {
    const uint32_t q = (uint32_t)((uint64_t)x * inv >> 32), less = (int32_t)(x - q * d) < 0 ? 1u : 0u;
    return inv ? q - less : x;
}

// How the workgroups of a pass over K share the keys out, in quads of 128 keys (four 32-key tiles, one per wave).
struct SplitArgs {
    int32_t n, total;   // evenly: workgroup c of n takes positions c * total / n .. (c + 1) * total / n - 1 of the row of all quads,
    int32_t gap;        // with a gap of this many between sequences, for the start-up that a change of sequence costs
    int32_t per_layer;  // positions per layer (the gap behind it included), or workgroups per layer
    int32_t whole;      // 1: whole workgroups for every sequence
    int32_t q;          // total / n
    uint32_t inv_n, inv_total, inv_layer;  // inverse() of n, total, per_layer
};
inline uint32_t inverse(int32_t d) { return d == 1 ? 0u : (uint32_t)((0x100000000ull + (uint32_t)d - 1) / (uint32_t)d); }  // of the device's udiv()
struct Split {
    SplitArgs args;
    int32_t n_wg;       // workgroups per KV head (and group of query rows)
    int32_t n_sets;     // sets of statistics per KV head that a first pass shared out like this leaves
    int32_t max_sets;   // ... of one (layer, sequence) at most
    bool fewer;         // there are fewer workgroups than the chip has room for, for no more than kMergedSets sets
    int32_t cu[JQ_MAX_SEQ + 1];  // first position, or workgroup, of every sequence in a layer
};

// How the passes over K share the keys out.  `chunk` (keys per wave, a knob) gives every sequence whole workgroups of four waves
// with about that many.  Without it as many workgroups as make one per CU, or two, share the quads: whole ones for every
// (layer, sequence), as many as keep the longest of them shortest, or all quads dealt evenly, whichever has the shorter longest
// workgroup.  Many short sequences get a workgroup each.  `first`: the split is a first pass's (the second pass alone has no
// statistics to merge).
template <class P>
static Split make_split(const P& p, int32_t chunk, int32_t max_quads, bool tight, bool first = true) {
    Split x{};
    const int64_t n_quads = (int64_t)p.n_layers * p.cu_quad[p.n_seq], units = (int64_t)p.n_layers * p.n_seq;
    auto pieces = [&](int32_t keys) {
        for (int s = 0; s < p.n_seq; ++s) {
            const int32_t L = p.tab.cu_seq[s + 1] - p.tab.cu_seq[s], n = (L - 1) / (kScoreWaves * keys) + 1;
            x.cu[s + 1] = x.cu[s] + n;
            x.max_sets = std::max(x.max_sets, n);
        }
        x.args.whole = 1;
        x.args.per_layer = x.cu[p.n_seq];
        x.args.inv_layer = inverse(x.args.per_layer);
        x.n_wg = x.n_sets = p.n_layers * x.args.per_layer;
        return x;
    };
    if (chunk) return pieces(chunk);
    const int64_t per = (int64_t)p.h_kv * p.row_groups;
    // A workgroup's time in quads of either pass (1.25 us each where the whole chip streams); a change of sequence (query rows,
    // statistics, another merge) costs about as much as kStartUp of them (5.6 us in the first pass, 7 in the second).  More than
    // kMergedSets sets of a (layer, sequence) take a launch that merges them and two for the passes.
    constexpr double kStartUp = 5.0, kMerge = 2.7;
    struct Deal {
        int64_t n;      // workgroups per head (and group of query rows)
        int64_t steps;  // whole workgroups with at most that many quads each; 0: dealt evenly
        int64_t gap;
        double cost;    // of the longest workgroup
    };
    // The best of n workgroups at `quad` a quad and `start` a share.
    auto deal = [&](int64_t n, double quad, double start) {
        Deal d{n, 0, 0, 0.0};
        auto whole = [&](int64_t steps) {  // workgroups per layer with at most that many quads each
            int64_t wgs = 0;
            for (int s = 0; s < p.n_seq; ++s) wgs += (p.cu_quad[s + 1] - p.cu_quad[s] + steps - 1) / steps;
            return wgs;
        };
        int64_t steps = 0;  // the fewest that n workgroups can do with; 0: more (layer, sequence)s than workgroups
        if (units <= n) {
            int64_t lo = (n_quads + n - 1) / n, hi = max_quads;
            while (lo < hi) {
                const int64_t mid = (lo + hi) / 2;
                if (p.n_layers * whole(mid) <= n) hi = mid; else lo = mid + 1;
            }
            steps = lo;
        }
        auto longest = [&](int64_t gap) {
            const int64_t total = n_quads + (units - 1) * gap;
            double worst = 0.0;
            int64_t u0 = 0;
            int32_t s = 0;
            for (int64_t c = 0, b0 = 0; c < n; ++c) {
                const int64_t b1 = (c + 1) * total / n;
                int64_t quads = 0, shares = 0;
                for (;;) {
                    const int64_t nq = p.cu_quad[s + 1] - p.cu_quad[s], lo = std::max(b0, u0), hi = std::min(b1, u0 + nq);
                    if (hi > lo) { quads += hi - lo; ++shares; }
                    if (b1 < u0 + nq + gap || (b1 == total && u0 + nq >= total)) break;
                    u0 += nq + gap;
                    if (++s == p.n_seq) s = 0;
                    if (u0 >= b1) break;
                }
                worst = std::max(worst, quad * (double)quads + start * (double)shares);
                b0 = b1;
            }
            return worst;
        };
        // (A workgroup that comes to more than one sequence may take fewer keys: a gap between sequences in the row that is dealt.)
        const double one = quad * (double)steps + start;  // whole workgroups
        d.cost = 1e300;
        if (units > 1 && units <= 1024 && n > 1) {
            d.cost = longest(0);
            const double gapped = n_quads / n > (int64_t)kStartUp ? longest((int64_t)kStartUp) : 1e300;
            if (gapped < d.cost) { d.cost = gapped; d.gap = (int64_t)kStartUp; }
        } else if (units > 1) {  // many sequences, a few to every workgroup
            d.cost = quad * (double)(n_quads / n) + start * (double)(units / n + 1);
        }
        if (steps && one <= d.cost) d = Deal{n, steps, 0, one};
        const int64_t each = d.steps ? d.steps : n_quads / n;  // quads of a (layer, sequence) that one workgroup takes, at least
        if (first && !p.by_rows && (d.steps ? (max_quads - 1) / each + 1 : (max_quads - 2) / each + 2) > kMergedSets) d.cost += kMerge;
        return d;
    };
    // Of n workgroups per head as many as there are keys for, down to a quad each: 4096 tokens and 8 heads 17.6 us a call, with two
    // quads each 19.0; 2000 tokens 17.2 / 19.0.  With many query rows two, which halves the sets of statistics (1024 rows x 2048
    // keys 34.7 / 34.8), but a workgroup for every (layer, sequence): 256 rows, 8 layers of 37 keys 22.1 us, two to a workgroup 27.4.
    auto at_most = [&](int64_t n) {
        n = std::min(n, n_quads);
        return p.by_rows ? std::min(n, std::max(units, (n_quads + 1) / 2)) : n;
    };
    // (With many query rows the keys come out of the caches and arithmetic is the bound: two workgroups per CU hide each other's
    // start-ups, 1024 rows x 16384 keys 94.4 -> 93.3 us per evaluation step, x 131072 keys 531 -> 511, training forward 88.6 -> 86.3;
    // three and four lose that again.  With more than about twelve workgroups per head merging takes it back unless they have
    // long to run: 256 rows x 65536 keys of 8 heads 91.6 against 89.6, x 131072 167.9 / 168.8, 1024 rows x 131072 of one head 84.7 / 83.2.)
    const bool pairs = p.by_rows && (per >= 40 || n_quads * per >= 24 * 512);
    const int64_t one_per_cu = tight ? 1 : std::max<int64_t>(1, (pairs ? 512 : 256) / per), n1 = at_most(one_per_cu);
    // 84 % of the CUs take what memory delivers: more make every quad slower, fewer leave it idle.
    constexpr double kEnough = 0.84;
    auto busy = [&](int64_t n, int64_t places) { return std::max(kEnough, (double)(n * per) / (double)places); };
    // Two workgroups per CU hide part of each other's start-ups, and their sweeps take 6 % longer; one for each sequence, 4 %.
    constexpr double kPairStart = 3.55, kPairQuad = 1.065, kEachQuad = 1.04;
    auto one = [&](int64_t n, int64_t per_cu) { return deal(n, p.by_rows || tight ? 1.0 : std::min(1.0, busy(per_cu, 256)), kStartUp); };
    auto two = [&](int64_t n, int64_t per_cu) {
        Deal d = deal(n, kPairQuad * busy(per_cu, 512), kPairStart);
        d.cost *= 2.0;
        return d;
    };
    Deal best = pairs && !tight ? two(n1, one_per_cu) : one(n1, one_per_cu);
    // One or two KV heads: fewer workgroups than CUs, but no sets that a launch of its own would have to merge.  In us, all / at most 64
    // a sequence: 16384 tokens of one head 29.3 / 26.1, 32768 31.7 / 31.5, 50000 147.1 / 149.0; of two heads 24000 35.9 / 32.6, 65536 173.6 /
    // 175.1; of three 131072 46.1 / 42.6 (scores alone).
    if (n1 > kMergedSets && max_quads > kMergedSets && !p.by_rows && first) {
        const int64_t fewer = units == 1 ? kMergedSets : std::max<int64_t>(1, n_quads / ((max_quads + kMergedSets - 3) / (kMergedSets - 2)));
        if (fewer < n1) {
            const Deal d = one(fewer, fewer);
            if (d.cost < best.cost) { best = d; x.fewer = true; }
        }
    }
    // Two workgroups per CU, which takes a launch for either pass (unless there are many query rows), where sequences are short or the
    // heads do not divide the chip.  Where sequences are many and alike, one workgroup for each, which the chip takes up as it
    // has room, beats even portions.  The constants are fitted to 580 calls of 1 to 200 KV heads, 1 to 128 sequences and 1 to
    // 128 layers, each timed all three ways (0.4 % slower than the best of them on average).  Whole calls in us, one workgroup per CU /
    // two, even portions / one for each (layer, sequence):
    //   8 KV heads, 1024 x 512 tokens 769 / 655 / 628, 512 x 3000 1490 / 1463 / 1433, 256 x 300 157 / 129 / 129, 128 x 1024 144 / 137 / 132,
    //   64 x 4096 223 / 229 / 232, 80 x 3000 230 / 222 / 240, 256 of 100 to 3000 292 / 276 / 292;  96 heads, 32 x 2048 907 / 790 / 771,
    //   131072 1371 / 1304, 32768 340 / 337, 8192 77 / 85;  72 heads, 131072 945 / 962;  130 heads, 8192 128 / 113, 32768 550 / 438.
    if (!tight && (2 * units > n1 || (double)(per * n1) < kEnough * 256)) {
        const int64_t n2 = at_most(512 / per);
        if (n2 > n1) {
            const Deal d = two(n2, 512 / per);
            if (d.cost < best.cost) { best = d; x.fewer = false; }
        }
        if (units > n1) {
            // rounds of 512 workgroups, of which the last takes two thirds of the time where its workgroups are alone on a CU; of
            // unequal sequences a long one may come last
            const double rounds = (double)(units * per) / 512.0, rest = rounds - std::floor(rounds);
            const double mean = kEachQuad * (double)n_quads / (double)units + kPairStart, longest = kEachQuad * max_quads + kPairStart;
            const double r = rounds < 1.0 ? 1.0 : std::floor(rounds) + (rest > 0.0 ? 0.67 + 0.66 * std::max(0.0, rest - 0.5) : 0.0);
            const double cost = std::max(2.0 * mean * r, 2.0 * mean * (r - 1.0) + 1.1 * longest + 0.75 * mean) + 0.65;
            if (cost <= best.cost) { best = Deal{units, max_quads, 0, cost}; x.fewer = false; }
        }
    }
    const int64_t n = best.n;
    if (best.steps) {
        x.args.whole = 1;
        for (int s = 0; s < p.n_seq; ++s) {
            const int32_t w = (int32_t)(p.n_seq == 1 && !x.fewer ? n / units : (p.cu_quad[s + 1] - p.cu_quad[s] + best.steps - 1) / best.steps);
            x.cu[s + 1] = x.cu[s] + w;
            x.max_sets = std::max(x.max_sets, w);
        }
        x.args.per_layer = x.cu[p.n_seq];
        x.args.inv_layer = inverse(x.args.per_layer);
        if (p.n_seq == 1) x.args.inv_n = inverse(x.args.per_layer);
        x.n_wg = x.n_sets = p.n_layers * x.args.per_layer;
        return x;
    }
    // The arithmetic of even portions is one of 32 bits: n * total has to stay below 2^32.  A call of 2^24 quads or more (2^31 tokens
    // over all layers, which a paged cache reaches where sequences share pages) has whole workgroups of 2048 quads instead, some
    // 2.5 ms of either pass each: thousands of them, at most 64 per sequence, and no start-up that counts.
    const int64_t total = n_quads + (units - 1) * best.gap;
    if (n * total >= (int64_t)1 << 32) return pieces(2048 * kKeyTile);
    x.args.gap = (int32_t)best.gap;
    x.args.n = (int32_t)n;
    x.args.total = (int32_t)total;
    x.args.per_layer = p.cu_quad[p.n_seq] + p.n_seq * x.args.gap;
    for (int s = 0; s < p.n_seq; ++s) x.cu[s + 1] = p.cu_quad[s + 1] + (s + 1) * x.args.gap;
    x.args.q = x.args.total / x.args.n;
    x.args.inv_n = inverse(x.args.n); x.args.inv_total = inverse(x.args.total); x.args.inv_layer = inverse(x.args.per_layer);
    x.n_wg = (int32_t)n;
    x.n_sets = (int32_t)(units + n - 1);
    x.max_sets = (int32_t)std::min<int64_t>(n, max_quads < 2 ? 1 : (max_quads - 2) / x.args.q + 2);
    return x;
}

// ---- which keys a workgroup sweeps ----------------------------------------------------------------
// The keys of a head, over all layers and sequences of the call, are shared out in steps of four tiles (one per wave), called
// quads; a quad never straddles sequences.  Either every sequence gets whole workgroups, or (evenly) all quads in a row are
// dealt to the workgroups in equal, contiguous portions, whatever sequences those touch: then all finish together, and a
// workgroup has a SHARE of one (layer, sequence) or of several in turn.
// The workgroups that share a (layer, sequence) take its quads in the order in which they reach them, counted in steps on
// every workgroup's own clock, so that all waves that run at the same time sweep one moving window of the key tensor, which
// DRAM serves at close to its streaming rate (one contiguous range per workgroup instead took 49 us cold against 45 on the
// 128K layer).  Dealt evenly, a (layer, sequence) has at most one workgroup that comes to it late (the first), workgroups that
// work on nothing else, and one that leaves early (the last), so the number of quads taken before a workgroup's step i has a
// closed form.
constexpr int kWhole = 0x7FFFFFFF;  // Share::q of a whole workgroup
struct Share {
    int layer, seq, L, seq_tiles;  // seq_tiles: 32-key tiles of the sequence
    int64_t tok0;                  // first token of the sequence in the flattened T axis
    int set0, n_sets, rank;        // sets of statistics of the (layer, sequence): set0 .. set0 + n_sets - 1, here set0 + rank
    int x, len;                    // the workgroup's steps for it: x .. x + len - 1
    int full, at, at_last, q;      // workgroups with nothing else; of those, how many come before this one in a step; in step q
    int late_from, late_n, early;  // first step (counted with its place in a step) and steps of the late one; steps of the early one
    JQ_HD int quad(int i) const {
        return (i < q ? full * i + at : full * q + at_last) + lesser(greater(i - late_from, 0), late_n) + lesser(i, early);
    }
};
template <class S>
JQ_HD int split_start(S& sp, int c) { return (int)udiv((uint32_t)c * (uint32_t)sp.total, (uint32_t)sp.n, sp.inv_n); }
template <class S>
JQ_HD int split_owner(S& sp, int pos) {  // the largest c with split_start(c) <= pos
    return (int)udiv(((uint32_t)pos + 1u) * (uint32_t)sp.n - 1u, (uint32_t)sp.total, sp.inv_total);
}
template <class A>
JQ_HD int quads_of(A& a, int seq) { return a.one_L ? a.layer_quads : a.cu_quad[seq + 1] - a.cu_quad[seq]; }
// sets of statistics of a (layer, sequence); `cu`: the split's table
template <class A, class S, class Table>
JQ_HD void sets_of(A& a, S& sp, Table cu, int layer, int seq, int& set0, int& n) {
    const int at = layer * sp.per_layer + (a.one_L ? 0 : cu[seq]);
    if (sp.whole) {
        set0 = at;
        n = a.one_L ? sp.per_layer : cu[seq + 1] - cu[seq];
        return;
    }
    const int ca = split_owner(sp, at), cb = split_owner(sp, at + quads_of(a, seq) - 1);
    set0 = layer * a.n_seq + seq + ca;  // along the row either the sequence or the workgroup (or both) steps on: no number twice
    n = cb - ca + 1;
}
// the first (or last) (layer, sequence) of workgroup c
template <class A>
JQ_HD void first_share(A& a, int c, bool last, int& layer, int& seq) {
    auto& sp = a.own;
    const int pos = sp.whole ? c : last ? split_start(sp, c + 1) - 1 : split_start(sp, c);
    layer = a.n_layers == 1 ? 0 : (int)udiv((uint32_t)pos, (uint32_t)sp.per_layer, sp.inv_layer);
    seq = a.one_L ? 0 : find_seq(a.cu_wg, a.n_seq, pos - layer * sp.per_layer);
    if (!last && !sp.whole && pos - layer * sp.per_layer - (a.one_L ? 0 : a.cu_wg[seq]) >= quads_of(a, seq))  // in the gap behind it
        if (++seq == a.n_seq) { seq = 0; ++layer; }
}
template <class A>
JQ_HD Share share_of(A& a, int c, int layer, int seq) {
    auto& sp = a.own;
    Share h;
    h.layer = layer; h.seq = seq;
    h.tok0 = a.one_L ? 0 : a.cu_seq[seq];
    h.L = a.one_L ? a.one_L : a.cu_seq[seq + 1] - a.cu_seq[seq];
    h.seq_tiles = (h.L + kKeyTile - 1) / kKeyTile;
    const int nq = (h.seq_tiles + kScoreWaves - 1) / kScoreWaves;
    sets_of(a, sp, a.cu_wg, layer, seq, h.set0, h.n_sets);
    h.late_from = h.late_n = h.early = h.at_last = 0;
    if (sp.whole) {
        h.rank = c - h.set0;
        h.x = 0;
        const uint32_t steps = (uint32_t)(nq - h.rank + h.n_sets - 1);  // >= n_sets: no more workgroups than quads
        h.len = (int)(sp.inv_n ? udiv(steps, (uint32_t)h.n_sets, sp.inv_n) : steps / (uint32_t)h.n_sets);
        h.full = h.n_sets; h.at = h.rank; h.q = kWhole;
        return h;
    }
    const int ca = h.set0 - (layer * a.n_seq + seq), cb = ca + h.n_sets - 1;
    const int q0 = layer * sp.per_layer + (a.one_L ? 0 : a.cu_wg[seq]), b0 = split_start(sp, c), b1 = split_start(sp, c + 1);
    h.rank = c - ca;
    h.x = greater(b0, q0) - b0;
    h.len = lesser(b1, q0 + nq) - b0 - h.x;
    h.q = sp.q;
    if (h.n_sets == 1) {
        h.full = h.at = 0;
        h.late_from = h.x; h.late_n = h.len;
    } else {
        h.full = h.n_sets - 2;
        h.at = lesser(greater(h.rank - 1, 0), h.full);
        const int s1 = split_start(sp, ca + 1);
        h.at_last = c == ca ? 0 : b0 - s1 - h.q * h.at;
        h.late_from = q0 - split_start(sp, ca) - (c > ca ? 1 : 0);
        h.late_n = s1 - q0;
        h.early = q0 + nq - split_start(sp, cb);
    }
    return h;
}

// The tiles of one wave of a share in the order in which it takes them, forwards or backwards: their numbers rise evenly but for
// the few steps at which another workgroup joins or leaves (Share::quad for every tile cost the sweeps a twentieth: a wave
// issues in order, and the matrix core waits meanwhile).
template <bool BACK>
struct Walk {
    int i, t, stride, left;  // step, its tile, distance to the next step's and for how many more steps it holds
    JQ_HD void turn(const Share& h) {
        if (h.q == kWhole) {  // whole workgroups: one distance throughout (2048 tokens 15.3 -> 15.0 us a call, 32768 41.3 -> 40.8)
            stride = kScoreWaves * (BACK ? -h.full : h.full);
            left = 0x7FFFFFFF;
            return;
        }
        const int at[5] = {h.q - 1, h.q, h.late_from, h.late_from + h.late_n, h.early};
        int next = BACK ? -1 : 0x7FFFFFFF;
#pragma unroll
        for (int k = 0; k < 5; ++k)
            if (BACK ? at[k] < i : at[k] > i) next = BACK ? greater(next, at[k]) : lesser(next, at[k]);
        stride = kScoreWaves * (BACK ? h.quad(i - 1) - h.quad(i) : h.quad(i + 1) - h.quad(i));
        left = BACK ? i - next : next - i;
    }
    JQ_HD void start(const Share& h, int from, int wave) {
        i = from;
        t = kScoreWaves * h.quad(i) + wave;
        turn(h);
    }
    JQ_HD void step(const Share& h) {
        i += BACK ? -1 : 1;
        t += stride;
        if (__builtin_expect(--left == 0, 0)) turn(h);
    }
};

// Where workgroup `b` of the launch (below 2^31: 32-bit arithmetic) starts: its KV head, group of query rows, number among their
// workgroups, and its first share (`last`: it takes its shares from the end, and `b` counts the launch's workgroups from there).
struct Place { int g, rg, c, layer, seq; };
template <class A>
JQ_HD Place place_of(A& a, uint32_t b, bool last) {
    Place at;
    uint32_t rest = udiv(b, (uint32_t)a.h_kv, a.inv_h_kv);
    at.g = (int)(b - rest * (uint32_t)a.h_kv);  // heads vary fastest: neighbouring workgroups read neighbouring 256-byte pieces of a token row
    at.rg = a.rg0;
    if (a.n_rg > 1) {  // row groups next: the workgroups that read the same keys run side by side (with eight heads on one XCD)
        at.rg += (int)(rest % (uint32_t)a.n_rg);
        rest /= (uint32_t)a.n_rg;
    }
    at.c = (int)rest;
    first_share(a, at.c, last, at.layer, at.seq);
    return at;
}
// on to the workgroup's next share (the one before it with `last`); false if `h` was the final one
template <class A>
JQ_HD bool next_share(A& a, const Share& h, bool last, Place& at) {
    auto& sp = a.own;
    if (sp.whole) return false;
    if (last) {
        if (h.x <= sp.gap) return false;  // what precedes the (layer, sequence) here is a gap at most
        if (--at.seq < 0) { at.seq = a.n_seq - 1; --at.layer; }
    } else {
        if (h.x + h.len + sp.gap >= split_start(sp, at.c + 1) - split_start(sp, at.c)) return false;
        if (++at.seq == a.n_seq) { at.seq = 0; ++at.layer; }
    }
    return true;
}

// ---- where requests lie ---------------------------------------------------------------------------
// A tile is 32 key rows of 256 B.  Load i (0..7) of a wave moves rows 4i..4i+3: lane l fetches 16 B
// of row r = 4i + (l >> 4), and the hardware stores them at slot + 1024 i + 16 l, i.e. at row r,
// physical 16-byte chunk (l & 15).  To realise the swizzle "logical chunk c lives at physical chunk
// c ^ (r & 15)" the lane therefore fetches logical chunk (l & 15) ^ (r & 15) from global memory.
// With (r & 15) = 4 (i & 3) + (l >> 4) the lane's byte offset takes four values over the 8 loads, which differ by an
// exclusive or of 64 (i & 3) (row_bytes is a multiple of 256): one register; the rest of the address is wave-uniform
// (buffer resource + scalar offset).
// Of a partial tile -- the last of a sequence -- only the requests whose first row exists lie inside the sequence; the others
// repeat the last of these (row 0 of it exists, and its rows past the end lie past the end of the resource by the lane part
// of the address, where the hardware returns zeros).  So no request starts outside what the resource covers: a scalar
// minimum per request, nothing else.
JQ_HD uint32_t tile_lane(int lane, uint32_t row_bytes) {  // the offset at i = 0
    const uint32_t a = (uint32_t)lane >> 4;
    return a * row_bytes + ((((uint32_t)lane & 15u) ^ a) << 4);
}
// offset of the last group of four rows that begins inside `n_rows` rows
JQ_HD uint32_t last_request(int n_rows, uint32_t row_bytes) { return ((uint32_t)(n_rows - 1) & ~3u) * row_bytes; }
JQ_HD uint32_t request_offset(uint32_t tile_off, int i, uint32_t row_bytes, uint32_t last) {
    const uint32_t off = tile_off + 4u * (uint32_t)i * row_bytes;
    return off < last ? off : last;
}
// Query rows r0 .. r0 + 31 of a head with 1 << gs query heads per KV head (gs <= 5, r0 a multiple of 32): the same for rows of
// `group` consecutive 256-byte pieces per token.  A tile behind the last token reads from the first one instead.
struct QueryTile {
    int first;             // token the resource starts with
    uint32_t bytes, last;  // its length, and the offset of the last request
};
JQ_HD uint32_t query_offset(int i, int gs, uint32_t tok_bytes, uint32_t group) {
    return ((uint32_t)(4 * i) >> gs) * tok_bytes + ((uint32_t)(4 * i) & (group - 1)) * (kHeadDim * 2);
}
JQ_HD QueryTile query_tile(int n_q, int r0, int gs, uint32_t tok_bytes, uint32_t group) {
    QueryTile q;
    q.first = (r0 >> gs) < n_q ? r0 >> gs : 0;
    const int left = lesser(n_q - q.first, kRowTile);  // tokens that the tile reaches, none past the end
    q.bytes = (uint32_t)(left - 1) * tok_bytes + group * (kHeadDim * 2);
    q.last = query_offset(lesser(((left << gs) - 1) >> 2, 7), gs, tok_bytes, group);
    return q;
}

}  // namespace jq
