// Walks every workgroup of a pass over K through its shares, as the kernels do, and checks that the keys are shared out exactly
// once.  Reads calls from stdin, one a line:
//   n_layers n_seq h_kv rows rows2 chunk full L_1 .. L_n_seq
// (query rows per KV head of either set; keys per wave or 0; 1: every quad, 0: share by share).  Prints one line per call:
//   "ok <workgroups per head> <sets> <longest workgroup's quads> <all quads>" or "bad <what>".
#include <cstdio>
#include <string>
#include <vector>

#include "jq_sweep.h"

using namespace jq;

struct Tab { std::vector<int32_t> cu_seq; };
struct Call {  // what make_split reads of a plan
    int32_t n_layers, n_seq, h_kv, row_tiles, row_groups;
    bool by_rows;
    std::vector<int32_t> cu_quad;
    Tab tab;
};
struct Args {  // what a share is found by in a kernel's arguments
    int32_t n_layers, n_seq, h_kv;
    uint32_t inv_h_kv;
    int32_t n_rg, rg0, one_L, layer_quads;
    SplitArgs own;
    std::vector<int32_t> cu_seq, cu_quad, cu_wg;
};

static std::string walk(const Call& p, const Split& sp, bool full, int64_t& longest) {
    Args a{};
    a.n_layers = p.n_layers; a.n_seq = p.n_seq; a.h_kv = p.h_kv; a.inv_h_kv = inverse(p.h_kv);
    a.n_rg = 1;
    a.one_L = p.n_seq == 1 ? p.tab.cu_seq[1] : 0;
    a.layer_quads = p.cu_quad[p.n_seq];
    a.own = sp.args;
    a.cu_seq = p.tab.cu_seq; a.cu_quad = p.cu_quad;
    a.cu_wg.assign(sp.cu, sp.cu + p.n_seq + 1);
    const int64_t units = (int64_t)p.n_layers * p.n_seq;
    std::vector<uint8_t> quad_seen(full ? (size_t)p.n_layers * a.layer_quads : 0), set_seen((size_t)sp.n_sets);
    std::vector<int64_t> taken((size_t)units);
    longest = 0;
    for (int c = 0; c < sp.n_wg; ++c) {
        const uint32_t b = (uint32_t)c * (uint32_t)p.h_kv + (uint32_t)(c % p.h_kv);
        Place at = place_of(a, b, false);
        if (at.c != c || at.g != c % p.h_kv) return "place of a workgroup";
        int64_t len = 0, n_shares = 0;
        std::vector<std::pair<int, int>> order;
        for (;;) {
            if (at.layer < 0 || at.layer >= p.n_layers || at.seq < 0 || at.seq >= p.n_seq) return "share outside the call";
            const Share h = share_of(a, c, at.layer, at.seq);
            const int nq = p.cu_quad[at.seq + 1] - p.cu_quad[at.seq];
            const int64_t unit = (int64_t)at.layer * p.n_seq + at.seq;
            if (h.len < 1 || h.len > nq || h.x < 0) return "length of a share";
            if (h.rank < 0 || h.rank >= h.n_sets || h.set0 < 0 || h.set0 + h.n_sets > sp.n_sets || h.n_sets > sp.max_sets) return "sets of a share";
            if (set_seen[(size_t)(h.set0 + h.rank)]++) return "set number used twice";
            taken[(size_t)unit] += h.len;
            len += h.len;
            for (int wave = 0; wave < kScoreWaves && full; ++wave) {
                Walk<false> to; Walk<true> fro;
                to.start(h, h.x, wave);
                fro.start(h, h.x + h.len - 1, wave);
                for (int k = 0; k < h.len; ++k) {
                    const int q = h.quad(h.x + k);
                    if (q < 0 || q >= nq) return "quad outside its sequence";
                    if (q == nq - 1 && k != h.len - 1) return "the last quad is not its owner's last step";
                    if (to.t != kScoreWaves * q + wave || fro.t != kScoreWaves * h.quad(h.x + h.len - 1 - k) + wave) return "walk and quad differ";
                    if (wave == 0 && quad_seen[(size_t)at.layer * a.layer_quads + p.cu_quad[at.seq] + q]++) return "quad taken twice";
                    to.step(h); fro.step(h);
                }
            }
            if (!full) {
                const int q0 = h.quad(h.x), q1 = h.quad(h.x + h.len - 1);
                if (q0 < 0 || q1 < q0 || q1 >= nq) return "quads of a share";
            }
            order.emplace_back(at.layer, at.seq);
            if (++n_shares > units) return "shares without end";
            if (!next_share(a, h, false, at)) break;
        }
        longest = len > longest ? len : longest;
        Place back = place_of(a, b, true);  // the second pass: the same shares, last one first
        for (;;) {
            if (order.empty() || back.c != c || order.back() != std::make_pair(back.layer, back.seq)) return "shares from the end";
            order.pop_back();
            if (!next_share(a, share_of(a, c, back.layer, back.seq), true, back)) break;
        }
        if (!order.empty()) return "shares from the end";
    }
    for (int64_t u = 0; u < units; ++u)
        if (taken[(size_t)u] != p.cu_quad[u % p.n_seq + 1] - p.cu_quad[u % p.n_seq]) return "quads left out";
    return "";
}

int main() {
    int n_layers, n_seq, h_kv, rows, rows2, chunk, full;
    while (std::scanf("%d %d %d %d %d %d %d", &n_layers, &n_seq, &h_kv, &rows, &rows2, &chunk, &full) == 7) {
        Call p;
        p.n_layers = n_layers; p.n_seq = n_seq; p.h_kv = h_kv;
        p.row_tiles = (rows + 31) / 32 + (rows2 + 31) / 32;
        p.row_groups = (p.row_tiles + 3) / 4;
        p.by_rows = p.row_groups > 1 || rows2 > 0;
        p.cu_quad.assign(1, 0); p.tab.cu_seq.assign(1, 0);
        int max_quads = 0;
        for (int s = 0; s < n_seq; ++s) {
            int L;
            if (std::scanf("%d", &L) != 1) return 1;
            const int n = (L + kScoreWaves * kKeyTile - 1) / (kScoreWaves * kKeyTile);
            p.tab.cu_seq.push_back(p.tab.cu_seq.back() + L);
            p.cu_quad.push_back(p.cu_quad.back() + n);
            max_quads = n > max_quads ? n : max_quads;
        }
        const Split sp = make_split(p, chunk, max_quads, false);
        int64_t longest = 0;
        const std::string bad = walk(p, sp, full != 0, longest);
        if (bad.empty()) std::printf("ok %d %d %lld %lld\n", sp.n_wg, sp.n_sets, (long long)longest, (long long)p.n_layers * p.cu_quad[n_seq]);
        else std::printf("bad %s\n", bad.c_str());
    }
    return 0;
}
