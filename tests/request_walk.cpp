// Where the requests for key tiles and query rows lie: every one starts inside what its buffer resource covers, a lane of an
// existing row reads that row, and any other lane reads rows of the same resource or falls behind its end by the lane part of its
// address alone.  Prints "ok", or what is wrong first.
#include <cstdio>
#include <cstdlib>

#include "jq_sweep.h"

using namespace jq;

static void bad(const char* what, int a, int b, int c, int i, int lane) {
    std::printf("bad %s: %d %d %d, request %d, lane %d\n", what, a, b, c, i, lane);
    std::exit(0);
}

int main() {
    for (uint32_t h_kv : {1u, 2u, 3u, 8u, 256u}) {
        const uint32_t rb = h_kv * kHeadDim * 2;
        for (int L = 1; L <= 200; ++L) {
            const uint32_t bytes = (uint32_t)(L - 1) * rb + kHeadDim * 2, last = last_request(L, rb);
            for (int t = 0; t * kKeyTile < L; ++t)
                for (int i = 0; i < 8; ++i) {
                    const uint32_t off = request_offset((uint32_t)t * kKeyTile * rb, i, rb, last);
                    if (off >= bytes) bad("key request behind the end", (int)h_kv, L, t, i, 0);
                    for (int lane = 0; lane < 64; ++lane) {
                        const uint32_t v = tile_lane(lane, rb) ^ (64u * (uint32_t)(i & 3)), at = off + v;
                        const int row = t * kKeyTile + 4 * i + (lane >> 4), chunk = (lane & 15) ^ (row & 15);
                        if (row < L ? at != (uint32_t)row * rb + 16u * (uint32_t)chunk : at + 16 > bytes && v < bytes - off) bad("key lane", (int)h_kv, L, t, i, lane);
                    }
                }
        }
    }
    for (int gs = 0; gs <= 5; ++gs)
        for (int h_kv : {1, 2, 3, 8})
            for (int n_q = 1; n_q <= 70; ++n_q) {
                const uint32_t group = 1u << gs, tok = (uint32_t)h_kv * group * kHeadDim * 2;
                const int rows = n_q << gs, tiles = (rows + kRowTile - 1) / kRowTile;
                for (int rt = 0; rt < tiles + 3; ++rt) {  // a launch of four tiles a group reaches past the last one
                    const QueryTile q = query_tile(n_q, rt * kRowTile, gs, tok, group);
                    if (q.first < 0 || (uint64_t)q.first * tok + q.bytes > (uint64_t)(n_q - 1) * tok + group * kHeadDim * 2) bad("query rows covered", gs, h_kv, n_q, rt, 0);
                    for (int i = 0; i < 8; ++i) {
                        const uint32_t full = query_offset(i, gs, tok, group), off = full < q.last ? full : q.last;
                        if (off >= q.bytes) bad("query request behind the end", gs, h_kv, n_q, i, rt);
                        for (int lane = 0; lane < 64; ++lane) {
                            const uint32_t rl = (uint32_t)lane >> 4, piece = ((uint32_t)lane & 15u) ^ rl;
                            const uint32_t v = ((rl >> gs) * tok + (rl & (group - 1)) * kHeadDim * 2 + (piece << 4)) ^ (64u * (uint32_t)(i & 3));
                            const int r = 4 * i + (lane >> 4), row = rt * kRowTile + r;
                            const uint64_t at = (uint64_t)q.first * tok + off + v;
                            if (row < rows && at != (uint64_t)(row >> gs) * tok + ((uint32_t)row & (group - 1)) * kHeadDim * 2 + 16u * ((uint32_t)(lane & 15) ^ (uint32_t)(r & 15)))
                                bad("query lane", gs, h_kv, n_q, i, lane);
                            if (row >= rows && off + v + 16 > q.bytes && v < q.bytes - off) bad("query lane across the end", gs, h_kv, n_q, i, lane);
                        }
                    }
                }
            }
    std::puts("ok");
    return 0;
}
