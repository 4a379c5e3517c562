"""Both passes over K in one launch (every eviction but the traced one, up to 64 workgroups per sequence and head), and how its
workgroups share the keys: contiguous, equal portions of all sequences in a row, so that workgroups come to several sequences
and sequences to several workgroups."""
import numpy as np
import pytest

import oracle
import paper_2509_10798_amd as jq
from parity import assert_scores_close, to_dev_bf16
from workloads import f32_to_bf16_bits

pytestmark = pytest.mark.gpu


def _inputs(n_layers, seq_lens, n_q, h_q, h_kv, seed=21):
    rng = np.random.default_rng(seed)
    Q = f32_to_bf16_bits(rng.standard_normal((n_layers, len(seq_lens), n_q, h_q, 128)).astype(np.float32))
    K = f32_to_bf16_bits(rng.standard_normal((n_layers, sum(seq_lens), h_kv, 128)).astype(np.float32))
    return Q, K


def _evict(sh, Q, K):
    """Scores (unpooled: pool_k is 1) and kept positions through the fused call."""
    _, _, idx, scores = jq.evict(sh, Q, K, K)
    return scores, idx


SHAPES = [
    (1, [129], 8, 8, 8),                      # two quads of 128 keys, the second with one key
    (1, [4099], 32, 8, 2),                    # whole workgroups for the one sequence, a partial last quad
    (3, [1000, 127, 1, 128, 2049], 16, 8, 8),  # portions that end inside sequences; sequences of a key, of less than and of exactly a quad
    (40, [300], 32, 8, 8),                    # more layers than workgroups per head
    (2, [70] * 30, 4, 4, 1),                  # thirty sequences of less than a quad: a workgroup has many shares
    (5, [9999], 32, 12, 4),                   # layers that do not divide the workgroups; a group of three
    (1, [5000, 200, 3000], 7, 9, 3),          # 21 rows; heads that do not divide the chip
    (9, [300, 1, 129] * 12, 16, 16, 8),       # many short sequences: a workgroup for each, two per CU
    (2, [6000], 4, 130, 130),                 # more heads than half the CUs: two workgroups per CU, even portions
    (12, [100, 1, 300] * 8, 64, 8, 2),        # 256 query rows: a workgroup for every sequence and group of rows
    (1, [9135], 8, 4, 1),                     # one head: 36 sets of statistics, not one for each of 72 quads
]


@pytest.mark.parametrize("n_layers,seq_lens,n_q,h_q,h_kv", SHAPES)
@pytest.mark.parametrize("wait_us", [None, 0])
def test_one_launch_equals_two_and_the_oracle(knobs, n_layers, seq_lens, n_q, h_q, h_kv, wait_us):
    # jq_score runs the passes one after the other on the same shares: the same bits.  Without patience a workgroup forms the
    # missing statistics itself, from the same keys in the same order: the same bits again.
    import torch
    assert torch.cuda.is_available(), "these tests need the GPU"
    print("one launch", n_layers, seq_lens, n_q, h_q, h_kv, wait_us, flush=True)
    Q, K = _inputs(n_layers, seq_lens, n_q, h_q, h_kv)
    Qd, Kd = to_dev_bf16(Q), to_dev_bf16(K)
    sh = jq.Shape(n_layers=n_layers, seq_lens=seq_lens, n_q=n_q, h_q=h_q, h_kv=h_kv, pool_k=1, budgets=[max(1, L // 8) for L in seq_lens])
    if wait_us is not None:
        knobs(JQ_WAIT_US=str(wait_us))
    got, _ = _evict(sh, Qd, Kd)
    two = jq.score(sh, Qd, Kd)
    torch.cuda.synchronize()
    assert torch.equal(got, two)
    got = got.cpu().numpy()
    cu = np.concatenate([[0], np.cumsum(seq_lens)])
    for layer in {0, n_layers - 1}:
        for s, L in enumerate(seq_lens):
            ref = oracle.score(Q[layer, s], K[layer, cu[s]:cu[s + 1]])
            assert_scores_close(got[layer, :, cu[s]:cu[s + 1]], ref, n_q * (h_q // h_kv) / L, "layer %d seq %d" % (layer, s))


@pytest.mark.parametrize("L", [3000, 40000])  # the flags are cleared by the short tail's kernel, by the pooling kernel
def test_replays_of_a_captured_eviction_wait_for_their_own_statistics(L):
    # A replay's flags have the same value as the one before it: they have to be cleared in between, or the second pass would
    # take the statistics of the keys that the buffers held before.
    import torch
    assert torch.cuda.is_available(), "these tests need the GPU"
    print("captured eviction", L, flush=True)
    gen = torch.Generator(device="cuda")
    gen.manual_seed(5)

    def new(*size):
        return torch.randn(size, generator=gen, device="cuda").bfloat16()
    sh = jq.Shape(n_layers=2, seq_lens=[L], n_q=16, h_q=16, h_kv=8, budgets=[200])
    Q, K = new(2, 1, 16, 16, 128), new(2, L, 8, 128)
    out = dict(zip(("K_out", "V_out", "idx_out", "scores_out"), jq.evict(sh, Q, K, K)))
    ws = jq.alloc_workspace(sh)
    side = torch.cuda.Stream()
    side.wait_stream(torch.cuda.current_stream())
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph, stream=side):
        jq.evict(sh, Q, K, K, ws=ws, **out)
    for i in range(4):
        Q.copy_(new(2, 1, 16, 16, 128) * (1.0 + i))  # other logits, other normalisers
        K.copy_(new(2, L, 8, 128))
        graph.replay()
        torch.cuda.synchronize()
        want = jq.evict(sh, Q, K, K)
        torch.cuda.synchronize()
        for a, b in zip(("K_out", "V_out", "idx_out", "scores_out"), want):
            assert torch.equal(out[a].view(torch.int16), b.view(torch.int16)), (i, a)


@pytest.mark.parametrize("seq_lens,n_q", [([70, 33, 129], 8), ([1], 8), ([200], 40)])  # 16 and 80 query rows per head; 160: streamed rows
@pytest.mark.parametrize("h_q", [4, 8])
def test_rest_of_a_page_may_hold_anything(seq_lens, n_q, h_q):
    # the last tile of a sequence is fetched whole: keys behind the sequence's end, NaN here, must not reach any score
    import torch
    assert torch.cuda.is_available(), "these tests need the GPU"
    print("rest of a page", seq_lens, n_q, h_q, flush=True)
    h_kv, page = 2, 64
    Q, K = _inputs(1, seq_lens, n_q, h_q, h_kv, seed=22)
    n_pages = sum(-(-L // page) for L in seq_lens) + 1
    pool = torch.full((1, n_pages, page, h_kv, 128), float("nan"), dtype=torch.bfloat16, device="cuda")
    table = torch.zeros((len(seq_lens), max(-(-L // page) for L in seq_lens)), dtype=torch.int32)
    Kd, at, nxt = to_dev_bf16(K), 0, 1
    for s, L in enumerate(seq_lens):
        for j in range(0, L, page):
            table[s, j // page] = nxt
            n = min(page, L - j)
            pool[0, nxt, :n] = Kd[0, at + j:at + j + n]
            nxt += 1
        at += L
    sh = jq.Shape(n_layers=1, seq_lens=seq_lens, n_q=n_q, h_q=h_q, h_kv=h_kv, pool_k=1, budgets=[max(1, L // 4) for L in seq_lens])
    pages = jq.Pages(page, n_pages, table.cuda())
    two = jq.score_paged(sh, pages, to_dev_bf16(Q), pool)
    got = jq.evict_paged(sh, pages, to_dev_bf16(Q), pool, pool)[3]
    torch.cuda.synchronize()
    cu = np.concatenate([[0], np.cumsum(seq_lens)])
    for x in (two.cpu().numpy(), got.cpu().numpy()):
        for s, L in enumerate(seq_lens):
            assert_scores_close(x[0, :, cu[s]:cu[s + 1]], oracle.score(Q[0, s], K[0, cu[s]:cu[s + 1]]), n_q * (h_q // h_kv) / L, "seq %d" % s)


@pytest.mark.parametrize("n_q,h_q,h_kv", [(5, 4, 2), (7, 8, 1), (33, 8, 2), (20, 2, 2), (3, 64, 1), (45, 8, 2), (3, 12, 4)])
@pytest.mark.parametrize("L", [1, 33, 131, 4099])
def test_nothing_behind_queries_and_keys_is_read(n_q, h_q, h_kv, L):
    # row and key tiles that end in the middle: what follows the tensors in memory, NaN here, must not reach any score
    import torch
    assert torch.cuda.is_available(), "these tests need the GPU"
    print("behind the tensors", n_q, h_q, h_kv, L, flush=True)
    Q, K = _inputs(1, [L], n_q, h_q, h_kv, seed=23)

    def at_the_start_of_more(x):
        d = to_dev_bf16(x)
        more = torch.full((d.numel() + 64 * 64 * 128 * 4,), float("nan"), dtype=torch.bfloat16, device="cuda")
        more[:d.numel()] = d.view(-1)
        return more[:d.numel()].view(d.shape)
    Qd, Kd = at_the_start_of_more(Q), at_the_start_of_more(K)
    sh = jq.Shape(n_layers=1, seq_lens=[L], n_q=n_q, h_q=h_q, h_kv=h_kv, pool_k=1, budgets=[max(1, L // 4)])
    two = jq.score(sh, Qd, Kd)
    one, _ = _evict(sh, Qd, Kd)
    torch.cuda.synchronize()
    ref = oracle.score(Q[0, 0], K[0])
    for x in (two, one):
        assert_scores_close(x[0].cpu().numpy(), ref, n_q * (h_q // h_kv) / L)


def _timed(torch, run):
    import time
    torch.cuda.synchronize()
    t = time.perf_counter()
    run()
    torch.cuda.synchronize()
    return time.perf_counter() - t


def _eviction(torch, n_layers, L, seed):
    gen = torch.Generator(device="cuda")
    gen.manual_seed(seed)
    Q = torch.randn((n_layers, 1, 32, 32, 128), generator=gen, device="cuda").bfloat16()
    K = torch.randn((n_layers, L, 8, 128), generator=gen, device="cuda").bfloat16()
    sh = jq.Shape(n_layers=n_layers, seq_lens=[L], n_q=32, h_q=32, h_kv=8, budgets=[256])
    out = dict(zip(("K_out", "V_out", "idx_out", "scores_out"), jq.evict(sh, Q, K, K)))
    ws = jq.alloc_workspace(sh)
    torch.cuda.synchronize()
    return lambda: jq.evict(sh, Q, K, K, ws=ws, **out), out


@pytest.mark.parametrize("wait_us", [None, 0])
@pytest.mark.parametrize("n_layers,L", [(1, 4096), (1, 32768), (3, 40000)])
def test_evictions_on_two_streams_share_the_chip(knobs, n_layers, L, wait_us):
    # workgroups of one call may find those that they share a sequence with not yet running: the same bits, and no time lost
    import torch
    assert torch.cuda.is_available(), "these tests need the GPU"
    print("two streams", n_layers, L, wait_us, flush=True)
    calls = [_eviction(torch, n_layers, L, seed) for seed in (1, 2)]
    want = [{k: x.clone() for k, x in out.items()} for _, out in calls]
    if wait_us is not None:
        knobs(JQ_WAIT_US=str(wait_us))
    streams = [torch.cuda.Stream(), torch.cuda.Stream()]

    def loop(which, n=50):
        for _ in range(n):
            for (call, _), st in zip(calls, which):
                with torch.cuda.stream(st):
                    call()
    loop([streams[0]] * 2, 3)
    alone = _timed(torch, lambda: loop([streams[0]] * 2))
    for _, out in calls:
        for x in out.values():
            x.zero_()
    torch.cuda.synchronize()
    both = min(_timed(torch, lambda: loop(streams)) for _ in range(3))
    for (_, out), w in zip(calls, want):
        for k in out:
            assert torch.equal(out[k].view(torch.int16), w[k].view(torch.int16)), k
    assert both < 2.0 * alone + 2e-3, (both, alone)


def test_more_workgroups_than_the_chip_runs_do_not_wait_for_each_other(knobs):
    # 512 keys per wave: 512 workgroups of a CU each.  With both passes in one launch the first half would wait for the other,
    # here a tenth of a second.
    import torch
    assert torch.cuda.is_available(), "these tests need the GPU"
    print("512 workgroups", flush=True)
    _, out = _eviction(torch, 1, 131072, 3)
    want = out["idx_out"].clone()
    knobs(JQ_CHUNK_KEYS="512", JQ_WAIT_US="100000")
    call, out = _eviction(torch, 1, 131072, 3)
    assert _timed(torch, call) < 0.05
    # (another cut, another order of the sums: 3e-6 of a score, far less than what stands between most kept and dropped sums)
    for got, ref in zip(out["idx_out"][0].tolist(), want[0].tolist()):
        assert len(set(got) & set(ref)) >= 250
