"""More than 128 query rows per KV head (response tokens as queries): the kernel that holds the keys and streams the
query rows, at the edges of its key groups (128 keys), row tiles (32 rows, four waves) and query grouping, in every form
that reaches it -- prompt-only softmax, supplied normalisers, the soft tokens' own keys, window queries, paged keys."""
import numpy as np
import pytest

import oracle
import paper_2509_10798_amd as jq
from parity import assert_scores_close, to_dev_bf16
from workloads import f32_to_bf16_bits, page_out

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n_layers,seq_lens,n_q,h_q,h_kv", [
    (1, [129], 33, 8, 2),            # 132 rows: a fifth tile with four rows; one key past the first group of 128
    (1, [128, 127, 1], 129, 2, 2),   # no grouping; key groups exactly full, one short, a single key
    (2, [513, 33], 43, 9, 3),        # three heads per KV head: rows of one token straddle row tiles; 129 rows
    (1, [260], 5, 64, 1),            # 64 query heads share one KV head: 320 rows, more heads than a row tile holds
    (1, [700], 97, 32, 4),           # 776 rows: 25 row tiles, waves with 7 and 6 of them
])
@pytest.mark.parametrize("form", ["prompt", "lse", "tail", "window", "paged"])
def test_many_query_rows_match_the_oracle(n_layers, seq_lens, n_q, h_q, h_kv, form):
    import torch
    assert torch.cuda.is_available(), "these tests need the GPU"
    if form == "window" and min(seq_lens) < n_q:
        seq_lens = [max(L, n_q + 1) for L in seq_lens]
    print("many rows", form, n_layers, seq_lens, n_q, h_q, h_kv, flush=True)
    rng = np.random.default_rng(7)
    ns, T, d, G = len(seq_lens), sum(seq_lens), 128, h_q // h_kv
    Q = f32_to_bf16_bits(rng.standard_normal((n_layers, ns, n_q, h_q, d)).astype(np.float32))
    K = f32_to_bf16_bits(rng.standard_normal((n_layers, T, h_kv, d)).astype(np.float32))
    tail = f32_to_bf16_bits(rng.standard_normal((n_layers, ns, n_q, h_kv, d)).astype(np.float32))
    lse = (np.log(np.asarray(seq_lens, dtype=np.float64))[None, :, None, None] + 0.5
           + 0.1 * rng.standard_normal((n_layers, ns, n_q, h_q))).astype(np.float32)
    sh = jq.Shape(n_layers=n_layers, seq_lens=seq_lens, n_q=n_q, h_q=h_q, h_kv=h_kv, window=form == "window")
    Qd, Kd = to_dev_bf16(Q), to_dev_bf16(K)
    if form == "paged":
        Kp, _, table = page_out(K, K, seq_lens, 32, 3)
        got = jq.score_paged(sh, jq.Pages(32, Kp.shape[1], torch.from_numpy(table).cuda()), Qd, to_dev_bf16(Kp))
    else:
        extra = {"lse": {"lse": torch.from_numpy(lse).cuda()}, "tail": {"k_tail": to_dev_bf16(tail)}}.get(form, {})
        got = jq.score(sh, Qd, Kd, **extra)
    torch.cuda.synchronize()
    got = got.cpu().numpy()
    cu = np.concatenate([[0], np.cumsum(seq_lens)])
    for layer in range(n_layers):
        for s, L in enumerate(seq_lens):
            q, k = Q[layer, s], K[layer, cu[s]:cu[s + 1]]
            ref = {"prompt": oracle.score, "paged": oracle.score, "window": oracle.score_window}[form](q, k) if form in ("prompt", "paged", "window") \
                else oracle.score_lse(q, k, lse[layer, s].astype(np.float64)) if form == "lse" else oracle.score_tail(q, k, tail[layer, s])
            seg = got[layer, :, cu[s]:cu[s + 1]]
            if form == "window":
                assert not seg[:, L - n_q:].any()
                seg, ref = seg[:, :L - n_q], ref[:, :L - n_q]
            assert_scores_close(seg, ref, n_q * G / L, "layer %d seq %d" % (layer, s))


@pytest.mark.parametrize("n_layers,seq_lens,n_q,h_q,h_kv", [
    (1, [16384], 64, 32, 8),                 # two groups of rows, eight sets each
    (3, [1000, 127, 1, 2049], 40, 8, 2),     # 160 rows: the last group is partial; workgroups with several sequences
    (40, [130], 33, 4, 1),                   # a set per sequence and group: every workgroup is the last
])
def test_replays_of_captured_scores_merge_their_own_statistics(n_layers, seq_lens, n_q, h_q, h_kv):
    # The workgroup that completes the sets of statistics merges them, by flags that have the same value in every replay: left over
    # from the one before, they would have it merge sets of the keys that the buffers held before.
    import torch
    assert torch.cuda.is_available(), "these tests need the GPU"
    print("captured scores", n_layers, seq_lens, n_q, h_q, h_kv, flush=True)
    gen = torch.Generator(device="cuda")
    gen.manual_seed(9)

    def new(*size):
        return torch.randn(size, generator=gen, device="cuda").bfloat16()
    T, n = sum(seq_lens), len(seq_lens)
    common = dict(n_layers=n_layers, seq_lens=seq_lens, h_q=h_q, h_kv=h_kv, pool_k=1)
    sh, few = jq.Shape(n_q=n_q, budgets=[max(1, L // 4) for L in seq_lens], **common), jq.Shape(n_q=8, **common)
    Q, Qf, K = new(n_layers, n, n_q, h_q, 128), new(n_layers, n, 8, h_q, 128), new(n_layers, T, h_kv, 128)

    def run():
        return (jq.score(sh, Q, K), jq.evict(sh, Q, K, K)[3], jq.map_mse_fused(few, Qf, Q, K))
    run()
    torch.cuda.synchronize()
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph):
        got = run()
    for i in range(4):
        Q.copy_(new(n_layers, n, n_q, h_q, 128) * (1.0 + i))
        K.copy_(new(n_layers, T, h_kv, 128))
        graph.replay()
        torch.cuda.synchronize()
        for a, b in zip(got, run()):
            assert torch.equal(a, b), i
        assert torch.equal(got[0], got[1])
        torch.cuda.synchronize()
        at = 0
        for L in seq_lens:  # every row's probabilities add up to one
            total = got[0][:, :, at:at + L].double().sum(-1)
            assert torch.allclose(total, torch.full_like(total, n_q * h_q / h_kv), rtol=1e-5)
            at += L
