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
