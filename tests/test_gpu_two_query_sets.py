"""Both query sets of the training objective's forward value in one sweep (jq_map_mse_fused): the row tiles of the sets follow
each other, so the edges are the sets' last, partly filled tiles, waves whose tiles are all of one set, and waves without any."""
import numpy as np
import pytest

import oracle
import paper_2509_10798_amd as jq
from parity import to_dev_bf16
from workloads import f32_to_bf16_bits

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n_layers,seq_lens,n_a,n_b,h_q,h_kv", [
    (1, [129], 8, 8, 8, 2),          # one tile each: two of the four waves have none; one key past the first group of 128
    (1, [300, 5], 37, 5, 8, 2),      # 148 + 20 rows: the larger set first, a partly filled tile in the middle of the rows
    (2, [513, 33], 11, 43, 9, 3),    # three heads per KV head: 33 + 129 rows, rows of one token straddle tiles
    (1, [260], 2, 5, 64, 1),         # 64 query heads share one KV head
    (3, [127], 32, 128, 4, 1),       # 4 + 16 tiles, every wave one of the first set and four of the second
])
def test_map_mse_of_two_sets_matches_the_oracle(n_layers, seq_lens, n_a, n_b, h_q, h_kv):
    import torch
    assert torch.cuda.is_available(), "these tests need the GPU"
    print("two query sets", n_layers, seq_lens, n_a, n_b, h_q, h_kv, flush=True)
    rng = np.random.default_rng(11)
    ns, T, d, G = len(seq_lens), sum(seq_lens), 128, h_q // h_kv
    K = f32_to_bf16_bits(rng.standard_normal((n_layers, T, h_kv, d)).astype(np.float32))
    Qa, Qb = (f32_to_bf16_bits(rng.standard_normal((n_layers, ns, n, h_q, d)).astype(np.float32)) for n in (n_a, n_b))
    sh = jq.Shape(n_layers=n_layers, seq_lens=seq_lens, n_q=n_a, h_q=h_q, h_kv=h_kv)
    got = jq.map_mse_fused(sh, to_dev_bf16(Qa), to_dev_bf16(Qb), to_dev_bf16(K))
    torch.cuda.synchronize()
    got = got.cpu().numpy()
    cu = np.concatenate([[0], np.cumsum(seq_lens)])
    for layer in range(n_layers):
        for s in range(ns):
            k = K[layer, cu[s]:cu[s + 1]]
            want = oracle.map_mse(oracle.score(Qa[layer, s], k), n_a * G, oracle.score(Qb[layer, s], k), n_b * G)
            # the maps agree with the oracle's to 2e-3 relative per entry (the bar for scores), and so does the mean square of
            # their difference as long as the maps differ by about their own size, twice over: 4e-3, doubled for the sum of both
            np.testing.assert_allclose(got[layer, s], want, rtol=8e-3)
