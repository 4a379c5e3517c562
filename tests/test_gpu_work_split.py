"""How the sequences are cut into workgroups is planned from the call's size (one workgroup per CU where they divide evenly,
several rounds of smaller ones otherwise).  Whatever the cut, every key is scored once and every statistic counted once:
scores agree with those of the smallest cut, 64 keys per wave, up to the rounding of differently grouped sums."""
import numpy as np
import pytest

import paper_2509_10798_amd as jq

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n_layers,seq_lens,h_q,h_kv", [
    (1, [32768], 32, 8),                     # 256 workgroups, eight tiles per wave
    (5, [9999], 16, 8),                      # an odd length over five layers: uneven waves, a partial last tile
    (3, [20011, 31, 4099, 1, 12345], 8, 8),  # ragged, with sequences of less than a tile and of less than a workgroup's waves
    (2, [9999, 70], 8, 8),                   # one query-row tile
    (16, [4097], 8, 2),                      # one key past a whole number of tiles
    (2, [54579], 16, 8),                     # 256 workgroups, 27 tiles in some waves and 26 in others
    (2, [65536], 8, 1),                      # one KV head: more than 64 workgroups per sequence (merged by a launch of their own)
])
def test_scores_do_not_depend_on_the_cut(knobs, n_layers, seq_lens, h_q, h_kv):
    import torch
    assert torch.cuda.is_available(), "these tests need the GPU"
    print("work split", n_layers, seq_lens, h_q, h_kv, flush=True)
    gen = torch.Generator(device="cuda")
    gen.manual_seed(3)
    T, n_q = sum(seq_lens), 32
    Q = torch.randn((n_layers, len(seq_lens), n_q, h_q, 128), generator=gen, device="cuda").bfloat16()
    K = torch.randn((n_layers, T, h_kv, 128), generator=gen, device="cuda").bfloat16()
    sh = jq.Shape(n_layers=n_layers, seq_lens=seq_lens, n_q=n_q, h_q=h_q, h_kv=h_kv)
    planned = jq.score(sh, Q, K)
    torch.cuda.synchronize()
    knobs(JQ_CHUNK_KEYS="64")
    small = jq.score(sh, Q, K)
    torch.cuda.synchronize()
    # A score sums n_q * group terms whose normalisers are fp32 sums in another order, each of a dozen levels of rounding (lane,
    # wave, workgroup, sequence) at 6e-8: 1.2e-6 is the most that cuts of 64 and 512 keys moved a score over the calls of
    # perf/cases.py, and 3e-6 two and a half times that.
    np.testing.assert_allclose(planned.cpu().numpy(), small.cpu().numpy(), rtol=3e-6)
    at = 0
    for L in seq_lens:
        np.testing.assert_allclose(planned[:, :, at:at + L].double().sum(-1).cpu().numpy(), n_q * h_q / h_kv, rtol=1e-5)
        at += L


@pytest.mark.parametrize("n_layers,seq_lens,h_q,h_kv", [(1, [16384], 4, 1), (2, [9999, 300], 4, 2)])
def test_scores_from_supplied_normalisers_do_not_depend_on_the_cut(knobs, n_layers, seq_lens, h_q, h_kv):
    # the second pass alone has no sets to merge and shares the keys out more finely than a call of both
    import torch
    assert torch.cuda.is_available(), "these tests need the GPU"
    print("work split with normalisers", n_layers, seq_lens, h_q, h_kv, flush=True)
    gen = torch.Generator(device="cuda")
    gen.manual_seed(4)
    T, n_q = sum(seq_lens), 32
    Q = torch.randn((n_layers, len(seq_lens), n_q, h_q, 128), generator=gen, device="cuda").bfloat16()
    K = torch.randn((n_layers, T, h_kv, 128), generator=gen, device="cuda").bfloat16()
    lse = 9.0 + torch.rand((n_layers, len(seq_lens), n_q, h_q), generator=gen, device="cuda")
    sh = jq.Shape(n_layers=n_layers, seq_lens=seq_lens, n_q=n_q, h_q=h_q, h_kv=h_kv)
    planned = jq.score(sh, Q, K, lse=lse)
    torch.cuda.synchronize()
    knobs(JQ_CHUNK_KEYS="64")
    small = jq.score(sh, Q, K, lse=lse)
    torch.cuda.synchronize()
    assert torch.equal(planned, small)  # a key's sum is formed by one wave, in the same order whatever the cut
