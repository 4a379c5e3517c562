"""Rows of pooled scores that start at any multiple of four bytes: every alignment, and sequence ends at every distance from a run's,
in the pooling kernel and in the one-kernel tail."""
import numpy as np
import pytest

import oracle
import paper_2509_10798_amd as jq

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("seq_lens", [[1021], [5, 1023, 2050, 1], [8191, 3], [33001, 6, 1025], [20003, 30]])
@pytest.mark.parametrize("n_layers,h_kv", [(1, 3), (5, 8)])
def test_pooled_scores_of_rows_at_any_alignment(seq_lens, n_layers, h_kv):
    import torch
    assert torch.cuda.is_available(), "these tests need the GPU"
    print("odd rows", seq_lens, n_layers, h_kv, flush=True)
    gen = torch.Generator(device="cuda")
    gen.manual_seed(2)
    T = sum(seq_lens)
    Q = torch.randn((n_layers, len(seq_lens), 4, h_kv, 128), generator=gen, device="cuda").bfloat16()
    K = torch.randn((n_layers, T, h_kv, 128), generator=gen, device="cuda").bfloat16()
    sh = jq.Shape(n_layers=n_layers, seq_lens=seq_lens, n_q=4, h_q=h_kv, h_kv=h_kv, budgets=[max(1, L // 8) for L in seq_lens])
    raw = jq.score(sh, Q, K)
    for off in range(4):  # the output's own alignment
        flat = torch.full((n_layers * h_kv * T + 8,), float("nan"), device="cuda")
        out = flat[off:off + n_layers * h_kv * T].view(n_layers, h_kv, T)
        got = jq.evict(sh, Q, K, K, scores_out=out)[3]
        alone = jq.pool(sh, raw)
        torch.cuda.synchronize()
        assert torch.equal(got, alone)
        assert torch.isnan(flat[:off]).all() and torch.isnan(flat[off + n_layers * h_kv * T:]).all()
    at = 0
    for L in seq_lens:
        ref = oracle.pool(raw[:, :, at:at + L].double().cpu().numpy(), 7)
        np.testing.assert_allclose(alone[:, :, at:at + L].cpu().numpy(), ref, rtol=2e-6)  # seven additions and a product in fp32
        at += L
