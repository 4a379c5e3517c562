"""Sequences of up to 32768 tokens: pooling, selection and gather in one kernel, at the edges of its instances (runs of
4 / 8 / 16 / 32 positions per thread, 512 and 1024 threads), against the oracle and against the two kernels that longer
sequences take, whose results must be the same bits."""
import numpy as np
import pytest

import oracle
import paper_2509_10798_amd as jq
from parity import to_dev_bf16
from workloads import f32_to_bf16_bits

pytestmark = pytest.mark.gpu


def torch_():
    import torch
    assert torch.cuda.is_available(), "these tests need the GPU"
    return torch


@pytest.mark.parametrize("L", [1, 3, 2047, 2048, 2049, 4096, 4097, 8192, 8193, 16384, 16385, 32767, 32768, 32769])
@pytest.mark.parametrize("kind", ["random", "flat", "ties", "octaves"])
def test_select_is_exact_at_the_edges(L, kind):
    torch = torch_()
    rng = np.random.default_rng(L)
    x = {"random": lambda: rng.standard_normal((1, 2, L)), "flat": lambda: 1.0 + 0.01 * rng.random((1, 2, L)),
         "ties": lambda: np.round(rng.random((1, 2, L)), 1) - 0.5, "octaves": lambda: np.exp(-60.0 * rng.random((1, 2, L)) ** 2)}[kind]().astype(np.float32)
    for B, kf, kl in ((1, 0, 0), (L, 0, 0), (max(1, L // 3), 0, 0), (max(1, L // 2), min(4, L // 4), L // 4)):
        print("short select", kind, L, B, kf, kl, flush=True)
        sh = jq.Shape(n_layers=1, seq_lens=[L], n_q=1, h_q=2, h_kv=2, budgets=[B], keep_first=kf, keep_last=kl)
        got = jq.select_topk(sh, torch.from_numpy(x).cuda())
        torch.cuda.synchronize()
        np.testing.assert_array_equal(got.cpu().numpy()[0], oracle.select_topk(x[0].astype(np.float64), B, kf, kl))


@pytest.mark.parametrize("L", [200, 5000, 20000, 32768])
@pytest.mark.parametrize("share", [0.01, 0.7, 1.0])
def test_select_keeps_apart_what_always_stays_and_nan_of_all_ones(L, share):
    # a caller's values may hold any bits: a NaN of all ones ranks above every number, is counted like any other value, and
    # the positions that come out are each a position of the sequence
    torch = torch_()
    rng = np.random.default_rng(L)
    bits = rng.random((1, 2, L)).astype(np.float32).view(np.uint32)
    ones = rng.random((1, 2, L)) < share
    bits[ones] = 0x7FFFFFFF
    rank = np.where(ones[0], 2.0, bits.view(np.float32)[0].astype(np.float64))  # numbers are below 1
    for B, kf, kl in ((L // 2, 0, 0), (max(1, L // 200), 0, 0), (L // 3, 5, 17), (L - 1, 0, 1)):
        print("NaN of all ones", L, share, B, kf, kl, flush=True)
        sh = jq.Shape(n_layers=1, seq_lens=[L], n_q=1, h_q=2, h_kv=2, budgets=[B], keep_first=kf, keep_last=kl)
        got = jq.select_topk(sh, torch.from_numpy(bits.view(np.float32).copy()).cuda())
        torch.cuda.synchronize()
        np.testing.assert_array_equal(got.cpu().numpy()[0], oracle.select_topk(rank, B, kf, kl))


@pytest.mark.parametrize("seq_lens,budgets,pool_k,kf,kl", [
    ([2048], [256], 7, 0, 0), ([2049, 5, 2048], [100, 5, 64], 7, 2, 1), ([4097], [3000], 5, 0, 0), ([4097], [70], 13, 4, 32),
    ([9000, 31], [1000, 1], 1, 0, 0), ([700], [200], 1399, 0, 0), ([16385], [513], 7, 4, 8), ([32768, 100], [2048, 50], 5, 0, 16),
    ([2048], [300], 63, 0, 0), ([4096], [300], 31, 3, 0), ([4096, 9], [300, 2], 63, 0, 2), ([8192], [300], 9, 0, 0), ([8193], [700], 3, 0, 0),
    ([8193], [700], 13, 0, 0), ([16384], [400], 3, 0, 5), ([16385], [400], 3, 0, 5), ([16385, 70], [400, 7], 63, 2, 0), ([32768], [1100], 13, 0, 0),
    ([16400] + [40] * 64, [300] + [3] * 64, 7, 0, 0),      # more than 256 problems above 16384 positions
    ([16400] + [5000] * 8, [1500] + [600] * 8, 7, 0, 0)])  # 36 problems: seven slices each, not eight
def test_evict_equals_the_two_kernel_path_bit_for_bit(knobs, seq_lens, budgets, pool_k, kf, kl):
    # a sequence of 32769 tokens in the same batch sends the others through the two kernels; one number of keys per wave for
    # both calls, so that their scores are the same bits
    torch = torch_()
    print("short evict", seq_lens, budgets, pool_k, kf, kl, flush=True)
    knobs(JQ_CHUNK_KEYS="1024")
    rng = np.random.default_rng(5)
    T, ns = sum(seq_lens), len(seq_lens)
    Q = to_dev_bf16(f32_to_bf16_bits(rng.standard_normal((2, ns, 8, 8, 128)).astype(np.float32)))
    K = to_dev_bf16(f32_to_bf16_bits(rng.standard_normal((2, T, 2, 128)).astype(np.float32)))
    V = to_dev_bf16(f32_to_bf16_bits(rng.standard_normal((2, T, 2, 128)).astype(np.float32)))
    sh = jq.Shape(n_layers=2, seq_lens=seq_lens, n_q=8, h_q=8, h_kv=2, pool_k=pool_k, budgets=budgets, keep_first=kf, keep_last=kl)
    long = jq.Shape(n_layers=2, seq_lens=seq_lens + [32769], n_q=8, h_q=8, h_kv=2, pool_k=pool_k, budgets=budgets + [max(1, kf + kl)], keep_first=kf, keep_last=kl)
    more = torch.randn((2, 32769, 2, 128), device="cuda").bfloat16()
    wide = jq.evict(long, torch.cat([Q, Q[:, :1]], dim=1), torch.cat([K, more], dim=1), torch.cat([V, more], dim=1))
    TB = sum(budgets)
    want = wide[0][:, :TB], wide[1][:, :TB], wide[2][:, :, :TB], wide[3][:, :, :T]
    want = [x.contiguous() for x in want]
    got = jq.evict(sh, Q, K, V)
    bare = jq.evict(sh, Q, K, V, want_idx=False, want_scores=False)  # pooled scores are not stored then
    Ki, Vi = K.clone(), V.clone()
    jq.evict_inplace(sh, Q, Ki, Vi)
    torch.cuda.synchronize()
    for a, b in zip(got, want):
        assert torch.equal(a.view(torch.int16), b.view(torch.int16))
    assert torch.equal(bare[0].view(torch.int16), want[0].view(torch.int16)) and torch.equal(bare[1].view(torch.int16), want[1].view(torch.int16))
    assert torch.equal(Ki[:, :TB].view(torch.int16), want[0].view(torch.int16)) and torch.equal(Vi[:, :TB].view(torch.int16), want[1].view(torch.int16))
