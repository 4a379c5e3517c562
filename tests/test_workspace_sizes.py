"""Workspace sizes (host logic only): a finer split of a small call over workgroups asks for no larger workspace."""
import pytest

import paper_2509_10798_amd as jq


def _up(n):
    return (n + 255) // 256 * 256


def _expected(nl, lens, n_q, h_q, h_kv, budgets):
    """One statistics set per workgroup of 4 waves x 64 keys, whatever split the call then takes, plus the other pieces."""
    rp = (n_q * (h_q // h_kv) + 31) // 32 * 32
    T, n_seg = sum(lens), sum((L + 1023) // 1024 for L in lens)
    head, dens = 128, max(b / L for L, b in zip(lens, budgets))
    while head < 1024 and head < 8.0 * dens * 1024:
        head *= 2
    pieces = [nl * h_kv * sum((L + 255) // 256 for L in lens) * rp * 8, nl * len(lens) * h_kv * rp * 8, nl * len(lens) * h_kv * (2048 + 16) * 4,
              nl * h_kv * T * 4, nl * h_kv * T * 4, nl * h_kv * sum(budgets) * 4, nl * h_kv * n_seg * head * 8, nl * h_kv * n_seg * 16]
    return sum(_up(p) for p in pieces)


@pytest.mark.parametrize("nl,lens,n_q,h_q,h_kv", [
    (1, [1], 1, 1, 1), (1, [129], 32, 4, 1), (1, [2048], 32, 8, 2), (1, [255, 129, 1, 257], 32, 8, 2), (2, [1000], 16, 32, 8), (64, [129], 32, 4, 1),
])
def test_small_calls_need_no_larger_workspace(nl, lens, n_q, h_q, h_kv):
    budgets = [max(1, L // 16) for L in lens]
    sh = jq.Shape(nl, lens, n_q, h_q, h_kv, budgets=budgets)
    assert jq.workspace_bytes(sh) <= _expected(nl, lens, n_q, h_q, h_kv, budgets)
