"""Scores held back in LDS and written together (second passes that read much of K from memory): the same bits as the scores that
smaller calls, which store every tile's at once, make of the same keys -- with the normalisers supplied a score depends on its
own key alone."""
import pytest

import paper_2509_10798_amd as jq

pytestmark = pytest.mark.gpu

HELD = 110_000_000  # bytes of K from which on one pass holds its scores back


@pytest.mark.parametrize("h_q,h_kv,n_q,window,page,chunk,n_layers,seq_lens", [
    (32, 8, 32, False, 0, None, 1, [30001, 20011, 77, 1, 4128, 12345]),   # a workgroup per CU, odd ends
    (8, 8, 8, False, 0, None, 2, [29999, 127]),                            # one tile of query rows
    (6, 2, 20, True, 0, None, 4, [50001, 4100]),                           # the window's own positions are 0; 60 rows
    (32, 8, 32, False, 64, None, 1, [30001, 20011, 77, 1, 4128, 12345]),   # paged
    (8, 1, 16, False, 0, 8192, 8, [53000, 1, 2000]),                       # 256 tiles a wave: more than are held at once
    (16, 8, 16, False, 0, 1312, 3, [40000, 20000]),                        # two workgroups per CU, 41 tiles a wave
])
def test_held_back_scores_equal_those_stored_at_once(knobs, h_q, h_kv, n_q, window, page, chunk, n_layers, seq_lens):
    import torch
    assert torch.cuda.is_available(), "these tests need the GPU"
    print("held back", h_q, h_kv, n_q, window, page, chunk, n_layers, seq_lens, flush=True)
    T = sum(seq_lens)
    assert n_layers * T * h_kv * 256 >= HELD
    gen = torch.Generator(device="cuda")
    gen.manual_seed(6)
    Q = torch.randn((n_layers, len(seq_lens), n_q, h_q, 128), generator=gen, device="cuda").bfloat16()
    K = torch.randn((n_layers, T, h_kv, 128), generator=gen, device="cuda").bfloat16()
    lse = 9.0 + torch.rand((n_layers, len(seq_lens), n_q, h_q), generator=gen, device="cuda")
    if chunk:
        knobs(JQ_CHUNK_KEYS=chunk, JQ_CHUNK_KEYS_2=chunk)
    common = dict(n_q=n_q, h_q=h_q, h_kv=h_kv, window=window)
    sh = jq.Shape(n_layers=n_layers, seq_lens=seq_lens, **common)
    out = torch.full((n_layers, h_kv, T), float("nan"), device="cuda")
    if page:
        per = [-(-L // page) for L in seq_lens]
        table = torch.full((len(seq_lens), max(per)), -1, dtype=torch.int32)
        pool = torch.zeros((n_layers, sum(per), page, h_kv, 128), dtype=torch.bfloat16, device="cuda")
        flat, at, nxt = pool.view(n_layers, -1, h_kv, 128), 0, 0
        for s, L in enumerate(seq_lens):
            table[s, :per[s]] = torch.arange(nxt, nxt + per[s])
            flat[:, nxt * page:nxt * page + L] = K[:, at:at + L]
            at, nxt = at + L, nxt + per[s]
        got = jq.score_paged(sh, jq.Pages(page, sum(per), table.cuda()), Q, pool, lse=lse, scores=out)
    else:
        got = jq.score(sh, Q, K, lse=lse, scores=out)
    at = 0
    for s, L in enumerate(seq_lens):
        for layer in range(n_layers):
            assert L * h_kv * 256 < HELD
            one = jq.score(jq.Shape(n_layers=1, seq_lens=[L], **common), Q[layer:layer + 1, s:s + 1].contiguous(),
                           K[layer:layer + 1, at:at + L].contiguous(), lse=lse[layer:layer + 1, s:s + 1].contiguous())
            torch.cuda.synchronize()
            assert torch.equal(got[layer, :, at:at + L], one[0]), (layer, s)
        at += L


def _paged(torch, K, seq_lens, page):
    """The same keys in a pool whose pages lie in reverse order, and its block table."""
    n_layers, _, h_kv, d = K.shape
    per = [-(-L // page) for L in seq_lens]
    n = sum(per)
    table = torch.full((len(seq_lens), max(per)), -1, dtype=torch.int32)
    pool = torch.zeros((n_layers, n, page, h_kv, d), dtype=K.dtype, device=K.device)
    at, left = 0, n
    for s, L in enumerate(seq_lens):
        for j in range(per[s]):
            left -= 1
            table[s, j] = left
            rows = min(page, L - j * page)
            pool[:, left, :rows] = K[:, at + j * page:at + j * page + rows]
        at += L
    return jq.Pages(page, n, table.cuda()), pool


@pytest.mark.parametrize("n_layers,seq_lens,n_q,h_q,h_kv,chunk", [
    (2, [40000, 129, 9000], 32, 32, 8, 4096),  # 128 tiles a wave: more than are held at once
    (5, [12000], 8, 64, 64, None),             # the same, over several layers a workgroup, whose query rows come where scores were
    (1, [7937], 16, 16, 4, 1984),              # as many as are held, 62, and one
    (1, [129], 8, 8, 8, None),                 # a tile of query rows; a wave has one tile of keys or none
    (1, [4099], 16, 8, 2, None),               # two
    (3, [1000, 127, 45, 128, 2049], 24, 8, 2, None),  # three; portions that end inside sequences
    (5, [9999], 32, 12, 4, None),              # three; layers that do not divide the workgroups
    (40, [300], 32, 8, 2, None),               # four; more layers than workgroups per head: several shares a workgroup
    (9, [300, 33, 129] * 12, 32, 32, 8, None),  # four; many short sequences, two workgroups per CU in two launches
    (1, [40000], 32, 32, 8, None),             # a workgroup per CU
])
@pytest.mark.parametrize("form", ["dense", "paged", "window"])
@pytest.mark.parametrize("wait_us", [None, 0])
def test_passes_that_form_their_statistics_hold_the_same_scores_back(knobs, n_layers, seq_lens, n_q, h_q, h_kv, chunk, form, wait_us):
    # both passes in one launch (evict) and one after the other (score), every number of row tiles; without patience a workgroup
    # finds sets missing, forms them itself and starts the second pass of its share again
    import torch
    assert torch.cuda.is_available(), "these tests need the GPU"
    print("held back, two passes", n_layers, seq_lens[:4], n_q, h_q, h_kv, chunk, form, wait_us, flush=True)
    gen = torch.Generator(device="cuda")
    gen.manual_seed(8)
    Q = torch.randn((n_layers, len(seq_lens), n_q, h_q, 128), generator=gen, device="cuda").bfloat16()
    K = torch.randn((n_layers, sum(seq_lens), h_kv, 128), generator=gen, device="cuda").bfloat16()
    sh = jq.Shape(n_layers=n_layers, seq_lens=seq_lens, n_q=n_q, h_q=h_q, h_kv=h_kv, pool_k=1, window=form == "window",
                  budgets=[max(n_q, L // 8) if form == "window" else max(1, L // 8) for L in seq_lens])
    if form == "paged":
        pages, pool = _paged(torch, K, seq_lens, 64)

    def run(hold):
        knobs(JQ_HOLD_BYTES=str(hold), **({} if wait_us is None else {"JQ_WAIT_US": str(wait_us)}), **({"JQ_CHUNK_KEYS": str(chunk)} if chunk else {}))
        if form == "paged":
            two, one = jq.score_paged(sh, pages, Q, pool), jq.evict_paged(sh, pages, Q, pool, pool)
        else:
            two, one = jq.score(sh, Q, K), jq.evict(sh, Q, K, K)
        torch.cuda.synchronize()
        return two, one[3], one[2]
    at_once = run(1 << 60)
    held = run(0)
    for name, a, b in zip(("two launches", "one launch", "positions"), held, at_once):
        assert torch.equal(a, b), name
    assert torch.equal(held[0], held[1])
    total = held[0].double().cpu()
    assert torch.isfinite(total).all() and float(total.sum()) > 0


@pytest.mark.parametrize("n_layers,L,lse,evicts,held", [
    (1, 120000, True, True, False),   # a tail of two kernels behind one pass over 246 MB: slower on some cards if held back
    (1, 120000, True, False, True),   # the scores alone
    (2, 32768, True, True, True),     # the one-kernel tail
    (1, 250000, True, True, True),
    (1, 120000, False, True, False),
    (1, 250000, False, True, True),
])
def test_which_calls_hold_their_scores_back(n_layers, L, lse, evicts, held):
    import torch
    from torch.profiler import ProfilerActivity, profile
    assert torch.cuda.is_available(), "these tests need the GPU"
    print("which kernel", n_layers, L, lse, evicts, flush=True)
    gen = torch.Generator(device="cuda")
    gen.manual_seed(4)
    Q = torch.randn((n_layers, 1, 32, 32, 128), generator=gen, device="cuda").bfloat16()
    K = torch.randn((n_layers, L, 8, 128), generator=gen, device="cuda").bfloat16()
    norms = torch.full((n_layers, 1, 32, 32), 12.0, device="cuda") if lse else None
    sh = jq.Shape(n_layers=n_layers, seq_lens=[L], n_q=32, h_q=32, h_kv=8, budgets=[256])
    jq.score(sh, Q, K, lse=norms)
    with profile(activities=[ProfilerActivity.CUDA]) as prof:
        for _ in range(3):  # (the profiler may miss one)
            jq.evict(sh, Q, K, K, lse=norms) if evicts else jq.score(sh, Q, K, lse=norms)
        torch.cuda.synchronize()
    ran = {e.name.split("(")[0] for e in prof.events() if "jq_score_kernel" in e.name or "jq_passes_kernel" in e.name}
    assert ran and all(("passes" in n) == (not lse) for n in ran), ran
    assert all(n.endswith("true>") == held for n in ran), ran
