"""The calls whose speed this repository answers for: what a user has the eviction path do, through its public entry
points, from the smallest prompt to a 128K-token layer.

Every case is one call (or the few calls of one evaluation step) on inputs made on the GPU from a seed.  Keys are
drawn so that the kept set is well defined at any rounding, as it is when a prompt's relevant passages stand out: the
soft tokens' queries share a direction per KV head, exactly as many keys as the call keeps carry it, in short spans at
positions of the head's own (single positions where nothing is pooled), and all other keys are noise of varying
length.  A pooled span of s tokens has exactly s positions that at least (pool_k + 1) / 2 of its tokens fall into, so
the budget's last place and the next one differ by a quarter (two tokens in five to two in seven), not by rounding.
"""
import math
import random

import torch

import paper_2509_10798_amd as jq

_D = 128
_SPAN = 16  # tokens per planted span


# ---------------------------------------------------------------------------------------------------------------
# cases
# ---------------------------------------------------------------------------------------------------------------
def _case(name, kind, layers, lens, budget, *, n_q=32, h_q=32, h_kv=8, pool_k=7, keep_first=0, page=0, n_resp=0):
    c = dict(name=name, kind=kind, layers=layers, lens=",".join(str(x) for x in lens), budget=budget, n_q=n_q, h_q=h_q,
             h_kv=h_kv, pool_k=pool_k, keep_first=keep_first, page=page, n_resp=n_resp)
    if name is None:
        del c["name"]
    return c


def listed():
    return [
        # the smallest call: a short prompt on a small model (16 soft tokens, 2 KV heads); launches and latency
        _case("tiny_2k", "evict", 1, [2048], 256, n_q=16, h_q=8, h_kv=2),
        # one layer evicted as soon as its prefill is done, at a usual and at the longest context
        _case("layer_32k", "evict", 1, [32768], 512),
        _case("layer_128k", "evict", 1, [131072], 2048),
        # all 32 layers of an 8K-token prompt in one call, as an engine that evicts after the whole prefill does
        _case("layers32_8k", "evict", 32, [8192], 1024),
        # the large multi-layer call: 8 layers of a 64K-token prompt
        _case("layers8_64k", "evict", 8, [65536], 1024),
        # a batch of 16 prompts of odd, very different lengths, one layer
        _case("ragged_16", "evict", 1, [21713, 102389, 4099, 77777, 58211, 9041, 131071, 34567, 120001, 15013, 66049,
                                        48017, 90173, 6151, 111119, 28657], 2048),
        # the prefill attention kernel hands its log-sum-exps over: one pass over K
        _case("lse_4x32k", "lse", 4, [32768], 1024),
        # a serving engine's paged cache, 8 sequences, pruned cache paged again
        _case("paged_8", "paged", 1, [30011, 8111, 16384, 45007, 2039, 60013, 12007, 24001], 1024, page=256),
        # eviction during decoding: 32 layers of a pruned cache of 3072 rows plus 768 decoded tokens, back to 3072
        _case("stream_32", "stream", 32, [3840], 3072, pool_k=1, keep_first=4),
        # the window-query baselines: the prompt's own last 32 tokens are the queries; sinks kept; an odd length
        _case("window_8x12k", "window", 8, [12345], 512, keep_first=4),
        # critical-KV hit rate: the kept set under 256 response tokens, stage by stage, against that of the soft tokens
        _case("response_hit_rate", "response", 1, [16384], 512, n_resp=256),
        # forward value of the training objective: maps of 32 soft and 128 response tokens over a prompt, 4 layers
        _case("train_forward", "train", 4, [6007], 0, n_resp=128),
    ]


_KINDS = ("evict", "evict", "evict", "evict", "lse", "paged", "stream", "window", "response", "train")
_HEADS = ((32, 8), (32, 8), (8, 2), (16, 8), (32, 4), (24, 8))
_COST = 8 * 65536 * 8 * 128  # (layer, key, KV head, query row) products of the largest listed single-pass case


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    kind = rng.choice(_KINDS)
    h_q, h_kv = rng.choice(_HEADS)
    group = h_q // h_kv
    n_q = rng.choice((16, 24, 32, 32))
    layers, n_resp, page, keep_first = 1, 0, 0, 0
    pool_k = rng.choice((7, 7, 7, 5, 1))
    if kind == "stream":
        pool_k, keep_first = 1, rng.choice((0, 4))
        budget = _log_int(rng, 512, 4096)
        lens = [budget + _log_int(rng, 64, 1024)]
        layers = _log_int(rng, 1, 32)
    elif kind in ("response", "train"):
        lens = [_log_int(rng, 1024, 16384)]
        n_resp = _log_int(rng, 48, 320 if kind == "response" else 192)
        budget = _log_int(rng, 128, 1024)
        layers = 1 if kind == "response" else _log_int(rng, 1, 4)
    elif kind in ("evict", "paged") and rng.random() < 0.4:  # a ragged batch
        lens = [_log_int(rng, 1024, 131072 if kind == "evict" else 65536) for _ in range(rng.randint(2, 16))]
        budget = _log_int(rng, 128, 3072)
    else:
        lens = [_log_int(rng, 1024, 131072)]
        budget = _log_int(rng, 128, 3072)
        layers = _log_int(rng, 1, 32) if kind != "paged" else 1
    if kind == "paged":
        page = rng.choice((64, 128, 256))
    if kind == "window":
        keep_first = rng.choice((0, 4))
    rows = max(n_q * group, 128) + n_resp * group
    while layers > 1 and layers * sum(lens) * h_kv * rows > _COST:
        layers -= 1
    while len(lens) > 1 and layers * sum(lens) * h_kv * rows > _COST:
        lens.pop()
    return _case(None, kind, layers, lens, 0 if kind == "train" else budget, n_q=n_q, h_q=h_q, h_kv=h_kv, pool_k=pool_k,
                 keep_first=keep_first, page=page, n_resp=n_resp)


def _lens(c):
    return [int(x) for x in c["lens"].split(",")]


def _budgets(c):
    """Kept rows per sequence: the asked budget, but at most an eighth of a short prompt (a decoding step: as asked)."""
    if c["kind"] == "stream":
        return [min(c["budget"], L) for L in _lens(c)]
    return [max(min(c["budget"], L // 8), 64) for L in _lens(c)]


def _shape(c, budgets=True):
    return jq.Shape(n_layers=c["layers"], seq_lens=_lens(c), n_q=c["n_q"], h_q=c["h_q"], h_kv=c["h_kv"], pool_k=c["pool_k"],
                    budgets=_budgets(c) if budgets else None, keep_first=c["keep_first"], window=c["kind"] == "window")


# ---------------------------------------------------------------------------------------------------------------
# inputs
# ---------------------------------------------------------------------------------------------------------------
def _planted(gen, c, L, B, layers):
    """Mask [layers, L, h_kv]: the keys that carry the head's direction, exactly as many as a head may choose freely."""
    k, first, last = c["pool_k"], c["keep_first"], c["n_q"] if c["kind"] == "window" else 0
    n, H = B - first - last, layers * c["h_kv"]
    lo, room = first + k, L - first - last - 2 * k
    mask = torch.zeros((H, L), dtype=torch.bool, device="cuda")
    if n <= 0:
        return mask.view(layers, c["h_kv"], L).transpose(1, 2)
    if k == 1:
        pick = torch.rand((H, L - first - last), generator=gen, device="cuda").topk(n, dim=1).indices + first
        mask.scatter_(1, pick, True)
    else:
        spans = max(1, min(-(-n // _SPAN), (room - n) // (2 * k)))
        slot = room // spans
        size = torch.full((spans,), n // spans, device="cuda") + (torch.arange(spans, device="cuda") < n % spans)
        free = (slot - k - size).clamp_min(0)
        at = (torch.rand((H, spans), generator=gen, device="cuda") * (free + 1)).long() + lo + torch.arange(spans, device="cuda") * slot
        for j in range(-(-n // spans)):
            mask.scatter_(1, torch.where(j < size, at + j, at), True)
    return mask.view(layers, c["h_kv"], L).transpose(1, 2)


def _inputs(c, seed, with_v=True):
    """Q [layers, n_seq, n_q, h_q, d], K and V [layers, T, h_kv, d] in bf16, the queries of the response tokens, and the
    mask of the last sequence's planted keys."""
    gen = torch.Generator(device="cuda")
    gen.manual_seed(seed)
    nl, hkv, G, lens = c["layers"], c["h_kv"], c["h_q"] // c["h_kv"], _lens(c)
    T, bf = sum(lens), torch.bfloat16

    def normal(*size):
        return torch.randn(size, generator=gen, device="cuda")

    K = torch.empty((nl, T, hkv, _D), dtype=bf, device="cuda")
    V = torch.empty_like(K) if with_v else None
    n_resp = c["n_resp"]
    Q = torch.empty((nl, len(lens), c["n_q"], c["h_q"], _D), dtype=bf, device="cuda")
    R = torch.empty((nl, len(lens), n_resp, c["h_q"], _D), dtype=bf, device="cuda") if n_resp else None
    buds = _budgets(c)
    at = 0
    for s, L in enumerate(lens):
        way = torch.nn.functional.normalize(normal(nl, hkv, _D), dim=-1)  # the head's direction
        shared = 4.0 * way.repeat_interleave(G, dim=1)[:, None]
        Q[:, s] = (normal(nl, c["n_q"], c["h_q"], _D) + shared).to(bf)
        if n_resp:
            R[:, s] = (normal(nl, n_resp, c["h_q"], _D) + shared).to(bf)
        heavy = _planted(gen, c, L, max(buds[s], 1), nl)
        for layer in range(nl):
            for t in range(0, L, 32768):
                u = min(L, t + 32768)
                x = normal(u - t, hkv, _D)
                noise = x * (0.25 * normal(u - t, hkv, 1)).exp().clamp(0.5, 1.75)
                K[layer, at + t:at + u] = torch.where(heavy[layer, t:u, :, None], 1.5 * math.sqrt(_D) * way[layer] + 0.1 * x, noise).to(bf)
                if with_v:
                    V[layer, at + t:at + u] = normal(u - t, hkv, _D).to(bf)
        at += L
    return Q, K, V, R, heavy


def _lse(c, Q, K):
    """The log-sum-exps that a prefill attention kernel keeps for the soft tokens, over the prompt's keys."""
    nl, G, at = c["layers"], c["h_q"] // c["h_kv"], 0
    out = torch.empty((nl, len(_lens(c)), c["n_q"], c["h_q"]), device="cuda")
    for s, L in enumerate(_lens(c)):
        for layer in range(nl):
            for g in range(c["h_kv"]):
                q = Q[layer, s, :, g * G:(g + 1) * G].reshape(-1, _D).float()
                x = (q @ K[layer, at:at + L, g].float().T) / math.sqrt(_D)
                out[layer, s, :, g * G:(g + 1) * G] = torch.logsumexp(x, dim=1).view(c["n_q"], G)
        at += L
    return out


def _pages(lens, page, seed):
    """A block table with the pages handed out in random order: (table, pages of the pool)."""
    per = [-(-L // page) for L in lens]
    order = list(range(sum(per) + 3))
    random.Random(seed).shuffle(order)
    table = torch.full((len(lens), max(per)), -1, dtype=torch.int32)
    for s, n in enumerate(per):
        table[s, :n] = torch.tensor([order.pop() for _ in range(n)], dtype=torch.int32)
    return table.cuda(), sum(per) + 3


def prepare(case, seed):
    kind, sh, train = case["kind"], _shape(case), case["kind"] == "train"
    Q, K, V, R, heavy = _inputs(case, seed, with_v=kind not in ("response", "train"))
    nl, hkv, dev = case["layers"], case["h_kv"], "cuda"
    st = {"kind": kind, "sh": sh, "Q": Q, "K": K, "V": V}

    def f32(*size):
        return torch.empty(size, dtype=torch.float32, device=dev)

    def i32(*size):
        return torch.empty(size, dtype=torch.int32, device=dev)

    if train:
        st.update(sh=_shape(case, budgets=False), R=R, mse=f32(nl, sh.n_seq, hkv))
        return st
    st.update(idx=i32(nl, hkv, sh.TB), scores=f32(nl, hkv, sh.T))
    if kind == "response":
        rs = jq.Shape(n_layers=nl, seq_lens=_lens(case), n_q=case["n_resp"], h_q=case["h_q"], h_kv=hkv, pool_k=case["pool_k"],
                      budgets=_budgets(case))
        st.update(sh=rs, Q=R, ws=jq.alloc_workspace(rs), pooled=f32(nl, hkv, sh.T), rate=f32(nl, sh.n_seq, hkv))
        # what the evaluation compares with: another method's kept set, three positions in four of them the same
        at = heavy.transpose(1, 2).nonzero()[:, 2].view(nl, hkv, sh.TB)
        other = torch.rand(at.shape, generator=torch.Generator(device=dev).manual_seed(seed + 1), device=dev) < 0.25
        st["soft"] = torch.where(other, (at * 7 + 3) % sh.T, at).sort(dim=-1).values.to(torch.int32).contiguous()
        return st
    st["ws"] = jq.alloc_workspace(sh)
    st.update(K_out=torch.zeros((nl, sh.TB, hkv, _D), dtype=torch.bfloat16, device=dev))
    if kind == "lse":
        st["lse"] = _lse(case, Q, K)
    if kind == "stream":
        gaps = torch.randint(1, 5, (nl, hkv, sh.T), generator=torch.Generator(device=dev).manual_seed(seed + 1), device=dev)
        st.update(pos=gaps.cumsum(-1).to(torch.int32), pos_out=i32(nl, hkv, sh.TB))
    if kind == "paged":
        page = case["page"]
        table, n = _pages(_lens(case), page, seed)
        pools, at = [torch.zeros((nl, n, page, hkv, _D), dtype=torch.bfloat16, device=dev) for _ in range(2)], 0
        for s, L in enumerate(_lens(case)):
            t = torch.arange(L, device=dev)
            where = table[s].long()[t // page] * page + t % page
            for pool, dense in zip(pools, (K, V)):
                pool.view(nl, n * page, hkv, _D)[:, where] = dense[:, at:at + L]
            at += L
        out_table, out_n = _pages(_budgets(case), page, seed + 1)
        st.update(K=pools[0], V=pools[1], pages=jq.Pages(page, n, table), out_pages=jq.Pages(page, out_n, out_table))
        st["K_out"] = torch.zeros((nl, out_n, page, hkv, _D), dtype=torch.bfloat16, device=dev)
    st["V_out"] = torch.zeros_like(st["K_out"])
    return st


def run(state):
    s, kind, sh = state, state["kind"], state["sh"]
    if kind == "train":
        return {"mse": jq.map_mse_fused(sh, s["Q"], s["R"], s["K"], mse=s["mse"])}
    if kind == "response":
        jq.score(sh, s["Q"], s["K"], scores=s["scores"], ws=s["ws"])
        jq.pool(sh, s["scores"], pooled=s["pooled"])
        jq.select_topk(sh, s["pooled"], idx=s["idx"], ws=s["ws"])
        jq.hit_rate(sh, s["soft"], s["idx"], rate=s["rate"])
        return {k: s[k] for k in ("scores", "pooled", "idx", "rate")}
    out = dict(K_out=s["K_out"], V_out=s["V_out"], idx_out=s["idx"], scores_out=s["scores"], ws=s["ws"])
    if kind == "paged":
        jq.evict_paged(sh, s["pages"], s["Q"], s["K"], s["V"], out_pages=s["out_pages"], **out)
    elif kind == "stream":
        jq.evict_stream(sh, s["Q"], s["K"], s["V"], s["pos"], pos_out=s["pos_out"], **out)
    else:
        jq.evict(sh, s["Q"], s["K"], s["V"], lse=s.get("lse"), **out)
    return {k: s[k] for k in ("K_out", "V_out", "idx", "scores", "pos_out") if k in s}


# ---------------------------------------------------------------------------------------------------------------
# what a pass cannot do without, and what it may be off by
# ---------------------------------------------------------------------------------------------------------------
def work(case):
    nl, hkv, hq, T, n_seq = case["layers"], case["h_kv"], case["h_q"], sum(_lens(case)), len(_lens(case))
    n_q = case["n_resp"] if case["kind"] == "response" else case["n_q"] + (case["n_resp"] if case["kind"] == "train" else 0)
    nbytes = nl * (T * hkv * _D * 2 + n_seq * n_q * hq * _D * 2)  # keys and queries once
    flops = 2 * nl * T * n_q * hq * _D                            # every logit once
    if case["kind"] == "train":
        return {"bytes": nbytes + nl * n_seq * hkv * 4, "flops": flops}
    TB = sum(_budgets(case))
    nbytes += nl * hkv * (T + TB) * 4  # pooled scores and kept positions written
    if case["kind"] == "response":
        return {"bytes": nbytes + nl * hkv * (T + TB) * 4, "flops": flops}  # unpooled scores too; the other set read
    nbytes += 4 * nl * TB * hkv * _D * 2  # kept rows of K and V read and written
    if case["kind"] == "lse":
        nbytes += nl * n_seq * n_q * hq * 4
    if case["kind"] == "stream":
        nbytes += 2 * nl * hkv * TB * 4
    return {"bytes": nbytes, "flops": flops}


def tolerance(case):
    # Measured: with other numbers of keys per wave (JQ_CHUNK_KEYS=64, 512), i.e. with the 32-bit sums behind every
    # normaliser taken in another order, scores move by up to 1.6e-7 (2-norm) and 1.2e-6 (single value) over the listed
    # and twelve drawn cases, and either way they are up to 4e-7 from the 64-bit result, so that two correct ways of
    # summing may be 4e-7 apart.  The objective squares differences of two maps: up to 6e-6.
    return {"rel": 2.4e-5, "max": 1e-4} if case["kind"] == "train" else {"rel": 1.6e-6, "max": 1e-5}


# ---------------------------------------------------------------------------------------------------------------
# the same in 64 bits
# ---------------------------------------------------------------------------------------------------------------
def _scores64(Q, K, window=False, lse=None):
    """[h_kv, L] in fp64 from Q [n_q, h_q, d], K [L, h_kv, d]."""
    n_q, h_q, _ = Q.shape
    L, h_kv, _ = K.shape
    G, out = h_q // h_kv, []
    for g in range(h_kv):
        q = Q[:, g * G:(g + 1) * G].reshape(-1, _D).double()
        k, total = K[:, g].double(), torch.zeros(L, dtype=torch.float64, device=K.device)
        for r in range(0, q.shape[0], 128):
            x = q[r:r + 128] @ k.T / math.sqrt(_D)
            if window:
                i = torch.arange(r, min(r + 128, q.shape[0]), device=K.device) // G
                x = x.masked_fill(torch.arange(L, device=K.device)[None] > L - n_q + i[:, None], -math.inf)
            if lse is None:
                x = torch.softmax(x, dim=1)
            else:
                x = (x - lse[:, g * G:(g + 1) * G].reshape(-1, 1)[r:r + 128].double()).exp()
            total += x.sum(dim=0)
        out.append(total)
    out = torch.stack(out)
    if window:
        out[:, L - n_q:] = 0
    return out


def _pool64(x, k):
    return torch.nn.functional.avg_pool1d(x[:, None], k, stride=1, padding=k // 2, count_include_pad=True)[:, 0]


def exact(case, seed):
    st = prepare(case, seed)
    nl, kind, lens, buds, hkv = case["layers"], case["kind"], _lens(case), _budgets(case), case["h_kv"]
    if kind == "train":
        out, rows = torch.empty((nl, len(lens), hkv), dtype=torch.float64), case["h_q"] // hkv
        for layer in range(nl):
            a = _scores64(st["Q"][layer, 0], st["K"][layer]) / (case["n_q"] * rows)
            b = _scores64(st["R"][layer, 0], st["K"][layer]) / (case["n_resp"] * rows)
            out[layer, 0] = ((a - b) ** 2).mean(dim=1).cpu()
        return {"mse": out}
    raw, pooled, idx, K_out, V_out, pos = ([] for _ in range(6))
    for layer in range(nl):
        at, per = 0, [[] for _ in range(6)]
        for s, (L, B) in enumerate(zip(lens, buds)):
            if kind == "paged":
                t = torch.arange(L, device="cuda")
                where = st["pages"].block_table[s].long()[t // case["page"]] * case["page"] + t % case["page"]
                K, V = (st[n][layer].reshape(-1, hkv, _D)[where] for n in ("K", "V"))
            else:
                K = st["K"][layer, at:at + L]
                V = st["V"][layer, at:at + L] if st["V"] is not None else K
            x = _scores64(st["Q"][layer, s], K, kind == "window", st["lse"][layer, s] if kind == "lse" else None)
            y = _pool64(x, case["pool_k"])
            z = y.clone()
            z[:, :case["keep_first"]] = math.inf
            if kind == "window":
                z[:, L - case["n_q"]:] = math.inf
            kept = z.topk(B, dim=1).indices.sort(dim=1).values
            rows = kept.T[:, :, None].expand(-1, -1, _D)
            for to, v in zip(per, (x, y, kept, K.gather(0, rows), V.gather(0, rows),
                                   st["pos"][layer, :, at:at + L].gather(1, kept) if kind == "stream" else kept)):
                to.append(v)
            at += L
        for to, v, dim in zip((raw, pooled, idx, K_out, V_out, pos), per, (1, 1, 1, 0, 0, 1)):
            to.append(torch.cat(v, dim=dim))
    scores, kept = torch.stack(pooled), torch.stack(idx).to(torch.int32)
    if kind == "response":
        soft = st["soft"]
        hits = torch.stack([torch.isin(kept[l, g], soft[l, g]).double().mean() for l in range(nl) for g in range(hkv)])
        return {"scores": torch.stack(raw), "pooled": scores, "idx": kept, "rate": hits.view(nl, 1, hkv)}
    ans = {"idx": kept, "scores": scores}
    if kind == "paged":  # the pools' rows outside the kept ones are the caller's
        ans.update(K_out=None, V_out=None)
    else:
        ans.update(K_out=torch.stack(K_out), V_out=torch.stack(V_out))
    if kind == "stream":
        ans["pos_out"] = torch.stack(pos).to(torch.int32)
    return ans
