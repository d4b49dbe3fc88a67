"""The decode-step workloads that performance work on this library is measured on.

A case is one call of the kind a serving loop makes for one layer and one step, through the public entry points
(`DecodeSession`, which holds a plan with its workspace and output buffers, as a serving process keeps it):

  op "decode"   vatt_decode, exact top-k from the score pass.
  op "step"     the step of a continuous-batching loop: the scheduler's sequence lengths of this step are put in
                place, vatt_append_kv adds the new token's rows, vatt_decode attends.
  op "given"    vatt_decode_given_topk: the top-k set comes from an approximate index outside the library.
  op "cached"   vatt_decode_given_topk_cached, the same with the base sample served by the random cache.
  op "dense"    vatt_dense_decode: exact attention on the same cache (layers or steps kept dense).

`q_len` > 1 are multi-query steps (the tokens of a question, or of a speculated continuation).

Inputs follow workloads/configs.py: q, V ~ N(0, 1); even KV heads "spiky" (K ~ N(0, 1) with 0.1 % planted keys along
the group's mean query), odd ones "flat" (K ~ N(0, 0.25)); everything is made on the GPU from the seed.
"""
import math

import torch

from paper_2510_05688_amd.session import DecodeSession

# Attention shapes (query heads, KV heads, head_dim): the repository's benchmark shape, then groups of 1, 2 and 8.
SHAPES = [(32, 8, 128), (32, 8, 128), (32, 8, 128), (32, 4, 128), (16, 16, 64), (16, 8, 64)]


def _case(op, batch, n, **over):
    c = dict(op=op, batch=batch, n=n, n_lo=n, hq=32, hkv=8, d=128, q_len=1, page=0, sink=128, window=128, topk_abs=0,
             topk_frac=0.025, base_abs=0, base_frac=0.025, epsilon=0.05, delta=0.05, target=0)
    c.update(over)
    return c


def listed():
    return [
        # the smallest call the tests and smoke() make: one head of a small model, launches and latency only
        _case("decode", 1, 1024, name="decode one head 1k", hq=1, hkv=1, d=64, sink=4, window=32, topk_abs=32,
              base_abs=32),
        # a chat-sized batch on a paged cache, odd ragged lengths far below a long capacity
        _case("decode", 8, 7001, name="decode 8 x 0.5k-7k paged", n_lo=517, page=64),
        # the benchmark's headline: one sequence at the paper's 32K context
        _case("decode", 1, 32768, name="decode 1 x 32k"),
        # the same with the budget rule, not the base sample, setting the sample size (tight epsilon)
        _case("decode", 2, 20011, name="decode 2 x 20k adaptive", base_abs=32, epsilon=0.02),
        # the batched benchmark
        _case("decode", 16, 32768, name="decode 16 x 32k"),
        # long context, the 128K capacity of the model family the shapes come from
        _case("decode", 4, 131072, name="decode 4 x 128k", window=512, topk_frac=0.01),
        # continuous batching: ragged sequences on 16-token pages, one token appended per step
        _case("step", 32, 32768, name="step 32 x 1k-32k paged", n_lo=1024, page=16, epsilon=0.1, delta=0.1),
        # the whole attention output verified instead of the denominator alone
        _case("decode", 4, 16384, name="decode 4 x 16k sdpa", target=2, epsilon=0.1, delta=0.1),
        # top-k from an approximate index: only attended rows are read
        _case("given", 16, 32768, name="given 16 x 32k"),
        _case("cached", 1, 32768, name="cached 1 x 32k"),
        # the tokens of a question, all in one call
        _case("decode", 1, 32768, name="decode 1 x 32k, 16 queries", q_len=16),
        # dense attention of a short question over a batch: layers that are not run sparsely
        _case("dense", 4, 32768, name="dense 4 x 32k, 8 queries", q_len=8),
    ]


def _log(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    """Any operation, shape, batch and length within the limits of the listed cases (at most 512K cached tokens per
    query token, contexts from 200 to 131072)."""
    op = rng.choice(["decode", "decode", "decode", "step", "given", "cached", "dense", "dense"])
    hq, hkv, d = rng.choice(SHAPES)
    n = _log(rng, 200, 131072)
    q_len = rng.choice([1, 1, 1, _log(rng, 2, 16)]) if op in ("decode", "given", "dense") else 1
    batch = min(_log(rng, 1, 32), max(1, 16 * 32768 // (n * q_len)))
    n = min(n, 16 * 32768 // (batch * q_len))
    paged = op == "step" or rng.random() < 0.4
    page = rng.choice([16, 16, 64]) if paged else 0
    ragged = batch > 1 and rng.random() < 0.6
    lo = max(q_len, n // 16) if ragged else n
    sink, window = rng.choice([(128, 128), (128, 128), (128, 512), (4, 64)])
    over = rng.choice([{}, {}, {}, dict(epsilon=0.1, delta=0.1), dict(topk_frac=0.01), dict(topk_frac=0.05, base_frac=0.05),
                       dict(base_abs=64, epsilon=0.02)])
    target = rng.choice([0, 0, 0, 2]) if op == "decode" and q_len == 1 else 0
    return _case(op, batch, n, n_lo=lo, hq=hq, hkv=hkv, d=d, q_len=q_len, page=page, sink=sink, window=window,
                 target=target, **over)


def _lengths(case):
    """Lengths of the sequences: the longest is n, the others spread evenly down to n_lo, in a scattered order."""
    b, n, lo = case["batch"], case["n"], case["n_lo"]
    if b == 1 or lo == n:
        return [n] * b
    lens = [n - (n - lo) * i // (b - 1) for i in range(b)]
    return [lens[(i * 7 + 3) % b] if math.gcd(7, b) == 1 else lens[i] for i in range(b)]


def _gen(seed, what):
    g = torch.Generator(device="cuda")
    g.manual_seed(1000003 * int(seed) + what)
    return g


def _randn(shape, g):
    return torch.randn(shape, generator=g, device="cuda", dtype=torch.float32).to(torch.bfloat16)


def _rows(t, table, page, b, n):
    """The first n rows of sequence b: [Hkv, n, d]."""
    if not page:
        return t[b, :, :n]
    p = t[table[b, :(n + page - 1) // page].long()]                      # [pages, Hkv, page, d]
    return p.transpose(0, 1).reshape(t.shape[1], -1, t.shape[3])[:, :n]


def _plant(k, q, table, case, lens, g):
    """Heavy keys of the spiky heads: 0.1 % of the tokens lie along the mean query of the head's group."""
    d, hkv, grp, page = case["d"], case["hkv"], case["hq"] // case["hkv"], case["page"]
    qf = q.float().reshape(case["batch"], case["q_len"], hkv, grp, d)[:, -1].mean(2)
    for b, n in enumerate(lens):
        m = max(1, n // 1000)
        at = torch.randint(0, n // m, (hkv, m), generator=g, device="cuda")
        at += (n // m) * torch.arange(m, device="cuda")
        noise = torch.randn((hkv, m, d), generator=g, device="cuda") * math.sqrt(0.1)
        dirn = qf[b] / qf[b].norm(dim=-1, keepdim=True)
        rows = (3.0 * math.sqrt(d) * dirn[:, None] + noise).to(torch.bfloat16)
        heads = torch.arange(hkv, device="cuda")[:, None].expand(hkv, m)
        even = torch.arange(0, hkv, 2, device="cuda")
        h, a, r = heads[even].reshape(-1), at[even].reshape(-1), rows[even].reshape(-1, d)
        if page:
            k[table[b, a // page].long(), h, a % page] = r
        else:
            k[b, h, a] = r


def _approximate_topk(sess, case, k, q, table, lens, g):
    """What an approximate index would hand over: the largest scores of the middle region after noise on them."""
    cap = sess.seg[3] - sess.seg[2]
    b_, ql, hq, hkv, d = case["batch"], case["q_len"], case["hq"], case["hkv"], case["d"]
    grp = hq // hkv
    idx = torch.zeros((b_ * ql, hq, cap), dtype=torch.int32, device="cuda")
    cnt = torch.zeros((b_ * ql, hq), dtype=torch.int32, device="cuda")
    for b, n in enumerate(lens):
        rows = _rows(k, table, case["page"], b, n).float()
        for t in range(ql):
            seen = n - (ql - 1 - t)
            lo, hi = case["sink"], seen - case["window"]
            kk = case["topk_abs"] or int(case["topk_frac"] * seen)
            kk = min(kk, max(0, hi - lo), cap)
            if kk <= 0:
                continue
            qf = q.reshape(b_, ql, hkv, grp, d)[b, t].float().transpose(1, 2).contiguous()
            s = torch.matmul(rows[:, lo:hi].contiguous(), qf) / math.sqrt(d)  # [Hkv, middle, group]
            s = s + 0.1 * torch.randn(s.shape, generator=g, device="cuda")
            best = torch.topk(s, kk, dim=1).indices + lo
            idx[b * ql + t, :, :kk] = best.transpose(1, 2).reshape(hq, kk).int()
            cnt[b * ql + t] = kk
    return idx, cnt


def prepare(case, seed):
    b, hq, hkv, d, page, ql = (case[x] for x in ("batch", "hq", "hkv", "d", "page", "q_len"))
    lens = _lengths(case)
    room = max(lens) + (1 if case["op"] == "step" else 0)
    n_max = -(-room // page) * page if page else room
    blocks = b * (n_max // page) if page else 0
    params = dict(batch=b, n_q_heads=hq, n_kv_heads=hkv, head_dim=d, n_max=n_max, kv_layout=1 if page else 0, page_size=page,
                  num_blocks=blocks, sink=case["sink"], window=case["window"], topk_abs=case["topk_abs"],
                  topk_frac=case["topk_frac"], base_abs=case["base_abs"], base_frac=case["base_frac"],
                  epsilon=case["epsilon"], delta=case["delta"], target=case["target"], sm_scale=0.0, budget_cap_frac=1.0)
    sess = DecodeSession(params, q_len=ql)
    for t in (sess.out_o, sess.out_lse, sess.out_idx, sess.out_counts, sess.out_budget_raw, sess.out_stats, sess.dense_o,
              sess.dense_lse):
        t.zero_()  # index lists are shorter than their buffer
    table = None
    if page:
        table = torch.randperm(blocks, generator=_gen(seed, 1), device="cuda").int().reshape(b, n_max // page)
    shape = (blocks, hkv, page, d) if page else (b, hkv, n_max, d)
    q = _randn((b, ql, hq, d) if ql > 1 else (b, hq, d), _gen(seed, 2))
    k = torch.empty(shape, dtype=torch.bfloat16, device="cuda")
    v = torch.empty(shape, dtype=torch.bfloat16, device="cuda")
    k.normal_(generator=_gen(seed, 3))
    v.normal_(generator=_gen(seed, 4))
    k[:, 1::2] *= 0.5
    if case["target"] == 2:
        v += 1.0  # with zero-mean values the output's budget is the whole residual
    _plant(k, q, table, case, lens, _gen(seed, 5))
    sess.q, sess.k, sess.v, sess.block_table = q, k, v, table
    sess.seq_lens = torch.tensor(lens, dtype=torch.int32, device="cuda")
    sess.seq_seeds = torch.tensor([(int(seed) * 7919 + i) & 0x7fffffff for i in range(b)], dtype=torch.int64, device="cuda")
    state = dict(case=dict(case), sess=sess)
    if case["op"] == "step":
        state["lens"] = sess.seq_lens.clone()
        state["new"] = (_randn((b, hkv, d), _gen(seed, 6)), _randn((b, hkv, d), _gen(seed, 7)))
    if case["op"] in ("given", "cached"):
        state["topk"] = _approximate_topk(sess, case, k, q, table, lens, _gen(seed, 8))
    if case["op"] == "cached":
        sess.make_random_cache(torch.arange(b, dtype=torch.int64).numpy() + int(seed) % 100003)
    return state


def run(state):
    sess, op = state["sess"], state["case"]["op"]
    if op == "dense":
        sess.dense()
        return dict(o=sess.dense_o, lse=sess.dense_lse)
    if op == "given":
        sess.decode_given_topk(*state["topk"])
    elif op == "cached":
        sess.decode_given_topk_cached(*state["topk"])
    else:
        if op == "step":
            sess.seq_lens.copy_(state["lens"])
            sess.append_device(*state["new"])
        sess.decode()
    return dict(o=sess.out_o, lse=sess.out_lse, idx=sess.out_idx, counts=sess.out_counts, budget=sess.out_budget_raw,
                stats=sess.out_stats)


def work(case):
    """K (and V) rows that must be read once, lists and outputs written once; the final sample at its least size."""
    hq, hkv, d, ql = case["hq"], case["hkv"], case["d"], case["q_len"]
    grp, row = hq // hkv, 2 * case["d"]
    nbytes = flops = 0.0
    for n in _lengths(case):
        nbytes += ql * hq * (2 * d + 4 * d + 4)
        if case["op"] == "dense":
            nbytes += 2 * hkv * n * row
            flops += 4.0 * n * d * hq * ql
            continue
        fixed = min(n, case["sink"] + case["window"])
        k = min(case["topk_abs"] or int(case["topk_frac"] * n), n - fixed)
        rest = n - fixed - k
        base = min(rest, case["base_abs"] or max(2, int(case["base_frac"] * rest)))
        scored = min(n, fixed + ql * grp * (k + 2 * base)) if case["op"] in ("given", "cached") else n
        gathered = min(n, fixed + ql * grp * (k + base))
        nbytes += hkv * row * (scored + gathered) + ql * hq * (4 * (fixed + k + 2 * base) + 60)
        flops += 2.0 * d * hq * ql * (scored if case["op"] == "decode" or case["op"] == "step" else fixed + k + 2 * base)
        flops += 2.0 * d * hq * ql * (fixed + k + base)
    return dict(bytes=nbytes, flops=flops)


def tolerance(case):
    if case["op"] == "dense":
        return dict(rel=2e-5)      # 32-bit sums of 32-bit weights over up to 128K tokens
    if case["op"] in ("given", "cached"):
        return dict(rel=1e-4, differ=1e-3)  # the same, and n_s / b of a budget next to a whole number
    # Two scores closer than their rounding at the edge of the top-k set may change places: one token then moves
    # between the exact and the sampled part of its head, and the head's list shifts between the two places.
    return dict(rel=1e-3, differ=5e-3)
