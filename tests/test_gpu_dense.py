"""vatt_dense_decode against plain fp32 attention: every number of query-vector waves, ragged and large batches."""
import numpy as np
import pytest

import workloads
from workloads.configs import default_params

pytestmark = pytest.mark.gpu

CASES = [
    # (batch, lengths low .. high, q_len, Hq, Hkv, d, page)
    (1, 1, 1, 1, 1, 1, 64, 0), (1, 1, 2, 1, 4, 4, 128, 0), (3, 31, 33, 2, 8, 8, 64, 16),
    (2, 127, 129, 4, 8, 2, 128, 0), (2, 300, 1500, 5, 8, 2, 128, 16), (3, 20, 900, 16, 4, 1, 128, 0),
    (2, 100, 700, 17, 8, 2, 64, 8), (2, 200, 260, 33, 4, 1, 128, 64), (1, 300, 600, 40, 8, 1, 64, 0),
    (1, 3000, 4001, 1, 32, 8, 128, 0), (70, 1, 400, 1, 4, 2, 128, 0), (130, 1, 90, 2, 2, 1, 64, 16),
    (300, 1, 60, 1, 2, 1, 128, 0), (2, 5, 3000, 1, 8, 1, 128, 16), (1, 3, 3, 8, 4, 1, 128, 0),
]


@pytest.mark.parametrize("case", CASES, ids=lambda c: "-".join(map(str, c)))
def test_dense_against_fp32_attention(case):
    import torch
    from paper_2510_05688_amd.session import DecodeSession

    batch, lo, hi, q_len, hq, hkv, d, page = case
    rng = np.random.default_rng(sum(case))
    lens = rng.integers(lo, hi + 1, size=batch)
    lens[0] = hi
    n_max = -(-hi // page) * page if page else hi
    wl = workloads.make_workload("dense", batch=batch, n_q_heads=hq, n_kv_heads=hkv, head_dim=d, n_max=n_max,
                                 seq_lens=lens, seed=5, params=default_params(d), plant_frac=0.01)
    q_bits = workloads.chunk_queries(wl, q_len, seed=2) if q_len > 1 else wl.q_bits
    k_bits, v_bits, table = workloads.to_paged(wl, page) if page else (wl.k_bits, wl.v_bits, None)
    sess = DecodeSession(dict(batch=batch, n_q_heads=hq, n_kv_heads=hkv, head_dim=d, n_max=n_max, kv_layout=1 if page else 0,
                              page_size=page, num_blocks=k_bits.shape[0] if page else 0, sink=4, window=8, topk_abs=0,
                              topk_frac=0.02, base_abs=0, base_frac=0.02, epsilon=0.1, delta=0.1, target=0, sm_scale=0.0,
                              budget_cap_frac=1.0), q_len=q_len)
    sess.upload(q_bits, k_bits, v_bits, wl.seq_lens, wl.seeds, table)
    sess.dense()
    torch.cuda.synchronize()
    o, lse = sess.dense_o.cpu().double(), sess.dense_lse.cpu().double()
    q = torch.from_numpy(workloads.bf16_bits_to_f32(q_bits)).reshape(batch, q_len, hq, d).double()
    for b in range(batch):
        for t in range(q_len):
            seen = max(int(lens[b]) - (q_len - 1 - t), 1)
            for j in range(hkv):
                k = torch.from_numpy(wl.k_f32(b, j, seen)).double()
                v = torch.from_numpy(wl.v_f32(b, j, seen)).double()
                g = hq // hkv
                s = q[b, t, j * g:(j + 1) * g] @ k.T / np.sqrt(d)
                want = torch.softmax(s, dim=-1) @ v
                got = o[b * q_len + t, j * g:(j + 1) * g]
                assert float((got - want).norm() / want.norm()) < 2e-5, (b, t, j)
                assert float((lse[b * q_len + t, j * g:(j + 1) * g] - torch.logsumexp(s, -1)).abs().max()) < 2e-5, (b, t, j)
    sess.close()


def _dense(batch, lens, q_len, hq, hkv, d, page, touch=None, seed=5, q_first=None):
    """Outputs of one dense call and the workload's values; touch(k_bits, v_bits, b, n) edits a sequence's rows."""
    import torch
    from paper_2510_05688_amd.session import DecodeSession

    lens = np.asarray(lens)
    n_max = -(-int(lens.max()) // page) * page if page else int(lens.max())
    wl = workloads.make_workload("dense", batch=batch, n_q_heads=hq, n_kv_heads=hkv, head_dim=d, n_max=n_max,
                                 seq_lens=lens, seed=seed, params=default_params(d), plant_frac=0.01)
    for b in range(batch if touch else 0):
        touch(wl.k_bits, wl.v_bits, b, int(lens[b]))
    q_bits = workloads.chunk_queries(wl, q_len, seed=2) if q_len > 1 else wl.q_bits
    if q_first is not None:
        q_bits = q_bits.copy()
        q_bits[..., 0] = q_first
    k_bits, v_bits, table = workloads.to_paged(wl, page) if page else (wl.k_bits, wl.v_bits, None)
    sess = DecodeSession(dict(batch=batch, n_q_heads=hq, n_kv_heads=hkv, head_dim=d, n_max=n_max, kv_layout=1 if page else 0,
                              page_size=page, num_blocks=k_bits.shape[0] if page else 0, sink=4, window=8, topk_abs=0,
                              topk_frac=0.02, base_abs=0, base_frac=0.02, epsilon=0.1, delta=0.1, target=0, sm_scale=0.0,
                              budget_cap_frac=1.0), q_len=q_len)
    sess.upload(q_bits, k_bits, v_bits, wl.seq_lens, wl.seeds, table)
    sess.dense()
    torch.cuda.synchronize()
    o = sess.dense_o.cpu().double().reshape(batch, q_len, hq, d)
    lse = sess.dense_lse.cpu().double().reshape(batch, q_len, hq)
    sess.close()
    q = torch.from_numpy(workloads.bf16_bits_to_f32(q_bits)).reshape(batch, q_len, hq, d).double()
    return wl, q, o, lse


def _check(wl, q, o, lse, lens):
    """Against attention in 64 bits over the tokens that each query sees; an Inf or a NaN where that has one, and no other."""
    import torch
    batch, q_len, hq, d = o.shape
    g = hq // wl.n_kv_heads
    for b in range(batch):
        for j in range(wl.n_kv_heads):
            n = int(lens[b])
            k, v = torch.from_numpy(wl.k_f32(b, j, n)).double(), torch.from_numpy(wl.v_f32(b, j, n)).double()
            fin = torch.isfinite(v)
            odd = (~fin).any(1).nonzero()[:, 0]
            v_fin, v_odd = torch.where(fin, v, 0.0), torch.where(fin, 0.0, v)
            for t in range(q_len):
                seen = max(n - (q_len - 1 - t), 1)
                s = q[b, t, j * g:(j + 1) * g] @ k[:seen].T / np.sqrt(d)
                p, rows = torch.softmax(s, -1), odd[odd < seen]
                want = p @ v_fin[:seen] + (p[:, rows, None] * v_odd[rows]).sum(1)
                got, ok = o[b, t, j * g:(j + 1) * g], torch.isfinite(want)
                assert torch.equal(got[~ok].nan_to_num(3.0, 1.0, 2.0), want[~ok].nan_to_num(3.0, 1.0, 2.0)), (b, t, j)
                err, size = torch.where(ok, got - want, 0.0).norm(dim=1), torch.where(ok, want, 0.0).norm(dim=1)
                assert float((err / size).max()) < 2e-5, (b, t, j)
                assert float((lse[b, t, j * g:(j + 1) * g] - torch.logsumexp(s, -1)).abs().max()) < 2e-5, (b, t, j)


INF, NINF, NAN = 0x7F80, 0xFF80, 0x7FC1


@pytest.mark.parametrize("case", [
    # (batch, length, q_len, Hq, Hkv, d, page): one and more tiles, waves and rounds of query vectors; whole and cut sequences
    (2, 333, 4, 8, 2, 128, 0), (2, 90, 1, 4, 1, 64, 0), (1, 1500, 8, 8, 2, 128, 16), (2, 700, 12, 4, 1, 64, 16),
    (1, 400, 33, 4, 1, 128, 0), (1, 130, 40, 8, 1, 64, 0), (3, 257, 3, 2, 2, 128, 0),
], ids=lambda c: "-".join(map(str, c)))
def test_rows_with_inf_and_nan_reach_only_the_queries_that_see_them(case):
    batch, n, q_len, hq, hkv, d, page = case
    lens = [n - 7 * b for b in range(batch)]

    def touch(k, v, b, m):
        v[b, :, m - 1, 3], v[b, :, m - 1, 4], v[b, :, m - 1, 11] = NAN, INF, INF   # the newest token, seen by the last query only
        v[b, :, max(m - q_len // 2 - 2, 0), 11] = NINF                              # seen by some
        v[b, 0, m // 3, 20], v[b, 0, m // 2, 21], v[b, 0, m // 2 + 1, 21] = INF, INF, NINF
    wl, q, o, lse = _dense(batch, lens, q_len, hq, hkv, d, page, touch)
    _check(wl, q, o, lse, lens)


@pytest.mark.parametrize("hq,hkv,d,q_len,page", [(8, 2, 128, 1, 0), (4, 2, 64, 1, 0), (4, 4, 128, 1, 16), (8, 1, 64, 5, 16)])
def test_pieces_whose_scores_are_all_minus_infinity(hq, hkv, d, q_len, page):
    """In the middle of the sequence (its pieces are 64 to 512 keys here), and in all of it but the last keys."""
    lens = [2300, 1100]

    def touch(k, v, b, n):
        k[b, :, (600 if b == 0 else 0):(1800 if b == 0 else n - 9), 0] = NINF
    wl, q, o, lse = _dense(2, lens, q_len, hq, hkv, d, page, touch, q_first=0x3F80)
    _check(wl, q, o, lse, lens)


def _deal(lens, q_len, hq, hkv, d, page):
    """How the keys of a batch are dealt out on 256 CUs: (every sequence starts a new run, units per run, pieces of each
    sequence), or None for equal ranges."""
    vectors = q_len * hq // hkv
    unit = 128 // (1 if vectors <= 32 else 2 if vectors <= 64 else 4)
    jobs = hkv * -(-vectors // 128)
    share = -(-(512 if page else 256) // jobs)
    if len(lens) > 256:
        return None
    units = [-(-int(n) // unit) for n in lens]
    most = -(-int(max(lens)) // unit)
    splits = min(most, max(2, min(128, share + 1, 65536 // (len(lens) * q_len * hq))))
    run = -(-sum(units) // share)
    if max(units) > splits and max(units) > run * (splits - 1):
        run = -(-max(units) // (splits - 1))
    short = 384 * 1024 // (4 * d * unit)
    whole = run <= short or sum(-(-u // run) for u in units) <= share
    at, pieces = 0, []
    for u in units:
        pieces.append((at + u - 1) // run - at // run + 1)
        at += -(-u // run) * run if whole else u
    assert max(pieces) <= splits
    return whole, run, pieces


DEALS = [
    # (mode, lengths, q_len, Hq, Hkv, d, page)
    ("end to end", [1500, 1400, 1600, 1333, 1700, 1290, 1555, 1420, 1601], 1, 64, 16, 128, 0),
    ("end to end", [150 + 37 * (i * 11 % 9) for i in range(70)], 1, 64, 16, 128, 0),       # a second group of 64 sequences
    ("end to end", [5000, 33, 1200, 4100, 2600, 64, 700], 12, 64, 16, 128, 0),             # 48 vectors: two waves of them
    ("end to end", [600 + 61 * (i * 5 % 8) for i in range(16)], 4, 128, 32, 128, 16),
    ("end to end", [13000, 200, 9000, 4000], 9, 128, 16, 64, 0),                             # 72 vectors: four waves
    ("whole runs", [6000, 100, 100, 100], 1, 8, 2, 128, 0),
    ("whole runs", [20000, 3], 1, 4, 1, 64, 16),                                           # more units than partial sums
    ("equal ranges", [2300] + [1 + 7 * (i % 60) for i in range(299)], 1, 4, 1, 128, 0),
    ("equal ranges", [1 + 5 * (i % 50) for i in range(257)], 2, 8, 2, 64, 16),
    ("equal ranges", [3000] + [1 + 3 * (i % 70) for i in range(256)], 1, 16, 4, 64, 0),
]


@pytest.mark.parametrize("odd", [False, True])
@pytest.mark.parametrize("case", DEALS, ids=lambda c: "-".join([c[0].replace(" ", "_"), str(len(c[1])), str(max(c[1]))]))
def test_every_way_the_keys_are_dealt_out(case, odd):
    """With and without rows that hold an Inf or a NaN, whose pieces the merge takes again."""
    mode, lens, q_len, hq, hkv, d, page = case
    deal = _deal(lens, q_len, hq, hkv, d, page)
    assert (deal is None) == (mode == "equal ranges")
    if deal:
        assert deal[0] == (mode == "whole runs") and max(deal[2]) > 1

    def touch(k, v, b, n):
        if b % 3 == 0:
            v[b, :, n - 1, 3], v[b, :, n // 2, 11], v[b, 0, n // 3, 20] = NAN, NINF, INF
    wl, q, o, lse = _dense(len(lens), lens, q_len, hq, hkv, d, page, touch if odd else None)
    _check(wl, q, o, lse, lens)
