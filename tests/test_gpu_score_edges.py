"""Score pass against fp32 dot products at the edges of its pieces: keys per wave (16, 32, 64), per workgroup (64 to 512),
and rounds of query vectors."""
import numpy as np
import pytest

import workloads
from workloads.configs import default_params

pytestmark = pytest.mark.gpu

CASES = [
    # (lengths, q_len, Hq, Hkv, d, page)
    ((1, 15, 16, 17), 1, 4, 1, 128, 0), ((63, 64, 65, 66), 1, 8, 8, 64, 0), ((129, 31, 33, 47), 1, 16, 2, 128, 0),
    ((5, 64, 193, 257), 1, 16, 8, 64, 0), ((31, 32, 33, 127), 1, 4, 2, 128, 16), ((128, 129, 255, 1), 1, 8, 1, 64, 16),
    ((500, 512, 513, 9), 1, 2, 2, 128, 64), ((3, 1025, 70, 700), 1, 32, 8, 128, 0),
    ((63, 64, 65, 1), 2, 4, 1, 128, 0), ((255, 256, 257, 40), 3, 8, 8, 64, 16), ((511, 512, 513, 64), 5, 8, 1, 64, 0),
    ((300, 17, 18, 200), 17, 8, 2, 128, 16), ((100, 33, 20, 65), 16, 16, 2, 128, 0), ((200, 1, 9, 64), 9, 8, 1, 128, 64),
]


@pytest.mark.parametrize("case", CASES, ids=lambda c: "-".join(map(str, c[0] + c[1:])))
def test_scores_against_fp32(case):
    import torch
    from paper_2510_05688_amd.session import DecodeSession

    lens, q_len, hq, hkv, d, page = case
    batch, g = len(lens), hq // hkv
    n_max = -(-max(lens) // page) * page if page else max(lens)
    wl = workloads.make_workload("scores", batch=batch, n_q_heads=hq, n_kv_heads=hkv, head_dim=d, n_max=n_max,
                                 seq_lens=np.array(lens), seed=7, params=default_params(d), plant_frac=0.01)
    q_bits = workloads.chunk_queries(wl, q_len, seed=2) if q_len > 1 else wl.q_bits
    k_bits, v_bits, table = workloads.to_paged(wl, page) if page else (wl.k_bits, wl.v_bits, None)
    sess = DecodeSession(dict(batch=batch, n_q_heads=hq, n_kv_heads=hkv, head_dim=d, n_max=n_max, kv_layout=1 if page else 0,
                              page_size=page, num_blocks=k_bits.shape[0] if page else 0, sink=4, window=8, topk_abs=0,
                              topk_frac=0.02, base_abs=0, base_frac=0.02, epsilon=0.1, delta=0.1, target=0, sm_scale=0.0,
                              budget_cap_frac=1.0), q_len=q_len)
    sess.upload(q_bits, k_bits, v_bits, wl.seq_lens, wl.seeds, table)
    sess.score()
    torch.cuda.synchronize()
    got = sess.scores_host()
    q = workloads.bf16_bits_to_f32(q_bits).reshape(batch, q_len, hq, d)
    for b, n in enumerate(lens):
        for t in range(q_len):
            seen = max(n - (q_len - 1 - t), 1)
            for h in range(hq):
                want = (wl.k_f32(b, h // g, seen).astype(np.float64) @ q[b, t, h].astype(np.float64)) / np.sqrt(d)
                np.testing.assert_allclose(got[b * q_len + t, h, :seen], want, rtol=0, atol=1e-5 * max(1.0, np.abs(want).max()))
    sess.close()
