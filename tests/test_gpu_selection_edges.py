"""Selection kernel at the edges of its sizes: draws that repeat many tokens, mail slots shared by two tokens, few and
many candidates of the top-k set, candidates with equal scores; every head against the oracle."""
import numpy as np
import pytest

import workloads
from workloads.configs import default_params
from parity import check_all
from util import plan_params

pytestmark = pytest.mark.gpu

# (longest row, shortest row, k, b0, epsilon): middle regions of 0 .. a few times the 2048 mail slots; base samples of a
# few tokens up to half of the residual (the whole first batch of draws, and more than one batch)
CASES = [
    (40, 33, 3, 4, 0.3), (300, 290, 5, 60, 0.05), (1024, 517, 32, 32, 0.05), (2079, 2080 - 3, 100, 700, 0.02),
    (2081, 2079, 256, 40, 0.3), (4200, 3000, 257, 1900, 0.1), (6000, 5121, 513, 300, 0.01), (9001, 8200, 1100, 1000, 0.05),
]


@pytest.mark.parametrize("fused", [True, False])
@pytest.mark.parametrize("case", CASES, ids=lambda c: "-".join(map(str, c)))
def test_selection_at_the_edges_of_its_sizes(case, fused):
    from paper_2510_05688_amd import binding as vb
    from paper_2510_05688_amd.session import DecodeSession
    hi, lo, k, b0, eps = case
    p = default_params(64, sink=4, window=28, topk_abs=k, topk_frac=0.0, base_abs=b0, base_frac=0.0, epsilon=eps)
    wl = workloads.make_workload("edges", batch=3, n_q_heads=4, n_kv_heads=2, head_dim=64, n_max=hi,
                                 seq_lens=[hi, lo, (hi + lo) // 2], seed=sum(map(int, case[:4])), params=p, plant_frac=0.003)
    sess = DecodeSession(plan_params(wl))
    if not fused:
        vb.vatt_plan_set_option(sess.plan, vb.VATT_OPT_FUSED_GATHER, 0)
    sess.upload(wl.q_bits, wl.k_bits, wl.v_bits, wl.seq_lens, wl.seeds)
    sess.decode()
    check_all(wl, sess.results_host(), label="edges %s" % (case,))
    sess.close()


def test_equal_scores_among_the_candidates():
    # rows of one repeated key: every candidate has the same score and the lower tokens win; and rows of two keys
    from paper_2510_05688_amd.session import DecodeSession
    p = default_params(64, sink=4, window=28, topk_abs=300, topk_frac=0.0, base_abs=50, base_frac=0.0, epsilon=0.1)
    wl = workloads.make_workload("equal", batch=2, n_q_heads=2, n_kv_heads=1, head_dim=64, n_max=3000, seq_lens=[3000, 2500],
                                 seed=8, params=p, plant_frac=0.0)
    wl.k_bits[0, 0, :] = wl.k_bits[0, 0, 0]
    wl.k_bits[1, 0, 0::2] = wl.k_bits[1, 0, 0]
    wl.k_bits[1, 0, 1::2] = wl.k_bits[1, 0, 1]
    sess = DecodeSession(plan_params(wl))
    sess.upload(wl.q_bits, wl.k_bits, wl.v_bits, wl.seq_lens, wl.seeds)
    sess.decode()
    res = sess.results_host()
    seg = res["seg"]
    for h in range(2):
        got = res["idx"][0, h, seg[2]:seg[2] + 300]
        assert np.array_equal(got, np.arange(4, 304)), "equal scores: the lower tokens win"
    check_all(wl, res, label="equal scores")
    sess.close()


@pytest.mark.parametrize("k", [1900, 2048, 2049, 5500])
def test_more_candidates_than_the_list_holds(k):
    # long rows (1024 threads): the candidates fit the list, do not, and (5500 of 7500 sub-tiles) nearly all sub-tiles qualify
    from paper_2510_05688_amd.session import DecodeSession
    p = default_params(64, sink=5, window=30, topk_abs=k, topk_frac=0.0, base_abs=200, base_frac=0.0, epsilon=0.2)
    wl = workloads.make_workload("wide", batch=2, n_q_heads=2, n_kv_heads=1, head_dim=64, n_max=60003, seq_lens=[60003, 45001],
                                 seed=k, params=p, plant_frac=0.003)
    sess = DecodeSession(plan_params(wl))
    sess.upload(wl.q_bits, wl.k_bits, wl.v_bits, wl.seq_lens, wl.seeds)
    sess.decode()
    check_all(wl, sess.results_host(), label="wide %d" % k)
    sess.close()


# (longest row, shortest row, k, b0, epsilon): samples within the first batch of draws, of several batches, complements, whole
# residuals, no residual; top-k sets from the candidate list, from the wide list and from the general path
@pytest.mark.parametrize("case", [(45, 33, 6, 3, 0.3), (1200, 700, 64, 32, 0.05), (9001, 8200, 200, 300, 0.05), (9001, 5000, 2300, 40, 0.02),
                                  (16003, 12000, 400, 100, 0.006), (33001, 30000, 5000, 300, 0.1)], ids=lambda c: "-".join(map(str, c)))
def test_two_workgroups_per_head_leave_what_one_leaves(case):
    from paper_2510_05688_amd import binding as vb
    from paper_2510_05688_amd.session import DecodeSession
    hi, lo, k, b0, eps = case
    p = default_params(64, sink=4, window=28, topk_abs=k, topk_frac=0.0, base_abs=b0, base_frac=0.0, epsilon=eps)
    wl = workloads.make_workload("pair", batch=2, n_q_heads=4, n_kv_heads=2, head_dim=64, n_max=hi, seq_lens=[hi, lo],
                                 seed=sum(map(int, case[:4])), params=p, plant_frac=0.003)
    got = []
    for repeat in (1, 20):  # 8 heads; 160, more than half of the compute units: one workgroup each
        sess = DecodeSession(dict(plan_params(wl), batch=wl.batch * repeat))
        vb.vatt_plan_set_option(sess.plan, vb.VATT_OPT_HEAD_THREADS, 1024)
        tile = lambda a: np.concatenate([a] * repeat)
        sess.upload(tile(wl.q_bits), tile(wl.k_bits), tile(wl.v_bits), tile(wl.seq_lens), tile(wl.seeds))
        sess.workspace.fill_(0xff)  # (scores that nobody left would be NaN)
        sess.out_idx.zero_()
        sess.decode()
        got.append(sess.results_host())
        sess.close()
    one, many = got
    check_all(wl, one, label="pair %s" % (case,))
    for name in ("idx", "counts", "b_star", "stats"):
        assert np.array_equal(many[name][:wl.batch], one[name]), name
    # (another number of partial sums of the same 32-bit products)
    np.testing.assert_allclose(many["O"][:wl.batch], one["O"], rtol=0, atol=4e-6 * np.abs(one["O"]).max())
