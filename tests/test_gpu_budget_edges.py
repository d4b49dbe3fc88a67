"""Budget and final sample of the targets N and SDPA at the edges of their sizes: samples that the first batch of draws holds, that take
several, complements, whole residuals and none; every head against the oracle, and few heads, which have two workgroups each in the first
selection phase, against many."""
import numpy as np
import pytest

import workloads
from workloads.configs import default_params
from parity import check_all
from util import plan_params

pytestmark = pytest.mark.gpu

# (longest row, shortest row, k, b0, epsilon, target): budgets from the base sample up to the whole residual; residuals around
# 1024 and 4096 draws, and (30 tokens of a row of 62) none
CASES = [
    (62, 31, 30, 2, 0.3, 2), (700, 530, 20, 30, 0.5, 1), (2100, 1500, 100, 64, 0.2, 2), (5003, 4099, 64, 40, 0.12, 2),
    (9001, 8200, 200, 300, 0.1, 1), (16387, 12000, 400, 390, 0.1, 2), (30000, 20011, 0, 100, 0.06, 2),
]


def _launches(sess):
    """Kernels of one decode call: the nodes of a graph that it is captured into."""
    import ctypes
    import torch
    side = torch.cuda.Stream()
    side.wait_stream(torch.cuda.current_stream())
    graph = torch.cuda.CUDAGraph(keep_graph=True)
    with torch.cuda.graph(graph, stream=side):
        sess.decode()
    count = ctypes.c_size_t(0)
    hip = ctypes.CDLL("libamdhip64.so")
    assert hip.hipGraphGetNodes(ctypes.c_void_p(graph.raw_cuda_graph()), None, ctypes.byref(count)) == 0
    return count.value


def _run(wl, threads, repeat=1, paged=False):
    from paper_2510_05688_amd.session import DecodeSession
    from paper_2510_05688_amd import binding as vb
    k_bits, v_bits, table = workloads.to_paged(wl, 16) if paged else (wl.k_bits, wl.v_bits, None)
    params = dict(plan_params(wl, paged=paged, num_blocks=len(k_bits) if paged else 0), batch=wl.batch * repeat)
    sess = DecodeSession(params)
    vb.vatt_plan_set_option(sess.plan, vb.VATT_OPT_HEAD_THREADS, threads)
    tile = lambda a: np.concatenate([a] * repeat)
    # (on a paged cache the copies of a sequence read the same pages)
    sess.upload(tile(wl.q_bits), k_bits if paged else tile(k_bits), v_bits if paged else tile(v_bits), tile(wl.seq_lens), tile(wl.seeds),
                tile(table) if paged else None)
    sess.workspace.fill_(0xff)  # (scores and sums that nobody left would be NaN)
    sess.out_idx.zero_()
    sess.decode()
    res = sess.results_host()
    launches = _launches(sess)
    sess.close()
    return res, launches


@pytest.mark.parametrize("head_dim, threads, paged", [(64, 512, False), (128, 512, False), (128, 1024, False), (64, 512, True), (128, 512, True)])
@pytest.mark.parametrize("case", CASES, ids=lambda c: "-".join(map(str, c)))
def test_budgets_at_the_edges_of_their_sizes(case, head_dim, threads, paged):
    hi, lo, k, b0, eps, target = case
    p = default_params(head_dim, sink=4, window=28, topk_abs=k, topk_frac=0.0, base_abs=b0, base_frac=0.0, epsilon=eps, target=target)
    wl = workloads.make_workload("budgets", batch=2, n_q_heads=4, n_kv_heads=2, head_dim=head_dim, n_max=-(-hi // 16) * 16 if paged else hi,
                                 seq_lens=[hi, lo], seed=sum(map(int, case[:4])), params=p, v_mean=1.0, plant_frac=0.003)
    res, _ = _run(wl, threads, paged=paged)
    check_all(wl, res, label="budgets %s" % (case,))
    # The same sequences among more heads than the card has compute units, one workgroup each: the same lists, counts and flags.  The
    # statistics pass is cut at other places there, so its 32-bit sums of a few hundred rows differ by rounding, the unrounded budgets by
    # some 1e-6 and a budget next to a whole number by one.  A head with the same budget has the same output up to that rounding.
    repeat = 40
    many, _ = _run(wl, threads, repeat, paged)
    seg, counts = res["seg"], res["counts"]
    for r in (0, repeat - 1):
        rows = slice(r * wl.batch, (r + 1) * wl.batch)
        np.testing.assert_allclose(many["b_star"][rows], res["b_star"], rtol=1e-5)
        np.testing.assert_allclose(many["stats"][rows], res["stats"], rtol=1e-5)
        agree = many["counts"][rows, :, 4] == counts[..., 4]
        assert agree.sum() >= 6, agree
        np.testing.assert_allclose(many["O"][rows][agree], res["O"][agree], rtol=0, atol=4e-6 * np.abs(res["O"]).max())
        np.testing.assert_allclose(many["lse"][rows][agree], res["lse"][agree], rtol=0, atol=4e-6)
        for b in range(wl.batch):
            for h in range(4):
                one, other = counts[b, h], many["counts"][r * wl.batch + b, h]
                assert abs(int(one[4]) - int(other[4])) <= 1
                if one[4] == other[4]:
                    assert np.array_equal(one, other)
                n_dyn = int(min(one[4], other[4]))
                if not int(one[7]) & 2:  # (a complement leaves out another token if one fewer is left out)
                    assert np.array_equal(many["idx"][r * wl.batch + b, h, seg[4]:seg[4] + n_dyn], res["idx"][b, h, seg[4]:seg[4] + n_dyn])


@pytest.mark.parametrize("paged", [False, True])
@pytest.mark.parametrize("head_dim", [64, 128])
def test_one_gather_workgroup_per_head_finishes_it(head_dim, paged):
    """Sixteen heads per compute unit and more: the gather of the final sample adds the sums over I_f itself, with an empty sample (30
    tokens) too, and no merge is launched."""
    p = default_params(head_dim, sink=4, window=28, topk_abs=20, topk_frac=0.0, base_abs=16, base_frac=0.0, epsilon=0.3, target=2)
    wl = workloads.make_workload("alone", batch=2, n_q_heads=4, n_kv_heads=2, head_dim=head_dim, n_max=320, seq_lens=[317, 30], seed=9, params=p,
                                 v_mean=1.0)
    repeat = 512
    one, launches_one = _run(wl, 512, 1, paged)
    many, launches_many = _run(wl, 512, repeat, paged)
    check_all(wl, one, label="alone")
    assert (launches_one, launches_many) == (6, 5)
    assert not one["counts"][1, :, 4].any() and (one["counts"][0, :, 4] > 0).all()
    for r in range(0, repeat, 73):
        rows = slice(2 * r, 2 * r + 2)
        assert np.array_equal(many["counts"][rows], one["counts"])
        # (sums of some hundred 32-bit products cut at other places: a few units in the last place of the largest value)
        np.testing.assert_allclose(many["O"][rows], one["O"], rtol=0, atol=4e-6 * np.abs(one["O"]).max())
        np.testing.assert_allclose(many["lse"][rows], one["lse"], rtol=0, atol=4e-6)
