"""Gather and merge at the edges of the rows a workgroup takes per step (128 of 128 columns, 256 of 64): contexts short
enough to be selected whole, so that the output is plain attention."""
import numpy as np
import pytest

import workloads
from workloads.configs import default_params
from util import plan_params

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("given", [False, True])
@pytest.mark.parametrize("paged", [False, True])
@pytest.mark.parametrize("d", [64, 128])
def test_whole_contexts_around_a_step(d, paged, given):
    import torch
    from paper_2510_05688_amd import binding as vb
    from paper_2510_05688_amd.session import DecodeSession
    lens = [1, 127, 128, 129, 255, 256, 257, 511, 513, 1025, 2048, 2049]
    p = default_params(d, sink=16, window=48, topk_abs=2049, topk_frac=0.0, base_abs=8, base_frac=0.0)
    n_max = 2064 if paged else 2049
    wl = workloads.make_workload("whole", batch=len(lens), n_q_heads=4, n_kv_heads=2, head_dim=d, n_max=n_max,
                                 seq_lens=lens, seed=3, params=p, plant_frac=0.01)
    k_bits, v_bits, table = workloads.to_paged(wl, 16) if paged else (wl.k_bits, wl.v_bits, None)
    sess = DecodeSession(plan_params(wl, paged=paged, num_blocks=k_bits.shape[0] if paged else 0))
    vb.vatt_plan_set_option(sess.plan, vb.VATT_OPT_GIVEN_FUSED if given else vb.VATT_OPT_FUSED_GATHER, 0)
    sess.upload(wl.q_bits, k_bits, v_bits, wl.seq_lens, wl.seeds, table)
    if given:  # all tokens between sink and window
        counts = torch.tensor([max(n - 64, 0) for n in lens], dtype=torch.int32, device="cuda")[:, None].repeat(1, 4)
        sess.decode_given_topk((torch.arange(2049, dtype=torch.int32, device="cuda") + 16).repeat(len(lens), 4, 1), counts)
    else:
        sess.decode()
    res = sess.results_host()
    q = torch.from_numpy(workloads.bf16_bits_to_f32(wl.q_bits)).reshape(len(lens), 4, d).double()
    for b, n in enumerate(lens):
        for h in range(4):
            assert res["counts"][b, h, :5].sum() - res["counts"][b, h, 3] == n
            s = torch.from_numpy(wl.k_f32(b, h // 2, n)).double() @ q[b, h] / np.sqrt(d)
            want = torch.softmax(s, 0) @ torch.from_numpy(wl.v_f32(b, h // 2, n)).double()
            got = torch.from_numpy(res["O"][b, h]).double()
            assert float((got - want).norm() / want.norm()) < 2e-5, (n, h)
            assert abs(float(torch.logsumexp(s, 0)) - float(res["lse"][b, h])) < 2e-5, (n, h)
    sess.close()


@pytest.mark.parametrize("fused", [False, True])
@pytest.mark.parametrize("d,rows", [(64, 1), (64, 700), (128, 1), (128, 400)])
def test_a_nan_among_the_listed_scores_is_not_left_out(d, rows, fused):
    """One K row, and enough of them to fill the whole run of a workgroup, hold a NaN: every output of the heads that list
    them is NaN, whichever kernels take the step, and the others are as without."""
    import torch
    from paper_2510_05688_amd import binding as vb
    from paper_2510_05688_amd.session import DecodeSession
    n, first = 2000, 900
    p = default_params(d, sink=16, window=48, topk_abs=n, topk_frac=0.0, base_abs=8, base_frac=0.0)
    wl = workloads.make_workload("nan", batch=1, n_q_heads=4, n_kv_heads=2, head_dim=d, n_max=n, seq_lens=[n], seed=3, params=p)
    wl.k_bits[0, 0, first:first + rows, 5] = 0x7FC0
    sess = DecodeSession(plan_params(wl))
    if not fused:
        vb.vatt_plan_set_option(sess.plan, vb.VATT_OPT_GIVEN_FUSED, 0)
    sess.upload(wl.q_bits, wl.k_bits, wl.v_bits, wl.seq_lens, wl.seeds)
    counts = torch.full((1, 4), n - 64, dtype=torch.int32, device="cuda")
    sess.decode_given_topk((torch.arange(n, dtype=torch.int32, device="cuda") + 16).repeat(1, 4, 1), counts)
    res = sess.results_host()
    assert np.isnan(res["O"][0, :2]).all() and np.isnan(res["lse"][0, :2]).all()
    for h in (2, 3):
        s = torch.from_numpy(wl.k_f32(0, 1, n)).double() @ torch.from_numpy(wl.q_f32()[0, h]).double() / np.sqrt(d)
        want = torch.softmax(s, 0) @ torch.from_numpy(wl.v_f32(0, 1, n)).double()
        assert float((torch.from_numpy(res["O"][0, h]).double() - want).norm() / want.norm()) < 2e-5
    sess.close()


@pytest.mark.parametrize("fused", [False, True])
@pytest.mark.parametrize("d,n", [(64, 700), (128, 321), (128, 1000)])
def test_an_inf_in_the_last_listed_row_stays_an_inf(d, n, fused):
    """A workgroup's last step repeats its last row where it has no more; with weight 0, which must not make a NaN of it."""
    import torch
    from paper_2510_05688_amd import binding as vb
    from paper_2510_05688_amd.session import DecodeSession
    p = default_params(d, sink=16, window=48, topk_abs=n, topk_frac=0.0, base_abs=8, base_frac=0.0)
    wl = workloads.make_workload("inf", batch=1, n_q_heads=4, n_kv_heads=2, head_dim=d, n_max=n, seq_lens=[n], seed=3, params=p)
    wl.v_bits[0, :, n - 49, 7] = 0x7F80   # the largest token before the window: the last of the list
    sess = DecodeSession(plan_params(wl))
    if not fused:
        vb.vatt_plan_set_option(sess.plan, vb.VATT_OPT_GIVEN_FUSED, 0)
    sess.upload(wl.q_bits, wl.k_bits, wl.v_bits, wl.seq_lens, wl.seeds)
    counts = torch.full((1, 4), n - 64, dtype=torch.int32, device="cuda")
    sess.decode_given_topk((torch.arange(n, dtype=torch.int32, device="cuda") + 16).repeat(1, 4, 1), counts)
    o = sess.results_host()["O"][0]
    assert np.all(o[:, 7] == np.inf) and np.isfinite(np.delete(o, 7, axis=1)).all()
    sess.close()


@pytest.mark.parametrize("splits", [1, 2])
@pytest.mark.parametrize("paged", [False, True])
@pytest.mark.parametrize("d", [64, 128])
def test_fused_gather_around_its_rounds(d, paged, splits):
    """Lists that end at, before and behind a quarter, half and all of the rows that the fused gather requests at a time (64,
    128 and 256 rows of 128 columns, twice as many of 64)."""
    import torch
    from paper_2510_05688_amd import binding as vb
    from paper_2510_05688_amd.session import DecodeSession
    lens = [m * splits + e for m in (64, 128, 256, 512) for e in (-1, 0, 1)] + [1, 640 * splits]
    n_max = 640 * splits
    p = default_params(d, sink=16, window=48, topk_abs=n_max, topk_frac=0.0, base_abs=8, base_frac=0.0)
    wl = workloads.make_workload("rounds", batch=len(lens), n_q_heads=4, n_kv_heads=2, head_dim=d, n_max=n_max,
                                 seq_lens=lens, seed=4, params=p, plant_frac=0.01)
    k_bits, v_bits, table = workloads.to_paged(wl, 16) if paged else (wl.k_bits, wl.v_bits, None)
    sess = DecodeSession(plan_params(wl, paged=paged, num_blocks=k_bits.shape[0] if paged else 0))
    vb.vatt_plan_set_option(sess.plan, vb.VATT_OPT_FUSED_GATHER, splits)
    sess.upload(wl.q_bits, k_bits, v_bits, wl.seq_lens, wl.seeds, table)
    sess.decode()
    res = sess.results_host()
    q = torch.from_numpy(workloads.bf16_bits_to_f32(wl.q_bits)).reshape(len(lens), 4, d).double()
    for b, n in enumerate(lens):
        for h in range(4):
            s = torch.from_numpy(wl.k_f32(b, h // 2, n)).double() @ q[b, h] / np.sqrt(d)
            want = torch.softmax(s, 0) @ torch.from_numpy(wl.v_f32(b, h // 2, n)).double()
            got = torch.from_numpy(res["O"][b, h]).double()
            assert float((got - want).norm() / want.norm()) < 2e-5, (n, h)
            assert abs(float(torch.logsumexp(s, 0)) - float(res["lse"][b, h])) < 2e-5, (n, h)
    sess.close()


@pytest.mark.parametrize("splits", [1, 2, 4])
@pytest.mark.parametrize("d,epsilon", [(64, 0.02), (64, 0.004), (128, 0.03), (128, 0.008)])
def test_budgets_beyond_the_first_draws_are_paged_as_they_are_contiguous(d, epsilon, splits):
    """Final samples that the first batch of draws holds, that need further ones and that are complements, on a paged cache
    (whose lists name rows by their place in the pool) and on a contiguous one: the same bits."""
    from paper_2510_05688_amd import binding as vb
    from paper_2510_05688_amd.session import DecodeSession
    p = default_params(d, sink=16, window=48, topk_abs=0, topk_frac=0.02, base_abs=32, base_frac=0.0, epsilon=epsilon)
    wl = workloads.make_workload("budgets", batch=3, n_q_heads=4, n_kv_heads=2, head_dim=d, n_max=8192,
                                 seq_lens=[8192, 5001, 700], seed=6, params=p, plant_frac=0.01)
    got = []
    for paged in (False, True):
        k_bits, v_bits, table = workloads.to_paged(wl, 16) if paged else (wl.k_bits, wl.v_bits, None)
        sess = DecodeSession(plan_params(wl, paged=paged, num_blocks=k_bits.shape[0] if paged else 0))
        sess.upload(wl.q_bits, k_bits, v_bits, wl.seq_lens, wl.seeds, table)
        for fused in (0, splits):
            vb.vatt_plan_set_option(sess.plan, vb.VATT_OPT_FUSED_GATHER, fused)
            sess.out_idx.zero_()
            sess.decode()
            got.append(sess.results_host())
        sess.close()
    assert (got[0]["counts"][..., 4] > 1024).any() or epsilon > 0.01
    for key in ("counts", "idx", "b_star"):
        assert all(np.array_equal(got[0][key], g[key]) for g in got[1:]), key
    assert np.array_equal(got[1]["O"], got[3]["O"]) and np.array_equal(got[1]["lse"], got[3]["lse"])
    for b in range(3):
        for h in range(4):
            want = got[0]["O"][b, h]
            assert np.linalg.norm(got[1]["O"][b, h] - want) <= 2e-6 * np.linalg.norm(want)


def _decode(wl, paged, splits, v_bits, copies=1):
    from paper_2510_05688_amd import binding as vb
    from paper_2510_05688_amd.session import DecodeSession
    kept, wl.v_bits = wl.v_bits, v_bits
    k_bits, v_bits, table = workloads.to_paged(wl, 16) if paged else (wl.k_bits, wl.v_bits, None)
    wl.v_bits = kept
    sess = DecodeSession(dict(plan_params(wl, paged=paged, num_blocks=k_bits.shape[0] if paged else 0), batch=wl.batch * copies))
    vb.vatt_plan_set_option(sess.plan, vb.VATT_OPT_FUSED_GATHER, splits)
    tile = lambda a: np.concatenate([a] * copies)
    sess.upload(tile(wl.q_bits), k_bits if paged else tile(k_bits), v_bits if paged else tile(v_bits), tile(wl.seq_lens), tile(wl.seeds),
                tile(table) if paged else None)
    sess.decode()
    res = sess.results_host()
    sess.close()
    return res


@pytest.mark.parametrize("splits", [0, 1, 4])
@pytest.mark.parametrize("paged", [False, True])
@pytest.mark.parametrize("d,n,epsilon", [(64, 700, 0.05), (128, 2000, 0.05), (64, 5000, 0.02), (128, 5000, 0.01)])
def test_a_row_that_no_head_lists_adds_nothing(d, n, epsilon, paged, splits):
    """An Inf and a NaN in the V rows of token 0, which the heads compared here do not list (no sink): the same bits as without,
    whether the first draws hold the final sample or not."""
    p = default_params(d, sink=0, window=48, topk_abs=0, topk_frac=0.02, base_abs=32, base_frac=0.0, epsilon=epsilon)
    wl = workloads.make_workload("unlisted", batch=1, n_q_heads=8, n_kv_heads=2, head_dim=d, n_max=5008, seq_lens=[n], seed=5, params=p)
    spoilt = wl.v_bits.copy()
    spoilt[0, :, 0, 5], spoilt[0, :, 0, d - 1] = 0x7FC0, 0x7F80
    want, got = _decode(wl, paged, splits, wl.v_bits), _decode(wl, paged, splits, spoilt)
    seg, compared = got["seg"], 0
    for h in range(8):
        c, idx = got["counts"][0, h], got["idx"][0, h]
        listed = np.concatenate([idx[seg[2]:seg[2] + c[2]], idx[seg[4]:seg[4] + c[4]]])
        if 0 not in listed:
            compared += 1
            assert np.array_equal(got["O"][0, h], want["O"][0, h]) and np.isfinite(got["O"][0, h]).all(), h
    assert compared >= 4 and ((got["counts"][..., 4] > 1024).any() or epsilon > 0.01)


@pytest.mark.parametrize("splits", [0, 1, 2])
@pytest.mark.parametrize("paged", [False, True])
@pytest.mark.parametrize("d,n", [(64, 700), (128, 321), (128, 1000)])
def test_an_inf_in_a_listed_row_stays_an_inf(d, n, paged, splits):
    """The first row of the list and the last: what fills a batch of rows behind the list's end must not make a NaN of it."""
    p = default_params(d, sink=16, window=48, topk_abs=n, topk_frac=0.0, base_abs=8, base_frac=0.0)
    wl = workloads.make_workload("inf", batch=1, n_q_heads=4, n_kv_heads=2, head_dim=d, n_max=1008, seq_lens=[n], seed=3, params=p)
    for tok in (0, n - 49):
        spoilt = wl.v_bits.copy()
        spoilt[0, :, tok, 7] = 0x7F80
        o = _decode(wl, paged, splits, spoilt)["O"][0]
        assert np.all(o[:, 7] == np.inf) and np.isfinite(np.delete(o, 7, axis=1)).all(), tok


@pytest.mark.parametrize("paged", [False, True])
@pytest.mark.parametrize("d", [64, 128])
def test_an_inf_in_the_last_base_sample_row_stays_an_inf(d, paged):
    """Output target: the statistics pass reads the base sample's rows last, the gather behind it the final sample's.  Both are the whole
    residual here and end with the largest token before the window; an Inf in its V row makes the numerator's norm and the output
    Inf, not NaN, with several gather workgroups per head and with one."""
    n = 300
    p = default_params(d, sink=16, window=48, topk_abs=8, topk_frac=0.0, base_abs=n, base_frac=0.0, target=2)
    wl = workloads.make_workload("inf_base", batch=1, n_q_heads=4, n_kv_heads=2, head_dim=d, n_max=304, seq_lens=[n], seed=3, params=p)
    spoilt = wl.v_bits.copy()
    spoilt[0, :, n - 49, 7] = 0x7F80
    for copies in (1, 1024):  # (4096 heads have one workgroup each)
        res = _decode(wl, paged, 0, spoilt, copies)
        seg, counts, idx = res["seg"], res["counts"][-1], res["idx"][-1]
        heads = [h for h in range(4) if idx[h, seg[3] + counts[h, 3] - 1] == n - 49]
        assert heads
        for h in heads:
            assert idx[h, seg[4] + counts[h, 4] - 1] == n - 49
            assert res["stats"][-1, h, 3] == np.inf and res["O"][-1, h, 7] == np.inf
            assert np.isfinite(np.delete(res["O"][-1, h], 7)).all()
