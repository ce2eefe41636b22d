"""The fused call pools, adds the prior and selects in one kernel where one workgroup holds a request: same bits as the
separate calls (each of which is checked against the oracle elsewhere) at the edges of every workgroup shape."""
import numpy as np
import pytest

from paper_2604_10235_amd import workloads as wl
from tests import parity_util as pu

pytestmark = pytest.mark.gpu

W = 16


def both(w, **kw):
    import torch
    from paper_2604_10235_amd import binding as b
    q, k, v, prior = wl.make_all(w)
    steps, fused = (b.DeviceProblem(w, q, k, v, prior, **kw) for _ in range(2))
    steps.score(); steps.select(); steps.gather()
    fused.workspace.fill_(0xFF)                                    # nothing may be read before it is written
    fused.scores.fill_(float("nan")); fused.idx.fill_(-1); fused.k_out.fill_(0)
    fused.compress()
    torch.cuda.synchronize()
    assert torch.equal(steps.scores.view(torch.int32), fused.scores.view(torch.int32))
    assert torch.equal(steps.idx, fused.idx)
    cu, cb = w.cu_seqlens(), w.cu_budgets()
    assert np.array_equal(b.DeviceProblem.bits(fused.k_out), pu.host_gather(k, fused.idx.cpu().numpy(), cu, cb))
    return fused


def batch(lens, heads=2, **over):
    budgets = [max(W, W + (n - W) * (1 + i % 3) // 7) for i, n in enumerate(lens)]
    return wl.scaled(wl.tiny(), seqlens=lens, budgets=budgets, window=W, n_q_heads=heads, n_kv_heads=heads, **over)


@pytest.mark.parametrize("edge", [1024, 2048, 4096, 8192, 16384, 32768, 49152, 65536])
@pytest.mark.parametrize("off", [-1, 0, 1])
def test_edges_of_the_workgroup_shapes(edge, off):
    n = edge + off
    both(batch([n, W + 5, W, W + 1]))                              # the longest request picks the shape
    both(batch([n], prior_weight=0.0), select_mode=1, span_budget_ratio=0.5)


@pytest.mark.parametrize("candidates", [0, 1, 2, 3, 4, 5])
def test_prefixes_about_one_group_of_four(candidates):
    for window in (1, 2, 3, 4, W):                                 # the end of the prefix inside a group of four tokens, and of the request
        n = window + candidates
        for kept in range(candidates + 1):
            w = wl.scaled(wl.tiny(), seqlens=[n, window], budgets=[window + kept, window], window=window, n_q_heads=2, n_kv_heads=2)
            both(w)
        both(w, select_mode=1, span_budget_ratio=0.5)


@pytest.mark.parametrize("longest", [2048, 4096, 8192, 16384])
def test_many_problems_take_the_small_workgroups(longest):
    both(batch([longest, longest - 3, 700, W + 2], heads=128))     # 512 problems


@pytest.mark.parametrize("pool", [1, 3, 5, 7, 9, 11, 65, 1025])
@pytest.mark.parametrize("variant", [0, 4, 8, 16, 4 | 8 | 16])
def test_pooling_widths_and_readings(pool, variant):
    both(batch([5003, 300, 33041, W + 40], pool_kernel=pool), score_variant=variant)


@pytest.mark.parametrize("longest,quad,heads", [(8192, 4096, 2), (40000, 4096, 2), (2048, 1024, 86), (4096, 1024, 86), (8192, 2048, 86)])
@pytest.mark.parametrize("pool,variant", [(7, 0), (1025, 0), (7, 8), (7, 16), (1025, 8 | 16)])
def test_requests_whose_masses_end_just_below_a_quad_of_the_longest_one(longest, quad, heads, pool, variant):
    """The longest request makes every workgroup ask for several quads; the masses of others end one to three tokens below one of
    them, within the pooling reach of what lies past their row: the next request's masses, which must not come in."""
    trim = W if variant & (8 | 16) else 0
    both(batch([longest, quad - 1 + trim, W + 3, quad - 2 + trim, quad - 3 + trim, W + 1], heads=heads, pool_kernel=pool),
         score_variant=variant)


@pytest.mark.parametrize("pool", [1, 3, 7, 9, 11])
@pytest.mark.parametrize("variant", [0, 4])
def test_masses_that_are_not_finite_reach_no_further_than_the_pooling_width(pool, variant):
    """A query row whose logits all lie below the smallest softmax reference has infinite masses, NaN where a logit is -inf: the
    pooled scores of the fused call hold infinities and NaN at the same tokens as those of the separate calls."""
    import torch
    from paper_2604_10235_amd import binding as b
    w = batch([3000, 700, 41], pool_kernel=pool)
    q, k, v, prior = wl.make_all(w)
    as_bits = lambda x: int(torch.tensor(x, dtype=torch.bfloat16).view(torch.int16)) & 0xFFFF
    q[:, 0, 0] = 0                                                  # head 0 in the first request: even rows but for one ...
    q[:, 0, 0, 3, :] = as_bits(1e18)
    k[:, 0, :3000, :] = as_bits(-1e18)                             # ... that meets keys which give it about -6e37
    k[:, 0, [0, 1000, 1012, 2047, 2999], :] = as_bits(-3e38)       # ... and -inf
    steps, fused = (b.DeviceProblem(w, q, k, v, prior, score_variant=variant) for _ in range(2))
    steps.score(); steps.select(); fused.compress()
    torch.cuda.synchronize()
    want, got = steps.scores.cpu().numpy(), fused.scores.cpu().numpy()
    assert np.isinf(want[:, 0, :3000]).any() and np.isfinite(want[:, :, 3000:]).all() and np.isfinite(want[:, 1]).all()
    assert np.array_equal(np.isnan(want), np.isnan(got)) and np.array_equal(want[~np.isnan(want)], got[~np.isnan(want)])
    assert (np.diff(fused.idx.cpu().numpy()[:, :, :w.budgets[0]]) > 0).all()


# Widths above nine on both sides of the rule that gives them to the fused kernel (11 .. 215) or to the pooling kernel; quads of
# one, two and four rounds, requests that end just below one of them.
@pytest.mark.parametrize("longest,quad,heads,pool", [(150, 0, 2, 1025), (600, 0, 2, 257), (2000, 0, 2, 65), (4000, 0, 2, 33), (8192, 4096, 2, 19), (8192, 4096, 2, 21),
                                                     (14000, 8192, 2, 11), (14000, 8192, 2, 13), (2048, 1024, 86, 65), (2048, 1024, 86, 215),
                                                     (4096, 1024, 86, 65), (4096, 2048, 86, 129)])
@pytest.mark.parametrize("variant", [0, 4, 8, 8 | 16])
def test_wide_pooling_fused_and_separate(longest, quad, heads, pool, variant):
    trim = W if variant & (8 | 16) else 0
    lens = [quad - d + trim for d in (1, 2, 3)] if quad else [W + 1, W + 2, longest // 2]
    both(batch([longest, lens[0], W + 3, lens[1], lens[2], W + 1], heads=heads, pool_kernel=pool), score_variant=variant)


@pytest.mark.parametrize("pool", [7, 11, 19])
@pytest.mark.parametrize("variant", [0, 4 | 16])
def test_pooling_across_the_seam_of_two_fillings(pool, variant):
    """Requests beyond 32768 tokens pass through LDS in two fillings; with 256 of them the widths above nine are fused too."""
    import torch
    from paper_2604_10235_amd import binding as b
    heads, n, budget = 256, 33000, 3000
    g = torch.Generator(device="cuda:0").manual_seed(pool)
    q, k = (torch.randn((heads, rows, 64), generator=g, device="cuda:0").bfloat16() for rows in (W, n))
    prior = torch.rand((n,), generator=g, device="cuda:0")
    cu, cb = np.array([0, n], np.int32), np.array([0, budget], np.int32)
    cud, cbd = (torch.from_numpy(x).cuda() for x in (cu, cb))
    p = b.make_params(n_layers=1, n_q_heads=heads, n_kv_heads=heads, head_dim=64, window=W, pool_kernel=pool, prior_weight=1e-3,
                      cu_seqlens_host=cu, cu_budgets_host=cb, cu_seqlens_dev=cud.data_ptr(), cu_budgets_dev=cbd.data_ptr(), score_variant=variant)
    ws = torch.full((b.codecomp_workspace_bytes(p),), 0xFF, dtype=torch.uint8, device="cuda:0")
    scores, fused_scores = (torch.full((heads, n), float("nan"), device="cuda:0") for _ in range(2))
    idx, fused_idx = (torch.full((heads, budget), -1, dtype=torch.int32, device="cuda:0") for _ in range(2))
    out = torch.empty((heads, budget, 64), dtype=torch.bfloat16, device="cuda:0")
    b.codecomp_score(q, k, prior, p, scores, ws)
    b.codecomp_select(scores, p, idx, ws)
    b.codecomp_compress(q, k, k, prior, p, fused_scores, fused_idx, out, out.clone(), ws)
    torch.cuda.synchronize()
    assert torch.equal(scores.view(torch.int32), fused_scores.view(torch.int32)) and torch.equal(idx, fused_idx)


def test_masses_of_several_row_splits_are_added():
    both(wl.scaled(wl.qwen7b_32k(), n_layers=1, seqlens=[2000, 600], budgets=[700, 512], window=512, n_q_heads=8, n_kv_heads=2))
