"""Branches that short calls and crowded selections take: pass 2 folding the row statistics itself (workgroups of up to four
waves, few segments per request) against the merge kernel, one tile per workgroup, and the cut found in lists that just fit
and just do not fit the registers of the resolving workgroup."""
import numpy as np
import pytest

from oracle import codecomp_oracle as orc
from paper_2604_10235_amd import workloads as wl
from tests import parity_util as pu
from tests.test_gpu_select_cases import W, select_on_device

pytestmark = pytest.mark.gpu


# Workgroups of 1, 2, 3, 4 and 8 waves; 76 tiles of one head over 2 .. 76 workgroups, which is as many segments per row, on
# both sides of the limit (40, which counts two more); a last tile of one key; several requests.
@pytest.mark.parametrize("group,window", [(1, 32), (2, 50), (5, 32), (7, 32), (9, 32)])
@pytest.mark.parametrize("lens,wgs", [([4801], 0), ([4801], 2), ([4801], 33), ([4801], 38), ([4801], 39), ([700, 64, 65, 1300], 0),
                                      ([700, 64, 65, 1300], 5)])
def test_row_statistics_folded_by_the_second_pass(group, window, lens, wgs):
    import torch
    from paper_2604_10235_amd import binding as b
    w = wl.scaled(wl.qwen7b_32k(), n_layers=1, n_q_heads=group, n_kv_heads=1, window=window, seqlens=lens, budgets=lens)
    q, k, v, prior = wl.make_all(w)
    whole, steps = (b.DeviceProblem(w, q, k, v, prior, score_workgroups=wgs) for _ in range(2))
    whole.workspace.fill_(0xFF)                                    # nothing may be read before it is written
    whole.score()
    for stage in (b.STAGE_ROW_STATS, b.STAGE_ROW_MERGE, b.STAGE_MASS, b.STAGE_FINISH):
        steps.score_stages(stage)
    torch.cuda.synchronize()
    got = whole.scores.cpu().numpy()
    # the two fold the same (reference, sum) pairs in another order: a normaliser below 2^5 in units of log2 is rounded twice
    # on either side, 4 * 2^-19 * ln 2 = 5.3e-6
    np.testing.assert_allclose(got, steps.scores.cpu().numpy(), rtol=5.3e-6, atol=1e-30)
    pu.assert_scores_close(got, orc.score_packed(q, k, prior, w.cu_seqlens(), pool_kernel=w.pool_kernel, prior_weight=w.prior_weight))


@pytest.mark.parametrize("group,window", [(1, 32), (2, 50), (5, 32), (7, 32), (9, 32), (20, 32)])
@pytest.mark.parametrize("lens,variant", [([700, 64, 65, 1300], 0), ([50, 700, 51, 1300], 8)])
def test_stages_asked_for_again_after_a_whole_call(group, window, lens, variant):
    """Whatever the whole call merges on its way, it leaves what the mass kernel and the pooling alone read afterwards: the
    same bits from them (1, 2, 3, 4 and 8 waves, two row splits; requests without a key of their own included)."""
    import torch
    from paper_2604_10235_amd import binding as b
    w = wl.scaled(wl.qwen7b_32k(), n_layers=2, n_q_heads=2 * group, n_kv_heads=2, window=window, seqlens=[max(n, window) for n in lens],
                  budgets=[max(n, window) for n in lens])
    q, k, v, prior = wl.make_all(w)
    first_three = b.STAGE_ROW_STATS | b.STAGE_ROW_MERGE | b.STAGE_MASS
    for whole in (lambda p: p.score(), lambda p: p.compress(), lambda p: p.score_stages(first_three)):
        p = b.DeviceProblem(w, q, k, v, prior, score_variant=variant)
        p.score()
        want = p.scores.clone()
        p.workspace.fill_(0xFF)
        whole(p)
        p.scores.fill_(float("nan"))
        for stages in ((b.STAGE_MASS, b.STAGE_FINISH), (b.STAGE_MASS | b.STAGE_FINISH,), (b.STAGE_FINISH,)):
            for stage in stages:
                p.score_stages(stage)
            torch.cuda.synchronize()
            assert torch.equal(p.scores.view(torch.int32), want.view(torch.int32)), stages


@pytest.mark.parametrize("crowd", [1, 63, 65, 16383, 16384, 16385, 40000])
@pytest.mark.parametrize("together", [False, True])
def test_cut_inside_a_crowded_first_digit(crowd, together):
    """`crowd` candidates share the first digit (values in [1, 1.25)) and the cut lies among them; scattered over all parts or
    next to one another (whole wavefronts of one part, and the seams between parts)."""
    npre = 70001
    g = np.random.default_rng(crowd)
    rows = []
    for values in (np.full(crowd, 1.125), 1.0 + g.integers(0, 5, crowd) / 32, 1.0 + g.random(crowd) * 0.2):
        r = np.full(npre + W, 0.25, np.float32)
        at = 8192 - crowd // 3 if together else 0
        where = np.arange(max(at, 0), max(at, 0) + crowd) if together else g.choice(npre, size=crowd, replace=False)
        r[where] = values.astype(np.float32)
        rows.append(r)
    rows = np.stack(rows)
    for need in sorted({1, crowd // 2 + 1, crowd}):
        idx, _, _ = select_on_device(rows, [npre + W], [need + W])
        assert np.array_equal(idx[0].astype(np.int64), orc.select(rows.astype(np.float64), W, need + W)), need


@pytest.mark.parametrize("heads", [511, 512])
@pytest.mark.parametrize("pool,variant", [(1, 0), (7, 0), (1025, 0), (7, 4 | 8 | 16)])
def test_pooling_by_short_and_long_workgroups(heads, pool, variant):
    """Below 512 workgroups of 2048 tokens the scores are pooled by workgroups of 512: seams inside and between requests."""
    import torch
    from paper_2604_10235_amd import binding as b
    from tests.test_gpu_parity import oracle_variant
    lens = [509, 3, 70, 900]
    w = wl.scaled(wl.tiny(), n_q_heads=heads, n_kv_heads=heads, window=2, seqlens=lens, budgets=lens, pool_kernel=pool)
    q, k, v, prior = wl.make_all(w)
    p = b.DeviceProblem(w, q, k, v, prior, score_variant=variant)
    p.score()
    torch.cuda.synchronize()
    pu.assert_scores_close(p.scores.cpu().numpy(), orc.score_packed(q, k, prior, w.cu_seqlens(), pool_kernel=pool,
                                                                    prior_weight=w.prior_weight, **oracle_variant(variant)))
