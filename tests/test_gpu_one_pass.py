"""Requests of up to 768 keys, whose logits are formed once (one workgroup holds the keys): against the oracle and against the
two passes, which calls with a given number of workgroups take for every request."""
import numpy as np
import pytest

from oracle import codecomp_oracle as orc
from paper_2604_10235_amd import workloads as wl
from paper_2604_10235_amd.binding import ROUTE_FEW_ROWS, ROUTE_ONE_PASS, ROUTE_TWO_PASSES
from tests import parity_util as pu

pytestmark = pytest.mark.gpu

# Both ways round the argument of an exponential (below 2^6 in units of log2, scores of normal keys) and take a normaliser that
# is as exact: 2^6 * 2^-24 * ln 2 = 2.6e-6 a side; sums of up to 1200 rows of 768 keys add less than 1e-6 each.
TWO_WAYS = 8e-6


def both_ways(w, kv="bf16", q_scale=1.0, route=None, **over):
    """Scores by the library's own rules and by two passes; `route`: what the first call has to take for its requests (b.ROUTE_*, one for all or one each)."""
    import torch
    from paper_2604_10235_amd import binding as b
    q, k, v, prior = wl.make_all(w)
    if not np.isscalar(q_scale) or q_scale != 1.0:                       # one factor, or one per row of the window
        q = wl.f32_to_bf16_bits(orc.bf16_bits_to_f64(q).astype(np.float32) * np.float32(q_scale))
    if kv == "fp8":
        k, v = wl.bf16_bits_to_fp8_codes(k), wl.bf16_bits_to_fp8_codes(v)
    got = []
    for wgs in (0, 40):
        p = b.DeviceProblem(w, q, k, v, prior, score_workgroups=wgs, **over)
        if route is not None:
            got_route = b.codecomp_score_route(p.params)[0]
            assert (got_route == (b.ROUTE_TWO_PASSES if wgs else route)).all()
        p.workspace.fill_(0xFF)                                    # nothing may be read before it is written
        p.score()
        first = p.scores.clone()
        p.scores.fill_(float("nan"))
        p.score()
        torch.cuda.synchronize()
        assert torch.equal(first.view(torch.int32), p.scores.view(torch.int32))      # the same bits again
        got.append(p.scores.cpu().numpy())
    return q, k, prior, got


# Rows: one, a part of a block of 16, 1 .. 3 row splits, odd numbers of blocks; few problems (rows shared out), more problems than
# compute units; tiles of 16 keys: one key, full, one over, one tile per wave of four and of eight, the longest of each kind.
@pytest.mark.parametrize("heads,d,window,layers", [((1, 1), 64, 1, 1), ((5, 1), 128, 3, 2), ((14, 2), 128, 50, 1), ((4, 4), 64, 16, 70),
                                                   ((12, 1), 128, 100, 1), ((18, 2), 128, 64, 3)])
@pytest.mark.parametrize("lens", [[1, 15, 16, 17, 63, 64], [65, 128, 129, 384], [385, 767, 768, 200]])
@pytest.mark.parametrize("kv", ["bf16", "fp8"])
def test_short_requests(heads, d, window, layers, lens, kv):
    lens = [max(n, window) for n in lens]
    w = wl.scaled(wl.qwen7b_32k(), n_layers=layers, n_q_heads=heads[0], n_kv_heads=heads[1], head_dim=d, window=window, seqlens=lens, budgets=lens)
    q, k, prior, (one, two) = both_ways(w, kv, route=ROUTE_ONE_PASS)
    np.testing.assert_allclose(one, two, rtol=TWO_WAYS, atol=1e-30)
    some = slice(0, min(layers, 2))
    pu.assert_scores_close(one[some], orc.score_packed(q[some], k[some], prior, w.cu_seqlens(), pool_kernel=w.pool_kernel, prior_weight=w.prior_weight,
                                                        k_format="fp8_e4m3" if kv == "fp8" else "bf16"))


# More than 512 problems of short requests next to longer ones, which take two passes in the same call; a window that the
# softmax leaves out (a request that is nothing else among them)
@pytest.mark.parametrize("lens,variant", [([300, 769, 100, 768, 32, 2000, 500], 0), ([300, 801, 100, 32, 800, 500, 400], 8), ([33, 64, 900, 40, 41], 1 | 4 | 8 | 16)])
def test_short_requests_among_longer_ones(lens, variant):
    from tests.test_gpu_parity import oracle_variant
    w = wl.scaled(wl.qwen7b_32k(), n_layers=2, n_q_heads=140, n_kv_heads=70, head_dim=64, window=32, seqlens=lens, budgets=lens)
    q, k, prior, (one, two) = both_ways(w, score_variant=variant)
    np.testing.assert_allclose(one, two, rtol=TWO_WAYS, atol=1e-30)
    pu.assert_scores_close(one[:1], orc.score_packed(q[:1], k[:1], prior, w.cu_seqlens(), pool_kernel=w.pool_kernel, prior_weight=w.prior_weight,
                                                     **oracle_variant(variant)))


# Logits hundreds of nats apart: the exponentials outrun the references and the rows are done again from their largest logits.
# An argument below 2^10 in units of log2 is off by 2^10 * 2^-24 * ln 2 = 4.2e-5 a side, its logit (128 products) by as much again.
@pytest.mark.parametrize("lens", [[700, 130], [384, 200, 96]])
@pytest.mark.parametrize("kv", ["bf16", "fp8"])
def test_logits_far_apart(lens, kv):
    w = wl.scaled(wl.qwen7b_32k(), n_layers=1, window=64, seqlens=lens, budgets=lens, prior_weight=0.0)
    q, k, prior, (one, two) = both_ways(w, kv, q_scale=40.0, route=ROUTE_ONE_PASS)
    np.testing.assert_allclose(one, two, rtol=2e-4, atol=1e-30)
    # masses below 2^-126 are 0 in 32 bits
    ref = orc.score_packed(q, k, prior, w.cu_seqlens(), pool_kernel=w.pool_kernel, prior_weight=0.0,
                           k_format="fp8_e4m3" if kv == "fp8" else "bf16")
    np.testing.assert_allclose(one, ref, rtol=1e-3, atol=1e-30)


# One logit of 100 nats, all others 0.  Layer l has it in row 16 l and key 0: among the 16 keys that give that row its reference, but
# not those of the rows that repeat it where the row count is no multiple of 16.  Every other probability is 1 / n: an exponential
# of 0, a sum of up to 768 ones and one reciprocal (a few 2^-24), added up over up to 539 rows (539 * 2^-24 = 3.2e-5 at worst).
@pytest.mark.parametrize("window,rows_per_head", [(17, 1), (33, 1), (35, 2), (100, 1), (77, 7)])
@pytest.mark.parametrize("d,kv", [(64, "bf16"), (128, "bf16"), (64, "fp8"), (128, "fp8")])
@pytest.mark.parametrize("n", [100, 300, 500, 768])
def test_one_large_logit_beside_unfinished_row_blocks(window, rows_per_head, d, kv, n):
    import torch
    from paper_2604_10235_amd import binding as b
    R = window * rows_per_head
    layers = (R + 15) // 16
    w = wl.scaled(wl.qwen7b_32k(), n_layers=layers, n_q_heads=rows_per_head, n_kv_heads=1, head_dim=d, window=window, seqlens=[n], budgets=[n],
                  prior_weight=0.0, pool_kernel=1)
    q = np.zeros((layers, 1, rows_per_head, window, d), np.float32)
    k = np.zeros((layers, 1, n, d), np.float32)
    for l in range(layers):
        q[l, 0, 16 * l // window, 16 * l % window, 0] = 100.0 * np.sqrt(d) / 16
    k[:, :, 0, 0] = 16.0
    qb, kb = wl.f32_to_bf16_bits(q), wl.f32_to_bf16_bits(k)
    if kv == "fp8":
        kb = wl.bf16_bits_to_fp8_codes(kb)
    prior = np.zeros(n, np.float32)
    p = b.DeviceProblem(w, qb, kb, None, prior)
    assert (b.codecomp_score_route(p.params)[0] == ROUTE_ONE_PASS).all()
    p.workspace.fill_(0xFF)
    p.score()
    torch.cuda.synchronize()
    ref = orc.score_packed(qb, kb, prior, w.cu_seqlens(), pool_kernel=1, prior_weight=0.0, k_format="fp8_e4m3" if kv == "fp8" else "bf16")
    np.testing.assert_allclose(p.scores.cpu().numpy(), ref, rtol=4e-5)


# The second run from the largest logits on other shapes: row counts that are no multiple of 16, both widths of keys, 32 blocks in a
# workgroup (the ring of query blocks twice over), two chunks in turn, short requests beside longer ones.  Every row scaled, or every
# third: then the blocks in range wait for the others and are done again with them.
@pytest.mark.parametrize("heads,d,window,layers,lens", [((3, 1), 64, 37, 3, [70, 300, 384]), ((3, 1), 128, 37, 3, [500, 768, 40]), ((4, 4), 64, 17, 2, [17, 600, 33]),
                                                        ((16, 4), 64, 128, 65, [130]), ((8, 2), 128, 128, 130, [400]), ((14, 2), 64, 128, 200, [130]), ((14, 2), 64, 128, 200, [390]),
                                                        ((14, 2), 64, 17, 4, [100, 17, 384, 33] * 20 + [800, 1500])])
@pytest.mark.parametrize("kv,rows", [("bf16", "all"), ("fp8", "some")])
def test_logits_far_apart_on_other_shapes(heads, d, window, layers, lens, kv, rows):
    from paper_2604_10235_amd import binding as b
    lens = [max(n, window) for n in lens]
    w = wl.scaled(wl.qwen7b_32k(), n_layers=layers, n_q_heads=heads[0], n_kv_heads=heads[1], head_dim=d, window=window, seqlens=lens, budgets=lens, prior_weight=0.0)
    scale = np.full((window, 1), 40.0, np.float32)
    if rows == "some":
        scale[np.arange(window) % 3 != 0] = 1.0
    q, k, prior, (one, two) = both_ways(w, kv, q_scale=scale, route=[ROUTE_ONE_PASS if n <= 768 else ROUTE_TWO_PASSES for n in lens])
    np.testing.assert_allclose(one, two, rtol=2e-4, atol=1e-30)
    ref = orc.score_packed(q[:1], k[:1], prior, w.cu_seqlens(), pool_kernel=w.pool_kernel, prior_weight=0.0, k_format="fp8_e4m3" if kv == "fp8" else "bf16")
    np.testing.assert_allclose(one[:1], ref, rtol=1e-3, atol=1e-30)


def test_strided_queries_and_keys():
    """Token-major keys and queries, padded rows: the strides that the two passes take."""
    import torch
    from paper_2604_10235_amd import binding as b
    lens, L, HQ, H, W, d = [700, 64, 385], 2, 6, 2, 48, 128
    cu = np.concatenate([[0], np.cumsum(lens)]).astype(np.int32)
    T = int(cu[-1])
    g = torch.Generator(device="cuda").manual_seed(3)
    q = torch.randn((L, W, len(lens), HQ, d + 8), generator=g, device="cuda").bfloat16()
    k = torch.randn((L, T, H, d + 24), generator=g, device="cuda").bfloat16()
    prior = torch.rand(T, generator=g, device="cuda")
    dev = torch.from_numpy(cu).cuda()
    scores = []
    for layout in ("strided", "packed"):
        qq = q if layout == "strided" else q[..., :d].permute(0, 2, 3, 1, 4).contiguous()
        kk = k if layout == "strided" else k[..., :d].permute(0, 2, 1, 3).contiguous()
        strides = {} if layout == "packed" else dict(
            q_stride_layer=q.stride(0), q_stride_tok=q.stride(1), q_stride_seq=q.stride(2), q_stride_head=q.stride(3),
            kv_stride_layer=k.stride(0), kv_stride_tok=k.stride(1), kv_stride_head=k.stride(2))
        p = b.make_params(n_layers=L, n_q_heads=HQ, n_kv_heads=H, head_dim=d, window=W, pool_kernel=7, prior_weight=1.0, cu_seqlens_host=cu,
                          cu_budgets_host=cu, cu_seqlens_dev=dev.data_ptr(), cu_budgets_dev=dev.data_ptr(), **strides)
        ws = torch.empty(b.codecomp_workspace_bytes(p), dtype=torch.uint8, device="cuda")
        out = torch.empty((L, H, T), dtype=torch.float32, device="cuda")
        b.codecomp_score(qq, kk, prior, p, out, ws)
        scores.append(out)
    torch.cuda.synchronize()
    assert torch.equal(scores[0].view(torch.int32), scores[1].view(torch.int32))


def test_replayed_in_a_graph():
    """The kernels (loads straight into LDS, no memset) under capture: every replay gives the eager result."""
    import torch
    from paper_2604_10235_amd import binding as b
    lens = [700, 100, 385]
    w = wl.scaled(wl.qwen7b_32k(), n_layers=2, seqlens=lens, budgets=[80, 64, 100])
    p = b.DeviceProblem(w, *wl.make_all(w))
    p.compress()
    torch.cuda.synchronize()
    want = [x.clone() for x in (p.scores, p.idx, p.k_out, p.v_out)]
    graph = torch.cuda.CUDAGraph()
    side = torch.cuda.Stream()
    with torch.cuda.graph(graph, stream=side):
        p.compress()
    for _ in range(4):
        for x in (p.scores, p.idx, p.k_out, p.v_out):
            x.zero_()
        p.workspace.fill_(0x7F)
        torch.cuda.synchronize()
        graph.replay()
        torch.cuda.synchronize()
        for got, ref in zip((p.scores, p.idx, p.k_out, p.v_out), want):
            assert torch.equal(got, ref)


# Few rows: all logits of a request of up to 4096 keys (16 rows) to 1024 (64 rows) at once, from 96 problems on.  Blocks of 16 rows
# full and begun; one tile more than fits the keys' own registers, the longest, the next longer (two passes), short ones among them.
@pytest.mark.parametrize("heads,d,window", [((50, 50), 64, 16), ((100, 100), 64, 7), ((100, 50), 64, 16), ((50, 50), 128, 17), ((50, 50), 128, 48),
                                            ((200, 50), 64, 16), ((50, 50), 128, 63)])
@pytest.mark.parametrize("which", ["shortest", "longest", "too long"])
@pytest.mark.parametrize("kv", ["bf16", "fp8"])
def test_few_rows(heads, d, window, which, kv):
    rows = heads[0] // heads[1] * window
    most = {1: 4096, 2: 2560, 3: 1536, 4: 1024}[(rows + 15) // 16]
    lens = {"shortest": [769, 20, 300], "longest": [most, most - 127], "too long": [most + 1, 100]}[which]
    lens = [max(n, window) for n in lens]
    w = wl.scaled(wl.qwen7b_32k(), n_layers=1, n_q_heads=heads[0], n_kv_heads=heads[1], head_dim=d, window=window, seqlens=lens, budgets=lens)
    q, k, prior, (one, two) = both_ways(w, kv, route=ROUTE_TWO_PASSES if which == "too long" else ROUTE_FEW_ROWS)
    np.testing.assert_allclose(one, two, rtol=TWO_WAYS, atol=1e-30)
    ref = orc.score_packed(q, k, prior, w.cu_seqlens(), pool_kernel=w.pool_kernel, prior_weight=w.prior_weight, k_format="fp8_e4m3" if kv == "fp8" else "bf16")
    pu.assert_scores_close(one, ref)


@pytest.mark.parametrize("variant", [8, 1 | 4 | 8 | 16])
def test_few_rows_other_readings(variant):
    from tests.test_gpu_parity import oracle_variant
    lens = [1500, 32, 40, 33]                                       # a request without a key of its own among them
    w = wl.scaled(wl.qwen7b_32k(), n_layers=2, n_q_heads=30, n_kv_heads=30, head_dim=64, window=32, seqlens=lens, budgets=lens)
    q, k, prior, (one, two) = both_ways(w, score_variant=variant)
    np.testing.assert_allclose(one, two, rtol=TWO_WAYS, atol=1e-30)
    pu.assert_scores_close(one, orc.score_packed(q, k, prior, w.cu_seqlens(), pool_kernel=w.pool_kernel, prior_weight=w.prior_weight,
                                                 **oracle_variant(variant)))


def scores_on_device(lens, layers, q_heads, kv_heads, d, window, q, k, pool=5):
    """The scores of packed q [layers][requests][..] and k [layers][heads][tokens][..], and the fastest of five calls (ms)."""
    import torch
    from paper_2604_10235_amd import binding as b
    cu = np.concatenate([[0], np.cumsum(lens)]).astype(np.int32)
    dev = torch.from_numpy(cu).cuda()
    p = b.make_params(n_layers=layers, n_q_heads=q_heads, n_kv_heads=kv_heads, head_dim=d, window=window, pool_kernel=pool, prior_weight=0.0,
                      cu_seqlens_host=cu, cu_budgets_host=cu, cu_seqlens_dev=dev.data_ptr(), cu_budgets_dev=dev.data_ptr(),
                      q_stride_layer=q.stride(0), kv_stride_layer=k.stride(0), kv_stride_head=k.stride(1))
    ws = torch.empty(b.codecomp_workspace_bytes(p), dtype=torch.uint8, device="cuda")
    ws.fill_(0xFF)
    out = torch.full((layers, kv_heads, int(cu[-1])), float("nan"), device="cuda")
    prior = torch.zeros(int(cu[-1]), device="cuda")
    best = float("inf")
    for _ in range(5):
        start, stop = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
        start.record()
        b.codecomp_score(q, k, prior, p, out, ws)
        stop.record()
        stop.synchronize()
        best = min(best, start.elapsed_time(stop))
    return out, best


@pytest.mark.parametrize("between", [1, 62, 63, 64, 65, 127, 128, 129, 1087, 1088, 1089, 2300])
def test_long_requests_behind_many_short_ones(between):
    """Long requests whose next long one lies any number of short ones further: the walk of a workgroup through the requests."""
    import torch
    layers, heads, d, window = 3, 5, 64, 16
    lens = []
    for n in (1400, 2100, 900, 1700):
        lens += [20 + i % 30 for i in range(between)] + [n]
    lens += [33] * 200                                               # so that the call has 512 short problems and more, and ends with some
    g = torch.Generator(device="cuda").manual_seed(5)
    q = torch.randn((layers, len(lens), heads, window, d), generator=g, device="cuda").bfloat16()
    k = torch.randn((layers, 1, sum(lens), d), generator=g, device="cuda").bfloat16()
    got, _ = scores_on_device(lens, layers, heads, 1, d, window, q, k)
    at = 0
    for i, n in enumerate(lens):
        if n > 768:
            alone, _ = scores_on_device([n], layers, heads, 1, d, window, q[:, i:i + 1], k[:, :, at:at + n])
            np.testing.assert_allclose(got[:, :, at:at + n].cpu().numpy(), alone.cpu().numpy(), rtol=TWO_WAYS)
        at += n


def test_many_short_requests_do_not_hold_up_long_ones():
    """A call with 20000 short requests ahead of forty long ones takes about as long as the two calls apart (8 times as long while a
    workgroup that came to the next head stepped over them one by one); half as long again leaves room for the machine."""
    import torch
    layers, heads, d, window = 3, 5, 64, 16
    short, long = [20] * 20000, [1000 + 61 * (7 * i % 40) for i in range(40)]
    g = torch.Generator(device="cuda").manual_seed(6)
    q = torch.randn((layers, len(short + long), heads, window, d), generator=g, device="cuda").bfloat16()
    k = torch.randn((layers, 1, sum(short + long), d), generator=g, device="cuda").bfloat16()
    cut = sum(short)
    both, t_both = scores_on_device(short + long, layers, heads, 1, d, window, q, k)
    first, t_first = scores_on_device(short, layers, heads, 1, d, window, q, k)
    then, t_then = scores_on_device(long, layers, heads, 1, d, window, q[:, len(short):], k[:, :, cut:])
    assert torch.equal(both[:, :, :cut], first)
    np.testing.assert_allclose(both[:, :, cut:].cpu().numpy(), then.cpu().numpy(), rtol=TWO_WAYS)
    print(f"{t_both:.3f} ms, apart {t_first:.3f} + {t_then:.3f}")
    assert t_both < 1.5 * (t_first + t_then)


# As many requests and heads as 2^32 threads on one axis of a launch do not hold: 65535 requests, all but one of a single key, whose
# only row gives it all its mass.
@pytest.mark.parametrize("first,heads", [(300, 257), (500, 129), (500, 257), (900, 129)])
def test_millions_of_problems(first, heads):
    import torch
    lens = [first] + [1] * 65534
    g = torch.Generator(device="cuda").manual_seed(7)
    q = torch.randn((1, len(lens), heads, 1, 64), generator=g, device="cuda").bfloat16()
    k = torch.randn((1, heads, sum(lens), 64), generator=g, device="cuda").bfloat16()
    got, _ = scores_on_device(lens, 1, heads, heads, 64, 1, q, k, pool=1)
    alone, _ = scores_on_device([first], 1, heads, heads, 64, 1, q[:, :1], k[:, :, :first], pool=1)
    assert float((got[:, :, first:] - 1.0).abs().max()) <= TWO_WAYS           # (NaN fails, too)
    np.testing.assert_allclose(got[:, :, :first].cpu().numpy(), alone.cpu().numpy(), rtol=TWO_WAYS)


# Requests of up to 384 keys apart while the longer short ones stay in the passes; both apart; more rows than one workgroup holds,
# chunks in turn.  Lengths on both sides of every line, a window that the softmax leaves out.
@pytest.mark.parametrize("heads,window,times,longer,variant", [((14, 2), 16, 24, 0, 0), ((14, 2), 16, 24, 62, 0), ((14, 2), 16, 24, 0, 8), ((14, 2), 100, 24, 62, 1 | 4 | 8 | 16)])
@pytest.mark.parametrize("kv", ["bf16", "fp8"])
def test_short_requests_apart(heads, window, times, longer, variant, kv):
    from tests.test_gpu_parity import oracle_variant
    trim = window if variant & 8 else 0
    lens = [n + trim for n in ([384, 20, 383, 17, 16, 65, 1, 300] * times + [385, 767, 768, 769, 1500] + [500, 768] * longer)]
    lens = [max(window, n) for n in lens]
    w = wl.scaled(wl.qwen7b_32k(), n_layers=4, n_q_heads=heads[0], n_kv_heads=heads[1], head_dim=64, window=window, seqlens=lens, budgets=lens)
    q, k, prior, (one, two) = both_ways(w, kv, score_variant=variant, route=[ROUTE_ONE_PASS if 0 < n - trim <= (768 if longer else 384) else ROUTE_TWO_PASSES for n in lens])
    np.testing.assert_allclose(one, two, rtol=TWO_WAYS, atol=1e-30)
    ref = orc.score_packed(q[:1], k[:1], prior, w.cu_seqlens(), pool_kernel=w.pool_kernel, prior_weight=w.prior_weight,
                           k_format="fp8_e4m3" if kv == "fp8" else "bf16", **oracle_variant(variant))
    pu.assert_scores_close(one[:1], ref)


@pytest.mark.parametrize("window,empty", [(512, 1500), (512, 40)])
def test_row_chunks_beside_requests_without_a_key(window, empty):
    """The last request alone has keys for the softmax: its chunks' arrays of masses, with a place for all tokens, stay inside the workspace."""
    import torch
    from paper_2604_10235_amd import binding as b
    lens = [window] * empty + [window + 700]
    cu = np.concatenate([[0], np.cumsum(lens)]).astype(np.int32)
    dev = torch.from_numpy(cu).cuda()
    g = torch.Generator(device="cuda").manual_seed(8)
    q = torch.randn((1, len(lens), 1, window, 64), generator=g, device="cuda").bfloat16()
    k = torch.randn((1, 1, sum(lens), 64), generator=g, device="cuda").bfloat16()
    prior, got = torch.zeros(sum(lens), device="cuda"), []
    for wgs in (0, 40):
        p = b.make_params(n_layers=1, n_q_heads=1, n_kv_heads=1, head_dim=64, window=window, pool_kernel=5, prior_weight=0.0, cu_seqlens_host=cu,
                          cu_budgets_host=cu, cu_seqlens_dev=dev.data_ptr(), cu_budgets_dev=dev.data_ptr(), score_variant=8, score_workgroups=wgs)
        route = b.codecomp_score_route(p)[0]
        assert (route[:-1] == ROUTE_TWO_PASSES).all() and route[-1] == (ROUTE_TWO_PASSES if wgs else ROUTE_ONE_PASS)
        need = b.codecomp_workspace_bytes(p)
        ws = torch.full((need + 65536,), 0x5A, dtype=torch.uint8, device="cuda")
        ws[:need] = 0xFF
        out = torch.full((1, 1, sum(lens)), float("nan"), device="cuda")
        b.codecomp_score(q, k, prior, p, out, ws)
        got.append(out.cpu().numpy())
        assert bool((ws[need:] == 0x5A).all())
    np.testing.assert_allclose(got[0], got[1], rtol=TWO_WAYS, atol=1e-30)
