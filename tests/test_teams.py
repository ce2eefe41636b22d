"""Requests whose logits are formed once by teams of workgroups that wait for one another: against the oracle and
against the two passes, which calls with a given number of workgroups take; and that what happens when a team can not do its work
(logits out of range, members kept from starting) gives the same bits."""
import numpy as np
import pytest

from oracle import codecomp_oracle as orc
from paper_2604_10235_amd import binding as b, workloads as wl
from tests import parity_util as pu

# Both ways round the argument of an exponential (below 2^6 in units of log2, scores of normal keys) and take a normaliser that is as
# exact: 2^6 * 2^-24 * ln 2 = 2.6e-6 a side; a sum of up to 1024 rows, all positive, in chains of 64 adds, adds less than 64 * 2^-24 =
# 3.8e-6 where every error has the same sign.
TWO_WAYS = 1.3e-5


def problem(lens, heads=(28, 4), window=64, layers=1, **over):
    return wl.scaled(wl.qwen7b_32k(), n_layers=layers, n_q_heads=heads[0], n_kv_heads=heads[1], window=window, seqlens=lens, budgets=[window] * len(lens), **over)


def test_which_calls_are_given_to_teams():
    def members(lens, heads=(28, 4), window=64, layers=28, head_dim=128, **over):
        cu = np.concatenate([[0], np.cumsum(lens)]).astype(np.int32)
        p = b.make_params(n_layers=layers, n_q_heads=heads[0], n_kv_heads=heads[1], head_dim=head_dim, window=window, pool_kernel=7, prior_weight=1.0, cu_seqlens_host=cu,
                          cu_budgets_host=np.arange(len(lens) + 1, dtype=np.int32) * window, cu_seqlens_dev=0x1000, cu_budgets_dev=0x2000, **over)
        assert (b.codecomp_score_route(p)[0] == b.ROUTE_TWO_PASSES).all() or b.codecomp_score_teams(p) == 0
        return b.codecomp_score_teams(p)
    assert members([32768]) == 64 and members([65536]) == 128 and members([1536], layers=42) == 3
    assert members([65537]) == 0                                           # 129 members
    assert members([32768], head_dim=64) == 0
    assert members([32768], score_workgroups=256) == 0 and members([32768], score_lead_tiles=-1) == 0
    assert members([32768], score_variant=2) == 0                          # largest head mass
    assert members([32768, 700]) == 0 and members([32768, 784], score_variant=8) == 0      # a request of one workgroup beside it
    assert members([32768], window=27) == 0 and members([32768], window=147) == 0          # 189 rows, 1029
    assert members([32768], window=28) == 64 and members([32768], window=146) == 64        # 196, 1022
    assert members([8192], layers=1) == 0                                  # a quarter of a round
    # 3 members of 22 tiles (waves with fewer than 3), of 24 (the request's last, begun tile were a wave's third), of 25
    assert [members([8192, 4096, n, 3000, 16384, 2049], layers=6, window=100) for n in (1040, 1137, 1152, 1185)] == [0, 0, 0, 32]
    assert members([5000, 2000, 12345], layers=6) == 25
    # rows far apart: the kernel's table of them counts pieces of 16 bytes, in 16 bits (6 heads and 63 tokens away)
    far = dict(q_stride_head=136, q_stride_seq=64 * 8400, q_stride_layer=64 * 8400)
    assert members([32768], q_stride_tok=8 * 1038, **far) == 64 and members([32768], q_stride_tok=8 * 1039, **far) == 0


# Short requests beside longer ones, too few to be taken apart: teams of one where a member is full enough (385 to 512 keys).
ONE_MEMBER = [([32768, 500], 6), ([9000, 385, 512, 400], 12)]


def test_which_short_requests_are_teams_of_one():
    def members(lens, layers, **over):
        cu = np.concatenate([[0], np.cumsum(lens)]).astype(np.int32)
        p = b.make_params(n_layers=layers, n_q_heads=28, n_kv_heads=4, head_dim=128, window=64, pool_kernel=7, prior_weight=1.0, cu_seqlens_host=cu,
                          cu_budgets_host=np.arange(len(lens) + 1, dtype=np.int32) * 64, cu_seqlens_dev=0x1000, cu_budgets_dev=0x2000, **over)
        route = b.codecomp_score_route(p)[0]
        return b.codecomp_score_teams(p), (route == b.ROUTE_TWO_PASSES).all()
    for lens, layers in ONE_MEMBER:
        for kv in (b.KV_BF16, b.KV_FP8_E4M3):
            assert members(lens, layers, kv_dtype=kv) == (-(-max(lens) // 512), True)
    assert members([9000, 384, 512, 400], 12) == (0, True)                 # 24 tiles: waves with fewer than three
    assert members([9000, 576, 576], 12, score_variant=8) == (18, True) and members([9000, 576, 576, 64], 12, score_variant=8) == (0, True)      # one without a key
    assert members([9000, 500] + [500] * 40, 12) == (0, False)             # enough of them: each in a workgroup by itself


@pytest.mark.gpu
@pytest.mark.parametrize("lens,layers", ONE_MEMBER)
@pytest.mark.parametrize("kv", ["bf16", "fp8"])
def test_teams_of_one(lens, layers, kv):
    w = problem(lens, layers=layers)
    data = inputs(w, kv)
    one, two = (scores(w, data, wgs).scores.cpu().numpy() for wgs in (0, 256))
    np.testing.assert_allclose(one, two, rtol=TWO_WAYS, atol=1e-30)
    q, k, _, prior = data
    pu.assert_scores_close(one[-1:], orc.score_packed(q[-1:], k[-1:], prior, w.cu_seqlens(), pool_kernel=w.pool_kernel, prior_weight=w.prior_weight,
                                                       k_format="fp8_e4m3" if kv == "fp8" else "bf16"))


# A program whose calls share the device refuses teams, and nothing else: what one workgroup or a few rows take stays where it is.
def test_teams_refused_by_the_caller():
    def routes(lens, layers, window=64, heads=(28, 4), **over):
        cu = np.concatenate([[0], np.cumsum(lens)]).astype(np.int32)
        p = b.make_params(n_layers=layers, n_q_heads=heads[0], n_kv_heads=heads[1], head_dim=128, window=window, pool_kernel=7, prior_weight=1.0, cu_seqlens_host=cu,
                          cu_budgets_host=np.arange(len(lens) + 1, dtype=np.int32) * window, cu_seqlens_dev=0x1000, cu_budgets_dev=0x2000, **over)
        route, chunks, turn = b.codecomp_score_route(p)
        return list(route), chunks, turn, b.codecomp_workspace_bytes(p)
    for lens, layers, window, heads, kind in (([32768], 28, 64, (28, 4), b.ROUTE_TWO_PASSES), ([700] * 8, 4, 64, (28, 4), b.ROUTE_ONE_PASS),
                                              ([300, 2000] * 64, 8, 64, (28, 4), b.ROUTE_ONE_PASS), ([2000], 64, 16, (4, 4), b.ROUTE_FEW_ROWS)):
        default = routes(lens, layers, window, heads)
        assert kind in default[0] and routes(lens, layers, window, heads, score_variant=b.VARIANT_NO_TEAMS) == default
    def members(**over):
        p = problem([32768], layers=28)
        cu, cb = p.cu_seqlens(), p.cu_budgets()
        return b.codecomp_score_teams(b.make_params(n_layers=28, n_q_heads=28, n_kv_heads=4, head_dim=128, window=64, pool_kernel=7, prior_weight=1.0, cu_seqlens_host=cu,
                                                    cu_budgets_host=cb, cu_seqlens_dev=0x1000, cu_budgets_dev=0x2000, **over))
    assert members() == 64 and members(score_variant=1 | 4 | 8 | 16) > 0
    assert members(score_variant=b.VARIANT_NO_TEAMS) == 0 and members(score_variant=b.VARIANT_NO_TEAMS | 1 | 4 | 8 | 16) == 0


@pytest.mark.gpu
def test_teams_refused_take_two_passes():
    import torch
    w = problem([20011, 2000], layers=4)
    q, k, v, prior = data = inputs(w)
    p = b.DeviceProblem(w, *data, score_variant=b.VARIANT_NO_TEAMS)
    p.score()
    one = p.scores.cpu().numpy()
    pu.assert_scores_close(one[-1:], orc.score_packed(q[-1:], k[-1:], prior, w.cu_seqlens(), pool_kernel=w.pool_kernel, prior_weight=w.prior_weight))
    # the row normalisers are there: the mass kernel alone gives the same bits again
    b.codecomp_score_stages(p.q, p.k, p.prior, p.params, p.scores, p.workspace, 1 | 2 | 4)
    p.scores.fill_(float("nan"))
    b.codecomp_score_stages(p.q, p.k, p.prior, p.params, p.scores, p.workspace, 4 | 8)
    torch.cuda.synchronize()
    np.testing.assert_array_equal(one.view(np.int32), p.scores.cpu().numpy().view(np.int32))
    teams = scores(w, data, 0).scores.cpu().numpy()
    np.testing.assert_allclose(one, teams, rtol=TWO_WAYS, atol=1e-30)


def scores(w, data, wgs, **over):
    import torch
    p = b.DeviceProblem(w, *data, score_workgroups=wgs, **over)
    assert (b.codecomp_score_teams(p.params) > 0) == (wgs == 0)
    p.workspace.fill_(0xFF)                                                # nothing may be read before it is written
    p.scores.fill_(float("nan"))
    p.score()
    first = p.scores.clone()
    p.scores.fill_(float("nan"))
    p.score()
    torch.cuda.synchronize()
    assert torch.equal(first.view(torch.int32), p.scores.view(torch.int32))
    return p


def inputs(w, kv="bf16", q_scale=None):
    q, k, v, prior = wl.make_all(w)
    if q_scale is not None:
        q = wl.f32_to_bf16_bits(orc.bf16_bits_to_f64(q).astype(np.float32) * q_scale)
    return (q, wl.bf16_bits_to_fp8_codes(k), wl.bf16_bits_to_fp8_codes(v), prior) if kv == "fp8" else (q, k, v, prior)


# Rows: the fewest, an odd number of blocks, a begun block, two row splits, the most.  Keys: members that are full, one key in the last
# tile, waves with 3 tiles and with 4; 2, 3, 64, 65 .. 85 and 128 members; a second round that is not full; rounds of unlike requests.
@pytest.mark.gpu
@pytest.mark.parametrize("lens,heads,window,layers", [([1536], (112, 28), 48, 12), ([1521], (140, 20), 64, 17), ([1350], (140, 20), 128, 17), ([1024], (160, 40), 50, 25), ([32768], (28, 4), 64, 2),
                                                      ([32753], (16, 2), 128, 2), ([43520], (21, 3), 64, 2), ([65536], (16, 4), 64, 2), ([40000] * 3, (28, 4), 100, 1),
                                                      ([5000, 2000, 12345], (28, 4), 64, 6), ([8192, 4096, 1185, 3000, 16384, 2049], (28, 4), 100, 6)])
@pytest.mark.parametrize("kv", ["bf16", "fp8"])
def test_teams(lens, heads, window, layers, kv):
    w = problem(lens, heads, window, layers)
    data = inputs(w, kv)
    one, two = (scores(w, data, wgs).scores.cpu().numpy() for wgs in (0, 256))
    np.testing.assert_allclose(one, two, rtol=TWO_WAYS, atol=1e-30)
    q, k, _, prior = data
    pu.assert_scores_close(one[-1:], orc.score_packed(q[-1:], k[-1:], prior, w.cu_seqlens(), pool_kernel=w.pool_kernel, prior_weight=w.prior_weight,
                                                       k_format="fp8_e4m3" if kv == "fp8" else "bf16"))


@pytest.mark.gpu
@pytest.mark.parametrize("variant", [8, 1 | 4 | 8 | 16])
def test_other_readings(variant):
    from tests.test_gpu_parity import oracle_variant
    w = problem([20011, 9000], layers=4)
    q, k, v, prior = data = inputs(w)
    one, two = (scores(w, data, wgs, score_variant=variant).scores.cpu().numpy() for wgs in (0, 256))
    np.testing.assert_allclose(one, two, rtol=TWO_WAYS, atol=1e-30)
    pu.assert_scores_close(one[:1], orc.score_packed(q[:1], k[:1], prior, w.cu_seqlens(), pool_kernel=w.pool_kernel, prior_weight=w.prior_weight, **oracle_variant(variant)))


# Logits hundreds of nats apart: the rows' references are outrun, their problems are done again from the largest logits.  An argument
# below 2^10 in units of log2 is off by 2^10 * 2^-24 * ln 2 = 4.2e-5 a side, its logit (128 products) by as much again.
@pytest.mark.gpu
@pytest.mark.parametrize("rows", ["all", "some"])
@pytest.mark.parametrize("lens,heads,window,layers,kv", [([1200], (140, 20), 128, 17, "bf16"), ([32753], (16, 2), 128, 2, "fp8"), ([5000, 2000, 12345], (28, 4), 50, 6, "bf16"), ([65536], (16, 4), 64, 2, "bf16")])
def test_logits_far_apart(lens, heads, window, layers, kv, rows):
    w = problem(lens, heads, window, layers, prior_weight=0.0)
    scale = np.full((window, 1), 40.0, np.float32)
    if rows == "some":
        scale[np.arange(window) % 3 != 0] = 1.0
    data = inputs(w, kv, scale)
    one, two = (scores(w, data, wgs).scores.cpu().numpy() for wgs in (0, 256))
    np.testing.assert_allclose(one, two, rtol=2e-4, atol=1e-30)


# One KV head with a key that outruns the references, or holds a NaN: the others keep their bits.
@pytest.mark.gpu
@pytest.mark.parametrize("lens", [[5000], [5000, 12345, 2000]])
@pytest.mark.parametrize("what", ["large", "nan", "inf"])
def test_other_problems_keep_their_bits(lens, what):
    import torch
    w = problem(lens, layers=12, prior_weight=0.0)
    p = scores(w, inputs(w), 0)
    clean = p.scores.clone()
    key = p.k[5, 2, 777]
    key.copy_(key * 80 if what == "large" else torch.full_like(key, float(what)))
    p.score()
    hit = p.scores.clone()
    torch.cuda.synchronize()
    keep = torch.ones(clean.shape, dtype=torch.bool, device="cuda")
    keep[5, 2, :lens[0]] = False
    assert torch.equal(clean[keep], hit[keep])
    if what == "large":
        assert torch.isfinite(hit).all() and not torch.equal(clean[5, 2], hit[5, 2])
    else:
        assert torch.isnan(hit[5, 2, :lens[0]]).all()


# Calls side by side on three streams: members of one keep those of another from starting, waits end, and the work is done without them.
@pytest.mark.gpu
def test_side_by_side():
    import torch
    shapes = [problem([20011], layers=8), problem([16384], layers=8), problem([5000, 9000], layers=8)]
    ps = [scores(w, inputs(w), 0) for w in shapes]
    want = [p.scores.clone() for p in ps]
    torch.cuda.synchronize()
    streams = [torch.cuda.Stream() for _ in ps]
    for _ in range(6):
        for p, s in zip(ps, streams):
            with torch.cuda.stream(s):
                p.scores.fill_(float("nan"))
                p.score()
        torch.cuda.synchronize()
        for p, x in zip(ps, want):
            assert torch.equal(p.scores, x)


# Beside copies, whose workgroups hold every compute unit in turn: members are missing more often than not.
@pytest.mark.gpu
@pytest.mark.parametrize("lens,layers", [([20011], 8), ([5000, 2000, 12345], 6)])
def test_beside_copies(lens, layers):
    import torch
    p = Made(lens, (28, 4), 64, layers)
    want = p.score()
    x = torch.zeros(1 << 27, device="cuda")
    y = torch.empty_like(x)
    params, got = p.make(), [torch.empty_like(want) for _ in range(6)]
    assert b.codecomp_score_teams(params) > 0
    copies, calls = torch.cuda.Stream(), torch.cuda.Stream()
    torch.cuda.synchronize()
    with torch.cuda.stream(copies):
        for _ in range(20):
            y.copy_(x)
    with torch.cuda.stream(calls):
        for out in got:
            b.codecomp_score(p.q, p.k, p.prior, params, out, p.ws)
    torch.cuda.synchronize()
    for out in got:
        assert torch.equal(out.view(torch.int32), want.view(torch.int32))


@pytest.mark.gpu
def test_replayed_in_a_graph():
    import torch
    w = problem([12000, 5000], layers=8)
    p = b.DeviceProblem(w, *inputs(w))
    assert b.codecomp_score_teams(p.params) == 24
    p.compress()
    torch.cuda.synchronize()
    want = [x.clone() for x in (p.scores, p.idx, p.k_out, p.v_out)]
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph, stream=torch.cuda.Stream()):
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


@pytest.mark.gpu
def test_strided_queries_and_keys():
    """Token-major keys and queries, padded rows: the strides that the two passes take."""
    import torch
    lens, L, HQ, H, W, d = [16370], 4, 28, 4, 64, 128
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
        assert b.codecomp_score_teams(p) == 32
        ws = torch.empty(b.codecomp_workspace_bytes(p), dtype=torch.uint8, device="cuda")
        out = torch.empty((L, H, T), dtype=torch.float32, device="cuda")
        b.codecomp_score(qq, kk, prior, p, out, ws)
        scores.append(out)
    torch.cuda.synchronize()
    assert torch.equal(scores[0].view(torch.int32), scores[1].view(torch.int32))


class Made:
    """A problem whose inputs are made on the GPU: N(0, 1) keys and queries, keys in 8 bits where kv says so."""

    def __init__(self, lens, heads, window, layers, kv="bf16", **over):
        import torch
        cu = np.concatenate([[0], np.cumsum(lens)]).astype(np.int32)
        g = torch.Generator(device="cuda").manual_seed(11)
        self.q = torch.randn((layers, len(lens), heads[0], window, 128), generator=g, device="cuda").bfloat16()
        self.k = torch.empty((layers, heads[1], cu[-1], 128), dtype=torch.uint8 if kv == "fp8" else torch.bfloat16, device="cuda")
        for layer in range(layers):
            x = torch.randn(self.k.shape[1:], generator=g, device="cuda")
            self.k[layer] = x.to(torch.float8_e4m3fn).view(torch.uint8) if kv == "fp8" else x
        self.prior = torch.zeros(int(cu[-1]), device="cuda")
        self.dev = torch.from_numpy(cu).cuda()
        self.make = lambda **more: b.make_params(n_layers=layers, n_q_heads=heads[0], n_kv_heads=heads[1], head_dim=128, window=window, pool_kernel=1, prior_weight=0.0,
                                                 cu_seqlens_host=cu, cu_budgets_host=cu, cu_seqlens_dev=self.dev.data_ptr(), cu_budgets_dev=self.dev.data_ptr(),
                                                 kv_dtype=b.KV_FP8_E4M3 if kv == "fp8" else b.KV_BF16, **over, **more)
        self.ws = torch.empty(b.codecomp_workspace_bytes(self.make()), dtype=torch.uint8, device="cuda")

    def score(self, variant=0, **more):
        """Scores, with scratch memory full of ones."""
        import torch
        p = self.make(score_variant=variant, **more)
        self.ws.fill_(0xFF)
        out = torch.full(tuple(self.k.shape[:2]) + (len(self.prior),), float("nan"), device="cuda")
        b.codecomp_score(self.q, self.k, self.prior, p, out, self.ws)
        torch.cuda.synchronize()
        return out


def test_teams_apart_is_a_flag_of_its_own():
    cu = np.array([0, 32768], np.int32)
    make = lambda variant: b.make_params(n_layers=28, n_q_heads=28, n_kv_heads=4, head_dim=128, window=64, pool_kernel=7, prior_weight=1.0, cu_seqlens_host=cu,
                                         cu_budgets_host=np.array([0, 64], np.int32), cu_seqlens_dev=0x1000, cu_budgets_dev=0x2000, score_variant=variant)
    assert b.codecomp_score_teams(make(b.VARIANT_TEAMS_APART)) == 64 and b.codecomp_workspace_bytes(make(b.VARIANT_TEAMS_APART)) == b.codecomp_workspace_bytes(make(0))
    assert b.codecomp_validate(make(b.VARIANT_TEAMS_APART | b.VARIANT_NO_TEAMS)) == -11 and b.codecomp_validate(make(128)) == -11 and b.codecomp_validate(make(1024)) == -11


# All of the work by the kernel that steps in where members can not run: one place for the sums of each problem, fewer places than
# problems (36 problems of 64 members and 1024 rows, 39 of 128 members and 224 rows, 72 of 64 members and 512 rows: the statistics hold 33, 37
# and 66 of them), requests of unlike lengths, 8-bit keys; and with rows whose logits outrun the references (the same scores as by two passes, as in test_logits_far_apart).
@pytest.mark.gpu
@pytest.mark.parametrize("lens,heads,window,layers,kv", [([20011], (28, 4), 64, 4, "bf16"), ([32753], (16, 2), 128, 18, "bf16"), ([65521], (21, 3), 32, 13, "bf16"), ([32768], (8, 2), 128, 36, "fp8"),
                                                         ([5000, 2000, 12345], (28, 4), 50, 6, "bf16"), ([1536], (28, 4), 48, 42, "fp8")])
def test_members_that_can_not_run(lens, heads, window, layers, kv):
    import torch
    p = Made(lens, heads, window, layers, kv)
    assert b.codecomp_score_teams(p.make()) > 0
    assert torch.equal(p.score().view(torch.int32), p.score(b.VARIANT_TEAMS_APART).view(torch.int32))
    p.q[:, :, :, ::3] *= 40.0
    far = p.score(b.VARIANT_TEAMS_APART)
    assert torch.equal(far.view(torch.int32), p.score().view(torch.int32))
    np.testing.assert_allclose(far.cpu().numpy(), p.score(b.VARIANT_NO_TEAMS).cpu().numpy(), rtol=2e-4, atol=1e-30)


# More problems with rows out of range than the list of them holds (1024): all are done again.
@pytest.mark.gpu
def test_more_problems_out_of_range_than_are_listed():
    import torch
    p = Made([1536], (32, 16), 128, 65)
    assert b.codecomp_score_teams(p.make()) == 3
    p.q[:, :, :, 5] *= 40.0
    far = p.score()
    assert torch.equal(far.view(torch.int32), p.score(b.VARIANT_TEAMS_APART).view(torch.int32))
    np.testing.assert_allclose(far.cpu().numpy(), p.score(b.VARIANT_NO_TEAMS).cpu().numpy(), rtol=2e-4, atol=1e-30)


# Some problems out of range, far from one another: their place in the list is not their number.  Key and query logits as in test_logits_far_apart.
@pytest.mark.gpu
@pytest.mark.parametrize("lens", [[9000], [5000, 12345, 2000]])
def test_problems_done_again_alone(lens):
    import torch
    p = Made(lens, (28, 4), 64, 12)
    assert b.codecomp_score_teams(p.make()) > 0
    clean = p.score()
    keep = torch.ones(clean.shape, dtype=torch.bool, device="cuda")
    first = np.concatenate([[0], np.cumsum(lens)])
    for layer, head, request in ((0, 1, 0), (5, 2, len(lens) - 1), (5, 3, len(lens) // 2), (11, 3, 0)):
        p.k[layer, head, first[request] + 777] *= 80
        keep[layer, head, first[request]:first[request + 1]] = False
    hit = p.score()
    assert torch.equal(clean[keep], hit[keep])
    np.testing.assert_allclose(hit.cpu().numpy(), p.score(b.VARIANT_NO_TEAMS).cpu().numpy(), rtol=2e-4, atol=1e-30)
    assert torch.equal(hit.view(torch.int32), p.score(b.VARIANT_TEAMS_APART).view(torch.int32))
