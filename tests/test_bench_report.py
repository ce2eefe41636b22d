"""What bench.py reports from the committed counter summaries."""
import bench


def test_counter_summary_names_its_build_as_text(tmp_path, monkeypatch):
    (tmp_path / "profiles").mkdir()
    (tmp_path / "profiles" / "pmc_some.txt").write_text(
        "# bytes per launch\ncommit = 12095e6\ndate = 2026-11-28\nscore_mass_hbm_bytes_per_launch = 1472732 (read + write)\n")
    monkeypatch.setattr(bench, "ROOT", str(tmp_path))
    got = bench.read_traffic("some")
    assert got["commit"] == "12095e6" and got["date"] == "2026-11-28"        # a commit that reads like a number stays a commit
    assert got["score_mass_hbm_bytes_per_launch"] == 1472732.0
    assert bench.read_traffic("other") is None


def test_share_of_logits_formed_twice_follows_the_library():
    from paper_2604_10235_amd import binding as b, workloads as wl

    def share(w):
        cu, cb = w.cu_seqlens(), w.cu_budgets()
        p = b.make_params(n_layers=w.n_layers, n_q_heads=w.n_q_heads, n_kv_heads=w.n_kv_heads, head_dim=w.head_dim, window=w.window, pool_kernel=w.pool_kernel,
                          prior_weight=w.prior_weight, cu_seqlens_host=cu, cu_budgets_host=cb, cu_seqlens_dev=0x1000, cu_budgets_dev=0x2000)
        return bench.two_pass_share(w, p, b)
    chunks = wl.paper_chunks()
    assert share(chunks) == sum(n for n in chunks.seqlens if n > 768) / chunks.total_tokens
    assert share(wl.qwen7b_32k()) == 1.0
    short = wl.scaled(chunks, seqlens=[300, 768], budgets=[150, 300])
    assert share(short) == 0.0
    few_rows = wl.scaled(wl.tiny(), n_layers=28)                            # 112 problems of 2048 tokens, 32 rows
    assert share(few_rows) == 0.0 and share(wl.tiny()) == 1.0


def test_floors_are_those_of_the_passes_that_ran():
    from paper_2604_10235_amd import binding as b, workloads as wl
    w = wl.qwen7b_32k()
    p = b.make_params(n_layers=w.n_layers, n_q_heads=w.n_q_heads, n_kv_heads=w.n_kv_heads, head_dim=w.head_dim, window=w.window, pool_kernel=w.pool_kernel,
                      prior_weight=w.prior_weight, cu_seqlens_host=w.cu_seqlens(), cu_budgets_host=w.cu_budgets(), cu_seqlens_dev=0x1000, cu_budgets_dev=0x2000)
    assert b.codecomp_score_teams(p) > 0
    assert bench.formed_twice(w, p, b, {"score_row_stats": 0.005, "score_mass": 0.63}) == 0.0
    assert bench.formed_twice(w, p, b, {"score_row_stats": 0.076, "score_mass": 0.64}) == 0.0        # under a profiler
    assert bench.formed_twice(w, p, b, {"score_row_stats": 0.43, "score_mass": 0.42}) == 1.0         # a device that the teams do not fit
    peaks = dict(mfma_bf16_tflops=1700.0, exp_per_s=1.6e13, read_gb_per_s=6000.0, mix_logits_per_s=6e12)
    ab = bench.algorithmic_bytes(w)
    for twice, name, times in ((0.0, "one_pass", 1.0), (1.0, "two_passes", 2.0), (0.5, "mixed_passes", 1.5)):
        got = bench.binding_roofline(4e11, 1.6e9, twice, ab, ab["k_read"], 0.7, peaks)["measured"]
        assert set(got["floors_ms"]) == {f"mfma_{name}", f"exp_{name}", f"issue_mix_{name}", "hbm_one_read"} | ({"hbm_two_reads"} if twice else set())
        assert got["binding"] == f"issue_mix_{name}" and abs(got["floors_ms"][got["binding"]] - times * 1.6e9 / 6e12 * 1e3) < 1e-3
