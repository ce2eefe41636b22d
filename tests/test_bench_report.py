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
