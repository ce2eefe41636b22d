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
