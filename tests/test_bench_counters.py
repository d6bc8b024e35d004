"""The counters that bench.py quotes belong to one kernel source: with any other they are left out (no GPU needed)."""
import bench


def test_counters_are_quoted_for_their_own_source_only(monkeypatch):
    now = bench.step_source_digest()
    monkeypatch.setattr(bench, "COUNTERS", {"own": {"source": now}, "other": {"source": "0" * len(now)}})
    assert bench.counters_of("own") == {"source": now}
    assert bench.counters_of("other") is None
    assert bench.counters_of("unknown") is None


def test_digest_follows_code_and_not_comments(monkeypatch, tmp_path):
    csrc = tmp_path / "paper_1905_12799_amd" / "csrc"
    csrc.mkdir(parents=True)
    (csrc / "rls_internal.h").write_text("int a;  // note\n")
    (csrc / "kmeans_lloyd.hip").write_text("int b = 1; /* text */\n")
    monkeypatch.setattr(bench, "ROOT", str(tmp_path))
    first = bench.step_source_digest()
    (csrc / "kmeans_lloyd.hip").write_text("int b  =  1; /* other text,\n two lines */ // more\n")
    assert bench.step_source_digest() == first
    (csrc / "kmeans_lloyd.hip").write_text("int b = 2; /* text */\n")
    assert bench.step_source_digest() != first
