"""bench.py takes counters only from a summary of the kernels that ran, built from the same sources."""
import os

import bench


def test_counters_are_those_of_the_kernels_that_ran(tmp_path, monkeypatch):
    digest = bench.source_digest()
    monkeypatch.setattr(bench, "ROOT", str(tmp_path))
    monkeypatch.setattr(bench, "source_digest", lambda: digest)
    os.mkdir(tmp_path / "profiles")
    path = tmp_path / "profiles" / "pmc_w.md"
    assert bench.profile_counters("w", ["tb::a<1>"])[0] == {}                 # no summary
    body = ("## `tb::a<1>`\n\n* SQ_INSTS_VALU: 1,000\n* HBM traffic per launch (scaled): fetch 1.0 MB + "
            "write 0.5 MB = 1.50 MB\n* LDS bank-conflict cycles / LDS-active cycles: 0.76\n\n"
            "## `tb::b`\n\n* SQ_INSTS_VALU: 20\n* HBM traffic per launch (scaled): = 0.25 MB\n")
    path.write_text(f"kernel sources: {digest}\n\n{body}")
    counters, source = bench.profile_counters("w", ["tb::a<1>", "tb::b"])
    assert counters["SQ_INSTS_VALU"] == 1020 and abs(counters["hbm_traffic_bytes"] - 1.75e6) < 1
    assert source == "profiles/pmc_w.md (tb::a<1> + tb::b)"
    for names in (["tb::a"], ["tb::a<1, 2>"], ["tb::a<1>", "tb::c"], None, []):  # other instantiations
        assert bench.profile_counters("w", names)[0] == {}, names
    path.write_text(f"kernel sources: {digest[::-1]}\n\n{body}")              # other sources
    assert bench.profile_counters("w", ["tb::a<1>"])[0] == {}


def test_digest_ignores_comments_only(tmp_path, monkeypatch):
    src = tmp_path / "paper_2510_05485_amd" / "csrc"
    os.makedirs(src)
    monkeypatch.setattr(bench, "ROOT", str(tmp_path))
    digests = []
    for text in ("int f() { return 1; }  // one\n", "/* two\n */ int f()\n{ return 1; }", "int f() { return 2; }"):
        (src / "a.hip").write_text(text)
        digests.append(bench.source_digest())
    assert digests[0] == digests[1] != digests[2]


def test_route_names():
    assert bench.route_of(["tb::fused_kernel<6, true, false, false>"], 2) == "fused"
    assert bench.route_of(["tb::runs_sort_kernel<4>", "tb::runs_count_kernel<4096>"], 2) == "sorted runs"
    assert bench.route_of(["tb::pack_kernel"], 1) == "global"
    assert bench.route_of(None, 1) == "fused" and bench.route_of(None, 2) == "global"


def test_route_of_dealt_positions():
    names = ["tb::deal_kernel<2>", "tb::tally_kernel<(tb::Counters)0>"]
    assert bench.route_of(names, 2) == "dealt"
    assert bench.route_of(["tb::deal_kernel<2>"], 2) == "global"      # (half of a call)
