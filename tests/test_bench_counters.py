"""bench.py's counter accounting of builds whose rounds or layers share a launch (CPU only)."""
import json
import re
import os

import bench

CSRC = os.path.join(bench.ROOT, "paper_1312_0526_amd", "csrc")


def rows(names):
    return [(i, n, 10.0 ** (i % 3) + i) for i, n in enumerate(names)]


def sums(seq, lo, hi):
    return sum(b for i, _, b in seq if lo <= i < hi)


def test_windows_of_a_claim_list_build_with_shared_rounds():
    """2^27 keys: lists first, small rounds in one launch, layers in one launch."""
    seq = rows(["k_gen_u64", "k_zero16", "k_hash_u64_tiles", "k_part_accum", "k_round0_updates", "k_update_accum", "k_apply",
                "k_claims_resolve", "k_fill_u32", "k_rounds_resume", "k_rounds", "k_copy_ctrl", "k_zero16", "k_mphf_finish",
                "k_pack_count", "k_scan_local"])
    w = bench.build_windows(seq)
    assert w["builds"] == 1
    assert w["hash_build"] == sums(seq, 2, 4) and w["peel"] == sums(seq, 4, 13) and w["assign_rank"] == sums(seq, 13, 16)


def test_windows_of_binned_builds():
    """10^6 keys, u64 (hashed by the tiles that sort them) and strings, twice each, with a launch for a large
    layer in one of them."""
    one = ["k_run_init", "k_bins", "k_bins_accum", "k_bins_again", "k_bins_round0", "k_rounds", "k_mphf_finish", "k_copy_ctrl"]
    strs = ["k_run_init", "k_hash_str_words", "k_bins", "k_bins_accum", "k_bins_again", "k_bins_round0", "k_apply",
            "k_rounds_from", "k_rounds", "k_sf_solve"]
    seq = rows(one + strs + one + ["k_hash_str_words", "k_bins", "k_bins_round0"])  # the last has no end
    w = bench.build_windows(seq)
    assert w["builds"] == 3
    # from each build's hashing kernel to its round 0, to its layers, to the next build's hashing kernel
    starts = [(1, 4, 6, 9), (9, 13, 17, 19), (19, 22, 24, 26)]
    assert w["hash_build"] == sum(sums(seq, a, b) for a, b, _, _ in starts) / 3
    assert w["peel"] == sum(sums(seq, b, c) for _, b, c, _ in starts) / 3
    assert w["assign_rank"] == sum(sums(seq, c, d) for _, _, c, d in starts) / 3


def test_every_timed_kernel_has_a_phase_and_its_sources():
    want = {"k_rounds": "apply", "k_apply": "apply", "k_mphf_finish": "assign", "k_sf_solve": "assign",
            "k_assign_round": "assign", "k_bins_round0": "frontier", "k_round0": "frontier", "k_round0_updates": "frontier",
            "k_bins_accum": "build", "k_bins_again": "build", "k_part_accum": "build", "k_rounds_resume": None,
            "k_rounds_from": None, "k_copy_ctrl": None}
    assert {k: bench.phase_of(k) for k in want} == want
    # the file that holds a phase's kernel is one of its sources
    where = {}
    for f in sorted(os.listdir(CSRC)):
        for k in re.findall(r"\b(k_\w+)\(", open(os.path.join(CSRC, f)).read()) if f.endswith(".hip") else ():
            where.setdefault(k, set()).add(f)
    for kernel, phase in want.items():
        if phase:
            assert where[kernel] & set(bench.PHASE_SOURCES[phase]), kernel
    assert all("grid.h" in bench.PHASE_SOURCES[p] for p in ("apply", "assign"))


def counter_csv(path, names):
    path.mkdir(parents=True)
    lines = ["Dispatch_Id,Kernel_Name,Counter_Name,Counter_Value"]
    lines += [f'{i},"void mphx::{n}<3, true>(int)",X,{100 + i}' for i, n in enumerate(names)]
    (path / "p_counter_collection.csv").write_text("\n".join(lines) + "\n")
    return str(path)


def test_summary_holds_every_phase_of_a_build(tmp_path, monkeypatch):
    """A summary of a 2^27 build's counters serves the step's traffic, and says what it lacks where it cannot."""
    names = ["k_hash_u64_tiles", "k_part_accum", "k_round0_updates", "k_update_accum", "k_apply", "k_claims_resolve",
             "k_rounds_resume", "k_rounds", "k_mphf_finish", "k_pack_count"]
    build, copy = counter_csv(tmp_path / "b", names), counter_csv(tmp_path / "c", ["k_copy"])
    monkeypatch.setattr(bench, "COUNTERS_FILE", str(tmp_path / "hbm_{workload}.json"))
    assert bench.summarize_counters(build, build, copy, copy, "w", "command") == 0
    doc = json.load(open(tmp_path / "hbm_w.json"))
    assert set(doc["phases"]) == set(bench.PHASE_SOURCES)
    assert doc["phases"]["apply"]["kernels"] == ["k_apply", "k_rounds"] and doc["phases"]["apply"]["launches"] == 2
    assert doc["phases"]["assign"]["kernels"] == ["k_mphf_finish"] and doc["windows"]["builds"] == 1
    total = bench.counters_step_traffic("w")
    assert total and abs(total - sum(v["fetch_bytes"] + v["write_bytes"] for v in doc["kernels"].values())) < 1
    digest = bench.sources_digest
    monkeypatch.setattr(bench, "sources_digest", lambda p: "0" if p == "apply" else digest(p))
    assert bench.counters_step_traffic("w") is None
    assert "sources changed since: apply" in bench.counters_missing("w")
    assert "never taken" in bench.counters_missing("other")


def test_rank_bytes_where_one_launch_assigns_and_ranks():
    st = dict(n=1 << 20, kind="u64")
    assert bench.algorithmic_bytes("assign", st) == 16 * st["n"]
    assert bench.algorithmic_bytes("assign", dict(st, rank_in_assign=True)) == 16 * st["n"] + 2.8 * st["n"]
