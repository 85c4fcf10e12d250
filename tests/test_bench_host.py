"""Host logic of bench.py (no GPU): the one-GPU guard, the algorithmic byte
counts of a round's phases, the roofline record and the traffic summaries'
source-hash gate."""
import hashlib
import json
import os
import subprocess
import sys

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
sys.path.insert(0, ROOT)

import bench  # noqa: E402


def test_more_than_one_gpu_is_refused():
    r = subprocess.run([sys.executable, os.path.join(ROOT, "bench.py"), "--gpus", "2"],
                       capture_output=True, text=True, timeout=120)
    assert r.returncode == 2
    assert "one GPU" in r.stderr
    assert r.stdout == ""


def test_no_timed_steps_is_refused():
    r = subprocess.run([sys.executable, os.path.join(ROOT, "bench.py"), "--steps", "0"],
                       capture_output=True, text=True, timeout=120)
    assert r.returncode == 2 and "--steps" in r.stderr


def test_phase_bytes_by_hand():
    st = {"boundary": 2, "active_pins": 5, "candidates": 1, "approved": 1, "moved_pins": 3,
          "touched_nets": 4, "touched_pins": 9}
    # n/8 + 16 per active vertex + (12 + 4 ceil(k/32)) per active incidence + 16 per candidate
    assert bench.select_bytes(st, 64, 16) == 8 + 32 + 5 * 16 + 16
    assert bench.select_bytes(st, 64, 64) == 8 + 32 + 5 * 20 + 16
    assert bench.approve_bytes(st, 64, 16) == 32 + 20 + 60
    assert bench.finalize_bytes(st, 64, 16) == 32 + 36 + 8


def test_roofline_record():
    r = bench.roofline_of("x", 8e9, 1000.0)       # 8 GB in one second
    assert r["achieved"] == pytest.approx(8.0)
    assert r["frac"] == pytest.approx(8.0 / bench.HBM_PEAK_GBS)
    assert r["unit"] == "GB/s" and r["bound"] == "hbm"


def _profile(tmp_path, sources, digest, value=123456):
    text = ("select_traffic_bytes_per_launch: %d\nselect_sources: %s\n"
            "select_sources_sha256: %s\n" % (value, sources, digest))
    (tmp_path / "p.md").write_text(text)


def test_traffic_gate(tmp_path, monkeypatch):
    monkeypatch.setattr(bench, "PROFILES", str(tmp_path))
    rel = "paper_2010_10272_amd/csrc/hg_lp.hip"
    digest = hashlib.sha256(open(os.path.join(ROOT, rel), "rb").read()).hexdigest()
    _profile(tmp_path, rel, digest)
    assert bench.measured_traffic("p.md", "select") == 123456.0
    _profile(tmp_path, rel, "0" * 64)                 # sources changed since the counters
    assert bench.measured_traffic("p.md", "select") is None
    _profile(tmp_path, "no/such/file.hip", digest)
    assert bench.measured_traffic("p.md", "select") is None
    assert bench.measured_traffic("missing.md", "select") is None
    assert bench.measured_traffic("p.md", "approve") is None


@pytest.mark.parametrize("profile", ["plain_vlsi_traffic.md", "plain_sparse_matrix_traffic.md"])
def test_committed_traffic_summaries_parse(profile):
    """Each committed summary records the three phases' bytes and their
    sources; the figures are positive wherever the hash still matches."""
    text = open(os.path.join(ROOT, "profiles", profile)).read()
    for prefix in ("select", "approve", "finalize"):
        assert prefix + "_traffic_bytes_per_launch:" in text
        assert prefix + "_sources_sha256:" in text
        v = bench.measured_traffic(profile, prefix)
        assert v is None or v > 0


def _full_record():
    """A record of every leg's shape, each number with all its digits."""
    x = 12345678901.234567
    roof = {"kernel": "k" * 40, "bound": "hbm", "achieved": x, "peak": 8000.0, "unit": "GB/s",
            "frac": x, "alg_bytes": x, "ms": x, "traffic": 123456789}
    host = {"cpu_model": "c" * 20, "compiler": "g" * 45, "flags": "f" * 40}
    cpu = {"value": x, "unit": "pins/s", "cores": 1, "kind": "oracle", "sample": "s" * 190,
           "seconds": x, "host": host}
    latency = {"p50_ms": x, "p99_ms": x, "round1_p50_ms": x}

    def plain(ks):
        return {"value": x, "unit": "pins/s", "ms_per_step": x, "cpu_baseline": cpu,
                "roofline": dict(roof, phases={"select": roof}, round=roof),
                "per_k": {k: {"records": [{"f%d" % i: 123456789 for i in range(12)}] * 10}
                          for k in ks},
                "round_latency": {k: latency for k in ks}, "graph_refine_ms": {k: x for k in ks},
                "km1_final": {k: 1234567 for k in ks}, "config": "c" * 190}

    times = {"refine_ms": x, "round_ms": x, "pins_per_s": x, "km1_after_rounds": [1234567] * 10}
    run = dict(latency, value=x, unit="pins/s", makespan_s=x, server={"steps": 1234567})
    rec = {"metric": bench.METRIC, "value": x, "unit": "pins/s", "n_gpus": 1, "steps": 20,
           "warmup": 5, "ms_per_step": x, "higher_is_better": True, "scaling": "weak",
           "vs_baseline": None, "dtype": "int32", "data": "synthetic",
           "config": {"workload": "w" * 200, "n": 4000000, "k": [16], "eps": 0.03},
           "roofline": dict(roof, phases={"select": roof}, round=roof, copy_reference=roof),
           "cpu_baseline": cpu, "vlsi": plain(["k16"]), "sparse_matrix": plain(["k8", "k64"]),
           "tiny": plain(["k2"]),
           "batched": {"value": x, "batch_ms": x, "sequential_ms": x, "round_latency": latency,
                       "speedup_vs_sequential": x, "schedule_tuned": [{"a": 1}] * 20,
                       "cpu_baseline": cpu},
           "served": {"open_loop": {"served": run, "plain": run},
                      "burst": {"served": run, "plain": run}}}
    for leg, other in (("monotone", "monotone"), ("cached", "cached")):
        rec[leg] = {k: {"plain": times, other: times, "roofline": roof, "cpu_baseline": cpu}
                    for k in ("k8", "k64")}
    rec["rebalance"] = {k: dict(times, ms=x, roofline=roof, cpu_baseline=cpu)
                        for k in ("k8", "k64")}
    rec["contract"] = dict(times, ms=x, roofline=roof, cpu_baseline=cpu)
    return rec


def test_printed_line_is_short():
    """The whole line has to be seen by who reads only the last few thousand
    characters of the output, the progress lines (about 1,200) among them."""
    rec = _full_record()
    assert len(json.dumps(rec)) > 20000
    line = bench.contract_line(rec)
    assert len(json.dumps(line)) < 6000
    for key in bench.HEADLINE_KEYS:
        if key != "roofline":
            assert line[key] == rec[key]
    for key in ("kernel", "bound", "unit", "peak", "traffic"):
        assert line["roofline"][key] == rec["roofline"][key]
    assert set(line) == set(rec)
    assert line["served"]["burst"]["plain"]["p99_ms"] == 12345700000.0
    assert line["sparse_matrix"]["graph_refine_ms"] == {"k8": 12345700000.0, "k64": 12345700000.0}
