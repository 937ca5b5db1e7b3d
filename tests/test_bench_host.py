"""Host-side logic of bench.py that decides what it reports: a counter record
is attached to a bench line only when it was taken on the same workload, the
same plan and the kernel's current sources."""
import json
import os
import sys
import types

import pytest
import torch

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
sys.path.insert(0, ROOT)

import bench  # noqa: E402
import paper_2607_04489_amd as eg  # noqa: E402

PLAN = {"variant": "global_hash", "predicted_out": 1000, "load_factor": 0.25}


def write_record(path, **over):
    rec = {"workload": "w", "kernel": "hash_probe", "plan": PLAN,
           "sources_sha": bench.sources_digest("hash_probe"),
           "fetch_bytes_per_launch": 3000, "write_bytes_per_launch": 500}
    rec.update(over)
    with open(path, "w") as f:
        json.dump({"hash_probe": rec}, f)


def test_traffic_needs_same_workload_plan_and_sources(tmp_path, monkeypatch):
    path = str(tmp_path / "traffic.json")
    monkeypatch.setattr(bench, "TRAFFIC_FILE", path)
    write_record(path)
    assert bench.traffic_for("hash_probe", "w", PLAN) == 3500
    assert bench.traffic_for("hash_probe", "other", PLAN) is None
    assert bench.traffic_for("hash_probe", "w", dict(PLAN, load_factor=0.5)) is None
    assert bench.traffic_for("radix_join", "w", PLAN) is None
    write_record(path, sources_sha="0" * 16)
    assert bench.traffic_for("hash_probe", "w", PLAN) is None
    write_record(path, plan=None)
    assert bench.traffic_for("hash_probe", "w", PLAN) is None


def test_missing_or_broken_record_file(tmp_path, monkeypatch):
    monkeypatch.setattr(bench, "TRAFFIC_FILE", str(tmp_path / "absent.json"))
    assert bench.traffic_for("hash_probe", "w", PLAN) is None
    bad = tmp_path / "bad.json"
    bad.write_text("{not json")
    monkeypatch.setattr(bench, "TRAFFIC_FILE", str(bad))
    assert bench.traffic_for("hash_probe", "w", PLAN) is None


def test_committed_records_name_their_plan():
    with open(os.path.join(ROOT, "profiles", "traffic.json")) as f:
        recs = json.load(f)
    for name, rec in recs.items():
        assert rec["kernel"] == name and isinstance(rec.get("plan"), dict) and rec["plan"]["variant"]


@pytest.mark.parametrize("rows", [bench.WIDE_DIGIT_ROWS - 1, bench.WIDE_DIGIT_ROWS])
def test_radix_bytes_follow_the_passes_that_ran(rows):
    """Ten bits of int32 keys, 4-byte payloads: the join's own single pass, or the radix
    sort's, one from WIDE_DIGIT_ROWS rows a side on and two below."""
    col = torch.empty(0, dtype=torch.int32)
    inp = types.SimpleNamespace(n_build=1000, n_probe=rows, build_keys=col, build_payload=col, probe_payload=col)
    plan = eg.make_plan(eg.RADIX, 10, 1, 0.5)
    own = bench.kernel_bytes(plan, inp, 7, {"radix_hist": 0, "radix_scatter": 0, "radix_join": 0})
    assert "sort_scatter" not in own and own["radix_scatter"] == (1000 + rows) * 20
    got = bench.kernel_bytes(plan, inp, 7, {"sort_hist": 0, "sort_scatter": 0, "radix_join": 0})
    n = 1 if rows >= bench.WIDE_DIGIT_ROWS else 2
    assert "radix_scatter" not in got
    assert got["sort_hist"] == 4 * (2 * 1000 + n * rows)
    assert got["sort_scatter"] == 20 * (1000 + rows) + 24 * (1000 + (n - 1) * rows)


def test_traffic_record_is_of_the_probe_that_ran(tmp_path, capsys):
    """Of the two probes launched for 32-byte slots the record takes the working one."""
    def write(sub, fname, text):
        os.makedirs(tmp_path / sub, exist_ok=True)
        (tmp_path / sub / fname).write_text(text)

    head = "Kernel_Name,Grid_Size,Counter_Name,Counter_Value\n"
    for sub, counter, value in (("p_fetch", "FETCH_SIZE", 2000), ("p_write", "WRITE_SIZE", 700)):
        rows = [
            ("void eiger::(anonymous namespace)::k_probe<eiger::(anonymous namespace)::HashTab<long; long> >", 300, 3),
            ("void eiger::(anonymous namespace)::k_probe_rows<long; long; long>", 200, value),
            ("void eiger::(anonymous namespace)::k_probe_rows<long; long; long>", 100, 9999)]
        write(sub, "run_counter_collection.csv", head + "".join(f"{n},{g},{counter},{v}\n" for n, g, v in rows))
        write("p_c" + sub[2:], "run_counter_collection.csv", head + f"copy,1,{counter},{1 << 20}\n")
    write("p_trace", "run_kernel_stats.csv", "Name,TotalDurationNs,Calls,AverageNs\n")
    bench.summarize_profile(str(tmp_path), "w", "hash_probe", PLAN)
    rec = json.loads(capsys.readouterr().out.splitlines()[0])
    assert (rec["fetch_bytes_per_launch"], rec["write_bytes_per_launch"]) == (2000 * 1024, 700 * 1024)
