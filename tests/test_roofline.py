"""The roofline that bench.py prints: the nearer of two measured ceilings, never
Alg. 2's bytes, which screened calls answer without reading."""

import csv
import os

from paper_2307_01716_amd import profiling


def test_nearer_ceiling():
    valu = {"frac": 0.57, "issue_rate": 0.57 * profiling.VALU_ISSUE_PEAK, "peak": profiling.VALU_ISSUE_PEAK,
            "unit": "wave64 VALU instructions/s"}
    r = profiling.roofline(0.73, 2.05e9, valu)
    assert r["bound"] == "valu_issue" and r["frac"] == 0.57 and r["traffic"] == 2.05e9
    r = profiling.roofline(0.73, 5.0e9, valu)
    assert r["bound"] == "hbm" and abs(r["frac"] - 5.0e9 / 0.73e-3 / 8e12) < 1e-12 and r["unit"] == "GB/s"
    r = profiling.roofline(0.73, 2.05e9, None)
    assert r["bound"] == "hbm" and abs(r["achieved"] - 2.05 / 0.73e-3) < 1e-9


def test_nothing_claimed_without_records():
    r = profiling.roofline(0.73, None, None)
    assert r["bound"] is None and r["frac"] is None and r["achieved"] is None


def test_bench_takes_it():
    with open(os.path.join(os.path.dirname(profiling.PKG), "bench.py")) as f:
        src = f.read()
    assert src.count('"roofline": profiling.roofline(') == 2 and '"roofline": {' not in src


def test_calls_of_several_dispatches(tmp_path):
    """Two launches of three dispatches: summed over the launches."""
    copy, kern = profiling.COPY_KERNEL, "void april::(anonymous namespace)::k_open<256, 2, 0>(X)"
    for name, ctr in (("fetch", "FETCH_SIZE"), ("write", "WRITE_SIZE"), ("valu", "SQ_INSTS_VALU")):
        os.makedirs(tmp_path / name)
        with open(tmp_path / name / "x_counter_collection.csv", "w", newline="") as f:
            w = csv.DictWriter(f, fieldnames=["Dispatch_Id", "Kernel_Name", "Counter_Name", "Counter_Value"])
            w.writeheader()
            rows = [(1, copy, 1048576)] + [(2 + k, kern, 100 * (k + 1)) for k in range(6)]
            for d, n, v in rows:
                w.writerow({"Dispatch_Id": d, "Kernel_Name": n, "Counter_Name": ctr, "Counter_Value": v})
    t = profiling.traffic(str(tmp_path / "fetch"), str(tmp_path / "write"), "k_open", parts=["k_open"], calls=2)
    assert t["fetch_bytes"] == t["write_bytes"] == 2100 / 2 * 1024
    assert profiling.valu(str(tmp_path / "valu"), "k_open", parts=["k_open"], calls=2)["insts_per_launch"] == 1050


def test_parts_of_the_dispatches(tmp_path):
    os.makedirs(tmp_path / "valu")
    with open(tmp_path / "valu" / "x_counter_collection.csv", "w", newline="") as f:
        w = csv.DictWriter(f, fieldnames=["Dispatch_Id", "Kernel_Name", "Counter_Name", "Counter_Value"])
        w.writeheader()
        for d in range(5):
            w.writerow({"Dispatch_Id": d, "Kernel_Name": "april::k_screen<0>(X)", "Counter_Name": "SQ_INSTS_VALU",
                        "Counter_Value": 10 ** d})
    got = profiling.valu(str(tmp_path / "valu"), "k_screen", parts=["k_screen[1:3]"], calls=2)
    assert got["insts_per_launch"] == 110 / 2 and got["dispatches"] == 2
