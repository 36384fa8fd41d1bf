"""The traffic summary holds every kernel of the library that the counters saw, those
of the coarse levels among them, and the benchmark's M2L bytes include them (no GPU)."""
import csv
import json
import os

import bench
from paper_1110_2921_amd import rocprof_summary as R

KERNELS = ["k_keys", "k_m2l_orbits<float, 10, 2>", "k_m2l_sym<10>", "k_m2m_coarse<float, false>",
           "k_l2l_coarse<float, false>", "k_sym_pack<float>", "k_lattice<float>"]


def _counters(path, counter, copy):
    os.makedirs(os.path.dirname(path))
    rows = [("__amd_rocclr_copyBuffer", copy)] + [(f"void vmfmm::(anonymous namespace)::{k}(int)", 8.0) for k in KERNELS]
    with open(path, "w", newline="") as f:
        w = csv.DictWriter(f, ["Kernel_Name", "Grid_Size", "Counter_Name", "Counter_Value"])
        w.writeheader()
        for name, v in rows:
            w.writerow({"Kernel_Name": name, "Grid_Size": 64, "Counter_Name": counter, "Counter_Value": v})


def test_every_kernel_of_the_library_is_summarised(tmp_path, monkeypatch):
    _counters(str(tmp_path / "f" / "run_counter_collection.csv"), "FETCH_SIZE", float(1 << 19))
    _counters(str(tmp_path / "w" / "run_counter_collection.csv"), "WRITE_SIZE", float(1 << 20))
    d = R.traffic_summary(str(tmp_path / "f"), str(tmp_path / "w"), "toy", "cmd")
    assert len(d["kernels"]) == len(KERNELS)
    os.makedirs(tmp_path / "profiles")
    (tmp_path / "profiles" / "hbm_traffic_toy_mixed.txt").write_text(json.dumps(d))
    monkeypatch.setattr(bench, "ROOT", str(tmp_path))
    per_kernel = 1024 * (2 * 8.0 + 8.0)
    got = bench.measured_phase_bytes("toy", "mixed", ("k_m2l_sym<", "k_m2l_orbits<float", "k_sym_pack<float>"))
    assert got == 3 * per_kernel


def test_tree_bytes_count_template_instances(tmp_path, monkeypatch):
    """The radix passes' kernels are templates; their bytes belong to the tree's."""
    one = {"dispatches": 4, "hbm_bytes_per_launch": 3.0}
    body = {"sources_sha256": R.sources_sha256(), "kernels": {
        "k_keys": {"dispatches": 2, "hbm_bytes_per_launch": 5.0}, "k_radix_hist<16>": one, "k_radix_scatter<4>": one,
        "k_permute": one, "k_p2p32<false,true>": one}}
    os.makedirs(tmp_path / "profiles")
    (tmp_path / "profiles" / "hbm_traffic_toy_mixed.txt").write_text(json.dumps(body))
    monkeypatch.setattr(bench, "ROOT", str(tmp_path))
    assert bench.measured_tree_bytes("toy", "mixed") == 5.0 + 3 * 6.0
