"""Host-side logic of bench.py (no GPU): the single-GPU guard, the lookup of measured
HBM traffic, which must refuse counter figures taken on other kernel sources, and
the library's rules for what a forward pass launches."""
import hashlib
import json
import os
import subprocess
import sys

import pytest

import bench
from helpers import gathers_signs

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


def test_more_than_one_gpu_is_refused_with_a_message():
    res = subprocess.run([sys.executable, os.path.join(ROOT, "bench.py"), "--gpus", "2"],
                         capture_output=True, text=True, timeout=60)
    assert res.returncode == 2
    assert "single GPU" in res.stderr
    assert res.stdout == ""          # no JSON line for an unsupported run


def _fake_tree(tmp_path, kernels_src, record_sources):
    csrc = tmp_path / "paper_2010_07565_amd" / "csrc"
    csrc.mkdir(parents=True)
    (csrc / "bigcn_kernels.hip").write_bytes(kernels_src)
    (csrc / "bigcn_api.hip").write_bytes(b"// api\n")
    h = hashlib.sha256()
    for part in record_sources:
        h.update(part)
    rec = {"sources_sha256": h.hexdigest(),
           "entries": [{"layer": 0, "entry": "spmm", "fetch_bytes": 1000, "write_bytes": 24},
                       {"layer": 1, "entry": "pack", "fetch_bytes": 7, "write_bytes": 5}]}
    prof = tmp_path / "profiles"
    prof.mkdir()
    (prof / "hbm_traffic_toy.md").write_text(
        "# toy\n\n```json\n" + json.dumps(rec) + "\n```\n")


def test_measured_traffic_matches_entry_and_sources(tmp_path, monkeypatch):
    _fake_tree(tmp_path, b"// kernels\n", [b"// kernels\n", b"// api\n"])
    monkeypatch.setattr(bench, "ROOT", str(tmp_path))
    assert bench.measured_traffic("toy", 0, "spmm") == 1024
    assert bench.measured_traffic("toy", 1, "pack") == 12
    assert bench.measured_traffic("toy", 1, "spmm") is None      # no such entry
    assert bench.measured_traffic("other", 0, "spmm") is None    # no summary


def test_measured_traffic_is_dropped_when_kernels_changed(tmp_path, monkeypatch):
    _fake_tree(tmp_path, b"// kernels, edited\n", [b"// kernels\n", b"// api\n"])
    monkeypatch.setattr(bench, "ROOT", str(tmp_path))
    assert bench.measured_traffic("toy", 0, "spmm") is None


def test_measured_traffic_is_dropped_when_any_device_source_changed(tmp_path, monkeypatch):
    # the figures of a pass with sign aggregations depend on their file and headers too
    sources = [("bigcn_kernels.hip", b"// kernels\n"), ("bigcn_api.hip", b"// api\n"),
               ("bigcn_e2m1.hip", b"// signs\n"), ("bigcn_device.h", b"// device\n"),
               ("bigcn_internal.h", b"// internal\n")]
    _fake_tree(tmp_path, b"// kernels\n", [text for _, text in sources])
    csrc = tmp_path / "paper_2010_07565_amd" / "csrc"
    for name, text in sources:
        (csrc / name).write_bytes(text)
    monkeypatch.setattr(bench, "ROOT", str(tmp_path))
    assert bench.measured_traffic("toy", 0, "spmm") == 1024
    for name, text in sources:
        (csrc / name).write_bytes(text + b"// edited\n")
        assert bench.measured_traffic("toy", 0, "spmm") is None, name
        (csrc / name).write_bytes(text)


def test_forward_route_follows_the_library():
    # the products-like model at its size and at a small one: what bench.py ranks
    import paper_2010_07565_amd as bg
    layers = [bg.Layer(a, b, None, None) for a, b in ((100, 256), (256, 256), (256, 47))]
    route = bg._lib.forward_route(2449029, 126149029, layers)
    assert [r["signs"] for r in route] == [True, False, False]
    assert [r["leaves"] for r in route] == ["signs", "products", None]
    route = bg._lib.forward_route(2000, 50000, layers)
    assert not any(r["signs"] for r in route)
    assert [r["leaves"] for r in route] == ["products", "products", None]


@pytest.mark.parametrize("n,nnz,dims,sage,signs", [
    (169_343, 2_469_343, [128, 256, 256, 40], False, True),    # leaves signs
    (700_000, 2_900_000, [65, 192, 65], False, False), (2_400_000, 12_000_000, [65, 192, 65], False, True),
    (169_343, 2_469_343, [100, 256, 47], False, False),        # leaves products: short rows
    (700_000, 2_100_000, [100, 256, 47], False, False),
    (1_200_000, 5_200_000, [100, 256, 47], False, False),
    (2_400_000, 12_000_000, [100, 256, 47], False, False),
    (300_000, 5_300_000, [100, 256, 47], False, True),
    (20_000, 2_400_000, [100, 256, 47], False, True),
    (700_000, 2_100_000, [100, 128], False, True),
    (300_000, 3_500_000, [128, 256], False, False), (1_200_000, 5_200_000, [128, 256], False, True),
    (250_000, 8_850_000, [200, 128], False, True), (2_400_000, 12_000_000, [256, 70], False, False),
    (2_400_000, 9_600_000, [100, 128], True, False), (250_000, 8_600_000, [100, 128], True, True),
    (1_200_000, 14_000_000, [200, 128], True, False)])
def test_layers_that_gather_signs(n, nnz, dims, sage, signs):
    """The lines of the rule at shapes measured on either side of them."""
    assert gathers_signs(n, nnz, dims, 0, sage) == signs


def test_committed_traffic_summaries_parse():
    # every committed summary carries a hash and per-entry byte counts
    import re
    prof = os.path.join(ROOT, "profiles")
    names = [f for f in os.listdir(prof) if f.startswith("hbm_traffic_")]
    assert names
    for f in names:
        m = re.search(r"```json\n(.*?)\n```", open(os.path.join(prof, f)).read(), re.S)
        assert m is not None, f
        rec = json.loads(m.group(1))
        assert len(rec["sources_sha256"]) == 64
        assert rec["entries"]
        for e in rec["entries"]:
            assert e["fetch_bytes"] > 0 and e["write_bytes"] > 0
            assert e["entry"] in ("pack", "bgemm", "spmm")


def test_cpu_baseline_times_small_graphs_on_one_thread_too():
    # the oracle's thread count is restored after the one-thread passes
    import oracle
    import workloads
    w = workloads.make_workload(1)
    before = oracle.threads()
    r = bench.cpu_baseline(w, budget_s=0.0)
    assert oracle.threads() == before
    assert r["kind"] == "oracle" and r["cores"] == before and r["value"] > 0
    one = r["single_thread"]
    assert one["cores"] == 1 and one["value"] > 0 and one["unit"] == "nodes/s"
    # above the size limit only the all-threads figure is taken
    r = bench.cpu_baseline(w, budget_s=0.0, single_thread_max_nodes=w.n - 1)
    assert "single_thread" not in r
