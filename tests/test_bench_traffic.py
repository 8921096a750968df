"""The table of memory traffic that the benchmark reads: it says which kernels it was measured with."""
import importlib.util
import json
import os
import shutil

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


def _bench():
    spec = importlib.util.spec_from_file_location("bench", os.path.join(ROOT, "bench.py"))
    m = importlib.util.module_from_spec(spec)
    spec.loader.exec_module(m)
    return m


def test_digest_of_the_kernels(tmp_path, monkeypatch):
    """Comments and blank space do not count, code does."""
    bench = _bench()
    csrc = tmp_path / "paper_1810_10962_amd" / "csrc"
    shutil.copytree(os.path.join(ROOT, "paper_1810_10962_amd", "csrc"), csrc, ignore=shutil.ignore_patterns("_build"))
    here = bench.kernel_sources_digest()
    monkeypatch.setattr(bench, "ROOT", str(tmp_path))
    assert bench.kernel_sources_digest() == here
    file = csrc / "bns_device.hpp"
    text = file.read_text()
    file.write_text("// another comment\n\n" + text.replace("#pragma once", "#pragma once   // once"))
    assert bench.kernel_sources_digest() == here
    file.write_text(text + "namespace bns { constexpr int kOneMore = 1; }\n")
    assert bench.kernel_sources_digest() != here


def test_the_table_names_its_kernels():
    table = json.load(open(os.path.join(ROOT, "profiles", "hbm_traffic.json")))
    assert len(table["kernel_sources_sha256"]) == 64 and table["measured_at_commit"]
