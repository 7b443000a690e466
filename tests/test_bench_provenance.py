"""bench.py reports counters that were profiled offline only for the kernel sources that they were taken on."""
import importlib.util
import json
import os

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


def bench():
    spec = importlib.util.spec_from_file_location("bench_module", os.path.join(ROOT, "bench.py"))
    m = importlib.util.module_from_spec(spec)
    spec.loader.exec_module(m)
    return m


def test_counters_of_other_sources_are_not_reported(tmp_path, monkeypatch):
    b = bench()
    path = str(tmp_path / "figures.txt")
    figures = {"sources": b.kernel_sources_hash(), "hbm_bytes_per_launch": 7.0, "valu_busy_frac": 0.5, "library_version": 1, "source": "x"}
    assert b.profiled_traffic(path, 1) == (None, None, None)
    json.dump(figures, open(path, "w"))
    assert b.profiled_traffic(path, 1)[:2] == (7.0, 0.5)
    json.dump(dict(figures, sources="0" * 16), open(path, "w"))          # the same version, other kernels
    assert b.profiled_traffic(path, 1)[:2] == (None, None)
    json.dump({k: v for k, v in figures.items() if k != "sources"}, open(path, "w"))
    assert b.profiled_traffic(path, 1)[:2] == (None, None)

    # a changed comment is the same kernel, a changed constant another
    csrc = tmp_path / "paper_2305_18627_amd" / "csrc"
    csrc.mkdir(parents=True)
    for name in ("quantize.hip", "gq_device.hpp", "gq_host.hpp"):
        with open(os.path.join(ROOT, "paper_2305_18627_amd", "csrc", name)) as f:
            (csrc / name).write_text("// another comment\n" + f.read())
    monkeypatch.setattr(b, "ROOT", str(tmp_path))
    assert b.kernel_sources_hash() == figures["sources"]
    text = (csrc / "quantize.hip").read_text()
    assert "kFusedBlock = 128" in text
    (csrc / "quantize.hip").write_text(text.replace("kFusedBlock = 128", "kFusedBlock = 256"))
    assert b.kernel_sources_hash() != figures["sources"]
