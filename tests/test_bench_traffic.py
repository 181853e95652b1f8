"""bench.py ties the recorded HBM traffic to the kernels it was measured on: to their sources and to no others."""
import os
import shutil

import bench


def test_traffic_belongs_to_the_sources_of_its_kernels(tmp_path, monkeypatch):
    csrc = tmp_path / "paper_2505_16162_amd" / "csrc"
    shutil.copytree(os.path.join(bench.ROOT, "paper_2505_16162_amd", "csrc"), csrc)
    for family, _ in bench.FAMILIES:
        name = family.split("<")[0]
        assert any("void " + name + "(" in (csrc / f).read_text() for f in bench.TRAFFIC_SOURCES), name
    monkeypatch.setattr(bench, "ROOT", str(tmp_path))
    note = tmp_path / "traffic.md"
    monkeypatch.setattr(bench, "TRAFFIC_FILE", str(note))
    assert bench.recorded_traffic() is None                       # no measurement
    note.write_text("traffic_bytes_per_launch: 160711245\nkernel_source_sha16: %s\n" % bench.kernel_source_sha16())
    assert bench.recorded_traffic() == 160711245.0
    for name in ("kernels_prefill.h", "kernels_generic.h"):
        with open(csrc / name, "a") as f:
            f.write("// changed\n")
    assert bench.recorded_traffic() == 160711245.0
    with open(csrc / "kernels_bf16.h", "a") as f:
        f.write("// changed\n")
    assert bench.recorded_traffic() is None
