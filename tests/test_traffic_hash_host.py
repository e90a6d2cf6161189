"""bench.py's hash of the device code, which ties measured traffic to the kernels it was measured on, covers
every file of device code."""
import os

import bench


def test_hash_covers_every_device_header(tmp_path, monkeypatch):
    src = os.path.join(bench.ROOT, "paper_1901_02211_amd", "csrc")
    csrc = tmp_path / "paper_1901_02211_amd" / "csrc"
    csrc.mkdir(parents=True)
    files = ("kernels.hip", "wilson_site.h", "tiles.h")
    for f in files:
        (csrc / f).write_text(open(os.path.join(src, f)).read())
    monkeypatch.setattr(bench, "ROOT", str(tmp_path))
    before = bench.kernel_source_hash()
    for f in files:
        text = (csrc / f).read_text()
        (csrc / f).write_text(text + "// a comment\n\n")
        assert bench.kernel_source_hash() == before
        (csrc / f).write_text(text + "int changed;\n")
        assert bench.kernel_source_hash() != before
        (csrc / f).write_text(text)
