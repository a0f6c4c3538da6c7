"""The source hash that ties counter records to the kernel covers every header
the kernel is built from (CPU)."""

import os
import shutil
import sys

from tests.conftest import ROOT

HEADERS = ["mc_block.h", "mc_direct.h", "mc_split.h", "mc_apply.h", "mc_internal.h", "mc_tiles.h"]


def test_a_change_in_any_header_changes_the_hash(tmp_path, monkeypatch):
    sys.path.insert(0, ROOT)
    import bench
    for d in ("paper_2005_13679_amd/csrc", "include"):
        shutil.copytree(os.path.join(ROOT, d), tmp_path / d)
    monkeypatch.setattr(bench, "ROOT", str(tmp_path))
    for p in bench.PATHS:
        before = bench.kernel_source_hash(p)
        for h in HEADERS:
            f = tmp_path / "paper_2005_13679_amd" / "csrc" / h
            text = f.read_text()
            f.write_text(text + "\n// changed\n")
            assert bench.kernel_source_hash(p) != before, (p, h)
            f.write_text(text)
        assert bench.kernel_source_hash(p) == before
