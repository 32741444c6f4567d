"""The source hash that ties a committed profile to its kernels changes with every
source a dslash launch is built from or chosen by.  No GPU."""
import os
import shutil
import sys

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
sys.path.insert(0, ROOT)
import bench  # noqa: E402


def test_every_kernel_source_is_hashed(tmp_path, monkeypatch):
    csrc = tmp_path / "paper_0911_3191_amd" / "csrc"
    shutil.copytree(os.path.join(ROOT, "paper_0911_3191_amd", "csrc"), csrc)
    now = bench.kernel_source_hash()
    monkeypatch.setattr(bench, "ROOT", str(tmp_path))
    assert bench.kernel_source_hash() == now
    names = [n for n in os.listdir(csrc) if n.endswith(".h")] + ["wd_dslash.hip", "wd_tune.cpp"]
    assert "wd_dslash_split.h" in names and "wd_finalize.h" in names
    for name in names:
        kept = (csrc / name).read_bytes()
        (csrc / name).write_bytes(kept + b"\n")
        assert bench.kernel_source_hash() != now, name
        (csrc / name).write_bytes(kept)
