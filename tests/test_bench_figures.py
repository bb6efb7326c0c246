"""The committed counters count as current only on the sources they were taken on: a
class's digest changes with its kernel's file and with every csrc header it includes."""
import os
import shutil

import pytest

import bench

CSRC = ("paper_2511_15022_amd", "csrc")


@pytest.mark.parametrize("cls,files", [
    ("col_pass", ["fft_chain.h", "fft_reg.h", "cgh_internal.h"]),
    ("row_loss", ["fft_chain.h", "fft_reg.h", "cgh_internal.h"]),
    ("raster_adjoint", ["raster_kernels.hip", "cgh_internal.h"]),
])
def test_digest_covers_included_headers(cls, files, tmp_path, monkeypatch):
    real = bench.kernel_digest(cls)
    shutil.copytree(os.path.join(bench.ROOT, *CSRC), tmp_path.joinpath(*CSRC))
    monkeypatch.setattr(bench, "ROOT", str(tmp_path))
    assert bench.kernel_digest(cls) == real
    for name in files:
        path = tmp_path.joinpath(*CSRC, name)
        text = path.read_text()
        path.write_text(text + "// changed\n")
        assert bench.kernel_digest(cls) != real, name
        path.write_text(text)
    assert bench.kernel_digest("preprocess") is None


def test_figures_of_other_sources_are_not_reported(tmp_path, monkeypatch):
    shutil.copytree(os.path.join(bench.ROOT, *CSRC), tmp_path.joinpath(*CSRC))
    monkeypatch.setattr(bench, "ROOT", str(tmp_path))
    (tmp_path / "profiles").mkdir()
    line = f"valu col_pass 1234 {bench.kernel_digest('col_pass')}\n"
    (tmp_path / "profiles" / "a_valu_counters.txt").write_text(line)
    assert bench.committed_figure("valu", "col_pass", "*valu_counters*.txt") == 1234.0
    header = tmp_path.joinpath(*CSRC, "fft_reg.h")
    header.write_text(header.read_text() + "// changed\n")
    assert bench.committed_figure("valu", "col_pass", "*valu_counters*.txt") is None
