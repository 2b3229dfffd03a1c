"""The hash that ties measured traffic to the decoder covers every file with
the kernels of csv_decode.hip."""
import os
import re
import shutil

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CSRC = os.path.join("paper_2308_16619_amd", "csrc")


def included():
    src = open(os.path.join(ROOT, CSRC, "csv_decode.hip")).read()
    # (csv_generic.hpp: another object's launch; csv.h: the interface)
    return [f for f in re.findall(r'#include "(csv_\w+\.hpp)"', src) if f != "csv_generic.hpp"] + ["csv_decode.hip"]


@pytest.mark.parametrize("name", included())
def test_a_change_changes_the_hash(tmp_path, monkeypatch, name):
    import bench
    shutil.copytree(os.path.join(ROOT, CSRC), str(tmp_path / CSRC))
    before = bench.decoder_hash()
    monkeypatch.setattr(bench, "ROOT", str(tmp_path))
    assert bench.decoder_hash() == before
    with open(str(tmp_path / CSRC / name), "a") as f:
        f.write("\n")
    assert bench.decoder_hash() != before
