"""The Python binding refuses a library without one of its functions as it
does one of another ABI version."""
import subprocess

import pytest


@pytest.mark.parametrize("source", ["unsigned csv_abi_version(void) { return 4; }",
                                    "unsigned csv_abi_version(void) { return 3; }", "int x;"])
def test_older_library_is_an_abi_mismatch(tmp_path, monkeypatch, source):
    import paper_2308_16619_amd as csv
    so = str(tmp_path / "libold.so")
    subprocess.run(["gcc", "-shared", "-fPIC", "-x", "c", "-", "-o", so], input=source, text=True, check=True)
    monkeypatch.setattr(csv, "LIB_PATH", so)
    monkeypatch.setattr(csv, "_lib", None)
    with pytest.raises(RuntimeError, match="ABI mismatch"):
        csv.lib()
