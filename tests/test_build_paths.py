"""Where the build looks for ROCm's headers."""
import os

from paper_2505_24133_amd import build as B


def test_headers_of_the_rocm_that_hipcc_belongs_to(monkeypatch, tmp_path):
    (tmp_path / "bin").mkdir()
    (tmp_path / "bin" / "hipcc").write_text("#!/bin/sh\n")
    (tmp_path / "bin" / "hipcc").chmod(0o755)
    monkeypatch.delenv("ROCM_PATH", raising=False)
    monkeypatch.setenv("PATH", str(tmp_path / "bin"))
    assert B.rocm_include() == str(tmp_path / "include")
    monkeypatch.setenv("ROCM_PATH", "/some/rocm")
    assert B.rocm_include() == "/some/rocm/include"
    monkeypatch.delenv("ROCM_PATH")
    monkeypatch.setenv("PATH", str(tmp_path))
    assert B.rocm_include() == os.path.join("/opt/rocm", "include")
