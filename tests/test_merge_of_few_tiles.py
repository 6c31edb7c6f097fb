"""The select kernels for calls of few tiles are the same code as the others: their merge, too, exchanges partials by
device-scope accesses alone (see test_abi.py)."""

import os
import re
import subprocess

import pytest

from paper_2510_18413_amd import build as B


def test_merge_uses_device_scope_accesses(tmp_path):
    hipcc = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")
    if not os.path.exists(hipcc):
        pytest.skip("no hipcc")
    out = tmp_path / "select.s"
    flags = [f for f in B.HIPCC_FLAGS if f != "-fPIC"]
    subprocess.run([hipcc] + flags + ["-w", "-DADAMAS_INST_D=128", "-DADAMAS_INST_METRIC=0", "-I", str(B.ROOT / "include"),
                                      "-I", str(B.CSRC), "-S", "--cuda-device-only", "-o", str(out),
                                      str(B.CSRC / "kernels_inst.hip")], check=True)
    text = out.read_text()
    starts = list(re.finditer(r"^_ZN6adamas13select_kernelILi(260|264|268)ELb1ELi0ELb[01]ELi128ELi\d+EEE\w*:", text, re.M))
    assert len(starts) == 8     # 4, 8, 12 tiles a pass at a time, 8 with eight passes; contiguous and paged
    for start in starts:
        one = text[start.end():text.index(".Lfunc_end", start.end())]
        kinds = {l.split()[0] for l in one.splitlines() if re.search(r"\bsc1\b", l)}
        assert any(k.startswith("global_store_dword") for k in kinds) and any(k.startswith("global_load_dword") for k in kinds)
        assert re.search(r"^\s*global_atomic_add\w* v\d+, .*\bsc0\b", one, re.M)
        assert "buffer_wbl2" not in one and "buffer_inv" not in one
