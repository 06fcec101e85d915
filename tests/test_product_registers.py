"""The prompt's matrix products keep everything in registers: no instantiation spills vector registers or keeps an array in
scratch memory (the kernels are held to two workgroups a compute unit, so a few more live values would)."""
import os
import re
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CSRC = os.path.join(ROOT, "paper_2504_08791_amd", "csrc")


@pytest.mark.parametrize("source,kernel,count", [("fmt_gemm.hip", "fmt_gemm_kernel", 16), ("q4k_gemm.hip", "q4k_gemm_kernel", 1)])
def test_products_use_no_scratch(tmp_path, source, kernel, count):
    assert shutil.which("hipcc") is not None, "hipcc not found"
    from paper_2504_08791_amd.build import FLAGS
    out = tmp_path / "k.s"
    flags = [f for f in FLAGS if f not in ("-fPIC", "-shared")]
    r = subprocess.run(["hipcc", *flags, "-I" + os.path.join(ROOT, "include"), "-I" + CSRC, "-S", "--cuda-device-only", "-o", str(out),
                        os.path.join(CSRC, source)], capture_output=True, text=True)
    assert r.returncode == 0, r.stderr[-2000:]
    found = {m.group(1): int(m.group(2)) for m in re.finditer(r"\.name: +(\S+).*?\.private_segment_fixed_size: (\d+)", out.read_text(), re.S)
             if kernel in m.group(1)}
    assert len(found) == count, found
    assert not any(found.values()), found
