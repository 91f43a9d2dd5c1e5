"""LDS of the span-loss kernel (no GPU): the partial tiles of its products
need more room than one of its matrices has, so one array holds them all;
separate arrays have no order that a program may rely on.  Sizes as the
compiler's front end declares them, before any layout."""
import os
import re
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
HIPCC = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")


@pytest.mark.skipif(shutil.which(HIPCC) is None, reason="needs hipcc")
def test_span_loss_tiles_lie_in_one_array(tmp_path):
    out = str(tmp_path / "k_learn.ll")
    subprocess.run([HIPCC, "-O0", "--offload-arch=gfx950", "-std=c++17", "-I" + os.path.join(ROOT, "include"),
                    "--offload-device-only", "-S", "-emit-llvm", "-Xclang", "-disable-llvm-passes", "-o", out,
                    os.path.join(ROOT, "paper_1512_04506_amd", "csrc", "k_learn.hip")], check=True)
    decl = re.compile(r"^@\w*net_span_loss_kernelILi(\d)E\S* = internal addrspace\(3\) global \[(\d+) x %\S*cx")
    arrays = {}
    with open(out) as f:
        for line in f:
            m = decl.match(line)
            if m:
                arrays.setdefault(int(m.group(1)), []).append(int(m.group(2)))
    assert set(arrays) == {1, 2}
    for mt, sizes in arrays.items():
        tiles = mt * (mt + 1) // 2 + mt * mt  # of G (upper triangle) and of C
        need = tiles * 8 * 64 * 8             # four real and four imaginary doubles per lane
        assert max(sizes) * 16 >= need, (mt, sizes, need)
