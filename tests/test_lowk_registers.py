"""The products for a handful of diagonals keep their weights and sums in registers: none of their kernels may spill to
scratch memory (a spill costs them a factor of four).  Compiled here for gfx950; needs hipcc, no GPU."""
import os
import re
import subprocess

import pytest

from paper_2506_11449_amd import build


def _scratch(source, tmp_path):
    """{kernel: bytes of scratch per lane} as the compiler reports them."""
    hipcc = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")
    if not os.path.exists(hipcc):
        pytest.skip("no hipcc")
    flags = [f for f in build.HIPCC_FLAGS if f != "-shared"]
    out = subprocess.run([hipcc, *flags, "-c", "--offload-device-only", "-Rpass-analysis=kernel-resource-usage", "-o",
                          str(tmp_path / "kernels.o"), os.path.join(build.CSRC, source)], capture_output=True, text=True)
    assert out.returncode == 0, out.stderr[-2000:]
    return {n: int(b) for n, b in re.findall(r"Function Name: (\S+)(?:(?!Function Name).)*?ScratchSize \[bytes/lane\]: (\d+)",
                                             out.stderr, flags=re.S)}


def test_products_for_a_handful_of_diagonals_do_not_spill(tmp_path):
    scratch = {n: b for n, b in _scratch("dd_lowk.hip", tmp_path).items() if "lowk_product_kernel" in n}
    assert len(scratch) >= 40
    assert {n: b for n, b in scratch.items() if b} == {}
