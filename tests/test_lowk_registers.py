"""The products for a handful of diagonals keep their weights and sums in registers, and so does the kernel that takes both gradients:
none of these may spill to scratch memory (a spill costs a product a factor of four).  Compiled here for gfx950; needs hipcc, no GPU."""
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


def test_kernels_for_a_handful_of_diagonals_do_not_spill(tmp_path):
    scratch = _scratch("dd_lowk.hip", tmp_path)
    products = {n: b for n, b in scratch.items() if "lowk_product_kernel" in n}
    both_gradients = {n: b for n, b in scratch.items() if re.search(r"lowk_wgrad_kernelILi\d+ELi\d+ELb1E", n)}
    assert len(products) >= 40 and len(both_gradients) == 24  # 1, 2, 4 column pairs a lane, 1 ... 8 diagonals
    assert {n: b for n, b in {**products, **both_gradients}.items() if b} == {}
