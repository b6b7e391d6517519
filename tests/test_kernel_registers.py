"""Host-side check of what the compiler gives the few-row kernel (mpgemm_rows8_kernel): no variant spills vector
registers.  Read from the kernel descriptions in the assembly.  No GPU needed."""
import os
import re
import subprocess

import pytest

from paper_2407_00088_amd import build as B


@pytest.fixture(scope="module")
def rows8(tmp_path_factory):
    """(integer tables, bits, activation rows, tables built in the kernel, variant) -> {vgpr_count, vgpr_spill_count}"""
    out = tmp_path_factory.mktemp("asm") / "rows.s"
    flags = [f for f in B.HIPCC_FLAGS if f not in ("-shared", "-fPIC")]
    subprocess.run([os.environ.get("HIPCC", "/opt/rocm/bin/hipcc"), *flags, "--offload-device-only", "-S", "-o", str(out),
                    os.path.join(B.CSRC, "tmac_rows.hip")], stderr=subprocess.DEVNULL, check=True)
    kernels = {}
    for block in out.read_text().split(".amdgpu_metadata")[1].split("\n  - .agpr_count")[1:]:
        m = re.search(r"\.symbol: +\S*mpgemm_rows8_kernelILb(\d)ELi(\d)ELi(\d)ELb(\d)ELi(\d)E", block)
        if m:
            kernels[tuple(int(x) for x in m.groups())] = {f: int(re.search(r"\.%s: +(\d+)" % f, block).group(1))
                                                          for f in ("vgpr_count", "vgpr_spill_count")}
    assert len(kernels) == 32 * len({k[4] for k in kernels}) > 32
    return kernels


def test_few_row_kernel_does_not_spill(rows8):
    assert not {k: v for k, v in rows8.items() if v["vgpr_spill_count"]}
