"""Host-side check of what the compiler gives the few-row kernel (mpgemm_rows8_kernel): no variant spills vector
registers, and a CU holds as many workgroups as the plan counts with.  Read from the kernel descriptions in the assembly.
No GPU needed."""
import os
import re
import subprocess

import pytest

from paper_2407_00088_amd import build as B
from plan_probe import wgs_by_registers


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


def test_plan_counts_with_the_registers_that_the_kernels_have(rows8):
    """Workgroups of four wavefronts, one on each SIMD of 512 registers, handed out in eights, at most eight wavefronts; the
    plan's number is that of the variant with most registers."""
    variants = max(k[4] for k in rows8)    # (the last one is that of longer slices)
    for nt in (4, 8):
        for bits in (1, 2, 3, 4):
            for longer in (False, True):
                held = [min(512 // (-(-v["vgpr_count"] // 8) * 8), 8) for k, v in rows8.items()
                        if k[1:3] == (bits, nt) and (k[4] == variants) == longer]
                assert min(held) == wgs_by_registers(nt, bits, longer), (nt, bits, longer, held)
