"""How the library would split a batched call (rows_plan of csrc/tmac_internal.h), asked of the built library on the host,
so that tests can say which side of a rule their shapes are on.  No GPU needed."""
import ctypes
import functools
import os
import subprocess
import tempfile
from types import SimpleNamespace

import paper_2407_00088_amd as T
from paper_2407_00088_amd import binding as B
from paper_2407_00088_amd import build

FIELDS = ["eight", "slices", "nt", "oct", "row_blocks", "n_tiles_n", "fix", "run_wgs", "n_chunks", "Mp", "builds_f16", "builds_i8"]
SOURCE = """
#include "tmac_internal.h"
extern "C" void plan_probe(const tmac_wdesc* d, int N, int from_act, int* o, size_t* part_bytes, size_t* srow_bytes) {
  const tmac::RowsPlan p = tmac::rows_plan(d, N, from_act != 0);
  const tmac::Geometry ge = tmac::geometry(d);
  const int v[] = {p.eight, p.slices, p.nt, p.oct, p.row_blocks, p.n_tiles_n, p.fix, p.run_wgs, ge.n_chunks, ge.Mp,
                   tmac::rows_builds_tables(d, N, false), tmac::rows_builds_tables(d, N, true)};
  for (int i = 0; i < (int)(sizeof(v) / sizeof(v[0])); ++i) o[i] = v[i];
  *part_bytes = p.part_bytes;
  *srow_bytes = p.srow_bytes;
}
extern "C" int wgs_by_registers(int nt, int bits, int longer) { return tmac::rows8_wgs_by_registers(nt, bits, longer != 0); }
"""


@functools.cache
def _probe():
    out = os.path.join(tempfile.mkdtemp(prefix="tmac_plan_"), "plan_probe.so")
    subprocess.run(["g++", "-O1", "-std=c++17", "-shared", "-fPIC", "-x", "c++", "-", "-x", "none", T.LIB_PATH,
                    "-I" + build.CSRC, "-I" + os.path.join(build.ROOT, "include"), "-o", out],
                   input=SOURCE.encode(), check=True)
    return ctypes.CDLL(out)


def rows_plan(N, M, K, bits, group, g=4, from_act=False):
    """The plan of a layout-3 call, with `longest`: 32-k chunks of the longest K slice of the eight-chunk kernel."""
    d = T.wdesc(M, K, bits, group, g=g, layout=B.TMAC_LAYOUT_R64K32)
    o, part, srow = (ctypes.c_int * len(FIELDS))(), ctypes.c_size_t(), ctypes.c_size_t()
    _probe().plan_probe(ctypes.byref(d), N, int(from_act), o, ctypes.byref(part), ctypes.byref(srow))
    p = SimpleNamespace(**dict(zip(FIELDS, o)), part_bytes=part.value, srow_bytes=srow.value, one_group=group in (0, K))
    cpg = 1 if p.one_group else max(group // 32, 1)
    p.longest = -(-(p.n_chunks // cpg) // p.slices) * cpg
    return p


def wgs_by_registers(nt, bits, longer):
    """Workgroups of the eight-chunk kernel that the plan takes a CU's registers to hold."""
    return _probe().wgs_by_registers(nt, bits, int(longer))
