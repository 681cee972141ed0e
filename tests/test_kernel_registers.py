"""Registers of the synchronisation kernels, as the compiler reports them: how
many wavefronts a SIMD holds decides how much of the memory latency is hidden,
and code that few launches run (rows of fewer than 4 coordinates) can take it
from all of them."""
import os
import re
import subprocess

import pytest

from paper_2607_21224_amd import build

UNIT = """
#include "cpdp_sync_impl.h"
namespace cpdp { namespace {
template int sync_w<Sync::CPDP, Opt::SGD, 0, ParamF32>(const OptParams&, const SyncArgs&, int);
template int sync_w<Sync::CPDP, Opt::ADAMW, 0, ParamF32>(const OptParams&, const SyncArgs&, int);
template int sync_w<Sync::CPDP, Opt::SGD, 16, ParamF32>(const OptParams&, const SyncArgs&, int);
template int sync_split<Sync::CPDP, Opt::ADAMW, ParamF32, false, ParamF32, ParamF32, DirectScalars>(
    const DirectScalars&, const SyncArgs&);
} }
"""


@pytest.fixture(scope="module")
def usage(tmp_path_factory):
    """{kernel name: (vector registers, wavefronts a SIMD, scratch bytes)}"""
    if not os.path.exists(build.HIPCC):
        pytest.skip("needs hipcc")
    d = tmp_path_factory.mktemp("regs")
    src = d / "unit.hip"
    src.write_text(UNIT)
    csrc = os.path.join(build.PKG, "csrc")
    r = subprocess.run([build.HIPCC, *build.COMPILE_FLAGS, "-I", csrc, "--cuda-device-only",
                        "-Rpass-analysis=kernel-resource-usage", "-c", "-o", str(d / "unit.o"),
                        str(src)], capture_output=True, text=True)
    assert r.returncode == 0, r.stderr
    out, name = {}, None
    for line in r.stderr.splitlines():
        m = re.search(r"remark: .*?(Function Name|VGPRs|ScratchSize \[bytes/lane\]|"
                      r"Occupancy \[waves/SIMD\]): (\S+)", line)
        if m and m[1] == "Function Name":
            name = m[2]
            out[name] = {}
        elif m and name:
            out[name][m[1].split()[0]] = int(m[2])
    return {k: (v["VGPRs"], v["Occupancy"], v["ScratchSize"]) for k, v in out.items()}


def _kernel(usage, *parts):
    names = [n for n in usage if all(p in n for p in parts)]
    assert len(names) == 1, (parts, sorted(usage))
    return usage[names[0]]


# the compiler's names: 11sync_kernel, then the template arguments
@pytest.mark.parametrize("opt,wt,waves", [("OptE0", "ELi0E", 6), ("OptE2", "ELi0E", 4),
                                          ("OptE0", "ELi16E", 3)])
def test_wavefronts_of_the_thread_per_coordinate_kernel(usage, opt, wt, waves):
    vgprs, occupancy, scratch = _kernel(usage, "11sync_kernel", opt, wt)
    assert scratch == 0
    assert occupancy >= waves, f"{vgprs} registers: {occupancy} wavefronts a SIMD"


def test_two_split_blocks_a_cu(usage):
    """AdamW above 16 replicas: two replicas a group, 16 wavefronts a block, and
    a CU holds 32 wavefronts."""
    vgprs, occupancy, scratch = _kernel(usage, "17sync_split_kernel", "OptE2", "ELi2E")
    assert scratch == 0 and occupancy == 8, f"{vgprs} registers: {occupancy} wavefronts a SIMD"
