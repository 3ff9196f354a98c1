"""The waves of a workgroup hand controls and states over through LDS slots and progress counters,
without a fence between a slot and its counter (small launches).  That holds for DS instructions,
which are carried out in the order in which a wave issues them, and not for FLAT ones.  The
counters are the only volatile (sc0 sc1) accesses of the sweep and set-up kernels, so no FLAT
instruction with these bits may be left in their listings, in the library built here."""

import os
import re
import shutil
import subprocess

import pytest

import paper_2607_25388_amd.sgtp as sg

OBJDUMP = "/opt/rocm/llvm/bin/llvm-objdump"


@pytest.fixture(scope="module")
def listing(tmp_path_factory):
    if not os.path.exists(sg.LIB_PATH) or not os.path.exists(OBJDUMP):
        pytest.skip("library not built, or no disassembler")
    d = tmp_path_factory.mktemp("listing")
    lib = shutil.copy(sg.LIB_PATH, d)
    subprocess.run([OBJDUMP, "--offloading", lib], cwd=d, check=True, stdout=subprocess.DEVNULL)
    kernels = {}
    for f in sorted(d.glob("*gfx950*")):
        out = subprocess.run([OBJDUMP, "-d", "--no-show-raw-insn", str(f)], check=True, text=True,
                             stdout=subprocess.PIPE).stdout
        for name, body in re.findall(r"^[0-9a-f]+ <(\w+)>:\n((?:[^\n]+\n)+)", out, re.M):
            kernels[name] = body
    return kernels


def test_counters_are_ds_accesses(listing):
    sweeps = {k: v for k, v in listing.items() if "k_sweep" in k or "k_setup" in k}
    teams = [k for k in sweeps if re.search(r"k_sweepILi\dELi\dELi\d+ELi6ELi1ELi1E", k)]
    assert len(sweeps) > 40 and len(teams) == 16  # models x discs x opponent tables
    for name, body in sweeps.items():
        flat = re.findall(r"\tflat_\w+ [^\n]*sc0 sc1", body)
        assert not flat, (name, len(flat), flat[:2])
        assert "ds_write_b32" in body and "ds_read_b32" in body
