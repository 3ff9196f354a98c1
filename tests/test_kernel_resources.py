"""Registers and scratch memory of the throughput sweep kernels (one lane per sample), read from the
library built here: what a lane spills is stored and loaded once per sample whatever the horizon,
and short horizons show it."""

import os
import re
import shutil
import subprocess

import pytest

import paper_2607_25388_amd.sgtp as sg

LLVM = "/opt/rocm/llvm/bin/"


@pytest.fixture(scope="module")
def kernels(tmp_path_factory):
    """(model, discs, opponents) -> (VGPRs, scratch bytes a lane) of k_sweep's throughput variants, and
    with a fourth entry 5 of k_sweep5's."""
    if not os.path.exists(sg.LIB_PATH) or not os.path.exists(LLVM + "llvm-readelf"):
        pytest.skip("library not built, or no reader of its notes")
    d = tmp_path_factory.mktemp("resources")
    subprocess.run([LLVM + "llvm-objdump", "--offloading", shutil.copy(sg.LIB_PATH, d)], cwd=d, check=True,
                   stdout=subprocess.DEVNULL)
    out = {}
    for f in sorted(d.glob("*gfx950*")):
        notes = subprocess.run([LLVM + "llvm-readelf", "--notes", str(f)], check=True, text=True,
                               stdout=subprocess.PIPE).stdout
        for block in notes.split("- .agpr_count")[1:]:
            name = re.search(r"\.name:\s+(\S+)", block)[1]
            m = re.search(r"k_sweepILi(\d)ELi(\d)ELi(\d+)ELi0ELi1ELi0E", name)
            m5 = re.search(r"k_sweep5ILi(\d)ELi(\d)ELi(\d+)E", name)
            if m or m5:
                out[tuple(map(int, (m or m5).groups())) + ((5,) if m5 else ())] = tuple(
                    int(re.search(rf"\.{k}:\s+(\d+)", block)[1]) for k in ("vgpr_count", "private_segment_fixed_size"))
    assert len(out) == 18
    return out


def test_dynamic_model_spills_nothing(kernels):
    """Up to nine opponents; with fifteen their distances alone fill the registers' rest."""
    for (model, discs, opp, *five), (vgprs, scratch) in kernels.items():
        if model == 0 and opp <= 9:
            assert vgprs <= 128 and scratch == 0, (discs, opp, vgprs, scratch)


def test_five_workgroups_per_cu(kernels):
    """512 registers a SIMD: 96 each in steps of 8; one value spilled around the sample loop at most."""
    for opp in (1, 3):
        vgprs, scratch = kernels[1, 1, opp, 5]
        assert vgprs <= 96 and scratch <= 8, (opp, vgprs, scratch)
