"""The key-owning attention launch off the 32-grid (csrc/unit_grid.h, built with g++): the units' blocks of rows and the gate gradients' workgroups
behind them, at the bound of 65535 units too, where a dimension that both share ends for y and z."""
import ctypes
import os
import re
import subprocess

import pytest

CSRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_2503_02495_amd", "csrc")
SHIM = """
#include "unit_grid.h"
extern "C" unsigned workgroups(int rows, int units, int behind) { return uoe::UnitGrid{rows, units, behind}.workgroups(); }
extern "C" unsigned own(int rows, int units, int behind) { return uoe::UnitGrid{rows, units, behind}.own(); }
extern "C" int unit(int rows, int units, int behind, unsigned id) { return uoe::UnitGrid{rows, units, behind}.unit(id); }
extern "C" int block(int rows, int units, int behind, unsigned id) { return uoe::UnitGrid{rows, units, behind}.block(id); }
"""


@pytest.fixture(scope="module")
def shim(tmp_path_factory):
    d = tmp_path_factory.mktemp("grid")
    (d / "shim.cc").write_text(SHIM)
    subprocess.run(["g++", "-std=c++17", "-O1", "-Wall", "-Werror", "-shared", "-fPIC", "-I", CSRC, str(d / "shim.cc"), "-o", str(d / "shim.so")], check=True)
    return ctypes.CDLL(str(d / "shim.so"))


@pytest.mark.parametrize("rows,units,gates", [(1, 1, 1), (1, 65535, 65535), (2, 43691, 43691), (3, 7, 0), (7, 384, 384), (33, 2, 2)])
def test_every_block_and_every_gate_once(shim, rows, units, gates):
    own, total = shim.own(rows, units, gates), shim.workgroups(rows, units, gates)
    assert (own, total - own) == (rows * units, gates)
    assert [(shim.unit(rows, units, gates, i), shim.block(rows, units, gates, i)) for i in range(own)] == [(u, r) for u in range(units) for r in range(rows)]


def test_launched_in_one_dimension():
    with open(os.path.join(CSRC, "bwd_any.hip")) as f:
        launches = re.findall(r"hipLaunchKernelGGL\(\(attention_bwd_f32_kernel<[^>]*>\), (.*?), dim3\(KS \* 64\)", f.read())
    assert launches == ["dim3(grid.workgroups())", "dim3(grid_kv.workgroups())"]
