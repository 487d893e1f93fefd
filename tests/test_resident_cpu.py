"""The number of workgroups per CU that a launch with a grid barrier may count
on (csrc/resident.h), compiled for the host."""
import ctypes
import os
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


@pytest.fixture(scope="module")
def resident(tmp_path_factory):
    cxx = shutil.which("g++") or shutil.which("c++")
    if not cxx:
        pytest.skip("no host compiler")
    d = tmp_path_factory.mktemp("resident")
    src, lib = d / "r.cpp", d / "libr.so"
    src.write_text('#include "resident.h"\n'
                   'extern "C" int f(int o, int w, int r) { return evlb::resident_per_cu(o, w, r); }\n')
    subprocess.run([cxx, "-std=c++17", "-shared", "-fPIC", "-I", os.path.join(ROOT, "paper_2503_15187_amd", "csrc"),
                    "-o", str(lib), str(src)], check=True)
    return ctypes.CDLL(str(lib)).f


def worst_case(wavefronts, slots):
    """Workgroups that surely fit four SIMDs of `slots` each, when a workgroup's
    wavefronts go round the SIMDs from any start: the smallest number placed,
    over all starts, before one does not fit."""
    best = 99
    todo = [((0, 0, 0, 0), 0)]
    seen = set(todo)
    while todo:
        load, n = todo.pop()
        for s in range(4):
            new = tuple(load[i] + (wavefronts + (3 - (i - s) % 4)) // 4 for i in range(4))
            if max(new) > slots:
                best = min(best, n)
            elif (new, n + 1) not in seen:
                seen.add((new, n + 1))
                todo.append((new, n + 1))
    return best


@pytest.mark.parametrize("wavefronts", [1, 4, 5, 6, 7, 8, 9, 10, 11, 12, 13, 14, 15, 16])
@pytest.mark.parametrize("registers", [64, 66, 72, 96, 120, 122, 128, 158, 168, 211, 255])
def test_never_more_than_any_placement_holds(resident, wavefronts, registers):
    slots = min(8, 512 // (8 * ((registers + 7) // 8)))
    occupancy = 4 * slots // wavefronts  # what the occupancy query counts
    got = resident(occupancy, wavefronts, registers)
    assert got <= occupancy
    if wavefronts == 1:
        assert got == occupancy
    elif occupancy and worst_case(wavefronts, slots):
        assert 1 <= got <= worst_case(wavefronts, slots)


def test_six_wavefronts_at_three_slots(resident):
    """Two workgroups of six wavefronts at 158 registers: twelve slots in sum,
    not in every placement."""
    assert resident(2, 6, 158) == 1
    assert resident(2, 6, 120) == 2
    assert resident(1, 12, 120) == 1
    assert resident(2, 8, 122) == 2
