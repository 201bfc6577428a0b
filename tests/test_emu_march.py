"""Index maps and wave-level data flow of the marching strips (lbm_march.h), checked on the CPU
(no GPU) by tests/emu/march_emu.cpp: a wave of 64 host threads with NaN in every slot that is not
state and at both ends of the cross-lane moves, under AddressSanitizer and UndefinedBehaviorSanitizer;
the steps of one launch must equal single steps of every node bit for bit. Lattices narrower than
the halo, ragged strips and segments of one to all rows, every geometry that marches; a copy of
the header with a planted mistake must fail."""
import os
import shutil
import subprocess

import pytest

HERE = os.path.dirname(os.path.abspath(__file__))
SRC = os.path.join(HERE, "emu", "march_emu.cpp")
CSRC = os.path.join(os.path.dirname(HERE), "paper_1410_2569_amd", "csrc")
CXX = os.environ.get("CXX_EMU", "/opt/rocm/llvm/bin/clang++")

pytestmark = pytest.mark.skipif(not shutil.which(CXX), reason=f"{CXX} not available")

# nx ny walls ghost eos wall_force
LATTICES = ["70 24 1 1 0 2", "130 17 0 1 0 0", "64 9 1 0 1 1", "101 12 2 1 1 2", "5 5 0 0 0 0",
            "109 16 2 0 0 1"]


def _build(out, *extra):
    subprocess.check_call([CXX, "-std=c++20", "-O1", "-g", "-pthread", "-w", "-ffp-contract=off",
                           "-I", os.path.join(HERE, "emu"), *extra, SRC, "-o", out])
    return out


def _run(exe, lattice, rows):
    return subprocess.run([exe, *lattice.split(), "3", str(rows)], capture_output=True, text=True,
                          timeout=300, env=dict(os.environ, ASAN_OPTIONS="detect_leaks=0"))


@pytest.fixture(scope="module")
def emulator(tmp_path_factory):
    return _build(str(tmp_path_factory.mktemp("march") / "march_emu"),
                  "-fsanitize=address,undefined", "-fno-sanitize-recover=all")


@pytest.mark.parametrize("rows", [1, 6, 100])
@pytest.mark.parametrize("lattice", LATTICES)
def test_marching_equals_single_steps(emulator, lattice, rows):
    r = _run(emulator, lattice, rows)
    assert r.returncode == 0 and "ok: 0 of" in r.stdout, (r.stdout[-2000:], r.stderr[-2000:])


@pytest.mark.parametrize("old,new", [
    ("f[8] = X::left(s[8]);", "f[8] = X::right(s[8]);"),
    ("M.a[0] = b ? s[4] : M.up[0];", "M.a[0] = M.up[0];"),
    ("constexpr int H = 2 * T - 1;", "constexpr int H = 2 * T - 2;"),
], ids=["lane", "wall", "halo"])
def test_emulator_catches_planted_mistakes(tmp_path, old, new):
    src = open(os.path.join(CSRC, "lbm_march.h")).read()
    assert src.count(old) == 1, old
    hdr = tmp_path / "lbm_march.h"
    hdr.write_text(src.replace(old, new).replace('#include "lbm_device.h"',
                                                 f'#include "{CSRC}/lbm_device.h"'))
    exe = _build(str(tmp_path / "mutant"), f'-DLBM_MARCH_HEADER="{hdr}"')
    r = _run(exe, "70 24 1 1 0 2", 6)
    assert r.returncode != 0 and "FAIL" in r.stdout, r.stdout
