"""Index maps of the two-reverse-steps tile (lbm_adj2.h), checked on the CPU (no GPU) by
tests/emu/adj2_emu.cpp: every workgroup on host threads with NaN in every slot that is not written
state and in the LDS before each tile, under AddressSanitizer and UndefinedBehaviorSanitizer; every
output must hold the bits of two single reverse steps. Ragged tiles, lattices smaller than the halo,
both equations of state and all wall forces; a copy of the header with a planted mistake must fail."""
import os
import shutil
import subprocess

import pytest

HERE = os.path.dirname(os.path.abspath(__file__))
SRC = os.path.join(HERE, "emu", "adj2_emu.cpp")
CSRC = os.path.join(os.path.dirname(HERE), "paper_1410_2569_amd", "csrc")
CXX = os.environ.get("CXX_EMU", "/opt/rocm/llvm/bin/clang++")

pytestmark = pytest.mark.skipif(not shutil.which(CXX), reason=f"{CXX} not available")

# nx ny walls ghost eos wall_force
LATTICES = ["33 19 1 1 0 2", "50 30 1 0 0 0", "24 13 1 1 1 1", "31 12 0 0 1 2", "3 4 1 1 0 2",
            "16 10 1 1 0 1"]


def _build(out, *extra):
    subprocess.check_call([CXX, "-std=c++20", "-O1", "-g", "-pthread", "-w", "-ffp-contract=off",
                           "-I", os.path.join(HERE, "emu"), *extra, SRC, "-o", out])
    return out


def _run(exe, lattice):
    return subprocess.run([exe, *lattice.split()], capture_output=True, text=True, timeout=300,
                          env=dict(os.environ, ASAN_OPTIONS="detect_leaks=0"))


@pytest.fixture(scope="module")
def emulator(tmp_path_factory):
    return _build(str(tmp_path_factory.mktemp("adj2") / "adj2_emu"),
                  "-fsanitize=address,undefined", "-fno-sanitize-recover=all")


@pytest.mark.parametrize("lattice", LATTICES)
def test_two_reverse_steps_equal_single_ones(emulator, lattice):
    r = _run(emulator, lattice)
    assert r.returncode == 0 and "ok: 0 differ" in r.stdout, (r.stdout[-2000:], r.stderr[-2000:])


@pytest.mark.parametrize("old,new", [
    ("if (t2 >= 0 && t2 < 2 * (W2 + 2) + 2 * H2) {", "if (t2 >= 0 && t2 < 2 * (W2 + 2) + 2 * H2 - 1) {"),
    ("l7 = bot ? l : l - W - sx", "l7 = bot ? l : l - W + sx"),
    ("L.rv1[2][lx] = rx;", "L.rv1[2][lx] = ry;"),
], ids=["ring", "gather", "wall"])
def test_emulator_catches_planted_mistakes(tmp_path, old, new):
    src = open(os.path.join(CSRC, "lbm_adj2.h")).read()
    assert src.count(old) == 1, old
    hdr = tmp_path / "lbm_adj2.h"
    hdr.write_text(src.replace(old, new).replace('#include "lbm_device.h"',
                                                 f'#include "{CSRC}/lbm_device.h"'))
    exe = _build(str(tmp_path / "mutant"), f'-DLBM_ADJ2_HEADER="{hdr}"')
    r = _run(exe, "33 19 1 1 0 2")
    assert r.returncode != 0 and "FAIL" in r.stdout, r.stdout
