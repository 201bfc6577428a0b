"""Index maps of the multi-step tiles (lbm_steps.h), checked on the CPU (no GPU) by
tests/emu/steps_emu.cpp: every workgroup on host threads with NaN in every slot that is not state
and in the LDS before each tile, under AddressSanitizer and UndefinedBehaviorSanitizer; the steps
of one launch must equal single steps of every node bit for bit. Every tile and geometry, lattices
smaller than the halo; a copy of the header with a planted mistake must fail."""
import os
import shutil
import subprocess

import pytest

HERE = os.path.dirname(os.path.abspath(__file__))
SRC = os.path.join(HERE, "emu", "steps_emu.cpp")
CSRC = os.path.join(os.path.dirname(HERE), "paper_1410_2569_amd", "csrc")
CXX = os.environ.get("CXX_EMU", "/opt/rocm/llvm/bin/clang++")

pytestmark = pytest.mark.skipif(not shutil.which(CXX), reason=f"{CXX} not available")

# nx ny walls ghost eos wall_force
LATTICES = ["33 19 1 1 0 2", "17 14 0 1 0 0", "31 12 2 1 1 2", "9 4 2 0 0 1", "40 21 3 0 1 2",
            "5 5 0 1 0 0"]


def _build(out, *extra):
    subprocess.check_call([CXX, "-std=c++20", "-O1", "-g", "-pthread", "-w", "-ffp-contract=off",
                           "-I", os.path.join(HERE, "emu"), *extra, SRC, "-o", out])
    return out


def _run(exe, lattice, tile):
    return subprocess.run([exe, *lattice.split(), str(tile)], capture_output=True, text=True,
                          timeout=300, env=dict(os.environ, ASAN_OPTIONS="detect_leaks=0"))


@pytest.fixture(scope="module")
def emulator(tmp_path_factory):
    return _build(str(tmp_path_factory.mktemp("steps") / "steps_emu"),
                  "-fsanitize=address,undefined", "-fno-sanitize-recover=all")


@pytest.mark.parametrize("tile", [0, 1, 2])
@pytest.mark.parametrize("lattice", LATTICES)
def test_multi_step_equals_single_steps(emulator, lattice, tile):
    r = _run(emulator, lattice, tile)
    assert r.returncode == 0 and "ok: 0 of" in r.stdout, (r.stdout[-2000:], r.stderr[-2000:])


@pytest.mark.parametrize("old,new", [
    ("h < NRING; h += NT", "h < NRING - 1; h += NT"),
    ("const int row = P.walls ? sy - (y0 - R - 2) : ly + 2;", "const int row = ly + 2;"),
    ("static constexpr int w(int k) { return TX + 4 * (N - k); }",
     "static constexpr int w(int k) { return TX + 4 * (N - k) - (k == 2); }"),
], ids=["ring", "ghost_row", "width"])
def test_emulator_catches_planted_mistakes(tmp_path, old, new):
    src = open(os.path.join(CSRC, "lbm_steps.h")).read()
    assert src.count(old) == 1, old
    hdr = tmp_path / "lbm_steps.h"
    hdr.write_text(src.replace(old, new).replace('#include "lbm_device.h"',
                                                 f'#include "{CSRC}/lbm_device.h"'))
    exe = _build(str(tmp_path / "mutant"), f'-DLBM_STEPS_HEADER="{hdr}"')
    r = _run(exe, "33 19 1 1 0 2", 0)
    assert r.returncode != 0, r.stdout
