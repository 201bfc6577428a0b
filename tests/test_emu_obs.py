"""The observables' tiles and final sums (lbm_obs.h), checked on the CPU (no GPU) by
tests/emu/obs_emu.cpp: every workgroup on host threads with NaN in every slot that is not state and
in the LDS before each tile, under AddressSanitizer and UndefinedBehaviorSanitizer; every partial row
must equal, bit for bit, the sums of the per-node values formed through fields of the lattice. Both
block heights, post- and pre-collision populations, every geometry, lattices narrower than a block
and around its edges; a copy of the header with a planted mistake must fail."""
import os
import shutil
import subprocess

import pytest

HERE = os.path.dirname(os.path.abspath(__file__))
SRC = os.path.join(HERE, "emu", "obs_emu.cpp")
CSRC = os.path.join(os.path.dirname(HERE), "paper_1410_2569_amd", "csrc")
CXX = os.environ.get("CXX_EMU", "/opt/rocm/llvm/bin/clang++")

pytestmark = pytest.mark.skipif(not shutil.which(CXX), reason=f"{CXX} not available")

# nx ny walls ghost eos wall_force, rows per block
CASES = [("65 12 1 1 0 2", 8), ("65 12 1 1 0 2", 4), ("63 9 0 1 0 0", 8), ("66 9 2 1 1 2", 4),
         ("9 5 2 0 0 1", 8), ("64 8 1 0 1 1", 4), ("3 4 1 1 0 0", 8), ("70 9 3 0 0 2", 8),
         ("40 7 3 0 1 0", 4)]


def _build(out, *extra):
    subprocess.check_call([CXX, "-std=c++20", "-O1", "-g", "-pthread", "-w", "-ffp-contract=off",
                           "-I", os.path.join(HERE, "emu"), *extra, SRC, "-o", out])
    return out


def _run(exe, lattice, pre, rows):
    return subprocess.run([exe, *lattice.split(), str(pre), str(rows)], capture_output=True,
                          text=True, timeout=300, env=dict(os.environ, ASAN_OPTIONS="detect_leaks=0"))


@pytest.fixture(scope="module")
def emulator(tmp_path_factory):
    return _build(str(tmp_path_factory.mktemp("obs") / "obs_emu"),
                  "-fsanitize=address,undefined", "-fno-sanitize-recover=all")


@pytest.mark.parametrize("lattice,rows", CASES)
def test_tiles_equal_the_sums_of_the_nodes(emulator, lattice, rows):
    r = _run(emulator, lattice, 0, rows)
    assert r.returncode == 0 and "ok: 0 differ" in r.stdout, (r.stdout[-2000:], r.stderr[-2000:])


@pytest.mark.parametrize("lattice,rows", [("40 11 2 1 1 2", 8), ("63 6 0 1 0 0", 4)])
def test_held_populations(emulator, lattice, rows):
    r = _run(emulator, lattice, 1, rows)
    assert r.returncode == 0 and "ok: 0 differ" in r.stdout, (r.stdout[-2000:], r.stderr[-2000:])


@pytest.mark.parametrize("old,new", [
    ("{ lx = h - LW; ly = ROWS + 1; }", "{ lx = h - LW; ly = ROWS; }"),
    ("L.rho[l + 1], L.rho[l + LW], v);", "L.rho[l + 1], L.rho[l + 2 * LW], v);"),
    ("(q == O_BAD && bad)", "(q == O_BAD && fit)"),
    ("for (int b = threadIdx.x; b < nblk; b += 256)", "for (int b = threadIdx.x; b < 256; b += 256)"),
], ids=["ring_top", "upper_neighbour", "bad_count", "final"])
def test_emulator_catches_planted_mistakes(tmp_path, old, new):
    src = open(os.path.join(CSRC, "lbm_obs.h")).read()
    assert src.count(old) == 1, old
    hdr = tmp_path / "lbm_obs.h"
    hdr.write_text(src.replace(old, new).replace('#include "lbm_device.h"',
                                                 f'#include "{CSRC}/lbm_device.h"'))
    exe = _build(str(tmp_path / "mutant"), f'-DLBM_OBS_HEADER="{hdr}"', "-fsanitize=address")
    r = _run(exe, "20 13 1 1 0 2", 0, 8)
    assert r.returncode != 0, r.stdout
