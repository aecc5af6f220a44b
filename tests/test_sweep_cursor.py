"""Host check (no GPU): the matrix-core stencil steps through a lattice in pairs of sites by carries
and keeps inputs from pair to pair; every site comes once and its neighbours are those found from
coordinates, for ranges that start anywhere in a row, rows of one pair up, and bricks smaller and larger
than a wave's range or of odd height."""
import os
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
BUILD = os.path.join(ROOT, "paper_1405_4524_amd", "_build")


@pytest.fixture(scope="module")
def exe(tmp_path_factory):
    hipcc = shutil.which("hipcc") or "/opt/rocm/bin/hipcc"
    if not os.path.exists(hipcc) or not os.path.exists(os.path.join(BUILD, "liba2a.so")):
        pytest.skip("hipcc or the built library is missing")
    out = str(tmp_path_factory.mktemp("sweep") / "sweep_check")
    subprocess.check_call([hipcc, "-x", "hip", "--offload-arch=gfx950", "-O1", "-std=c++17",
                           os.path.join(ROOT, "tests", "sweep_check.cpp"), "-L", BUILD, "-la2a",
                           "-Wl,-rpath," + BUILD, "-o", out], stderr=subprocess.DEVNULL)
    return out


@pytest.mark.parametrize("dims", [(2, 2, 2, 2), (4, 2, 6, 4), (6, 4, 4, 10), (10, 6, 14, 6), (8, 8, 8, 16), (34, 4, 2, 6),
                                  (32, 8, 8, 8)])
@pytest.mark.parametrize("brick", [(0, 0, 0), (1, 1, 1), (2, 1, 2)])
def test_pair_cursor_finds_every_neighbour(exe, dims, brick):
    for nsub in (1, 4, 16):
        r = subprocess.run([exe, *map(str, dims), *map(str, brick), str(nsub)], capture_output=True, text=True)
        assert r.returncode == 0 and r.stdout.strip() == "ok", (nsub, r.stdout)
