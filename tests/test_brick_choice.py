"""The choice between the brick and the tiled update (host code, no GPU),
compiled from the library's own header: no grid is given to the brick kernel
that its launch refuses, however narrow or large."""
import os
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
THREADS = 704  # of a brick's block; HIP takes fewer than 2^32 threads along an axis of a launch


@pytest.fixture(scope="module")
def choose(tmp_path_factory):
    hipcc = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")
    if not os.path.exists(hipcc) and not shutil.which("hipcc"):
        pytest.skip("hipcc not available")
    exe = str(tmp_path_factory.mktemp("brick") / "brick_check")
    subprocess.check_call([hipcc, "--cuda-host-only", "-x", "hip", "-std=c++20", "-O1",
                           "-I", os.path.join(ROOT, "paper_2401_17074_amd", "csrc"),
                           os.path.join(ROOT, "tests", "brick_check.cpp"), "-o", exe],
                          stderr=subprocess.DEVNULL)

    def run(grids):
        r = subprocess.run([exe] + [str(v) for g in grids for v in g], capture_output=True, text=True, timeout=120)
        assert r.returncode == 0
        return [list(map(int, ln.split())) for ln in r.stdout.strip().splitlines()]
    return run


def test_never_more_bricks_than_a_launch_takes(choose):
    grids = [(nx, ny, nz) for nx in (1, 3, 16, 17, 48) for ny in (1, 2, 4, 15, 2048, 16384)
             for nz in (1, 3, 64, 16400, 4 << 20, 24_800_000, 100_000_000) if nx * ny * nz < 1 << 30]
    grids += [(300_000_000, 1, 3), (1 << 28, 1, 3), (1, 1, (1 << 30) - 1)]
    rows = choose(grids)
    assert len(rows) == len(grids) and any(r[4] for r in rows) and any(r[3] * THREADS >= 1 << 32 for r in rows)
    for nx, ny, nz, bricks, chosen, chosen16 in rows:
        assert not chosen or (bricks + 7) // 8 * 8 * THREADS < 1 << 32, (nx, ny, nz, bricks)
        assert not chosen16


def test_small_grids_in_bricks(choose):
    for r in choose([(16, 16, 16), (24, 24, 24), (32, 32, 32), (40, 40, 40), (48, 48, 48), (16, 90, 90), (1, 1, 1)]):
        assert r[4], r
    for r in choose([(64, 64, 64), (96, 96, 96), (256, 256, 256), (384, 192, 192)]):
        assert not r[4], r


def test_narrow_grids_by_time(choose):
    """Bricks only where they were measured to be no slower than the tiles."""
    for r in choose([(16, 4, 262144), (3, 3, 1 << 20), (8, 500, 500), (17, 100, 100), (16, 200, 256), (64, 4, 1024)]):
        assert r[4], r
    for r in choose([(64, 4, 4096), (64, 4, 12000), (64, 1, 16384), (48, 4, 12000), (128, 4, 4096), (512, 4, 1024),
                     (52, 52, 52), (64, 4, 65536)]):
        assert not r[4], r
