"""Line passes are taken only where each launch holds fewer than 2^32 threads (no GPU)."""
import os
import subprocess

from paper_1907_12834_amd.build import CSRC, hipcc

HERE = os.path.dirname(os.path.abspath(__file__))


def _windows(n, lines):
    if n == 1:
        return -(-lines // 56)
    slots = min(n + 8, -(-n // 56) * 56)
    return -(-(lines * slots - 8) // 56)


def _threads(n, planes, nx, cols):
    """A launch along y or z: one window of `cols` columns per workgroup, a wavefront per column."""
    slots = planes * (1 if n == 1 else min(n + 8, -(-n // 56) * 56))
    fold = (56 // planes if planes <= 28 else 1) if n == 1 else 64 // slots if slots <= 32 else 1
    return -(-(-(-nx // cols)) // fold) * _windows(n, planes * fold) * 64 * cols


def test_launches_of_line_passes(tmp_path):
    exe = str(tmp_path / "launch_limits")
    subprocess.run([hipcc(), "-x", "hip", "--offload-host-only", "-O1", "-std=c++17", "-I", CSRC,
                    os.path.join(HERE, "host", "launch_limits.cpp"), "-o", exe], check=True)
    # sites, and the threads of columns that a narrow lattice does not have, around the limit
    shapes = [(64, 64, 1), (256, 256, 256), (1, 24000, 24000), (1, 21000, 21000), (1, 15000, 15000), (3, 12000, 12000),
              (8, 9000, 9000), (1, 4, 60000000), (1, 2, 70000000), (40000, 8, 1), (300000, 1, 1), (600, 600, 600)]
    cases = [s + (c,) for s in shapes for c in (4, 8)]
    out = subprocess.run([exe], input="\n".join("%d %d %d %d" % c for c in cases), text=True, capture_output=True, check=True)
    rows = [tuple(map(int, l.split())) for l in out.stdout.splitlines()]
    assert len(rows) == len(cases)
    verdicts = []
    for (nx, ny, nz, cols), (gx, gy, gz, fits) in zip(cases, rows):
        threads = [-(-_windows(nx, ny * nz) // 8) * 512, _threads(ny, nz, nx, cols), _threads(nz, ny, nx, cols)]
        assert [gx * 512, gy * 64 * cols, gz * 64 * cols] == threads, (nx, ny, nz, cols)
        verdicts.append(bool(fits))
        assert verdicts[-1] == (max(threads) < 2 ** 32), (nx, ny, nz, cols)
    assert True in verdicts and False in verdicts
