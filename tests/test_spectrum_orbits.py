"""The shell-spectrum kernel's walk over row orbits, replayed on the host.

A workgroup owns one window of 64 shells on one plane pair +-kz; its eight waves
share the window's row orbits (+-ky, +-kz), wave r taking ky = r, r + 8, ... up to
ny/2, and a wave reads the kx range of an orbit whose shells fall in the window in
chunks of 64 modes.  This replays the walk with the kernel's integer formulas and
checks that every stored mode is visited exactly once, through one row of one orbit,
by the window that holds its shell, and that the shells of a chunk never decrease
along the lanes (what the segmented scan relies on).
"""
import numpy as np
import pytest

ROWS, WIN, LANES = 8, 64, 64


def isqrt24(n):
    """The kernel's root: a float root settled in integers."""
    r = int(np.float32(np.sqrt(np.float32(n))))
    r -= r * r > n
    r += (r + 1) * (r + 1) <= n
    return r


def test_roots_are_exact():
    """floor(sqrt(n)) for n < 2^24, vectorised over all of them."""
    n = np.arange(1 << 24, dtype=np.int64)
    r = np.sqrt(n.astype(np.float32)).astype(np.int64)
    r -= r * r > n
    r += (r + 1) * (r + 1) <= n
    assert (r * r <= n).all() and ((r + 1) * (r + 1) > n).all()
    assert [isqrt24(k) for k in (0, 1, 3, 4, 16777215)] == [0, 1, 1, 2, 4095]


def shell_of_k2(k2):
    return (isqrt24(4 * k2) + 1) >> 1


def walk(ny, H, nshell, plane, win, wave):
    """(iy, base, kx1) of the wave's chunks, as the kernel's advance() makes them."""
    s0, s1 = WIN * win, min(WIN * win + WIN - 1, nshell - 1)
    lo2, hi2 = (2 * s0 - 1) ** 2, (2 * s1 + 1) ** 2
    iy, base, kx1 = wave - ROWS, 0, -1
    while True:
        base += LANES
        while base > kx1:
            iy += ROWS
            if 2 * iy > ny:
                return
            A4 = 4 * (iy * iy + plane * plane)
            if A4 >= hi2:
                return
            base = (isqrt24(lo2 - A4 - 1) + 2) // 2 if s0 > 0 and lo2 - A4 > 0 else 0
            kx1 = min(isqrt24(hi2 - A4 - 1) // 2, H - 1)
        yield iy, base, kx1


@pytest.mark.parametrize("grid", [(16, 16, 16), (12, 24, 16), (8, 8, 8), (128, 128, 8), (256, 16, 8), (8, 192, 96)])
def test_every_mode_once(grid):
    nx, ny, nz = grid
    H = nx // 2 + 1
    nshell = shell_of_k2((nx // 2) ** 2 + (ny // 2) ** 2 + (nz // 2) ** 2) + 1
    seen = np.zeros((nz, ny, H), np.int32)
    for plane in range(nz // 2 + 1):
        two_z = plane > 0 and 2 * plane < nz
        for win in range((nshell + WIN - 1) // WIN):
            for wave in range(ROWS):
                for iy, base, kx1 in walk(ny, H, nshell, plane, win, wave):
                    kx = np.arange(base, min(base + LANES, kx1 + 1))
                    shells = [shell_of_k2(int(k) ** 2 + iy * iy + plane * plane) for k in kx]
                    assert shells and shells == sorted(shells)
                    assert WIN * win <= shells[0] and shells[-1] < min(WIN * (win + 1), nshell)
                    two_y = iy > 0 and 2 * iy < ny
                    for r in range(4):
                        if ((r >> 1) == 0 or two_z) and ((r & 1) == 0 or two_y):
                            z = (nz - plane) if r >> 1 else plane
                            y = (ny - iy) if r & 1 else iy
                            seen[z, y, kx] += 1
    assert (seen == 1).all(), (grid, int(seen.min()), int(seen.max()))
