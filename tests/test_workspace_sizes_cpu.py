"""The sizes that the library asks for hold what it uses, and no more than
alignment beside it."""
import pytest


@pytest.fixture(scope="module")
def sph():
    from paper_2512_05516_amd import sphmi
    sphmi.lib()
    return sphmi


@pytest.mark.parametrize("n", [0, 1, 8192, 8193, 100003, 4194304])
def test_bin_workspace(sph, n):
    # four arrays of keys and values, h, and 512 counts for each 8192 keys
    use = 5 * 4 * n + 4 * 512 * max(-(-n // 8192), 1)
    assert use <= sph.bin_workspace_size(n, 16) <= use + 6 * 256


@pytest.mark.parametrize("n,n_c,ti", [(16, 4, 64), (100003, 16, 32), (4194304, 66, 64), (50, 200, 16)])
def test_worklist(sph, n, n_c, ti):
    # header, two prefixes over the cells, items
    cells = n_c ** 3
    use = 256 + 2 * 4 * (cells + 1) + 8 * ((n + (ti - 1) * min(cells, n)) // ti + 1)
    assert use - 256 <= sph.worklist_size(n, n_c, ti) <= use + 3 * 256
