"""Binning at the sizes where the sort's tiles change (one tile less one key,
one tile, one more, several, several prefix steps per thread), with few, many
and far more cells than particles, all particles in one cell, and each number
of passes: tables and permutation exactly as a stable sort has them."""
import numpy as np
import pytest

from paper_2512_05516_amd import inputs

from test_gpu_parity import sph  # noqa: F401

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n", [1, 63, 8191, 8192, 8193, 16385, 100003, 600001])
# keys of 5, 12, 15, 18 and 24 bits: one, two and three passes, 8- and 9-bit digits
@pytest.mark.parametrize("n_c,bits", [(3, 0), (16, 0), (5, 3), (64, 0), (63, 2)])
@pytest.mark.parametrize("crowd", [False, True])
def test_bin_sizes(sph, n, n_c, bits, crowd):  # noqa: F811
    import torch
    rng = np.random.default_rng(n + n_c)
    x = rng.uniform(0, 1, (n, 3))
    if crowd:       # nine of ten in one cell's corner
        x[: n * 9 // 10] = 0.5 + 1e-3 * x[: n * 9 // 10] / n_c
    h = rng.uniform(0.1, 1.0, n).astype(np.float32)
    h[rng.random(n) < 0.1] = 0.0
    ps = inputs.ParticleSet(x, np.zeros_like(x), np.ones(n), h.astype(np.float64), np.ones(n))
    cells = sph.DeviceCells(n, n_c, "cuda", sub_bits=bits)
    aos = torch.from_numpy(inputs.pack_aos(ps, "f32").view(np.uint8).reshape(-1).copy()).cuda()
    ws = torch.empty(sph.bin_workspace_size(n, n_c), dtype=torch.uint8, device="cuda")
    sph.bin(aos, sph.layout_from_dtype(inputs.AOS_F32), cells, ws)
    torch.cuda.synchronize()
    R = 1 << bits
    c = np.minimum(np.floor(x * n_c).astype(np.int64), n_c - 1)
    s = np.clip(np.floor(x * (n_c * R)).astype(np.int64) - c * R, 0, R - 1)
    cell = c[:, 0] + n_c * (c[:, 1] + n_c * c[:, 2])
    sub = np.zeros(n, np.int64)
    for b in range(bits):
        for a in range(3):
            sub |= ((s[:, a] >> b) & 1) << (3 * b + a)
    key = cell * R ** 3 + sub
    perm = np.argsort(key, kind="stable")
    C = n_c ** 3
    assert np.array_equal(cells.perm[:n].cpu().numpy(), perm)
    assert np.array_equal(cells.cell[:n].cpu().numpy(), cell[perm])
    assert np.array_equal(cells.cell_start.cpu().numpy(),
                          np.searchsorted(cell[perm], np.arange(C + 1)))
    if bits:
        assert np.array_equal(cells.sub_start.cpu().numpy(),
                              np.searchsorted(key[perm], np.arange(C * R ** 3 + 1)))
    hmax = np.zeros(C, np.float32)
    np.maximum.at(hmax, cell, h)
    assert np.array_equal(cells.hmax.cpu().numpy(), hmax)
