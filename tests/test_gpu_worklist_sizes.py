"""Work lists at the numbers of cells where their blocks change: one block,
cells of a block's end, many blocks, several rounds of cells per block.
Items and range boundaries as an independent rebuild on the host has them."""
import numpy as np
import pytest

from paper_2512_05516_amd import inputs

from test_gpu_parity import _read_worklist, _worklist_reference, sph  # noqa: F401

pytestmark = pytest.mark.gpu


# cells: 27, 216, 343 (blocks of 256), 4096, 32768, 274625 (1024 blocks and more: two rounds)
@pytest.mark.parametrize("n_c", [3, 6, 7, 16, 32, 65])
@pytest.mark.parametrize("merge,occ", [(1, (0, 2 ** 31 - 1)), (4, (0, 40)), (1, (10 ** 6, 2 ** 31 - 1))])
def test_worklist_cell_counts(sph, n_c, merge, occ):  # noqa: F811
    import torch
    ps = inputs.clustered_set(20000, 5, f_blob=0.5, sigma=0.05)
    cells = sph.DeviceCells(ps.n, n_c, "cuda")
    aos = torch.from_numpy(inputs.pack_aos(ps, "f32").view(np.uint8).reshape(-1).copy()).cuda()
    ws = torch.empty(sph.bin_workspace_size(ps.n, n_c), dtype=torch.uint8, device="cuda")
    sph.bin(aos, sph.layout_from_dtype(inputs.AOS_F32), cells, ws)
    w = sph.DeviceWork(ps.n, n_c, 64, "cuda", "grid", max_cells=merge)
    sph.worklist(cells, w, None, occ)
    torch.cuda.synchronize()
    items_ref, bounds_ref = _worklist_reference(cells.cell_start.cpu().numpy(), ps.n, n_c, 64,
                                                merge, occ)
    items, meta, _ = _read_worklist(w, ps.n, n_c)
    assert meta[0] == len(items_ref)
    assert np.array_equal(items, items_ref)
    assert np.array_equal(meta[1:10], bounds_ref)
