"""sph_tasks_run on tasks that no server has checked: cells that are not
neighbours have no pairs, at every task tile."""
import ctypes as C

import numpy as np
import pytest

from paper_2512_05516_amd import inputs

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def sph():
    torch = pytest.importorskip("torch")
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2512_05516_amd import sphmi
    sphmi.lib()
    return sphmi


@pytest.mark.parametrize("tile", [(64, 4), (32, 8), (16, 16)])
def test_cells_that_are_not_neighbours(sph, tile):
    import torch
    from paper_2512_05516_amd import serve
    from paper_2512_05516_amd.pipeline import Pipeline
    n, n_c = 5000, 5
    rng = np.random.default_rng(4)
    ps = inputs.ParticleSet(rng.uniform(0, 1, (n, 3)), rng.normal(0, 0.1, (n, 3)),
                            np.full(n, 1.0 / n), np.full(n, 0.9 / (n_c * sph.GAMMA_K[0])), np.ones(n))
    pipe = Pipeline(inputs.pack_aos(ps, "f32"), n_c)
    pipe.bin()
    pipe.convert("full")
    pipe.density()
    start = pipe.cells.cell_start.cpu().numpy()
    ci = 31
    a, b = int(start[ci]), int(start[ci + 1])
    k = b - a
    far, near = ci + 2, ci + 1
    tasks = np.array([(kind, ci, cj, a, b) for kind in (0, 1) for cj in (far, near)], np.int32)
    items = np.array([(t, f) for t in range(4) for f in range(a, b, tile[0])], np.int32)
    nd = int((items[:, 0] < 2).sum())
    dev = lambda v: torch.from_numpy(np.ascontiguousarray(v)).cuda()
    td, od, it = dev(tasks), dev(np.arange(4, dtype=np.int32) * k), dev(items)
    out = torch.full((4 * k * 8,), 7, dtype=torch.int32, device="cuda")
    p = lambda t: C.c_void_p(t.data_ptr())
    sph._check(sph.lib().sph_tasks_run(
        C.byref(pipe.soa.struct), C.byref(pipe.soa.prec), C.byref(pipe.cells.struct),
        C.byref(pipe.prm), sph.Tile(*tile), p(td), 4, p(od), p(it), nd, len(items) - nd, p(out),
        4 * k, None))
    torch.cuda.synchronize()
    r = out.cpu().numpy().view(serve.RESULT).reshape(4, k)
    for t, width in ((0, 3), (2, 5)):
        assert np.all(r[t]["v"][:, :width] == 0) and np.all(r[t]["count"] == 0)
    assert r[1]["count"].sum() > 0 and r[3]["count"].sum() > 0
