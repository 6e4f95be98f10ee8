"""Paths of the reductions and of the record loader: step totals where a
thread's next slot is loaded ahead and where several hundred partials hold the
minimum, reductions over records of mixed field types, and the pair loops on
records at the chunk layouts of the edge tests and with merged chunks."""
import math

import numpy as np
import pytest

from paper_2512_05516_amd import inputs

pytestmark = pytest.mark.gpu

N_C = 4
COUNTS = (0, 1, 2, 15, 16, 17, 31, 32, 33, 47, 63, 64, 65, 97, 129, 200)


@pytest.fixture(scope="module")
def sph():
    torch = pytest.importorskip("torch")
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2512_05516_amd import sphmi
    sphmi.lib()
    return sphmi


@pytest.mark.parametrize("at", ["first", "last"])
@pytest.mark.parametrize("n", [1, 256, 257, 65537, 262144, 262145, 600001])
def test_step_totals_sizes(sph, n, at):
    """The smallest Courant step in the first or last slot. Bars as for the
    reductions: n 2^-53 of the terms' magnitudes, the minimum to 2^-50."""
    import torch
    from paper_2512_05516_amd.pipeline import Pipeline
    rng = np.random.default_rng(n)
    ps = inputs.ParticleSet(rng.uniform(0, 1, (n, 3)), rng.normal(0, 1, (n, 3)),
                            rng.uniform(0.5, 1.5, n), np.full(n, 0.01), rng.uniform(0.5, 1.5, n))
    pipe = Pipeline(inputs.pack_aos(ps, "f32"), 3)
    pipe.bin()
    pipe.convert("full")
    vs = rng.uniform(1.0, 2.0, n).astype(np.float32)
    vs[rng.random(n) < 0.1] = 0.0
    vs[0 if at == "first" else n - 1] = 8.0
    pipe.soa["VSIG"].copy_(torch.from_numpy(vs))
    out = torch.zeros(8, dtype=torch.float64, device="cuda")
    sph.step_totals(pipe.soa, pipe.cells, out, pipe.red_ws)
    got = out.cpu().numpy()
    arr = lambda k: pipe.soa[k].cpu().numpy()[:n].astype(np.float64)
    m, u, v = arr("M"), arr("UK"), np.stack([arr(f"V_{a}") for a in "XYZ"], 1)
    terms = [m * v[:, 0], m * v[:, 1], m * v[:, 2], 0.5 * m * (v * v).sum(1), m * u, m]
    for q, t in enumerate(terms):
        bound = (n * 2.0 ** -53 + 2.0 ** -50) * math.fsum(np.abs(t)) + 1e-300
        assert abs(got[q] - math.fsum(t)) <= bound, q
    dt = sph.C_CFL * (pipe.prm.gamma_k * float(arr("H")[0])) / 8.0
    assert abs(got[6] / dt - 1) <= 2.0 ** -50 and got[7] == (vs > 0).sum()


def _mixed(order):
    """Records whose fields are FP32 or FP64 at random, in a random order."""
    rng = np.random.default_rng(order)
    fields = [("x", "<f8", 3)] + [(k, ("<f4", "<f8")[rng.integers(2)], c) for k, c in (
        ("v", 3), ("m", 1), ("h", 1), ("u", 1), ("rho", 1), ("wcount", 1), ("rho_dh", 1), ("f", 1),
        ("P", 1), ("c", 1), ("a", 3), ("du", 1), ("vsig", 1))]
    fields += [("nngb", "<i4", 1), ("nforce", "<i4", 1), ("cell", "<i4", 1)]
    names, formats, offsets, at = [], [], [], 0
    for name, t, k in [fields[i] for i in rng.permutation(len(fields))]:
        at = (at + 7) // 8 * 8 if t == "<f8" else at
        names.append(name)
        formats.append((t, (k,)) if k > 1 else t)
        offsets.append(at)
        at += k * np.dtype(t).itemsize
    return np.dtype({"names": names, "formats": formats, "offsets": offsets,
                     "itemsize": (at + 7) // 8 * 8})


def _records(dt, n, seed, n_c=N_C, cells=None):
    rng = np.random.default_rng(seed)
    rec = np.zeros(n, dt)
    if cells is None:
        rec["x"] = rng.uniform(0, 1, (n, 3))
    else:
        c = np.stack([cells % n_c, (cells // n_c) % n_c, cells // n_c ** 2], 1)
        rec["x"] = (c + rng.uniform(0, 1, (n, 3)) * (1 - 2 ** -20)) / n_c
    f32 = lambda a: a.astype(np.float32)
    for k in ("v", "a", "du"):
        rec[k] = f32(rng.normal(0, 1, rec[k].shape))
    rec["m"], rec["u"] = f32(rng.uniform(0.5, 1.5, n)), f32(rng.uniform(0.5, 1.5, n))
    rec["h"] = f32(rng.uniform(0.3, 0.99, n) / (n_c * 1.825742))
    rec["nngb"], rec["nforce"] = rng.integers(0, 100, n), rng.integers(0, 100, n)
    return rec


@pytest.mark.parametrize("order", range(4))
@pytest.mark.parametrize("n", [1, 257, 262145])
def test_reduce_mixed_records(sph, n, order):
    """The sums over records of mixed types are those over the FP32 slots, bit
    for bit (the records hold FP32 values)."""
    import torch
    from paper_2512_05516_amd.pipeline import Pipeline
    rec = _records(_mixed(order), n, n + order)
    pipe = Pipeline(rec, N_C)
    pipe.bin()
    pipe.convert("full")
    perm = pipe.cells.perm[:n].cpu().numpy()
    for k, v in (("A_X", rec["a"][:, 0]), ("A_Y", rec["a"][:, 1]), ("A_Z", rec["a"][:, 2]),
                 ("DU", rec["du"]), ("NNGB", rec["nngb"]), ("NFORCE", rec["nforce"])):
        pipe.soa[k].copy_(torch.from_numpy(v[perm].copy()).to(pipe.soa[k].dtype))
    pipe.reduce()
    want = pipe.red_out.cpu().numpy().copy()
    pipe.red_out.zero_()
    pipe.reduce_aos()
    assert np.array_equal(pipe.red_out.cpu().numpy(), want)


@pytest.mark.parametrize("dtype", ["f32", "f64", "mixed"])
@pytest.mark.parametrize("ti,k", [(64, 4), (32, 8), (128, 2), (64, 2), (64, 1), (16, 16), (16, 4),
                                  (32, 2)])
@pytest.mark.parametrize("which", ["cells", "sub_cells", "merged"])
def test_pair_loops_on_records(sph, ti, k, which, dtype):
    """Cells of 0 to 200 particles: the loops on records give the bits of those
    on FP32 slots, whole cells, sub-cells, and one to four cells a chunk."""
    from paper_2512_05516_amd.pipeline import Pipeline
    rng = np.random.default_rng(7)
    cnt = rng.permutation(np.resize(np.array(COUNTS), N_C ** 3)) // (16 if which == "merged" else 1)
    cells = rng.permutation(np.repeat(np.arange(N_C ** 3), cnt))
    dt = {"f32": inputs.AOS_F32, "f64": inputs.AOS_F64, "mixed": _mixed(5)}[dtype]
    rec = _records(dt, len(cells), 11, cells=cells)
    kw = {"cells": {}, "sub_cells": {"sub_bits": 1, "sched": "grid"},
          "merged": {"sched": "dynamic", "max_cells": 4}}[which]
    out = []
    for aos in (False, True):
        pipe = Pipeline(rec, N_C, til=sph.tile(ti, k), **kw)
        pipe.bin()
        if aos:
            pipe.density_aos()
            pipe.force_aos()
        else:
            pipe.convert("full")
            pipe.density()
            pipe.force()
            pipe.writeback("density")
            pipe.writeback("force")
        assert pipe.status() == 0
        out.append(pipe.records())
    for q in ("rho", "wcount", "rho_dh", "f", "P", "c", "nngb", "a", "du", "vsig", "nforce"):
        assert out[0][q].tobytes() == out[1][q].tobytes(), q
