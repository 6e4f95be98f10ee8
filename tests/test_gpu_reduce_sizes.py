"""The reductions at the sizes where their grid changes (one slot, one block
more or less, all blocks, a second slot per thread) and in each storage
format, SoA and records, against exactly rounded sums of the same values.

Bar: a sum of n FP64 terms in any order is within n 2^-53 of the sum of its
terms' magnitudes, and each term within 2^-50 of itself."""
import math

import numpy as np
import pytest

from paper_2512_05516_amd import inputs

from helpers import unpack_trunc

pytestmark = pytest.mark.gpu

SIZES = (1, 255, 256, 257, 1000, 262143, 262144, 262145, 600001)
FORMATS = (("f32", "f32"), ("f16", "bf16"), ("bf16", "f16"), ("f32", "bf16"), ("t20", "f32"),
           ("f16", "t14"))


@pytest.fixture(scope="module")
def sph():
    torch = pytest.importorskip("torch")
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2512_05516_amd import sphmi
    sphmi.lib()
    return sphmi


def _pipe(sph, n, mhu, vel, kind):
    import torch
    from paper_2512_05516_amd.pipeline import Pipeline
    rng = np.random.default_rng(n)
    ps = inputs.ParticleSet(rng.uniform(0, 1, (n, 3)), rng.normal(0, 1, (n, 3)),
                            rng.uniform(0.5, 1.5, n), rng.uniform(0.01, 0.02, n),
                            rng.uniform(0.5, 1.5, n))
    rec = inputs.pack_aos(ps, kind)
    rates = rng.normal(0, 1, (n, 5)).astype(np.float32)
    counts = rng.integers(0, 100, (n, 2)).astype(np.int32)
    rec["a"], rec["du"], rec["vsig"] = rates[:, :3], rates[:, 3], rates[:, 4]
    rec["nngb"], rec["nforce"] = counts[:, 0], counts[:, 1]
    pipe = Pipeline(rec, 4, prec=sph.precision("f32", vel, mhu))
    pipe.bin()
    pipe.convert("full")
    perm = pipe.cells.perm[:n].cpu().numpy()
    for i, k in enumerate(("A_X", "A_Y", "A_Z", "DU", "VSIG")):
        pipe.soa[k].copy_(torch.from_numpy(rates[perm, i]))
    for i, k in enumerate(("NNGB", "NFORCE")):
        pipe.soa[k].copy_(torch.from_numpy(counts[perm, i]))
    return pipe, rates.astype(np.float64), counts


def _slot(pipe, k):
    """The stored values of a field, in input order."""
    if k not in pipe.soa.packed:
        return np.asarray(pipe.slot(k), np.float64)
    out = np.empty(pipe.n)
    perm = pipe.cells.perm[:pipe.n].cpu().numpy()
    out[perm] = unpack_trunc(pipe.soa[k].cpu().numpy(), pipe.soa.packed[k], pipe.n)
    return out


def _close(got, terms):
    bound = (len(terms) * 2.0 ** -53 + 2.0 ** -50) * math.fsum(np.abs(terms)) + 1e-300
    assert abs(got - math.fsum(terms)) <= bound


def _check(out, m, v, r, counts):
    va = (v * r[:, :3]).sum(1)
    mag = (np.abs(v * r[:, :3])).sum(1)
    for c in range(3):
        _close(out[c], m * r[:, c])
    # the terms of the energy sum cancel inside: bounded by their parts
    e = m * (va + r[:, 3])
    assert abs(out[3] - math.fsum(e)) <= (len(m) * 2.0 ** -53 + 2.0 ** -50) * math.fsum(
        m * (mag + np.abs(r[:, 3])))
    _close(out[4], m * np.linalg.norm(r[:, :3], axis=1))
    assert abs(out[5] - math.fsum(m * (np.abs(va) + np.abs(r[:, 3])))) <= (
        len(m) * 2.0 ** -53 + 2.0 ** -50) * math.fsum(m * (mag + np.abs(r[:, 3])))
    assert out[6] == counts[:, 0].sum() and out[7] == counts[:, 1].sum()


@pytest.mark.parametrize("n", SIZES)
@pytest.mark.parametrize("kind", ["f32", "f64"])
def test_reduce_sizes(sph, n, kind):
    pipe, r, counts = _pipe(sph, n, "f32", "f32", kind)
    m = pipe.slot("M").astype(np.float64)
    v = np.stack([pipe.slot(f"VQ_{a}") for a in "XYZ"], 1).astype(np.float64)
    pipe.reduce()
    soa = pipe.red_out.cpu().numpy().copy()
    _check(soa, m, v, r, counts)
    pipe.reduce_aos()
    assert np.array_equal(pipe.red_out.cpu().numpy(), soa)


@pytest.mark.parametrize("mhu,vel", FORMATS)
def test_reductions_in_each_format(sph, mhu, vel):
    import torch
    n = 1000
    pipe, r, counts = _pipe(sph, n, mhu, vel, "f32")
    slot = lambda k: _slot(pipe, k)
    m, h, vs = slot("M"), slot("H"), r[:, 4]
    pipe.reduce()
    _check(pipe.red_out.cpu().numpy(), m, np.stack([slot(f"VQ_{a}") for a in "XYZ"], 1), r,
           counts)
    out = torch.zeros(8, dtype=torch.float64, device="cuda")
    sph.step_totals(pipe.soa, pipe.cells, out, pipe.red_ws)
    got = out.cpu().numpy()
    v, u = np.stack([slot(f"V_{a}") for a in "XYZ"], 1), slot("UK")
    for c in range(3):
        _close(got[c], m * v[:, c])
    _close(got[3], 0.5 * m * (v * v).sum(1))
    _close(got[4], m * u)
    _close(got[5], m)
    some = vs > 0
    dt = sph.C_CFL * (pipe.prm.gamma_k * h[some]) / vs[some]
    assert abs(got[6] / dt.min() - 1) <= 2.0 ** -50 and got[7] == some.sum()
