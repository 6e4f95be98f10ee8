"""Cells whose particles are all neighbours of each other, at the counts where
the lists of accepted candidates change their handling: a word of 32
candidates, a list of 32 entries, a group of 64 or 128, a batch, and chunks of
one, two and four threads per sum.

Bars: counts exact (every pair lies well inside the supports), fields within
1e-5 of the FP64 oracle on the same inputs, the FP32 bar of the parity tests."""
import numpy as np
import pytest

from paper_2512_05516_amd import inputs

from helpers import gpu_fields, max_rel, oracle_step, rel_rmse, run_gpu

pytestmark = pytest.mark.gpu

TILES = [(64, 4), (32, 8), (128, 2), (64, 2), (64, 1), (16, 16), (16, 4), (32, 2)]
N_C = 3


@pytest.fixture(scope="module")
def sph():
    torch = pytest.importorskip("torch")
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2512_05516_amd import sphmi
    sphmi.lib()
    return sphmi


def _dense(orc, n, own):
    """n particles within 0.35 H of each other around the centre of the box's
    middle cell, `own` of them in that cell and the others across its face."""
    rng = np.random.default_rng(n + 1000 * own)
    h = 0.9 / (N_C * orc.GAMMA_K)
    r = 0.1 * h * orc.GAMMA_K
    x = np.empty((n, 3))
    side = np.arange(n) < own
    x[:, 0] = 2 / 3 + np.where(side, -1, 1) * rng.uniform(1e-3 * r, r, n)
    x[:, 1:] = 0.5 + rng.uniform(-r, r, (n, 2))
    p = rng.permutation(n)
    ps = inputs.ParticleSet(x[p], rng.normal(0.0, 0.05, (n, 3)), rng.uniform(0.5, 1.5, n) / n,
                            np.full(n, h), rng.uniform(0.5, 1.5, n))
    return inputs.unpack_aos(inputs.pack_aos(ps, "f32"))


@pytest.mark.parametrize("n,own", [(16, 16), (31, 31), (32, 20), (33, 33), (48, 48), (64, 64),
                                   (65, 40), (96, 64), (97, 64), (128, 64), (129, 63), (160, 33),
                                   (192, 50), (257, 64), (520, 57), (1100, 130)])
@pytest.mark.parametrize("ti,k", TILES)
def test_all_pairs_accepted(sph, orc, ti, k, n, own):
    ps = _dense(orc, n, own)
    d, f = oracle_step(orc, ps, N_C, prm=orc.params(gradh=False))
    assert np.all(d["nngb"] == n) and np.all(f["nforce"] == n - 1)
    pipe = run_gpu(ps, N_C, "f32", til=sph.tile(ti, k), prm=sph.params(gradh=False))
    assert pipe.status() == 0
    got = gpu_fields(pipe)
    assert np.all(got["nngb"] == n) and np.all(got["nforce"] == n - 1)
    for q in ("rho", "wcount"):
        assert max_rel(got[q], d[q]) <= 1e-5, q
    assert max_rel(got["vsig"], f["vsig"]) <= 1e-5
    for q in ("a", "du"):
        assert rel_rmse(got[q], f[q]) <= 1e-5, q


@pytest.mark.parametrize("n", [3, 16, 24, 32])
@pytest.mark.parametrize("ti,k", [(64, 1), (64, 2), (32, 2), (16, 4)])
def test_lists_that_lanes_share(sph, orc, ti, k, n):
    """Chunks of few particles, whose lists are written by up to four lanes and
    read by others: the same bits on every launch."""
    import torch
    ps = _dense(orc, 10 * n, n)
    pipe = run_gpu(ps, N_C, "f32", til=sph.tile(ti, k), prm=sph.params(gradh=False))
    out = ("RHO", "WCOUNT", "RHO_DH", "NNGB", "A_X", "A_Y", "A_Z", "DU", "VSIG", "NFORCE")
    first = {q: pipe.soa[q].clone() for q in out}
    for _ in range(20):
        pipe.density()
        pipe.force()
        for q in out:
            assert torch.equal(pipe.soa[q].view(torch.int32), first[q].view(torch.int32)), q
