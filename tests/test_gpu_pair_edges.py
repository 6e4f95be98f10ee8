"""The pair loops at the sizes where their layout changes: chunks just below,
at and above 16, 32 and 64 particles (particles per matrix block, threads per
sum), above the tile, lists that overflow within a group of candidates,
batches with a few candidates, and candidates without a finite position.

Bars: neighbour counts as the FP64 definition gives them, fields within the
FP32 bar of the parity tests (1e-5 of the FP64 oracle on the same inputs)."""
import numpy as np
import pytest

from paper_2512_05516_amd import inputs

from helpers import assert_counts, gpu_fields, max_rel, oracle_step, rel_rmse, run_gpu

pytestmark = pytest.mark.gpu

TILES = [(64, 4), (32, 8), (128, 2), (64, 2), (64, 1), (16, 16), (16, 4), (32, 2)]
COUNTS = (0, 1, 2, 15, 16, 17, 31, 32, 33, 47, 48, 49, 63, 64, 65, 80, 96, 97, 127, 128, 129, 200)
N_C = 4


@pytest.fixture(scope="module")
def sph():
    torch = pytest.importorskip("torch")
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2512_05516_amd import sphmi
    sphmi.lib()
    return sphmi


def _set(orc, wide, thin=1):
    """Cells of every count of COUNTS (divided by thin) in a random order.
    wide: supports just within the cell side, so that most of a particle's
    candidates are pairs; else 0.3 to 0.9 of it."""
    rng = np.random.default_rng(31 + wide + 2 * thin)
    cnt = rng.permutation(np.resize(np.array(COUNTS), N_C ** 3)) // thin
    cell = np.repeat(np.arange(N_C ** 3), cnt)
    n = len(cell)
    c = np.stack([cell % N_C, (cell // N_C) % N_C, cell // N_C ** 2], axis=1)
    x = (c + rng.uniform(0.0, 1.0, (n, 3)) * (1 - 2 ** -20)) / N_C
    hmax = 0.99 / (N_C * orc.GAMMA_K)
    h = hmax * (rng.uniform(0.97, 1.0, n) if wide else rng.uniform(0.3, 0.9, n))
    p = rng.permutation(n)
    ps = inputs.ParticleSet(x[p], rng.normal(0.0, 0.05, (n, 3)), rng.uniform(0.5, 1.5, n) / n, h,
                            rng.uniform(0.5, 1.5, n))
    return inputs.unpack_aos(inputs.pack_aos(ps, "f32"))


@pytest.fixture(scope="module")
def sets(orc):
    out = {}
    for name, wide, thin in (("mixed", False, 1), ("wide", True, 1), ("sparse", True, 24)):
        ps = _set(orc, wide, thin)
        # without grad-h factors: on a few random neighbours those are 1 / (a
        # difference near zero), which no FP32 bar holds for
        out[name] = (ps,) + oracle_step(orc, ps, N_C, prm=orc.params(gradh=False))
    return out


@pytest.mark.parametrize("which", ["mixed", "wide", "sparse"])
@pytest.mark.parametrize("ti,k", TILES)
def test_chunk_and_list_sizes(sph, orc, sets, ti, k, which):
    ps, d, f = sets[which]
    kw = {"mixed": {}, "wide": {"sub_bits": 1, "sched": "grid"},
          "sparse": {"sched": "dynamic", "max_cells": 4}}[which]
    pipe = run_gpu(ps, N_C, "f32", til=sph.tile(ti, k), prm=sph.params(gradh=False), **kw)
    assert pipe.status() == 0
    got = gpu_fields(pipe)
    assert_counts(orc, got["nngb"], got["nforce"], d["nngb"], f["nforce"], ps, N_C, tag=which)
    for q in ("rho", "wcount", "P", "c"):
        assert max_rel(got[q], d[q]) <= 1e-5, q
    some = f["vsig"] > 0
    assert max_rel(got["vsig"][some], f["vsig"][some]) <= 1e-5
    for q in ("a", "du"):
        assert rel_rmse(got[q], f[q]) <= 1e-5, q


@pytest.mark.parametrize("ti,k", TILES)
def test_candidates_without_a_position(sph, orc, sets, ti, k):
    """A particle whose position is NaN is nobody's neighbour: all others
    have the counts and sums of the set without it."""
    ps, d, f = sets["mixed"]
    x = ps.x[:2].copy()
    x[0, 1], x[1, 2] = np.nan, np.inf
    more = inputs.ParticleSet(np.concatenate([ps.x, x]), np.concatenate([ps.v, ps.v[:2]]),
                              np.concatenate([ps.m, ps.m[:2]]), np.concatenate([ps.h, ps.h[:2]]),
                              np.concatenate([ps.u, ps.u[:2]]))
    pipe = run_gpu(more, N_C, "f32", til=sph.tile(ti, k), prm=sph.params(gradh=False))
    assert pipe.status() == sph.FLAG_BAD_POSITION
    got = {q: v[:ps.n] for q, v in gpu_fields(pipe).items()}
    assert_counts(orc, got["nngb"], got["nforce"], d["nngb"], f["nforce"], ps, N_C)
    for q in ("rho", "wcount"):
        assert max_rel(got[q], d[q]) <= 1e-5, q
    for q in ("a", "du"):
        assert rel_rmse(got[q], f[q]) <= 1e-5, q
