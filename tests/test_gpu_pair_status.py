"""The status flag of supports above the cell side: raised by each pair loop
for a single such particle, wherever it lies in its chunk, left down
otherwise, and no slower to raise where every chunk has cause to."""
import numpy as np
import pytest

from paper_2512_05516_amd import inputs

pytestmark = pytest.mark.gpu

TILES = [(64, 4), (32, 8), (128, 2), (64, 2), (64, 1), (16, 16), (16, 4), (32, 2)]
N_C = 4


@pytest.fixture(scope="module")
def sph():
    torch = pytest.importorskip("torch")
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2512_05516_amd import sphmi
    sphmi.lib()
    return sphmi


def _uniform(n, n_c, h, seed):
    rng = np.random.default_rng(seed)
    return inputs.ParticleSet(rng.uniform(0, 1, (n, 3)), np.zeros((n, 3)), np.full(n, 1.0 / n),
                              np.full(n, h), np.ones(n))


def _pipe(sph, ps, n_c, **kw):
    from paper_2512_05516_amd.pipeline import Pipeline
    pipe = Pipeline(inputs.pack_aos(ps, "f32"), n_c, **kw)
    pipe.bin()
    pipe.convert("full")
    return pipe


@pytest.mark.parametrize("n", [40, 900, 4500, 9000])      # up to 16, 32, 128 and more per cell
@pytest.mark.parametrize("ti,k", TILES)
def test_flag_of_one_particle(sph, ti, k, n):
    side = 1.0 / (N_C * sph.GAMMA_K[0])
    ps = _uniform(n, N_C, 0.5 * side, n)
    pipe = _pipe(sph, ps, N_C, til=sph.tile(ti, k))
    pipe.density()
    pipe.force()
    assert pipe.status() == 0
    for slot in (0, n // 2, n - 1):
        h = pipe.soa["H"].clone()
        pipe.soa["H"][slot] = 1.01 * side
        for loop in (pipe.density, pipe.force):
            pipe.cells.status.zero_()
            loop()
            assert pipe.status() == sph.FLAG_H_TOO_LARGE, (slot, loop.__name__)
            loop()                                        # up already
            assert pipe.status() == sph.FLAG_H_TOO_LARGE
        pipe.soa["H"].copy_(h)
    pipe.cells.status.zero_()
    pipe.density()
    pipe.force()
    assert pipe.status() == 0


def test_flag_costs_no_time(sph):
    """Every particle's support a thousandth above the cell side, as storage
    formats round it, against a thousandth below: the same pairs. Bar: half as
    long again (one atomic per wave and launch took twice as long)."""
    import torch
    n_c = 24
    side = 1.0 / (n_c * sph.GAMMA_K[0])
    pipes = [_pipe(sph, _uniform(12 * n_c ** 3, n_c, f * side, 3), n_c) for f in (0.999, 1.001)]
    t = {}
    for loop in ("density", "force"):
        for rep in range(8):
            for i, p in enumerate(pipes):
                e0, e1 = (torch.cuda.Event(enable_timing=True) for _ in range(2))
                e0.record()
                for _ in range(5):
                    getattr(p, loop)()
                e1.record()
                torch.cuda.synchronize()
                t.setdefault((loop, i), []).append(e0.elapsed_time(e1))
    assert pipes[0].status() == 0 and pipes[1].status() == sph.FLAG_H_TOO_LARGE
    for loop in ("density", "force"):
        below, above = (np.median(t[loop, i][2:]) for i in (0, 1))
        assert above <= 1.5 * below, (loop, below, above)
