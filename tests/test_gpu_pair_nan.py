"""What becomes of a sound speed that is not a number: v_sig of its particle's
neighbours, one lane per particle, is NaN too, whatever the size of their chunk."""
import numpy as np
import pytest

from paper_2512_05516_amd import inputs

pytestmark = pytest.mark.gpu

N_C = 3


@pytest.fixture(scope="module")
def sph():
    torch = pytest.importorskip("torch")
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2512_05516_amd import sphmi
    sphmi.lib()
    return sphmi


@pytest.mark.parametrize("n", [2, 9, 15, 16, 17, 31, 32, 33, 48, 64, 65, 96, 150])
def test_vsig_of_a_nan_sound_speed(sph, n):
    from paper_2512_05516_amd.pipeline import Pipeline
    rng = np.random.default_rng(n)
    h = 0.9 / (N_C * sph.GAMMA_K[0])
    x = 0.5 + 0.2 * h * rng.uniform(-1, 1, (n, 3))           # all are neighbours of all
    ps = inputs.ParticleSet(x, rng.normal(0, 0.1, (n, 3)), np.full(n, 1.0 / n), np.full(n, h),
                            np.ones(n))
    pipe = Pipeline(inputs.pack_aos(ps, "f32"), N_C, til=sph.tile(64, 1))
    pipe.bin()
    pipe.convert("full")
    pipe.density()
    for slot in {0, n // 2, n - 1}:
        c = pipe.soa["C"].clone()
        pipe.soa["C"][slot] = float("nan")
        pipe.force()
        assert np.all(np.isnan(pipe.soa["VSIG"].cpu().numpy()[:n])), slot
        assert np.all(pipe.soa["NFORCE"].cpu().numpy()[:n] == n - 1)
        pipe.soa["C"].copy_(c)
    pipe.force()
    assert np.all(pipe.soa["VSIG"].cpu().numpy()[:n] > 0)
