"""How a server's threads wait for batches on the device: asleep, and no longer
than a batch's own time."""
import glob
import os

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


def _cpu():
    """CPU time in ns of each of the process's threads."""
    out = {}
    for t in glob.glob("/proc/self/task/*"):
        try:
            with open(os.path.join(t, "schedstat")) as f:
                out[os.path.basename(t)] = int(f.read().split()[0])
        except (FileNotFoundError, ProcessLookupError):      # a thread that ended meanwhile
            pass
    return out


def test_threads_sleep_while_a_batch_runs(sph):
    """A task against a crowded cell, again and again. Bar: no thread of the
    server is on a core for more than half of the time that batches run (a
    completion thread that asks without sleeping: all of it)."""
    from paper_2512_05516_amd import serve
    from paper_2512_05516_amd.pipeline import Pipeline
    rng = np.random.default_rng(2)
    n, n_c = 10000, 3
    ps = inputs.ParticleSet(rng.uniform(0.36, 0.64, (n, 3)), np.zeros((n, 3)), np.full(n, 1.0 / n),
                            np.full(n, 0.9 / (n_c * sph.GAMMA_K[0])), np.ones(n))
    pipe = Pipeline(inputs.pack_aos(ps, "f32"), n_c)
    pipe.bin()
    pipe.convert("full")
    cell = 1 + n_c * (1 + n_c)
    before = _cpu()
    tasks = np.array([[0, cell, cell, 0, 64]], np.int32)
    ran = 0
    with serve.Server(pipe) as server:
        for k in range(120):
            if k == 20:
                start, ran = _cpu(), 0
            req, _ = serve.requests(tasks, serve.now_ns())
            done = server.run(req)
            ran += int(done["done_ns"][0] - done["launch_ns"][0])
        used = {t: v - start.get(t, 0) for t, v in _cpu().items() if t not in before}
    assert ran / 100 > 100_000                    # a batch of some length, or nothing is shown
    assert used and max(used.values()) <= 0.5 * ran, (used, ran)
