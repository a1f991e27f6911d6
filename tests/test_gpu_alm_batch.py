"""Batches of fits to spherical-harmonic data large enough for 8 private copies of
the bins: few fits (column jobs of 16 waves) and more (of 4), against the fits
alone."""

import numpy as np
import pytest

from workloads import workload

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


@pytest.mark.parametrize("count", [2, 5])
def test_batch_of_large_alm_fits(count):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_1202_2355_amd import _abi as A
    from paper_1202_2355_amd.batch import Batch
    from paper_1202_2355_amd.fit import Fit
    wl = workload(2)
    lay = dict(wl.layout, dens="alm", l_max=4, n_r=40)
    par = dict(wl.params, prior_every=3)
    V, S = np.zeros(lay["n_R"]), np.full(lay["n_R"], 0.4)
    before = A.m2m_get_launch()
    b = Batch(max_fits=count)
    alone, inside = [], []
    try:
        A.m2m_set_launch(1024, 2)
        for k in range(count):
            n = (1 << 18) + 77 * k
            print("[gpu-test] a_lm fit", count, n, flush=True)
            parts = wl.initial_particles(n=n, seed=30 + k)
            for into in (alone, inside):
                f = Fit(wl.potential, lay, par, parts, dtype="f32")
                y = f.observe(V, S)
                f.set_targets(y * (1 + 0.05 * np.sin(np.arange(y.size))),
                              0.05 * np.abs(y) + 1e-3 * np.abs(y).max(), V, S)
                into.append(f)
            assert b.admit(inside[k], 7)
        for steps in (4, 3):
            b.run(steps)
    finally:
        A.m2m_set_launch(*before)
    done, left = b.poll()
    assert left == 0 and len(done) == count
    b.close()
    for f, g in zip(alone, inside):
        f.step(7)
        np.testing.assert_allclose(g.particles()["u"], f.particles()["u"], rtol=1e-5)
        np.testing.assert_allclose(g.chi2_history(), f.chi2_history(), rtol=1e-5)
        f.close()
        g.close()
