"""Fits that refresh their priors on every step: the finalize reduces their cells
in blocks of their own, alone and among fits that refresh less often."""

import numpy as np
import pytest

from m2m_testlib import cast
from test_gpu_run import _fit, _say, _targets, _workload

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


@pytest.fixture(scope="module")
def Fit():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_1202_2355_amd import _abi
    _abi.lib()
    from paper_1202_2355_amd.fit import Fit
    return Fit


@pytest.mark.parametrize("grid", [(2, 1), (8, 8), (13, 5), (64, 32)])
@pytest.mark.parametrize("kin,dtype,tol", [("v2", "f64", 1e-10), ("gh", "f32", 1e-4), ("losvd", "f32", 1e-4)])
def test_every_step_refreshes(oracle, Fit, grid, kin, dtype, tol):
    """Fewer cells than observables, as many, and many more (50, 170 and 210 columns),
    against the oracle; then the same fit in a batch with one that refreshes every
    third step, against the fits alone."""
    from paper_1202_2355_amd.batch import Batch
    n = 9001
    _say("every step", grid, kin, dtype)
    alone, inside = [], []
    b = Batch(max_fits=2)
    for every in (1, 3):
        wl = _workload(kin, every)
        wl = wl.with_(params=dict(wl.params, n_E=grid[0], n_x=grid[1]))
        parts = cast(wl.initial_particles(n=n, seed=7), dtype)
        T = _targets(oracle, wl, parts, n)
        f, g = (_fit(Fit, wl, parts, T, dtype) for _ in range(2))
        for k in (1, 5):
            f.step(k)
        if every == 1:
            o = oracle.OracleFit(wl.potential, wl.layout, wl.params, parts, *T, track_flags=True,
                                 band=1e-5 if dtype == "f32" else 1e-12, nthreads=8)
            o.step(6)
            ok = o.flag == 0
            u = f.particles()["u"]
            assert np.max(np.abs(u[ok] / o.arr["u"][ok] - 1)) <= tol
        assert b.admit(g, 6)
        alone.append(f)
        inside.append(g)
    for _ in range(2):
        b.run(3)
    done, left = b.poll()
    assert left == 0 and len(done) == 2
    b.close()
    for f, g in zip(alone, inside):
        f.update_priors()
        g.update_priors()
        pf, pg = f.particles(), g.particles()
        for c in ("u", "uh"):
            np.testing.assert_allclose(pg[c], pf[c], rtol=1e-5 if dtype == "f32" else 1e-10)
        f.close()
        g.close()
