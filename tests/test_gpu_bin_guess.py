"""Bins of FP64 particles far from 1: the guess of a bin from an FP32
logarithm has to leave every point near an edge to the stored edges, whatever
the size of the radii."""

import numpy as np
import pytest

from workloads import workload

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


@pytest.mark.parametrize("scale", [1e-120, 1e-60, 1e-9, 1.0, 1e20, 1e60, 1e120])
def test_points_near_the_edges_are_in_their_bins(Fit, scale):
    """400 bins over a factor of 16 in r, points at 1e-4 to 3e-3 of a bin on both
    sides of every edge (3e-7 and more of the radius: unambiguous in FP64)."""
    wl = workload(1)
    n_r = 400
    lay = dict(wl.layout, n_r=n_r, r_min=scale, r_max=16.0 * scale, kin="none", n_R=0)
    d = np.concatenate([s * np.geomspace(1e-4, 3e-3, 60) for s in (-1, 1)])
    at = (np.arange(n_r)[:, None] + d[None, :]).reshape(-1)  # in bins
    at = at[at > 0]
    r = scale * 16.0 ** (at / n_r)
    parts = {k: np.zeros(r.size) for k in ("x", "y", "z", "vx", "vy", "vz")}
    parts["x"] = r
    f = Fit(wl.potential, lay, wl.params, parts, dtype="f64")
    want = np.bincount(np.floor(at).astype(int), minlength=n_r) * (wl.params["mass"] / r.size)
    np.testing.assert_allclose(f.observe(), want, rtol=1e-12)
    f.close()
