"""Fits whose tiles are bounded by the length of their partial rows (many
observables and cells): at sizes where the bounds meet (one tile, one particle
more than a whole number of tiles, the most tiles), alone and in batches that
would leave compute units idle, weights after 6 steps with two refreshes
against the FP64 oracle: to 1e-4 (FP32 state) and 1e-9 (FP64), the tolerances
of the other parity tests."""

import numpy as np
import pytest

from m2m_testlib import cast, weight_errors
from workloads import with_alm, with_scf, workload

pytestmark = pytest.mark.gpu


def _wl(kind):
    wl = workload(3 if kind == "losvd" else 2)
    if kind == "alm":
        wl = with_alm(wl, l_max=3)
    if kind == "scf":
        wl = with_scf(wl, l_max=2, every=3)
    return wl.with_(params=dict(wl.params, prior_every=3))


def _pair(oracle, wl, n, dtype):
    from paper_1202_2355_amd import Fit
    parts = cast(wl.initial_particles(n=n, seed=n), dtype)
    V = S = None
    if wl.layout["kin"] == "gh":
        V, S = np.zeros(wl.layout["n_R"]), np.full(wl.layout["n_R"], 0.4)
    Y = oracle.deposit(parts, np.ones(n), wl.layout, mass=wl.params["mass"], V_p=V, sigma_p=S)
    sig = 0.05 * np.abs(Y) + 1e-2 * np.abs(Y).max() + 1e-12
    Y = Y * (1.0 + 0.05 * np.sin(np.arange(Y.size)))
    f = Fit(wl.potential, wl.layout, wl.params, parts, dtype=dtype)
    f.set_targets(Y, sig, V, S)
    o = oracle.OracleFit(wl.potential, wl.layout, wl.params, parts, Y, sig, V, S,
                         track_flags=True, band=1e-5 if dtype == "f32" else 1e-12, nthreads=8)
    return f, o


def _check(f, o, dtype, what):
    _, rmax, _, _ = weight_errors(f.particles()["u"], o.arr["u"], o.flag)
    print(what, rmax, flush=True)
    assert rmax <= (1e-4 if dtype == "f32" else 1e-9)


CASES = [("losvd", "f32", 1023), ("losvd", "f32", 1025), ("losvd", "f32", 40_001), ("losvd", "f32", 170_001),
         ("losvd", "f64", 257), ("losvd", "f64", 20_011), ("alm", "f32", 255), ("alm", "f32", 30_001),
         ("alm", "f64", 9_001), ("alm", "f32", 262_144), ("scf", "f32", 20_011)]


@pytest.mark.parametrize("kind,dtype,n", CASES)
def test_tiles_match_oracle(oracle, kind, dtype, n):
    f, o = _pair(oracle, _wl(kind), n, dtype)
    f.step(6)
    o.step(6)
    _check(f, o, dtype, (kind, dtype, n))
    f.close()


@pytest.mark.parametrize("kind,dtype,ns", [("losvd", "f32", (3_001, 64, 20_011)), ("losvd", "f64", (3_001, 5_000)),
                                           ("alm", "f32", (9_001, 1_025, 5_000, 2_000))])
def test_batch_tiles_match_oracle(oracle, kind, dtype, ns):
    from paper_1202_2355_amd.batch import Batch
    wl = _wl(kind)
    pairs = [_pair(oracle, wl, n, dtype) for n in ns]
    b = Batch(max_fits=len(ns))
    for f, _ in pairs:
        assert b.admit(f, 6)
    b.run(6)
    done, left = b.poll()
    assert len(done) == len(ns) and left == 0
    b.close()
    for (f, o), n in zip(pairs, ns):
        o.step(6)
        _check(f, o, dtype, (kind, dtype, n))
        f.close()
