"""Fits of more than 1024 observables: calls of more than two steps by the run
kernel, shorter ones by the step and finalize kernels, in turn on one fit and on
a batch; weights after refreshes in both, and chi^2 of every step, against the
FP64 oracle: weights to 1e-4 (FP32 state) and 1e-10 (FP64), chi^2 to 1e-3 and
1e-9, the tolerances of the other run kernel tests."""

import numpy as np
import pytest

from m2m_testlib import cast, weight_errors
from workloads import workload

pytestmark = pytest.mark.gpu


def _pair(oracle, n, dtype, n_v):
    from paper_1202_2355_amd import Fit
    wl = workload(3)
    wl = wl.with_(layout=dict(wl.layout, n_v=n_v), params=dict(wl.params, prior_every=4))
    parts = cast(wl.initial_particles(n=n, seed=n), dtype)
    Y = oracle.deposit(parts, np.ones(n), wl.layout, mass=wl.params["mass"])
    sig = 0.05 * np.abs(Y) + 1e-2 * np.abs(Y).max() + 1e-12
    Y = Y * (1.0 + 0.05 * np.sin(np.arange(Y.size)))
    f = Fit(wl.potential, wl.layout, wl.params, parts, dtype=dtype)
    f.set_targets(Y, sig)
    o = oracle.OracleFit(wl.potential, wl.layout, wl.params, parts, Y, sig, None, None, track_flags=True,
                         band=1e-5 if dtype == "f32" else 1e-12, nthreads=8)
    return f, o


def _check(f, o, hist, dtype):
    _, rmax, _, _ = weight_errors(f.particles()["u"], o.arr["u"], o.flag)
    assert rmax <= (1e-4 if dtype == "f32" else 1e-10)
    np.testing.assert_allclose(f.chi2_history(), hist, rtol=1e-3 if dtype == "f32" else 1e-9)


# 1050 and 2610 observables; less than a block per job, one and several rounds
@pytest.mark.parametrize("dtype,n,n_v", [("f32", 999, 64), ("f32", 50_001, 64), ("f32", 300_007, 25),
                                         ("f64", 5_003, 64), ("f64", 90_001, 25)])
def test_calls_of_both_kinds(oracle, dtype, n, n_v):
    f, o = _pair(oracle, n, dtype, n_v)
    print("many observables", dtype, n, n_v, flush=True)
    hist = []
    for k in (1, 3, 2, 5, 1, 3):
        f.step(k)
        hist.extend(o.step(k))
    _check(f, o, hist, dtype)
    f.close()


@pytest.mark.parametrize("dtype,ns", [("f32", (3_001, 40_001)), ("f64", (2_003, 9_001, 500))])
def test_batch_calls_of_both_kinds(oracle, dtype, ns):
    from paper_1202_2355_amd.batch import Batch
    pairs = [_pair(oracle, n, dtype, 64) for n in ns]
    print("batch of many observables", dtype, ns, flush=True)
    b = Batch(max_fits=len(ns))
    for f, _ in pairs:
        assert b.admit(f, 11)
    for k in (3, 1, 5, 2):
        b.run(k)
    done, left = b.poll()
    assert len(done) == len(ns) and left == 0
    b.close()
    for f, o in pairs:
        hist = o.step(11)
        _check(f, o, hist, dtype)
        f.close()
