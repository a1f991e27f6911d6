"""The run kernel (several steps of a fit in one launch) around its edges: what
is reported of a launch that did not complete, and what the runs of several
streams wait for."""

import sys

import numpy as np
import pytest

from m2m_testlib import cast
from test_gpu_run import _fit, _say, _targets, _workload

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")

# byte offset of the error bits in the workspace (FitState comes first)
ERROR_AT = 28
# of the longest wait within a run, in the counters of its launches
WAIT_IN_SYNC = 16


@pytest.fixture(scope="module")
def Fit():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_1202_2355_amd import _abi
    _abi.lib()
    from paper_1202_2355_amd.fit import Fit
    return Fit


def _made(oracle, Fit, kin, dtype, n, every=4, **kw):
    wl = _workload(kin, every)
    parts = cast(wl.initial_particles(n=n, seed=n % 97), dtype)
    return _fit(Fit, wl, parts, _targets(oracle, wl, parts, n), dtype, **kw)


def _sync(f, at):
    """The counters of a fit's launches: they come last in the workspace, and a fit
    with a refresh on every step has the same workspace up to there."""
    from paper_1202_2355_amd import _abi as A
    base = A.m2m_workspace_bytes(f.layout, dict(f.params, prior_every=1), f.n, f.dtype)
    return f._ws[base + at:base + at + 4].view(torch.int32)


@pytest.mark.parametrize("kin,dtype,n", [("gh", "f32", 40_009), ("losvd", "f64", 20_011)])
def test_a_wait_without_its_value_fails_one_launch_only(oracle, Fit, kin, dtype, n):
    """The longest wait of a fit's launches set to 10 ns from the host: the next
    launch ends and is reported; a saved state taken up again steps as before."""
    from paper_1202_2355_amd import _abi as A
    _say("short wait", kin, dtype, n)
    a, b = (_made(oracle, Fit, kin, dtype, n) for _ in range(2))
    for f in (a, b):
        f.step(5)
    good, parts = b.get_state(), {k: v.clone() for k, v in b.t.items()}
    wait = _sync(b, WAIT_IN_SYNC)
    assert int(wait[0]) == 0
    wait.fill_(1)
    b.step(6)
    with pytest.raises(A.M2MError) as e:
        b.observables()
    assert e.value.status == A.M2M_EDEVICE
    wait.zero_()
    b.set_state(good)
    for k, v in parts.items():
        b.t[k].copy_(v)
    for f in (a, b):
        f.step(6)
    tol = 1e-5 if dtype == "f32" else 1e-10
    np.testing.assert_allclose(b.chi2_history(), a.chi2_history(), rtol=10 * tol)
    pa, pb = a.particles(), b.particles()
    for c in pa:
        np.testing.assert_allclose(pb[c], pa[c], rtol=tol, atol=1e-12)
    a.close()
    b.close()


@pytest.mark.parametrize("lagged", [False, True])
def test_a_run_that_did_not_complete_is_a_device_error(oracle, Fit, lagged):
    """The error bit of such a run set from the host: a batch hands the fit back
    with a device error, and every call that reads the fit's state reports it."""
    from paper_1202_2355_amd import _abi as A
    from paper_1202_2355_amd.batch import Batch
    _say("error bit", lagged)
    f = _made(oracle, Fit, "v2", "f64", 2001)
    b = Batch(max_fits=2)
    assert b.admit(f, 3)
    b.run(3)
    torch.cuda.synchronize()
    f._ws[ERROR_AT:ERROR_AT + 4].view(torch.int32).fill_(2)
    torch.cuda.synchronize()
    b.run(3)
    b.run(3)
    with pytest.raises(A.M2MError) as e:
        b.poll_lagged() if lagged else b.poll()
    assert e.value.status == A.M2M_EDEVICE
    b.close()
    for read in (f.observables, f.weights, f.chi2_history, f.get_state):
        with pytest.raises(A.M2MError) as e:
            read()
        assert e.value.status == A.M2M_EDEVICE, read
    f._ws[ERROR_AT:ERROR_AT + 4].view(torch.int32).zero_()
    assert np.isfinite(f.chi2_history()).all() and f.get_state()
    f.close()


def test_runs_wait_for_runs_only(oracle, Fit):
    """Other work on a stream that has stepped a fit holds up no fit of another
    stream: a step there ends while a kernel enqueued behind the first fit's
    steps still runs. Both before and after, steps in turn give what each fit
    gives alone."""
    n = (40_009, 270_001)  # 40 and 256 blocks
    alone = []
    for k in n:
        f = _made(oracle, Fit, "gh", "f32", k)
        f.step(22)
        alone.append(f.particles()["u"])
        f.close()
    fits = [_made(oracle, Fit, "gh", "f32", k, stream=torch.cuda.Stream()) for k in n]
    _say("two streams", n)

    def in_turn():
        for _ in range(5):
            for f in fits:
                f.step(2)

    in_turn()
    fits[0].step(1)
    busy = torch.cuda.Event()
    with torch.cuda.stream(fits[0].stream):
        torch.cuda._sleep(int(1e8))  # tens of ms at least
        busy.record()
    fits[1].step(1)
    fits[1].stream.synchronize()
    assert not busy.query()
    fits[1].step(1)
    fits[0].step(1)
    in_turn()
    for f, u in zip(fits, alone):
        np.testing.assert_allclose(f.particles()["u"], u, rtol=1e-5)
        f.close()


def test_many_streams_share_the_slots(oracle, Fit):
    """Fits of 16 to 256 blocks on streams of their own, calls of one to nine
    steps in a changing order."""
    n = (1001, 4003, 20_011, 33_001, 90_001, 262_147, 16_001, 50_021)
    rng = np.random.default_rng(3)
    alone, fits = [], []
    for k in n:
        f = _made(oracle, Fit, "gh", "f32", k)
        f.step(60)
        alone.append(f.particles()["u"])
        f.close()
        fits.append(_made(oracle, Fit, "gh", "f32", k, stream=torch.cuda.Stream()))
    _say("many streams", n)
    left = [60] * len(n)
    while any(left):
        k = int(rng.choice([j for j in range(len(n)) if left[j]]))
        m = min(left[k], int(rng.integers(1, 10)))
        fits[k].step(m)
        left[k] -= m
    for f, u in zip(fits, alone):
        np.testing.assert_allclose(f.particles()["u"], u, rtol=1e-5)
        f.close()
