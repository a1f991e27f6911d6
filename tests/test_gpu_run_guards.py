"""The run kernel (several steps of a fit in one launch) around its edges: what
is reported of a launch that did not complete."""

import sys

import numpy as np
import pytest

from m2m_testlib import cast
from test_gpu_run import _fit, _say, _targets, _workload

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")

# byte offset of the error bits in the workspace (FitState comes first)
ERROR_AT = 28


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
