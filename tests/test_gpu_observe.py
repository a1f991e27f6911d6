"""Observations with the fit's own and with given Gauss-Hermite centres: the
observables of each, the fit's centres afterwards, and several threads at once
(more than there are pinned blocks) against one after the other.

Both calls sum the same terms in FP64, each block's in the order its LDS
atomics arrive: a few rounding errors of 2^-52 of sum |w K| per deposit, far
below 1e-10 of it for 4096 particles; FP32 kernels are the same in both."""

import threading

import numpy as np
import pytest

from m2m_testlib import oracle_targets
from workloads import workload

pytestmark = pytest.mark.gpu


def make(wl, n, dtype, seed, stream=None):
    from paper_1202_2355_amd import Fit
    return Fit(wl.potential, wl.layout, wl.params, wl.initial_particles(n=n, seed=seed),
               dtype=dtype, stream=stream)


@pytest.mark.parametrize("dtype", ["f32", "f64"])
def test_given_centres_leave_the_fits_own(oracle, dtype):
    wl = workload(2)
    tg = oracle_targets(oracle, wl, n_target=1 << 14)
    f = make(wl, 4096, dtype, 11)
    f.set_targets(tg["Y"], tg["sigma"], tg["V_p"], tg["sigma_p"])
    own = f.observe()
    V, S = tg["V_p"] + 0.25, 1.5 * tg["sigma_p"]
    given = f.observe(V, S)
    again = f.observe()
    scale = np.abs(own).max()
    assert np.abs(again - own).max() <= 1e-10 * scale
    assert np.abs(given - own).max() > 1e-3 * scale
    g = make(wl, 4096, dtype, 11)
    g.set_targets(tg["Y"], tg["sigma"], V, S)
    assert np.abs(g.observe() - given).max() <= 1e-10 * scale


def test_more_threads_than_pinned_blocks():
    import torch
    wl = workload(3)
    fits = [make(wl, 20_000 + 77 * k, "f32", 20 + k, torch.cuda.Stream()) for k in range(6)]
    torch.cuda.synchronize()
    one = [f.observe() for f in fits]
    got = [[] for _ in fits]

    def run(k):
        for _ in range(8):
            got[k].append(fits[k].observe())

    th = [threading.Thread(target=run, args=(k,)) for k in range(len(fits))]
    for t in th:
        t.start()
    for t in th:
        t.join()
    for k, y in enumerate(one):
        assert len(got[k]) == 8
        for z in got[k]:
            assert np.abs(z - y).max() <= 1e-10 * np.abs(y).max()
