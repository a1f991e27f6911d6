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
# in the counters of a fit's launches: blocks started, the same before the next
# launch, longest wait within a run, patience with blocks that do not start
START, START0, WAIT, PATIENCE = 0, 8, 16, 20


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
    torch.cuda.synchronize()
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
    wait = _sync(b, WAIT)
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


# (kind, dtype, particles, smoothed priors)
CALLED_OFF = [("gh", "f32", 1001, False), ("gh", "f32", 40_009, False), ("gh6", "f64", 20_011, False),
              ("losvd", "f32", 100_003, False), ("gh", "f32", 262_147, False), ("gh", "f32", 30_011, True),
              ("v2", "f64", 9001, True)]


def _smoothed(oracle, Fit, kin, dtype, n, smooth, **kw):
    wl = _workload(kin, 4)
    wl = wl.with_(params=dict(wl.params, smooth=int(smooth)))
    parts = cast(wl.initial_particles(n=n, seed=n % 97), dtype)
    return _fit(Fit, wl, parts, _targets(oracle, wl, parts, n), dtype, **kw)


def _same(a, b, dtype):
    tol = 1e-5 if dtype == "f32" else 1e-10
    np.testing.assert_allclose(b.chi2_history(), a.chi2_history(), rtol=10 * tol)
    pa, pb = a.particles(), b.particles()
    for c in pa:
        np.testing.assert_allclose(pb[c], pa[c], rtol=tol, atol=1e-5 if dtype == "f32" else 1e-11)


@pytest.fixture(scope="module")
def hog(oracle, Fit):
    """A fit whose step kernels hold every compute unit for 0.16 ms each."""
    wl = _workload("v2", 4)
    wl = wl.with_(layout=dict(wl.layout, dens="alm", l_max=8, n_r=20))
    parts = cast(wl.initial_particles(n=1_500_000, seed=1), "f32")
    f = Fit(wl.potential, wl.layout, wl.params, parts, dtype="f32", stream=torch.cuda.Stream())
    y = f.observe()
    f.set_targets(y, 0.05 * np.abs(y) + 1e-3 * np.abs(y).max())
    yield f
    f.close()


@pytest.mark.parametrize("kin,dtype,n,smooth", CALLED_OFF)
def test_a_launch_called_off_before_it_started(oracle, Fit, kin, dtype, n, smooth):
    """A launch marked as called off from the host: no block of it has started, so
    the last to leave does its steps, refreshes and the assignment carried over
    among them; the launches after it run as usual."""
    _say("marked", kin, dtype, n, smooth)
    a, b = (_smoothed(oracle, Fit, kin, dtype, n, smooth) for _ in range(2))
    for f in (a, b):
        f.step(3)
    blocks = int(_sync(b, START)[0])
    _sync(b, START).add_(-(1 << 31))
    for f in (a, b):
        f.step(7)
    assert int(_sync(b, START)[0]) == 2 * blocks and int(_sync(b, PATIENCE)[0]) > 1
    for f in (a, b):
        f.step(5)
    assert int(_sync(b, START)[0]) == 3 * blocks and int(_sync(b, PATIENCE)[0]) == 0
    _same(a, b, dtype)
    a.close()
    b.close()


@pytest.mark.parametrize("kin,dtype,n,smooth", CALLED_OFF)
def test_a_launch_called_off_is_done_by_the_blocks_that_started(oracle, Fit, hog, kin, dtype, n, smooth):
    """Launches without patience for blocks that have not started (set from the
    host) beside kernels that hold the compute units. Streams that share the
    other kernels' hardware queue never meet them, so several are tried."""
    _say("no patience", kin, dtype, n, smooth)
    off = 0
    for _ in range(8):
        a = _smoothed(oracle, Fit, kin, dtype, n, smooth)
        b = _smoothed(oracle, Fit, kin, dtype, n, smooth, stream=torch.cuda.Stream())
        for k in range(16):
            _sync(b, PATIENCE).fill_(1)
            torch.cuda.synchronize()
            hog.step(6)
            b.step(2 + k % 4)
            a.step(2 + k % 4)
            off += int(_sync(b, PATIENCE)[0]) > 1
        _same(a, b, dtype)
        a.close()
        b.close()
        if off > 1:
            break
    _say("called off", off)
    assert off > 0


@pytest.mark.parametrize("kin,dtype", [("gh", "f32"), ("v2", "f64"), ("losvd", "f32")])
def test_fits_of_a_batch_called_off_one_by_one(oracle, Fit, hog, kin, dtype):
    """A batch of uneven fits with different numbers of steps beside such kernels,
    some fits without patience, one marked as called off: blocks that start late
    find the steps that the fit had left, however far the others are."""
    from paper_1202_2355_amd.batch import Batch
    plan = [(40_009, 33), (1003, 9), (90_001, 60)] if kin != "losvd" else [(40_009, 33), (9001, 60)]
    _say("batch called off", kin, plan)
    off = 0
    for attempt in range(8):
        st = torch.cuda.Stream()
        b = Batch(max_fits=4, stream=st)
        ref, fits = [], []
        for n, steps in plan:
            r = _made(oracle, Fit, kin, dtype, n)
            r.step(steps)
            ref.append(r)
            f = _made(oracle, Fit, kin, dtype, n, stream=st)
            assert b.admit(f, steps)
            fits.append(f)
        for k in range(16):
            for j, f in enumerate(fits):
                if j != k % 3:
                    _sync(f, PATIENCE).fill_(1)
            if k == 2:
                _sync(fits[-1], START).add_(-(1 << 31))
            torch.cuda.synchronize()
            hog.step(6)
            b.run(4)
            off += sum(int(_sync(f, PATIENCE)[0]) > 1 for f in fits)
        done, left = b.poll()
        assert left == 0 and len(done) == len(plan)
        b.close()
        for f, r in zip(fits, ref):
            f.step(2)
            r.step(2)
            _same(r, f, dtype)
            f.close()
            r.close()
        if off > 3 + attempt:  # more than the marked ones
            break
    _say("called off", off)
    assert off > 3


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


def test_a_stream_with_few_compute_units(oracle, Fit):
    """On a stream that may use 64 compute units, a fit whose runs have more blocks
    takes its steps one launch each, alone and in a batch; a small fit runs."""
    import ctypes as C
    from paper_1202_2355_amd.batch import Batch
    hip = C.CDLL("libamdhip64.so")
    h = C.c_void_p()
    mask = (C.c_uint32 * 8)(0xffffffff, 0xffffffff)
    assert hip.hipExtStreamCreateWithCUMask(C.byref(h), 8, mask) == 0
    st = torch.cuda.ExternalStream(h.value)
    for n, runs in ((1001, True), (300_007, False)):
        _say("64 compute units", n)
        a = _made(oracle, Fit, "gh", "f32", n)
        b = _made(oracle, Fit, "gh", "f32", n, stream=st)
        for f in (a, b):
            f.step(9)
        assert (int(_sync(b, START)[0]) > 0) == runs and int(_sync(b, PATIENCE)[0]) == 0
        _same(a, b, "f32")
        q = Batch(max_fits=1, stream=st)
        assert q.admit(b, 4)
        before = int(_sync(b, START)[0])
        q.run(4)
        assert (int(_sync(b, START)[0]) > before) == runs and int(_sync(b, PATIENCE)[0]) == 0
        q.poll()
        q.close()
        a.step(4)
        _same(a, b, "f32")
        a.close()
        b.close()
    torch.cuda.synchronize()


def test_the_tags_of_a_stream_come_round(oracle, Fit):
    """Two fits on one stream take 4200 steps each, one after the other, in calls
    that refresh the priors: the first round of tags ends within the second."""
    _say("tags")
    st = torch.cuda.Stream()
    a, b = (_made(oracle, Fit, "v2", "f64", 3001, stream=st) for _ in range(2))
    for f in (a, b):
        for _ in range(20):
            f.step(210)
    np.testing.assert_allclose(b.chi2_history(), a.chi2_history(), rtol=1e-8)
    a.close()
    b.close()


def test_the_count_of_blocks_begins_again(oracle, Fit):
    """The count of blocks started, set near its end from the host (a fit with
    smoothed priors reads it on the device), and one launch more."""
    _say("count of blocks")
    a, b = (_smoothed(oracle, Fit, "gh", "f32", 20_011, True) for _ in range(2))
    for f in (a, b):
        f.step(3)
    blocks = int(_sync(b, START)[0])
    last = (1 << 30) - blocks
    for at in (START, START0):
        _sync(b, at).fill_(last)
    for f in (a, b):
        f.step(5)
    assert int(_sync(b, START)[0]) == int(_sync(b, START0)[0]) == 1 << 30
    for k in range(1, 3):
        for f in (a, b):
            f.step(4)
        assert int(_sync(b, START)[0]) == int(_sync(b, START0)[0]) == (k - 1) * blocks
    _same(a, b, "f32")
    a.close()
    b.close()


def test_exchange_memory_is_not_in_the_workspace():
    """The workspace of a fit that steps by runs has the counters of its launches
    more than that of one that does not (a refresh on every step)."""
    from paper_1202_2355_amd import _abi as A
    for kin in ("v2", "gh", "losvd"):
        wl = _workload(kin, 4)
        for n in (1, 4001, 1_000_000):
            for dtype in ("f32", "f64"):
                more = (A.m2m_workspace_bytes(wl.layout, wl.params, n, dtype)
                        - A.m2m_workspace_bytes(wl.layout, dict(wl.params, prior_every=1), n, dtype))
                assert 0 < more <= 256, (kin, n, dtype)


def test_batches_and_fits_share_a_stream(oracle, Fit):
    """A batch, then a larger fit on the batch's stream (its exchange memory does
    not hold the fit's), then the batch again; another stream takes up memory that
    a first one has left."""
    from paper_1202_2355_amd.batch import Batch
    for kin, dtype, small, large in (("gh", "f32", 20_011, 262_147), ("losvd", "f64", 3001, 150_001)):
        _say("one stream", kin, dtype)
        for _ in range(2):
            st = torch.cuda.Stream()
            ref = [_made(oracle, Fit, kin, dtype, n) for n in (small, small + 7, large)]
            fits = [_made(oracle, Fit, kin, dtype, n, stream=st) for n in (small, small + 7, large)]
            b = Batch(max_fits=2, stream=st)
            for f in fits[:2]:
                assert b.admit(f, 12)
            for k in range(3):
                b.run(4)
                fits[2].step(3 + k)
                for r in ref[:2]:
                    r.step(4)
                ref[2].step(3 + k)
            b.poll()
            b.close()
            for f, r in zip(fits, ref):
                _same(r, f, dtype)
                f.close()
                r.close()


def _alm(oracle, Fit, n, **kw):
    wl = _workload("gh", 4)
    wl = wl.with_(layout=dict(wl.layout, dens="alm", l_max=2, n_r=20))
    parts = cast(wl.initial_particles(n=n, seed=n % 97), "f32")
    f = Fit(wl.potential, wl.layout, wl.params, parts, dtype="f32", **kw)
    V, S = np.zeros(wl.layout["n_R"]), np.full(wl.layout["n_R"], 0.4)
    y = f.observe(V, S)
    f.set_targets(y, 0.05 * np.abs(y) + 1e-3 * np.abs(y).max(), V, S)
    return f


def test_a_batch_counts_state_and_workspace(oracle, Fit):
    """The budget is the particle state and the workspace of the fits, to the byte,
    also of fits that have stepped alone; with a budget for two fits exactly, the
    batch steps them without memory of its own and the results are the same."""
    from paper_1202_2355_amd import _abi as A
    from paper_1202_2355_amd.batch import Batch
    for made, n, dtype in ((lambda n: _made(oracle, Fit, "losvd", "f64", n), 5003, "f64"),
                           (lambda n: _made(oracle, Fit, "gh", "f32", n), 40_009, "f32"),
                           (lambda n: _alm(oracle, Fit, n), 5003, "f32")):
        _say("budget", n, dtype)
        fits = [made(n + k) for k in range(3)]
        ref = [made(n + k) for k in range(2)]
        for f in fits[:2] + ref:
            f.step(3)
        want = [(64 if dtype == "f64" else 32) * f.n + A.m2m_workspace_bytes(f.layout, f.params, f.n, dtype)
                for f in fits]
        for budget in (want[0] + want[1], 0):
            b = Batch(max_fits=3, hbm_budget=budget)
            assert b.admit(fits[0], 6) and b.footprint == want[0]
            assert b.admit(fits[1], 6) and b.footprint == want[0] + want[1]
            if budget:
                assert not b.admit(fits[2], 6)
            b.run(6)
            b.poll()
            b.close()
            for f in ref:
                f.step(6)
        b = Batch(max_fits=3, hbm_budget=want[0] + want[1] - 1)
        assert b.admit(fits[0], 6) and not b.admit(fits[1], 6)
        b.cancel(fits[0])
        b.close()
        for f, r in zip(fits, ref):
            _same(r, f, dtype)
        for f in fits + ref:
            f.close()


@pytest.mark.parametrize("first", ["eager", "captured"])
def test_steps_in_a_graph_outlive_the_rows_of_a_fit_alone(oracle, Fit, first):
    """Steps recorded into a caller's graph before or after eager steps (which take
    rows outside the workspace), replayed when the fit has been in a batch."""
    from paper_1202_2355_amd.batch import Batch
    _say("graph and batch", first)
    st = torch.cuda.Stream()
    a, b = _alm(oracle, Fit, 20_011), _alm(oracle, Fit, 20_011, stream=st)
    if first == "eager":
        b.step(3)
    torch.cuda.synchronize()
    g = torch.cuda.CUDAGraph()
    with torch.cuda.graph(g, stream=st):
        b.step(35)
    if first == "captured":
        b.step(3)
    a.step(3)
    for _ in range(2):
        q = Batch(max_fits=1, stream=st)
        assert q.admit(b, 4)
        q.run(4)
        q.poll()
        q.close()
        with torch.cuda.stream(st):
            g.replay()
        torch.cuda.synchronize()
        other = _alm(oracle, Fit, 20_011)  # takes up the rows that b has left
        other.step(3)
        with torch.cuda.stream(st):
            g.replay()
        b.step(1)
        other.step(40)
        a.step(4 + 35 + 35 + 1)
        torch.cuda.synchronize()
        _same(a, b, "f32")
        other.close()
    a.close()
    b.close()


@pytest.mark.parametrize("kin,n", [("v2", 9001), ("alm", 20_011)])
def test_long_calls_captured_into_a_graph(oracle, Fit, kin, n):
    """Calls of 32 steps and more (which a fit takes by graphs of its own, or by runs)
    recorded into a caller's graph, with eager steps between the replays."""
    _say("long captured calls", kin)
    st = torch.cuda.Stream()
    make = (lambda **k: _alm(oracle, Fit, n, **k)) if kin == "alm" else (
        lambda **k: _made(oracle, Fit, kin, "f64", n, **k))
    a, b = make(), make(stream=st)
    b.step(1)
    torch.cuda.synchronize()
    g = torch.cuda.CUDAGraph()
    with torch.cuda.graph(g, stream=st):
        b.step(70)
    a.step(1)
    for _ in range(3):
        with torch.cuda.stream(st):
            g.replay()
        b.step(33)
        a.step(103)
        torch.cuda.synchronize()
        np.testing.assert_allclose(b.chi2_history(), a.chi2_history(), rtol=1e-4 if kin == "alm" else 1e-9)
    a.close()
    b.close()
