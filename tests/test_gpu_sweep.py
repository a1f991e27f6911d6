"""Interleaved tiles taken forward and backward in turn: every particle is
pushed exactly once a step. Positions and velocities depend on no other
particle here (mu scales only the weights), so they equal the contiguous
tiles' to the last bit, at particle counts around whole rounds of chunks (a
tile's first or last chunk missing, one particle long, or whole)."""

import numpy as np
import pytest

from workloads import rng, workload

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("block", [256, 1024])
@pytest.mark.parametrize("extra", [-1, 0, 1])
@pytest.mark.parametrize("chunks", [1, 256, 257, 3 * 256 + 100])
def test_both_directions_push_every_particle_once(block, extra, chunks):
    from paper_1202_2355_amd import Fit, _abi, tuning
    wl = workload(3)
    n = chunks * block + extra
    g = rng(n)
    parts = {k: g.standard_normal(n) for k in ("x", "y", "z")}
    parts.update({k: 0.3 * g.standard_normal(n) for k in ("vx", "vy", "vz")})
    print("interleaved, block", block, "n", n, flush=True)
    before = tuning.current()
    out = {}
    try:
        tuning.apply(dict(before, block=block, tiles_per_cu=1))
        for il in (0, 1):
            _abi.m2m_set_interleave(il)
            f = Fit(wl.potential, wl.layout, wl.params, parts, dtype="f32")
            Y = f.observe()
            f.set_targets(Y, 0.05 * np.abs(Y) + 0.01 * np.abs(Y).max())
            for k in (1, 1, 3, 32):  # 32: a captured graph of steps
                f.step(k)
            out[il] = f.particles()
            f.close()
    finally:
        _abi.m2m_set_interleave(-1)
        tuning.apply(before)
    for k in ("x", "y", "z", "vx", "vy", "vz"):
        np.testing.assert_array_equal(out[1][k], out[0][k], err_msg=k)
    # one weight update a step as well: FP32 weights from sums of another order
    np.testing.assert_allclose(out[1]["u"], out[0]["u"], rtol=1e-5)
