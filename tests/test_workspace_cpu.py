"""Sizes of a fit's workspace: what a batch and the server count against their
budgets."""

import pytest

from workloads import workload


def _layouts():
    v2, gh = workload(1), workload(2)
    losvd = dict(gh.layout, kin="losvd", n_r=50, n_R=40, n_v=64, v_min=-4.0, v_max=4.0, gh_nmax=0)
    alm = dict(gh.layout, dens="alm", l_max=4, n_r=60)
    scf = dict(gh.params, scf_lmax=4, scf_nr=32, scf_rmin=0.02, scf_rmax=100.0, scf_every=10)
    return {"v2": (v2.layout, v2.params), "gh": (gh.layout, gh.params),
            "losvd": (losvd, dict(gh.params, n_E=64, n_x=32)), "alm": (alm, gh.params),
            "scf": (gh.layout, scf), "scf losvd": (losvd, dict(scf, n_E=64, n_x=32))}


@pytest.mark.parametrize("kind", list(_layouts()))
def test_workspace_is_rows_and_tables(kind):
    """Tile rows of at most 16 bytes a particle (one row at least) and 2048 of them,
    the cell of every particle, and tables: 8192 steps of history, 8192 entries of the
    L_c table, and 16 values a column."""
    from paper_1202_2355_amd import _abi as A
    lay, par = _layouts()[kind]
    J = A.m2m_num_observables(lay)
    cols = J + 2 * par["n_E"] * par["n_x"] + (par.get("scf_nr", 0) * 2 * (par.get("scf_lmax", 0) + 1) ** 2)
    for n in (1, 1000, 4001, 20_000, 100_000, 1_000_000, 8_000_000):
        for dtype in ("f32", "f64"):
            ws = A.m2m_workspace_bytes(lay, par, n, dtype)
            assert 0 < ws <= max(16 * n, 8 * cols) + 2 * n + 8 * 2 * 8192 + 8 * 16 * cols + 65_536 + 48 * 2048
