"""The folded on-site kernels against the fp64 oracle over their degrees: every register and LDS
shape (lmax 0 to 20; 21 takes the matrix-core kernel, and so do few rows from 15), rank blocks with
remainders, and grids off the default one, whose Gauss-Legendre rows are not held in registers. fp32
bar of the other parity tests (2e-5 of the largest output)."""
from __future__ import annotations

import numpy as np
import pytest

import oracle
from paper_2605_15073_amd import inputs
from tests.gpu_util import ONSITE_KEYS, TOL_F32, rel_err, run_onsite, sample_rows, to_dev

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def cg():
    import torch

    assert torch.cuda.is_available(), "GPU tests need a GPU"
    import paper_2605_15073_amd as lib

    lib.load_library()
    return lib


@pytest.mark.parametrize("grid", ["default", "finer"])
@pytest.mark.parametrize("lmax,R", [(0, 3), (1, 70), (2, 8), (3, 43), (7, 22), (8, 20), (10, 17),
                                    (11, 15), (13, 13), (15, 12), (16, 11), (17, 1), (18, 10),
                                    (19, 9), (20, 9), (21, 3)])
def test_folded_onsite(cg, lmax, R, grid):
    d = inputs.onsite_inputs(3, lmax, 4, R, seed=500 + lmax, per_degree=True, distinct_out=True)
    kw = {} if grid == "default" else dict(n_theta=(3 * lmax + 3) // 2 + 5, n_phi=3 * lmax + 4)
    plan = cg.plan_create(lmax, 4, R, **kw)
    got = run_onsite(cg, plan, to_dev(d, ONSITE_KEYS))
    ref = oracle.onsite(lmax, d["A"], d["B"], d["U_A"], d["U_B"], d["U_out_even"], d["U_out_odd"])
    for a, b in zip(got, ref):
        assert rel_err(a, b) <= TOL_F32 or np.abs(b).max() == 0.0


@pytest.mark.parametrize("lmax,n,R", [(15, 64, 8), (15, 57, 9), (16, 96, 16), (16, 140, 11),
                                      (17, 64, 16), (17, 70, 15), (18, 41, 25), (19, 60, 18),
                                      (20, 1, 1), (20, 128, 8), (20, 79, 13)])
def test_onsite_rows(cg, lmax, n, R):
    """Degrees that the matrix-core kernel serves for few (node, rank) rows and the folded one for
    more: the last row count of the one and the first of the other."""
    d = inputs.onsite_inputs(n, lmax, 4, R, seed=540 + lmax, per_degree=True, distinct_out=True)
    rows = sample_rows(n, 4, seed=lmax)
    plan = cg.plan_create(lmax, 4, R)
    got = run_onsite(cg, plan, to_dev(d, ONSITE_KEYS))
    ref = oracle.onsite(lmax, d["A"][rows], d["B"][rows], d["U_A"], d["U_B"], d["U_out_even"],
                        d["U_out_odd"])
    for a, b in zip(got, ref):
        assert rel_err(a[rows], b) <= TOL_F32


@pytest.mark.parametrize("n,R,extra", [(1, 1, 0), (5, 300, 0), (5, 300, 4), (700, 17, 0)])
def test_degree_zero(cg, n, R, extra):
    """The constant product: even output against the oracle, odd output zero."""
    d = inputs.onsite_inputs(n, 0, 4, R, seed=580, per_degree=True, distinct_out=True)
    kw = dict(n_theta=1 + extra, n_phi=1 + extra) if extra else {}
    got = run_onsite(cg, cg.plan_create(0, 4, R, **kw), to_dev(d, ONSITE_KEYS))
    ref = oracle.onsite(0, d["A"], d["B"], d["U_A"], d["U_B"], d["U_out_even"], d["U_out_odd"])
    assert rel_err(got[0], ref[0]) <= TOL_F32
    assert float(got[1].abs().max()) == 0.0 and np.abs(ref[1]).max() == 0.0


@pytest.mark.parametrize("lmax,nu,extra", [(0, 2, 0), (3, 2, 0), (5, 3, 0), (9, 4, 0), (10, 4, 3),
                                           (4, 3, 6)])
def test_folded_nbody(cg, lmax, nu, extra):
    R = 11
    d = inputs.nbody_inputs(3, lmax, 4, R, seed=600 + lmax, nu=nu, self_coupled=False)
    nt, nph = cg.nbody_grid(lmax, nu)
    plan = cg.plan_create(lmax, 4, R, n_theta=nt + extra, n_phi=nph + extra)
    dev = to_dev({f"x{i}": x for i, x in enumerate(d["X"])} | {f"u{i}": u for i, u in
                 enumerate(d["U"])} | {"o": d["U_out"]},
                 [f"x{i}" for i in range(nu)] + [f"u{i}" for i in range(nu)] + ["o"])
    got = cg.onsite_nbody(plan, [dev[f"x{i}"] for i in range(nu)],
                          [dev[f"u{i}"] for i in range(nu)], dev["o"])
    ref = oracle.nbody(lmax, d["X"], d["U"], d["U_out"])
    assert rel_err(got, ref) <= TOL_F32


# Relative 2-norm errors against 64 bits, in 1e-7, that the sweep of the grid's own azimuths shows
# on these inputs (the folded one at half steps: 1.60 for two operands at lmax 2, the others 2.00,
# 2.26 and 2.05), and 1% for sums in another order.
GRID_AZIMUTHS = {(2, 2): 1.42, (2, 3): 2.01, (3, 4): 2.18, (4, 3): 1.93}


@pytest.mark.parametrize("lmax,nu", sorted(GRID_AZIMUTHS))
def test_low_degree_error(cg, lmax, nu):
    """The azimuths of the folded kernels are no further from 64 bits than the grid's own."""
    errors = []
    for seed in (1, 2, 3):
        if nu == 2:
            d = inputs.onsite_inputs(3000, lmax, 8, 8, seed=seed, per_degree=False,
                                     distinct_out=True)
            got = run_onsite(cg, cg.plan_create(lmax, 8, 8), to_dev(d, ONSITE_KEYS))[0]
            ref = oracle.onsite(lmax, d["A"], d["B"], d["U_A"], d["U_B"], d["U_out_even"],
                                d["U_out_odd"])[0]
        else:
            d = inputs.nbody_inputs(2000, lmax, 8, 8, seed=seed, nu=nu, self_coupled=False)
            nt, nph = cg.nbody_grid(lmax, nu)
            dev = to_dev({f"x{i}": x for i, x in enumerate(d["X"])} |
                         {f"u{i}": u for i, u in enumerate(d["U"])} | {"o": d["U_out"]},
                         [f"x{i}" for i in range(nu)] + [f"u{i}" for i in range(nu)] + ["o"])
            got = cg.onsite_nbody(cg.plan_create(lmax, 8, 8, n_theta=nt, n_phi=nph),
                                  [dev[f"x{i}"] for i in range(nu)],
                                  [dev[f"u{i}"] for i in range(nu)], dev["o"])
            ref = oracle.nbody(lmax, d["X"], d["U"], d["U_out"])
        errors.append(np.linalg.norm(got.cpu().numpy() - ref) / np.linalg.norm(ref))
    assert np.mean(errors) <= 1.01e-7 * GRID_AZIMUTHS[lmax, nu], errors
