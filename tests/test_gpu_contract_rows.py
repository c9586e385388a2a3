"""On-site products whose contractions run in whole rows, against the fp64 oracle: k chunks that
end inside a degree and ragged ones (K = 16, 25, 49, 121), nodes, inputs and outputs that no tile
divides, one and several reduction slices, weights of both orders (input and output side), and the
accumulating and gathering projections of the general call. Tolerance: the fp32 bar of the other
parity tests (2e-5 of the largest output)."""
from __future__ import annotations

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


# 256 workgroups (16 nodes x 16 k x 64 outputs) or more in each contraction; the last three on both
# sides of that line
SHAPES = [(3, 4090, 20, 9), (4, 2050, 33, 70), (6, 1030, 64, 40), (10, 515, 70, 96),
          (3, 4080, 16, 16), (3, 4081, 16, 16), (6, 500, 130, 20)]


@pytest.mark.parametrize("lmax,n,C,R", SHAPES)
def test_contract_rows_onsite(cg, lmax, n, C, R):
    d = inputs.onsite_inputs(n, lmax, C, R, seed=700 + lmax, per_degree=True, distinct_out=True)
    rows = sample_rows(n, 12, seed=lmax)
    plan = cg.plan_create(lmax, C, R)
    got = run_onsite(cg, plan, to_dev(d, ONSITE_KEYS))
    ref = oracle.onsite(lmax, d["A"][rows], d["B"][rows], d["U_A"], d["U_B"], d["U_out_even"],
                        d["U_out_odd"])
    for a, b in zip(got, ref):
        assert rel_err(a[rows], b) <= TOL_F32


# both sides of the rules for one problem and for accumulating projections (R no multiple of 32):
# below and from 512 workgroups, 64 and 65 outputs, 127 and 128, below and from 3,072 products
@pytest.mark.parametrize("lmax,n,C,R", [(4, 2050, 20, 24), (6, 1030, 64, 64), (3, 4090, 9, 32),
                                        (4, 4090, 64, 24), (4, 4090, 65, 24), (4, 2045, 65, 24),
                                        (3, 4090, 127, 24), (3, 4090, 128, 24), (3, 4090, 47, 65),
                                        (3, 4090, 48, 63), (3, 4090, 48, 64)])
def test_contract_rows_general(cg, lmax, n, C, R):
    """Ranks of a multiple of 32 gather a sector's input rows, the others accumulate."""
    keys = ("A", "B", "A_flip", "B_flip", "U_A", "U_B", "U_out_even", "U_out_odd")
    d = inputs.general_onsite_inputs(n, lmax, C, R, seed=720 + lmax)
    rows = sample_rows(n, 8, seed=lmax)
    plan = cg.plan_create(lmax, C, R)
    t = to_dev(d, keys)
    got = cg.onsite_general(plan, t["A"], t["B"], t["U_A"], t["U_B"], t["U_out_even"],
                            t["U_out_odd"], A_flip=t["A_flip"], B_flip=t["B_flip"])
    ref = oracle.onsite(lmax, d["A"][rows], d["B"][rows], d["U_A"], d["U_B"], d["U_out_even"],
                        d["U_out_odd"], A_flip=d["A_flip"][rows], B_flip=d["B_flip"][rows])
    for a, b in zip(got, ref):
        assert rel_err(a[rows], b) <= TOL_F32
