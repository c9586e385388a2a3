"""Operands at the ends of the fp32 range where products run on three bf16 parts: the whole-row
contraction (on-site calls of 256 workgroups and more) and the edge coefficients of the values-only
receiver. The parts lose bits below 2^-109 and have no infinity; a contraction then falls back to
fp32, and a finite coefficient stays finite. Reference: the fp64 oracle, with the fp32 bar of the
other parity tests, and for infinite weights the call on few nodes, which k_contract_mfma serves."""
from __future__ import annotations

import numpy as np
import pytest

import oracle
from paper_2605_15073_amd import inputs
from tests.gpu_util import MP_KEYS, ONSITE_KEYS, TOL_F32, rel_err, run_mp, run_onsite, sample_rows, to_dev

pytestmark = pytest.mark.gpu

LMAX, N, C, R = 4, 2050, 33, 40


@pytest.fixture(scope="module")
def cg():
    import torch

    assert torch.cuda.is_available(), "GPU tests need a GPU"
    import paper_2605_15073_amd as lib

    lib.load_library()
    return lib


def _onsite(seed):
    return inputs.onsite_inputs(N, LMAX, C, R, seed=seed, per_degree=True, distinct_out=True)


@pytest.mark.parametrize("key,shift", [("A", -100), ("A", -112), ("A", -120), ("U_A", -112),
                                       ("U_out_even", -115), ("A", 110), ("U_out_odd", 100)])
def test_scaled_operand(cg, key, shift):
    """A whole operand scaled by a power of two scales the outputs and keeps their error."""
    d = _onsite(800)
    d[key] = np.ldexp(d[key], shift).astype(np.float32)
    rows = sample_rows(N, 8, seed=1)
    got = run_onsite(cg, cg.plan_create(LMAX, C, R), to_dev(d, ONSITE_KEYS))
    ref = oracle.onsite(LMAX, d["A"][rows], d["B"][rows], d["U_A"], d["U_B"], d["U_out_even"],
                        d["U_out_odd"])
    for a, b in zip(got, ref):
        assert rel_err(a[rows], b) <= TOL_F32


def test_tiny_nodes_among_others(cg):
    """Some nodes' inputs tiny: those nodes keep their error too."""
    d = _onsite(801)
    rows = np.array([0, 17, 1000, N - 1])
    d["A"][rows] = np.ldexp(d["A"][rows], -120)
    got = run_onsite(cg, cg.plan_create(LMAX, C, R), to_dev(d, ONSITE_KEYS))
    ref = oracle.onsite(LMAX, d["A"][rows], d["B"][rows], d["U_A"], d["U_B"], d["U_out_even"],
                        d["U_out_odd"])
    for a, b in zip(got, ref):
        for i in range(len(rows)):
            assert rel_err(a[rows[i]], b[i]) <= TOL_F32


@pytest.mark.parametrize("value", [np.inf, -np.inf, 3.4e38, np.nan])
def test_weights_past_bf16(cg, value):
    """An output weight that is infinite, NaN or finite above bf16's largest value: every output is
    what the call on a few of the nodes gives, infinities with their signs."""
    d = _onsite(802)
    d["A"] *= np.float32(1e-3)
    d["U_out_even"][2, 5, 7] = value
    few = 30
    plan = cg.plan_create(LMAX, C, R)
    even, odd = (x.cpu().numpy() for x in run_onsite(cg, plan, to_dev(d, ONSITE_KEYS)))
    part = {k: (v[:few] if k in ("A", "B") else v) for k, v in d.items() if k in ONSITE_KEYS}
    even_few, odd_few = (x.cpu().numpy() for x in run_onsite(cg, plan, to_dev(part, ONSITE_KEYS)))
    assert np.isfinite(odd).all() and rel_err(odd[:few], odd_few) <= TOL_F32
    hit = np.zeros(even.shape, bool)
    hit[:, 5, 4:9] = True                       # channel 5, degree 2
    assert np.isfinite(even[~hit]).all()
    assert rel_err(np.where(hit[:few], 0, even[:few]), np.where(hit[:few], 0, even_few)) <= TOL_F32
    a, b = even[:few][hit[:few]], even_few[hit[:few]]
    if np.isfinite(value):
        assert np.isfinite(a).all() and rel_err(a, b) <= TOL_F32
    elif np.isnan(value):
        assert np.isnan(a).all() and np.isnan(b).all()
    else:
        assert np.isinf(a).all() and np.array_equal(a, b)


@pytest.mark.parametrize("shift", [-100, 60])
def test_scaled_edge_radial(cg, shift):
    """Edge coefficients in three parts over the range in which these are exact."""
    d = inputs.mp_inputs(700, 6, 5, 32, seed=803, r_cut=2.6, distinct_out=True)
    d["edge_radial"] = np.ldexp(d["edge_radial"], shift).astype(np.float32)
    rows = sample_rows(700, 8, seed=2)
    got = run_mp(cg, cg.plan_create(6, 5, 32), to_dev(d, MP_KEYS))
    ref = oracle.message_pass(6, *(d[k] for k in MP_KEYS), receivers=rows)
    for a, b in zip(got, ref):
        assert rel_err(a[rows], b) <= TOL_F32


def test_edge_coefficient_past_bf16(cg):
    """A coefficient of 3.4e38, finite in fp32 and above bf16's largest value (its derivative sum
    overflows, so the odd output does; the even one is finite)."""
    lmax, n = 6, 700
    d = inputs.mp_inputs(n, lmax, 1, 32, seed=804, r_cut=2.6, distinct_out=True)
    d["edge_radial"][:] = 0
    d["edge_radial"][:, 0, lmax] = 3.4e38 * 4 * np.pi / (2 * lmax + 1)
    d["U_E"][:] = 1
    d["node_feat"] *= np.float32(1e-35)
    rows = sample_rows(n, 8, seed=3)
    got = run_mp(cg, cg.plan_create(lmax, 1, 32), to_dev(d, MP_KEYS))
    ref = oracle.message_pass(lmax, *(d[k] for k in MP_KEYS), receivers=rows)
    assert rel_err(got[0][rows], ref[0]) <= TOL_F32
