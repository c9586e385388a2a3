"""The products on three bf16 parts against the fp64 oracle at a bound that a missing part product
fails, and the ranks that the values-only receiver adds on a workspace full of NaN.

A product of two operands in three parts each leaves out terms of 2^-26. Without any one of the six
part products that are formed, its relative 2-norm error is 2.2e-6 or more (the emulation below).
The whole calls measure 2e-7 to 4e-7 on site and, with radial degrees up to l in message passing,
about 2e-7 + 1e-7 l: so degrees up to 10 at most are given coefficients, of both groups of 8 that
the parts are then laid out in (from degree 16 on the recurrence's own error, 3e-6 and more, would
hide a missing product; the third group differs from the others in its lanes only)."""
from __future__ import annotations

import numpy as np
import pytest

import oracle
from paper_2605_15073_amd import inputs
from tests.gpu_util import MP_KEYS, ONSITE_KEYS, run_onsite, sample_rows, to_dev

BOUND = 1.5e-6


@pytest.fixture(scope="module")
def cg():
    import torch

    assert torch.cuda.is_available(), "GPU tests need a GPU"
    import paper_2605_15073_amd as lib

    lib.load_library()
    return lib


def _norm_err(got, ref):
    return float(np.linalg.norm(got.cpu().numpy() - ref) / np.linalg.norm(ref))


def _bf16(x):
    """Round to nearest even to the 8 significant bits of bf16."""
    u = x.astype(np.float32).view(np.uint32)
    return ((u + (((u >> 16) & 1) + 0x7fff)) & 0xffff0000).astype(np.uint32).view(np.float32)


def test_a_missing_part_product_shows():
    rng = np.random.default_rng(0)
    for n in (5, 33, 128):
        W = rng.standard_normal((200, n)).astype(np.float32)
        X = rng.standard_normal((n, 300)).astype(np.float32)
        split = []
        for x in (W, X):
            h = _bf16(x)
            m = _bf16(x - h)
            split.append([h.astype(np.float64), m.astype(np.float64),
                          _bf16(x - h - m).astype(np.float64)])
        exact = W.astype(np.float64) @ X.astype(np.float64)
        formed = [(0, 0), (0, 1), (1, 0), (1, 1), (0, 2), (2, 0)]

        def err(pairs):
            got = sum(split[0][i] @ split[1][j] for i, j in pairs)
            return np.linalg.norm(got - exact) / np.linalg.norm(exact)

        assert err(formed) < 1e-8
        for gone in formed:
            assert err([p for p in formed if p != gone]) > 1.4 * BOUND


# lmax and the radial degrees that are not zero
DEGREES = [(5, range(6)), (7, range(8)), (9, range(10)), (10, range(11)), (12, range(7)),
           (13, (8, 9)), (17, range(7)), (18, (8, 9)), (24, range(7)), (24, (8, 10))]


@pytest.mark.gpu
@pytest.mark.parametrize("slots", ["one", "two", "blocks"])
@pytest.mark.parametrize("lmax,degrees", DEGREES, ids=lambda x: str(x).replace(" ", ""))
def test_receiver_parts(cg, lmax, degrees, slots):
    n, C, R = 300 if lmax < 15 else 60, 5, 48
    kw = dict(seed=900 + lmax, r_cut=2.6)
    d = (inputs.general_mp_inputs(n, lmax, C, R, flip=True, **kw) if slots == "blocks" else
         inputs.mp_inputs(n, lmax, C, R, distinct_out=True, two_slot=slots == "two", **kw))
    keep = np.zeros(lmax + 1, bool)
    keep[list(degrees)] = True
    d["edge_radial"][:, :, ~keep] = 0
    rows = sample_rows(n, 8 if lmax < 15 else 3, seed=lmax)
    plan = cg.plan_create(lmax, C, R)
    t = to_dev(d, MP_KEYS)
    flip = d.get("node_flip")
    if flip is not None:
        t["node_flip"] = to_dev(d, ("node_flip",))["node_flip"]
    call = cg.message_pass_general if slots == "blocks" else cg.message_pass
    got = call(plan, *(t[k] for k in MP_KEYS), node_flip=t.get("node_flip"))
    ref = oracle.message_pass(lmax, *(d[k] for k in MP_KEYS), receivers=rows, node_flip=flip)
    errors = [_norm_err(a[rows], b) for a, b in zip(got, ref)]
    assert max(errors) <= BOUND, errors


@pytest.mark.gpu
@pytest.mark.parametrize("lmax,n,C,R", [(3, 4090, 20, 9), (4, 2050, 33, 70), (6, 1030, 64, 40),
                                        (10, 515, 70, 96)])
def test_contraction_parts(cg, lmax, n, C, R):
    """Both contractions of an on-site call in whole rows."""
    d = inputs.onsite_inputs(n, lmax, C, R, seed=700 + lmax, per_degree=True, distinct_out=True)
    rows = sample_rows(n, 12, seed=lmax)
    got = run_onsite(cg, cg.plan_create(lmax, C, R), to_dev(d, ONSITE_KEYS))
    ref = oracle.onsite(lmax, d["A"][rows], d["B"][rows], d["U_A"], d["U_B"], d["U_out_even"],
                        d["U_out_odd"])
    errors = [_norm_err(a[rows], b) for a, b in zip(got, ref)]
    assert max(errors) <= BOUND, errors


@pytest.mark.gpu
@pytest.mark.parametrize("slots", ["one", "two", "blocks"])
@pytest.mark.parametrize("lmax,R,n", [(2, 9, 60), (4, 40, 900), (5, 9, 900), (6, 40, 60),
                                      (9, 40, 300), (13, 9, 80), (17, 40, 60)])
def test_padded_ranks_on_nan_workspace(cg, lmax, R, n, slots):
    """The ranks added to fill the receiver's tiles are not all written before they are read;
    whatever the workspace holds there reaches no output."""
    import torch

    C = 5
    kw = dict(seed=950 + lmax, r_cut=2.6)
    d = (inputs.general_mp_inputs(n, lmax, C, R, flip=True, **kw) if slots == "blocks" else
         inputs.mp_inputs(n, lmax, C, R, distinct_out=True, two_slot=slots == "two", **kw))
    plan = cg.plan_create(lmax, C, R)
    t = to_dev(d, MP_KEYS + (("node_flip",) if slots != "one" else ()))
    E = t["col"].shape[0]
    if slots == "blocks":
        size = cg.workspace_bytes_general(plan, cg.CGTP_OP_MESSAGE_PASS_GENERAL, n, E, 2,
                                          1 if d["U_E"].ndim == 3 else d["U_E"].shape[0],
                                          1 if d["U_out_even"].ndim == 3 else d["U_out_even"].shape[0])
    else:
        op = cg.CGTP_OP_MESSAGE_PASS_TWO_SLOT if slots == "two" else cg.CGTP_OP_MESSAGE_PASS
        size = cg.workspace_bytes(plan, op, n, E)
    call = cg.message_pass_general if slots == "blocks" else cg.message_pass
    outs = []
    for fill in (0, 255):  # zeros; NaN in fp32 and in bf16
        ws = torch.full((size,), fill, dtype=torch.uint8, device="cuda")
        outs.append(call(plan, *(t[k] for k in MP_KEYS), node_flip=t.get("node_flip"),
                         workspace=ws))
    for a, b in zip(*outs):
        assert bool(torch.isfinite(a).all()) and torch.equal(a, b)
