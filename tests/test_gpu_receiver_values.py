"""The values-only message-passing receiver against the fp64 oracle at the edges of its tiling:
degree groups of 4, 8, 16 and 24 slots (lmax 3/4, 7/8, 15/16, 24), ranks padded to 16 and odd
numbers of rank tiles, the form that splits a receiver's edges over waves (small problems) and
the one that does not, each with one node slot, two slots and per-block factors. Tolerance: the
fp32 bar of the other parity tests (2e-5 of the largest output)."""
from __future__ import annotations

import numpy as np
import pytest

import oracle
from paper_2605_15073_amd import inputs
from tests.gpu_util import MP_KEYS, TOL_F32, rel_err, run_mp, sample_rows, to_dev

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def cg():
    import torch

    assert torch.cuda.is_available(), "GPU tests need a GPU"
    import paper_2605_15073_amd as lib

    lib.load_library()
    return lib


def _tiles(n, lmax, R):
    """Rank tiles x point tiles of all receivers: below 16384 (8192 with a single rank tile) the
    edges are split over waves."""
    uv = ((3 * lmax + 3) // 2) * (3 * lmax + 1)
    return n * ((R + 15) // 16) * ((uv + 31) // 32 * 2)


# (lmax, ranks, nodes): the first five split the edges, the others do not
SHAPES = [(0, 16, 60), (3, 9, 60), (7, 40, 40), (15, 16, 20), (24, 24, 20),
          (3, 16, 4200), (4, 100, 1100), (8, 48, 400), (16, 16, 300), (16, 72, 80)]


@pytest.mark.parametrize("slots", ["one", "two", "blocks"])
@pytest.mark.parametrize("lmax,R,n", SHAPES)
def test_receiver_values_tiles(cg, lmax, R, n, slots):
    split = _tiles(n, lmax, R) < (8192 if R <= 16 else 16384)
    assert split == (SHAPES.index((lmax, R, n)) < 5)
    check_receiver(cg, lmax, R, n, slots)


def check_receiver(cg, lmax, R, n, slots):
    C, r_cut = 5, 2.6
    rows = sample_rows(n, 10 if lmax < 15 else 3, seed=lmax)
    if slots == "blocks":
        d = inputs.general_mp_inputs(n, lmax, C, R, seed=300 + lmax, flip=True, r_cut=r_cut)
        plan = cg.plan_create(lmax, C, R)
        t = to_dev(d, MP_KEYS + ("node_flip",))
        got = cg.message_pass_general(plan, *(t[k] for k in MP_KEYS), node_flip=t["node_flip"])
    else:
        d = inputs.mp_inputs(n, lmax, C, R, seed=300 + lmax, r_cut=r_cut, distinct_out=True,
                             two_slot=slots == "two")
        plan = cg.plan_create(lmax, C, R)
        t = to_dev(d, MP_KEYS)
        kw = {}
        if slots == "two":
            kw["node_flip"] = to_dev(d, ("node_flip",))["node_flip"]
        got = run_mp(cg, plan, t, **kw)
    ref = oracle.message_pass(lmax, *(d[k] for k in MP_KEYS), receivers=rows,
                              node_flip=d.get("node_flip"))
    for a, b in zip(got, ref):
        assert rel_err(a[rows], b) <= TOL_F32


# Rank tiles that no group of two or four divides, one per way they are cut (3; 3 + 2; 4 + 3; with
# half a wave's tiles 2 + 1), a single one, and rows whose point tiles four do not divide (lmax 5
# and 7), each at a degree of one, two and three degree groups; nodes for the form that splits the
# edges and for the one that does not.
CUTS = [(5, 32, 30), (5, 32, 900), (7, 16, 500), (17, 80, 20), (17, 80, 60), (6, 112, 400),
        (9, 48, 200), (10, 144, 80), (20, 16, 150)]


@pytest.mark.parametrize("slots", ["one", "two", "blocks"])
@pytest.mark.parametrize("lmax,R,n", CUTS)
def test_receiver_values_cut_ranks(cg, lmax, R, n, slots):
    check_receiver(cg, lmax, R, n, slots)


# The form on fp32 products at every rest of its reduction steps of four degrees (lmax 5, 6, 7, 8),
# at the degrees of its one-step-shorter derivative sums (lmax 4, 8, 20), at the last degree, and on
# both sides of its rule: a single rank tile against two, lmax 4 and 8 against 5 and 9, and with
# per-block factors lmax 11, 12, 15 and 16. Ranks that no tile divides leave columns unwritten.
F32_SHAPES = [(1, 100, 700), (4, 16, 30), (4, 112, 700), (5, 10, 1000), (6, 16, 40), (7, 15, 600),
              (8, 64, 300), (8, 16, 30), (9, 16, 400), (11, 48, 120), (12, 32, 120), (15, 24, 90),
              (16, 33, 90), (20, 12, 90), (24, 16, 60), (24, 40, 40)]


@pytest.mark.parametrize("slots", ["one", "two", "blocks"])
@pytest.mark.parametrize("lmax,R,n", F32_SHAPES)
def test_receiver_values_f32(cg, lmax, R, n, slots):
    check_receiver(cg, lmax, R, n, slots)


@pytest.mark.parametrize("slots", ["one", "two", "blocks"])
@pytest.mark.parametrize("lmax,R", [(24, 16), (24, 48)])
def test_receiver_values_four_groups(cg, lmax, R, slots):
    """Few nodes on both sides of the degree from which a workgroup's waves do not share edges."""
    check_receiver(cg, lmax, R, 18, slots)


@pytest.mark.parametrize("n,lmax,R", [(17, 9, 16), (100, 12, 32), (130, 12, 32), (300, 9, 16)])
def test_sender_rank_blocks(cg, n, lmax, R):
    """The tiled sender's rank blocks of 4, 8 and 16 (fewer ranks with fewer nodes)."""
    check_receiver(cg, lmax, R, n, "one")


def test_receiver_without_edges_among_others(cg):
    """Receivers with no edges give zeros in both forms; the others are unchanged."""
    for n, lmax, R in ((40, 5, 32), (900, 5, 64)):
        d = inputs.mp_inputs(n, lmax, 4, R, seed=77, r_cut=1.2, distinct_out=True)
        assert (np.diff(d["row_ptr"]) == 0).any() and d["n_edges"] > 0
        plan = cg.plan_create(lmax, 4, R)
        got = run_mp(cg, plan, to_dev(d, MP_KEYS))
        ref = oracle.message_pass(lmax, *(d[k] for k in MP_KEYS))
        empty = np.diff(d["row_ptr"]) == 0
        for a, b in zip(got, ref):
            assert rel_err(a, b) <= TOL_F32
            assert float(a[np.where(empty)[0]].abs().max()) == 0.0
