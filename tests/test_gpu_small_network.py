"""Small networks, whose rows run whole in LDS, against the oracle: lattices at
the edges of the rule (boundaries of 2 and 8 sites, rows that one workgroup
takes, rows spread over their v values, the largest tensors that fit), with the
amplitude bars of parity_bars."""
import os
import sys

import numpy as np
import pytest

HERE = os.path.dirname(os.path.abspath(__file__))
sys.path[:0] = [os.path.dirname(HERE), HERE]

import rqcgen  # noqa: E402
from oracle import peps as opeps  # noqa: E402
from oracle import statevector as sv  # noqa: E402
from parity_bars import BAR, report  # noqa: E402

pytestmark = pytest.mark.gpu

FORMS = [("fp64", False), ("fp32", False), ("fp32", True), ("fp32_3m", False), ("fp32_3m", True)]
LATTICES = [
    (2, 2, 5, 16), (9, 2, 16, 40),          # two sites in a row
    (3, 6, 19, 33), (4, 4, 16, 50),         # bonds of 2, 4 and 8; whole rows
    (4, 5, 24, 20), (5, 4, 21, 7),          # spread rows, tensors of 4096 elements and mixed bonds
    (4, 3, 32, 9), (3, 3, 37, 5),           # bonds of 16 and 32 on three sites
    (5, 5, 20, 3),                          # the largest that fits in FP32; general path in FP64
]


@pytest.fixture(scope="module")
def ps():
    import torch
    if not torch.cuda.is_available():
        pytest.fail("no GPU")
    import paper_1905_08394_amd as p
    return p


@pytest.mark.parametrize("lv,lh,d,n", LATTICES)
def test_against_the_oracle(ps, lv, lh, d, n):
    c = rqcgen.generate(lv, lh, d, 3)
    bits = rqcgen.all_bitstrings(4) if lv * lh == 4 else rqcgen.bitstrings(lv, lh, 3, n)
    ref = sv.amplitudes(sv.run(c), bits) if lv * lh <= 20 else opeps.amplitudes(opeps.build(c), bits)
    peps = ps.Peps(c)
    for prec, split in FORMS:
        print(f"small {lv}x{lh} d{d} {prec} split={split}", flush=True)
        plan = ps.Plan(peps, prec=prec, split_acc=split, max_batch=len(bits), graph=True)
        a = plan.amplitudes(bits)
        assert report(f"small {lv}x{lh} {prec} {split}", a, ref, lv * lh) <= BAR[prec]
        # replays of the captured sweep, and a bitstring of the batch alone
        assert np.array_equal(plan.amplitudes(bits), a)
        assert np.array_equal(plan.amplitudes(bits[1:2]), a[1:2])
        plan.close()


def test_boundary_of_eight_sites(ps):
    c = rqcgen.generate(8, 8, 8, 1)
    bits = rqcgen.bitstrings(8, 8, 1, 3)
    ref = opeps.amplitudes(opeps.build(c), bits)
    for prec, split in FORMS:
        print(f"small 8x8 {prec} split={split}", flush=True)
        a = ps.Plan(ps.Peps(c), prec=prec, split_acc=split, max_batch=3).amplitudes(bits)
        assert report(f"small 8x8 {prec} {split}", a, ref, 64) <= BAR[prec]


def test_group_of_spread_and_whole_rows(ps):
    """Plans of every form in one group: each plan's own amplitudes bit for bit."""
    plans, bits = [], []
    for k, (lv, lh, d, n) in enumerate(LATTICES):
        prec, split = FORMS[k % len(FORMS)]
        c = rqcgen.generate(lv, lh, d, 3)
        bits.append(rqcgen.all_bitstrings(4) if lv * lh == 4 else rqcgen.bitstrings(lv, lh, 3, n))
        plans.append(ps.Plan(ps.Peps(c), prec=prec, split_acc=split, max_batch=len(bits[-1])))
    want = [p.amplitudes(b) for p, b in zip(plans, bits)]
    group = ps.Group(plans)
    for _ in range(2):
        got = group.amplitudes(bits)
        assert all(np.array_equal(g, w) for g, w in zip(got, want))
    group.close()


def test_error_estimate_of_a_small_plan(ps):
    """The companion sweep of a plan with sums over 64 products differs from it; with sums over at most 16 it cannot."""
    bits = rqcgen.bitstrings(4, 5, 3, 20)
    _, est = ps.Plan(ps.Peps(rqcgen.generate(4, 5, 24, 3)), prec="fp32", max_batch=20).amplitudes(bits, rel_err=True)
    assert np.all(np.isfinite(est)) and 0 < np.median(est) < 1e-5
    _, est = ps.Plan(ps.Peps(rqcgen.generate(4, 5, 16, 3)), prec="fp32", max_batch=20).amplitudes(bits, rel_err=True)
    assert np.all(est == 0)
