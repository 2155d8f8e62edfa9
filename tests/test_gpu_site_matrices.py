"""Site matrices built on the device: a doubled site (computed there from the
layer it doubles) against the same site held as a plain tensor on the host, in
every form that plans read, both sweeps and the square partition.

The two differ by the rounding of sums of four products, 2^-53 each, per site;
FP32 forms round the same values to within one unit of 2^-24."""
import os
import sys

import numpy as np
import pytest

sys.path.insert(0, os.path.dirname(os.path.dirname(os.path.abspath(__file__))))

import rqcgen  # noqa: E402

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def ps():
    import torch
    if not torch.cuda.is_available():
        pytest.fail("no GPU")
    import paper_1905_08394_amd as p
    return p


def _doubled(ps, lv, lh, d):
    rng = np.random.default_rng(5)
    P = ps.Peps(rqcgen.generate(lv, lh, d, 2))
    ops = rng.standard_normal((lv * lh, 2, 2, 2)) + 1j * rng.standard_normal((lv * lh, 2, 2, 2))
    return P, ops


@pytest.mark.parametrize("lv,lh,d", [(2, 3, 16), (4, 3, 13), (3, 4, 16)])
@pytest.mark.parametrize("prec,sweep", [("fp64", 1), ("fp64", 2), ("fp64", 3), ("fp32", 1), ("fp32_3m", 2),
                                        ("fp32_3m", 3), ("bf16x3", 1), ("bf16x3", 2)])
def test_doubled_site_equals_its_tensor(ps, lv, lh, d, prec, sweep):
    print(f"site matrices {lv}x{lh} d{d} {prec} sweep {sweep}", flush=True)
    P, ops = _doubled(ps, lv, lh, d)
    bits = rqcgen.bitstrings(lv, lh, 1, 6)
    a = ps.Plan(P.double_layer(ops), prec=prec, sweep=sweep, max_batch=6).amplitudes(bits)
    held = P.double_layer(ops)
    held.apply([])                       # no gates: the sites become plain tensors
    b = ps.Plan(held, prec=prec, sweep=sweep, max_batch=6).amplitudes(bits)
    tol = {"fp64": 1e-12, "fp32": 2e-5, "fp32_3m": 2e-5, "bf16x3": 1e-3}[prec]
    assert np.max(np.abs(a - b)) <= tol * np.max(np.abs(b))


def test_changes_to_a_doubled_network(ps):
    """Projection, gates and another double layer on a double-layer network."""
    P, ops = _doubled(ps, 2, 2, 9)
    bits = rqcgen.all_bitstrings(4)
    V = P.double_layer(ops)
    a = ps.Plan(V, prec="fp64", max_batch=16).amplitudes(bits)
    scale = np.max(np.abs(a))
    eye = np.zeros((4, 2, 2, 2), dtype=complex)
    eye[:, :] = np.eye(2)
    twice = ps.Plan(V.double_layer(eye), prec="fp64").amplitudes(np.zeros((1, 4), dtype=np.uint8))[0]
    assert abs(twice - np.sum(np.abs(a) ** 2)) <= 1e-12 * np.sum(np.abs(a) ** 2)
    V.apply([rqcgen.Gate(0, "U1", 1, -1, [1.0, 0, 0, 0, 0, 0, 1.0, 0])])
    assert np.max(np.abs(ps.Plan(V, prec="fp64", max_batch=16).amplitudes(bits) - a)) <= 1e-12 * scale
    W = P.double_layer(ops)
    W.project(2, 1)
    b = ps.Plan(W, prec="fp64", max_batch=16).amplitudes(bits)
    keep = bits[:, 2] == 1
    assert np.max(np.abs(b[keep] - a[keep])) <= 1e-12 * scale and not np.any(b[~keep])
