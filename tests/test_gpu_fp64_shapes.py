"""FP64 site contractions at the edges of their tiles and stages, against the
product in numpy.  Bound per component: 2 K products and as many roundings of the
sum, 2^-53 each, times the sum of magnitudes."""
import os
import sys

import numpy as np
import pytest

sys.path.insert(0, os.path.dirname(os.path.dirname(os.path.abspath(__file__))))

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def ps():
    import torch
    if not torch.cuda.is_available():
        pytest.fail("no GPU")
    import paper_1905_08394_amd as p
    return p


@pytest.mark.parametrize("trans", [False, True])
@pytest.mark.parametrize("M,K1,K2,N", [
    (1, 1, 1, 1), (63, 7, 1, 31), (64, 8, 1, 32), (65, 9, 1, 33),      # K-major, one and two stages
    (128, 1, 8, 16), (129, 1, 9, 17), (127, 3, 5, 15), (200, 4, 3, 40),  # odd K2, k past the end
    (128, 2, 8, 64), (256, 3, 8, 64), (300, 2, 24, 70),                # even and odd numbers of whole stages
])
def test_fp64_site(ps, M, K1, K2, N, trans):
    import torch
    print(f"fp64 M={M} K1={K1} K2={K2} N={N} trans={trans}", flush=True)
    rng = np.random.default_rng(M + 7 * K1 + 11 * K2 + N)
    A = rng.standard_normal((3, K1, M, K2)) + 1j * rng.standard_normal((3, K1, M, K2))
    W = rng.standard_normal((K1 * K2, N)) + 1j * rng.standard_normal((K1 * K2, N))
    C = ps.contract_site("fp64", torch.from_numpy(A.reshape(-1)).cuda(), W, M, K1, K2, N, batch=3, transpose_out=trans)
    flat = A.transpose(0, 2, 1, 3).reshape(3, M, K1 * K2)
    ref = flat @ W
    got = C.cpu().numpy().reshape((3, N, M) if trans else (3, M, N))
    if trans:
        got = got.transpose(0, 2, 1)
    mag = lambda x: np.abs(x.real) + np.abs(x.imag)  # noqa: E731
    bound = (2 * (4 * K1 * K2 + 4)) * 2.0 ** -53 * (mag(flat) @ mag(W))
    d = got - ref
    assert np.all(np.abs(d.real) <= bound) and np.all(np.abs(d.imag) <= bound)
