"""First sites of a row (K2 = 1) on their own kernel, against the general path
and against the product in numpy.

The general path takes the same call when A starts at an odd complex number (8
bytes off 16); its products and sums are the same, in the same order, for FP32 4M
and BF16x3, so those results agree bit for bit.  Against numpy, per component: 2 K
products and as many roundings of the sum, 2^-24 each, times the sum of
magnitudes, plus the rounding of the operands (2 2^-24)."""
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


@pytest.mark.parametrize("prec,split", [("fp32_4m", False), ("fp32_4m", True), ("fp32_3m", False), ("fp32_3m", True),
                                        ("bf16x3", False)])
@pytest.mark.parametrize("M,K1,N", [
    (2, 8, 1), (126, 8, 63), (128, 16, 64), (130, 24, 65),   # one, two and three stages; edges of the 128 x 64 tiles
    (256, 32, 1024), (512, 40, 100),                          # several tiles, even and odd numbers of stages
])
def test_first_site(ps, prec, split, M, K1, N):
    import torch
    print(f"first {prec} split={split} M={M} K1={K1} N={N}", flush=True)
    rng = np.random.default_rng(M + 7 * K1 + 11 * N)
    nb = 3
    A = (rng.standard_normal((nb, K1, M)) + 1j * rng.standard_normal((nb, K1, M))).astype(np.complex64)
    W = rng.standard_normal((K1, N)) + 1j * rng.standard_normal((K1, N))
    buf = torch.empty(nb * K1 * M + 1, dtype=torch.complex64, device="cuda")
    out = []
    for off in (0, 1):
        a = buf[off:off + nb * K1 * M]
        a.copy_(torch.from_numpy(A.reshape(-1)))
        out.append(ps.contract_site(prec, a, W, M, K1, 1, N, batch=nb, split_acc=split).cpu().numpy().reshape(nb, M, N))
    flat = A.astype(np.complex128).transpose(0, 2, 1)
    ref = flat @ W
    mag = lambda x: np.abs(x.real) + np.abs(x.imag)  # noqa: E731
    bound = (4 * K1 + 2) * 2.0 ** -24 * (mag(flat) @ mag(W))
    d = out[0] - ref
    assert np.all(np.abs(d.real) <= bound) and np.all(np.abs(d.imag) <= bound)
    if prec != "fp32_3m":
        np.testing.assert_array_equal(out[0].view(np.int32), out[1].view(np.int32))
