"""Last sites of a row (transposed stores of up to 32 columns) on their own kernel,
against the general path (A off 16 bytes, the same products and sums in the same
order: bit for bit) and against the product in numpy: per component 2 K products
and as many roundings, 2^-24 each, times the sum of magnitudes, plus the rounding
of the operands (2 2^-24)."""
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


@pytest.mark.parametrize("prec,split", [("fp32_4m", False), ("fp32_4m", True), ("bf16x3", False)])
@pytest.mark.parametrize("M,K1,K2,N", [
    (1, 2, 8, 1), (127, 2, 8, 7), (128, 8, 4, 16), (129, 3, 16, 17),   # edges of the 128 x 16 and 128 x 32 tiles
    (130, 8, 2, 15), (256, 4, 16, 32), (300, 2, 48, 31),               # even and odd numbers of stages
])
def test_last_site(ps, prec, split, M, K1, K2, N):
    import torch
    print(f"last {prec} split={split} M={M} K1={K1} K2={K2} N={N}", flush=True)
    rng = np.random.default_rng(M + 7 * K1 + 11 * N + K2)
    nb = 3
    A = (rng.standard_normal((nb, K1, M, K2)) + 1j * rng.standard_normal((nb, K1, M, K2))).astype(np.complex64)
    W = rng.standard_normal((K1 * K2, N)) + 1j * rng.standard_normal((K1 * K2, N))
    buf = torch.empty(A.size + 1, dtype=torch.complex64, device="cuda")
    out = []
    for off in (0, 1):
        a = buf[off:off + A.size]
        a.copy_(torch.from_numpy(A.reshape(-1)))
        out.append(ps.contract_site(prec, a, W, M, K1, K2, N, batch=nb, transpose_out=True,
                                    split_acc=split).cpu().numpy().reshape(nb, N, M))
    flat = A.astype(np.complex128).transpose(0, 2, 1, 3).reshape(nb, M, K1 * K2)
    ref = (flat @ W).transpose(0, 2, 1)
    mag = lambda x: np.abs(x.real) + np.abs(x.imag)  # noqa: E731
    bound = (4 * K1 * K2 + 2) * 2.0 ** -24 * (mag(flat) @ mag(W)).transpose(0, 2, 1)
    d = out[0] - ref
    assert np.all(np.abs(d.real) <= bound) and np.all(np.abs(d.imag) <= bound)
    np.testing.assert_array_equal(out[0].view(np.int32), out[1].view(np.int32))
