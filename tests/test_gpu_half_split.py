"""Site contractions of FP32 plans on the half-precision matrix units: every
operand split into two halves, three products per real product, FP32 sums.

Bound, per real component of an output, with S = sum |a| |w| over its real
products: the split leaves |a - hi - lo| <= 2^-23 |a| (likewise w) and drops
lo * lo <= 2^-22 |a| |w|, together 2^-21 S; each of the 6 K / 16 matrix
instructions of a component adds 16 products in at most four roundings of the
running sum, 2^-24 S each (twice that if it truncates); partial sums add one
rounding per two stages, and the scaled result one more.
"""
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


def _inputs(M, K1, K2, N, batch, scales, w_scale=1.0):
    rng = np.random.default_rng(M + 31 * K1 + 7 * K2 + N)
    A = rng.standard_normal((batch, K1, M, K2)) + 1j * rng.standard_normal((batch, K1, M, K2))
    A *= np.asarray(scales, dtype=float).reshape(batch, 1, 1, 1)
    W = (rng.standard_normal((K1 * K2, N)) + 1j * rng.standard_normal((K1 * K2, N))) * w_scale
    return A.astype(np.complex64), W.astype(np.complex64)


def _bound(A, W):
    """(batch, M, N): S and the exact product."""
    batch, K1, M, K2 = A.shape
    K = K1 * K2
    A = A.astype(complex).transpose(0, 2, 1, 3).reshape(batch, M, K)
    W = W.astype(complex)
    mag = lambda x: np.abs(x.real) + np.abs(x.imag)  # noqa: E731  bounds both components' sums
    tol = 2.0 ** -21 + 2.0 ** -23 * (4 * 6 * K / 16 + K / 32 + 1)
    return A @ W, tol * (mag(A) @ mag(W))


def _check(C, A, W):
    ref, bound = _bound(A, W)
    d = C.astype(complex).reshape(ref.shape) - ref
    assert np.all(np.abs(d.real) <= bound) and np.all(np.abs(d.imag) <= bound)


SHAPES = [
    (1, 1, 16, 1), (127, 1, 16, 63), (128, 2, 16, 64), (129, 3, 16, 65),    # tile edges; 1, 2 and 3 stages
    (130, 8, 2, 5), (64, 4, 4, 129), (257, 6, 8, 127),                      # stages of several k1 blocks
    (33, 1, 48, 128), (300, 5, 64, 200),                                    # several stages per k1 block
]


@pytest.mark.parametrize("prec,split", [("fp32", False), ("fp32", True), ("fp32_3m", False), ("fp32_3m", True)])
@pytest.mark.parametrize("M,K1,K2,N", SHAPES)
def test_edges_of_tiles_and_stages(ps, prec, split, M, K1, K2, N):
    import torch
    print(f"half split {prec} split={split} M={M} K1={K1} K2={K2} N={N}", flush=True)
    A, W = _inputs(M, K1, K2, N, 3, [1.0, 2.0 ** -90, 2.0 ** 60], 2.0 ** 40)
    C = ps.contract_site(prec, torch.from_numpy(A.reshape(-1)).cuda(), W.astype(complex), M, K1, K2, N, batch=3,
                         split_acc=split).cpu().numpy().reshape(3, M, N)
    for z in range(3):   # each batch entry has its own scale
        _check(C[z:z + 1], A[z:z + 1], W)


def test_large_tile_and_its_group(ps):
    """Enough tiles for the 128 x 128 form; every batch entry alone takes the
    128 x 64 form and gives the same bits."""
    import torch
    M, K1, K2, N, batch = 4096, 2, 16, 256, 16
    A, W = _inputs(M, K1, K2, N, batch, np.ones(batch))
    Ad = torch.from_numpy(A.reshape(batch, -1)).cuda()
    C = ps.contract_site("fp32_3m", Ad.reshape(-1), W.astype(complex), M, K1, K2, N, batch=batch)
    _check(C.reshape(batch, M, N)[5:6].cpu().numpy(), A[5:6], W)
    for z in (0, 5, 15):
        one = ps.contract_site("fp32_3m", Ad[z].contiguous(), W.astype(complex), M, K1, K2, N)
        assert torch.equal(one, C.reshape(batch, -1)[z])


def test_strides_alignment_zero_and_non_finite(ps):
    import torch
    M, K1, K2, N = 200, 2, 16, 40
    A, W = _inputs(M, K1, K2, N, 2, [1.0, 1e-3])
    Wc = W.astype(complex)
    flat = torch.from_numpy(A.reshape(2, -1)).cuda()
    want = ps.contract_site("fp32_3m", flat.reshape(-1), Wc, M, K1, K2, N, batch=2)
    # entries further apart than their size; the gap holds NaN
    gap = torch.full((2, flat.shape[1] + 6), complex("nan"), dtype=torch.complex64, device="cuda")
    gap[:, :-6] = flat
    got = ps.contract_site("fp32_3m", gap.reshape(-1), Wc, M, K1, K2, N, batch=2, a_batch_stride=gap.shape[1])
    assert torch.equal(got, want)
    # a start that is not a multiple of 16 bytes, and an odd stride: the FP32 kernels, same bound
    off = torch.zeros(2 * flat.shape[1] + 1, dtype=torch.complex64, device="cuda")
    off[1:] = flat.reshape(-1)
    _check(ps.contract_site("fp32_3m", off[1:], Wc, M, K1, K2, N, batch=2).cpu().numpy(), A, W)
    odd = torch.zeros(2, flat.shape[1] + 1, dtype=torch.complex64, device="cuda")
    odd[:, :-1] = flat
    got = ps.contract_site("fp32_3m", odd.reshape(-1), Wc, M, K1, K2, N, batch=2, a_batch_stride=odd.shape[1])
    _check(got.cpu().numpy(), A, W)
    # all zeros, in A and in W
    assert not ps.contract_site("fp32_3m", torch.zeros_like(flat[0]), Wc, M, K1, K2, N).abs().max().item()
    assert not ps.contract_site("fp32_3m", flat[0].contiguous(), 0 * Wc, M, K1, K2, N).abs().max().item()
    # an infinity or NaN stays in its row and does not set the others' scale
    for bad in (complex("inf"), complex("nan")):
        b = flat[0].clone().reshape(K1, M, K2)
        b[1, 7, 3] = 0
        clean = ps.contract_site("fp32_3m", b.reshape(-1).clone(), Wc, M, K1, K2, N).reshape(M, N)
        b[1, 7, 3] = bad
        dirty = ps.contract_site("fp32_3m", b.reshape(-1).clone(), Wc, M, K1, K2, N).reshape(M, N)
        rows = [m for m in range(M) if m != 7]
        assert torch.equal(dirty[rows], clean[rows])
        assert not torch.isfinite(torch.view_as_real(dirty[7])).any()


@pytest.mark.parametrize("M,K1,N,batch", [(257, 6, 127, 2), (128, 2, 64, 1), (1, 4, 1, 1), (4096, 2, 256, 16)])
def test_bf16x3_equals_the_register_staged_kernel(ps, M, K1, N, batch):
    """BF16x3 on these units against the kernel that takes K = 8 (mod 16): one
    more k1 of zero products leaves every sum, so the results agree bit for bit."""
    import torch
    print(f"bf16x3 M={M} K1={K1} N={N} batch={batch}", flush=True)
    A, W = _inputs(M, K1, 8, N, batch, np.ones(batch))
    C = ps.contract_site("bf16x3", torch.from_numpy(A.reshape(-1)).cuda(), W.astype(complex), M, K1, 8, N, batch=batch)
    A2 = np.concatenate([A, np.zeros_like(A[:, :1])], axis=1)
    W2 = np.concatenate([W, np.zeros_like(W[:8])], axis=0)
    C2 = ps.contract_site("bf16x3", torch.from_numpy(A2.reshape(-1)).cuda(), W2.astype(complex), M, K1 + 1, 8, N,
                          batch=batch)
    assert torch.equal(C, C2)
