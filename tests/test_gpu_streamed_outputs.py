"""Outputs on both sides of the size from which a site's stores bypass the caches
(2^25 complex numbers): the rows of one node equal the same node alone, bit for
bit, whichever store wrote them."""
import os
import sys

import numpy as np
import pytest

sys.path.insert(0, os.path.dirname(os.path.dirname(os.path.abspath(__file__))))

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("prec,split", [("fp32_3m", True), ("fp32_4m", False), ("bf16x3", False)])
@pytest.mark.parametrize("M,K1,K2,N", [(4096, 8, 8, 64), (4096, 8, 1, 64), (4097, 2, 8, 66)])
def test_streamed_stores(prec, split, M, K1, K2, N):
    import torch
    if not torch.cuda.is_available():
        pytest.fail("no GPU")
    import paper_1905_08394_amd as ps
    print(f"streamed {prec} split={split} M={M} K1={K1} K2={K2} N={N}", flush=True)
    nb = (1 << 25) // (M * N) + 2
    gen = torch.Generator("cuda").manual_seed(M + K1 + N)
    A = torch.randn(nb * K1 * M * K2, dtype=torch.complex64, device="cuda", generator=gen)
    W = np.random.default_rng(N).standard_normal((K1 * K2, N)) + 0.5j
    C = ps.contract_site(prec, A, W, M, K1, K2, N, batch=nb, split_acc=split).view(nb, M, N)
    for z in (0, nb - 1):
        one = ps.contract_site(prec, A.view(nb, -1)[z].contiguous(), W, M, K1, K2, N, split_acc=split).view(M, N)
        assert torch.equal(torch.view_as_real(C[z]).view(torch.int32), torch.view_as_real(one).view(torch.int32))
