"""The float GEMM: both of its variants (output blocks of 16, tiles of 64) at ragged sizes."""
import numpy as np
import pytest
import torch

from tests.harness import rel_err, to_np

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("epilogue", ["store", "add", "swiglu"])
@pytest.mark.parametrize("m,n,k", [(1, 1, 8), (17, 30, 24), (65, 1000, 688), (2051, 1030, 40), (1500, 1402, 264)])
def test_gemm_f32(m, n, k, epilogue):
    from paper_2603_13289_amd import binding as rc
    g = torch.Generator(device="cuda")
    g.manual_seed(m + n)
    a, w, u, c0 = (torch.empty(s, device="cuda").normal_(generator=g) for s in ((m, k), (n, k), (n, k), (m, n)))
    ad = to_np(a).astype(np.float64)
    prod = ad @ to_np(w).astype(np.float64).T
    want, epi = {"store": (prod, rc.RC_GEMM_STORE), "add": (to_np(c0) + prod, rc.RC_GEMM_ADD),
                 "swiglu": (prod / (1 + np.exp(-prod)) * (ad @ to_np(u).astype(np.float64).T), rc.RC_GEMM_SWIGLU)}[epilogue]
    c = c0.clone()
    rc.rc_gemm_rows_fused(rc.RC_F32, epi, a, w, u if epilogue == "swiglu" else None, c, m, n, k)
    # k roundings of 2^-24 of sums that grow like sqrt(k); the product of two such sums for the gated epilogue
    assert rel_err(to_np(c), want) <= (4e-6 if epilogue == "swiglu" else 2e-6) * max(np.sqrt(k), 4)
