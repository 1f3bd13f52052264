"""The few-row bf16 GEMM (decoding, LM head): one and two row tiles, both register-set sizes, remainders of the K loop."""
import numpy as np
import pytest
import torch

from tests.harness import rel_err, to_np

pytestmark = pytest.mark.gpu

# K steps per wavefront: K / 256.  Sets of four steps (K < 4096 or more than 512 column groups): shorter than two sets,
# two sets, a full round of the loop and remainders of one and two sets.  Sets of eight: the same from 16 steps on.
STEPS = [1, 2, 4, 5, 7, 8, 9, 13, 15, 16, 17, 25, 31, 32, 33, 45]


@pytest.mark.parametrize("epilogue", ["store", "add", "swiglu"])
@pytest.mark.parametrize("m", [1, 16, 17, 32])
@pytest.mark.parametrize("n,steps", [(48, s) for s in STEPS] + [(8208, 17), (8208, 8)])
def test_few_rows(m, n, steps, epilogue):
    from paper_2603_13289_amd import binding as rc
    k = 256 * steps
    g = torch.Generator(device="cuda")
    g.manual_seed(m * 131 + n + steps)
    a, w, u = (torch.empty(s, dtype=torch.bfloat16, device="cuda").normal_(generator=g) for s in ((m, k), (n, k), (n, k)))
    c0 = torch.empty((m, n), dtype=torch.float32, device="cuda").normal_(generator=g)
    gate, up = ((a.double() @ t.double().t()).cpu().numpy() for t in (w, u))
    epi, td, want, tol = {
        "store": (rc.RC_GEMM_STORE, torch.float32, gate, 2e-6 * np.sqrt(k)),
        "add": (rc.RC_GEMM_ADD, torch.float32, to_np(c0) + gate, 2e-6 * np.sqrt(k)),
        # result rounded to bf16 once (2^-9), __expf and the division on top
        "swiglu": (rc.RC_GEMM_SWIGLU, torch.bfloat16, gate / (1 + np.exp(-np.clip(gate, -700, 700))) * up, 4e-3),
    }[epilogue]
    c = c0.clone().to(td)
    rc.rc_gemm_rows_fused(rc.RC_BF16, epi, a, w, u if epilogue == "swiglu" else None, c, m, n, k, None)
    assert rel_err(to_np(c), want) <= tol
