"""The float GEMM: its variants (output blocks of 16, tiles of 64 and of 128) at ragged sizes."""
import numpy as np
import pytest
import torch

from tests.harness import TOL, rel_err, to_np

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


@pytest.mark.parametrize("epilogue", ["store", "add", "swiglu"])
@pytest.mark.parametrize("m,n,k", [(2100, 2060, 1032), (3000, 2900, 40)])
def test_gemm_f32_large_tile(m, n, k, epilogue):
    """The 128 x 128 tile (one workgroup per compute unit and more for K from 1024 on, two below) at ragged sizes."""
    test_gemm_f32(m, n, k, epilogue)


def test_prefill_f32_large_tile():
    """A float prefill whose gate/up product takes the large tile, RMS norm and gain inside the product."""
    from oracle import relay_oracle as R
    from paper_2603_13289_amd import binding as rc
    from synth import ModelShape, Workload, make_hidden, make_weights
    t, sh = 1530, ModelShape(2, 1024, 8, 2, 128, 1408, 512, 1.0e4, dtype="f32")
    w = Workload("f32_large_tile", sh, t, 0, 0, 0, 1, 1, 0)
    weights = make_weights(w)
    g = np.random.default_rng(5)
    for lw in weights["layers"]:
        lw["g_attn"], lw["g_ffn"] = (g.uniform(0.5, 1.5, sh.d_model).astype(np.float32) for _ in range(2))
    x = make_hidden(w, "x", t)
    want = R.full_prefill(R.OracleModel.from_shape(sh, weights), x)
    model = rc.rc_model_create(sh, weights)
    dst = rc.PagedKV.contiguous(2, 1, t, 2, 128, rc.RC_F32)
    logits = torch.zeros((1, sh.vocab), dtype=torch.float32, device="cuda")
    rc.rc_prefill(model, [torch.from_numpy(x).cuda()], [0], dst, logits, rc.alloc_workspace(rc.rc_prefill_workspace_bytes(model, [t])))
    for l in range(2):
        assert rel_err(to_np(dst.read("k", l, 0, t)), want.k_cache[l]) <= TOL["f32"]
        assert rel_err(to_np(dst.read("v", l, 0, t)), want.v_cache[l]) <= TOL["f32"]
    assert rel_err(to_np(logits)[0], want.logits) <= TOL["f32"]
    model.close()
