"""Products that the library sends to a special schedule by itself, against the same product on a forced tile type: the same K partition,
hence the same bits."""
import pytest
import torch

pytestmark = pytest.mark.gpu

# a ragged last tile row on the thin body behind at least one full round; few rows whose K, no multiple of 256, is cut in parts
THIN = [(1025, 16384, 192, "store"), (1088, 16384, 64, "add"), (1089, 16384, 64, "add"), (769, 11000, 128, "swiglu"), (2050, 16640, 128, "swiglu")]
FEW = [(1, 512, 1408, "add"), (3, 512, 1408, "add"), (16, 48, 1984, "store"), (17, 512, 1408, "add"), (32, 1408, 576, "swiglu"),
       (5, 80, 4160, "swiglu"), (31, 2064, 1088, "store")]


@pytest.mark.parametrize("m,n,k,epilogue", THIN + FEW)
def test_same_bits_as_a_forced_tile_type(m, n, k, epilogue):
    from paper_2603_13289_amd import binding as rc
    g = torch.Generator(device="cuda")
    g.manual_seed(m * 31 + n)
    a, w, u = (torch.empty(s, dtype=torch.bfloat16, device="cuda").normal_(generator=g) for s in ((m, k), (n, k), (n, k)))
    c0 = torch.empty((m, n), dtype=torch.float32, device="cuda").normal_(generator=g)
    epi = {"store": rc.RC_GEMM_STORE, "add": rc.RC_GEMM_ADD, "swiglu": rc.RC_GEMM_SWIGLU}[epilogue]
    ws = rc.alloc_workspace(rc.rc_gemm_workspace_bytes())
    out = []
    for tile in (0, 9, 12):
        c = c0.to(torch.bfloat16) if epilogue == "swiglu" else c0.clone()
        rc.rc_tune_set(rc.RC_TUNE_GEMM_TILE, tile)
        try:
            rc.rc_gemm_rows_fused(rc.RC_BF16, epi, a, w, u if epilogue == "swiglu" else None, c, m, n, k, ws)
        finally:
            rc.rc_tune_set(rc.RC_TUNE_GEMM_TILE, 0)
        out.append(c)
    assert torch.equal(out[1], out[2])
    assert torch.equal(out[0], out[1])
    if epilogue == "store":
        want = a.double() @ w.double().t()
        assert float((out[0].double() - want).norm() / want.norm()) <= 2e-6 * k ** 0.5
