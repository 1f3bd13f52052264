"""Products that the library sends to a special schedule by itself, against the same product on a forced tile type: the same K partition,
hence the same bits.  (That the shapes take these schedules: test_gemm_plan.py.)"""
import pytest
import torch

pytestmark = pytest.mark.gpu

# Products of other tile types: a ragged last tile row, with too few K steps for the thin body to pay; few rows, whole over K
OTHER = [(1025, 16384, 192, "store"), (1088, 16384, 64, "add"), (1089, 16384, 64, "add"), (769, 11000, 128, "swiglu"), (2050, 16640, 128, "swiglu"),
         (32, 1408, 576, "swiglu"), (31, 2064, 1088, "store")]
# a ragged last tile row on the thin body behind at least one full round, every tile summed whole
THIN = [(1025, 16384, 1024, "store"), (1088, 28672, 512, "add"), (1025, 14336, 512, "swiglu"), (1088, 14336, 1024, "swiglu")]
# the same where only the missing workspace leaves them whole
THIN_WHOLE = [(1025, 16384, 2048, "store"), (1088, 16384, 2048, "add"), (2112, 16384, 2048, "swiglu")]
# few rows whose K, no multiple of 256, is cut in parts: 4 to 16 of them, one and two row tiles; 16 parts of gate/up and 32 rows fill
# the 64 KB of LDS that a launch may ask for
FEW = [(1, 512, 1408, "add"), (3, 512, 1408, "add"), (16, 48, 1984, "store"), (17, 512, 1408, "add"), (5, 80, 4160, "swiglu"),
       (32, 512, 4160, "swiglu"), (32, 80, 1984, "swiglu"), (29, 16, 1984, "swiglu")]


@pytest.mark.parametrize("m,n,k,epilogue,workspace", [(*c, True) for c in OTHER + THIN + FEW] + [(*c, False) for c in THIN_WHOLE])
def test_same_bits_as_a_forced_tile_type(m, n, k, epilogue, workspace):
    from paper_2603_13289_amd import binding as rc
    g = torch.Generator(device="cuda")
    g.manual_seed(m * 31 + n)
    a, w, u = (torch.empty(s, dtype=torch.bfloat16, device="cuda").normal_(generator=g) for s in ((m, k), (n, k), (n, k)))
    c0 = torch.empty((m, n), dtype=torch.float32, device="cuda").normal_(generator=g)
    epi = {"store": rc.RC_GEMM_STORE, "add": rc.RC_GEMM_ADD, "swiglu": rc.RC_GEMM_SWIGLU}[epilogue]
    ws = rc.alloc_workspace(rc.rc_gemm_workspace_bytes()) if workspace else None
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
