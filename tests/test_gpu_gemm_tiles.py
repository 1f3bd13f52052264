"""All tile types of the bf16 GEMM: the same K partition, hence the same bits, at the edges of the tiles."""
import numpy as np
import pytest
import torch

from tests.harness import rel_err, to_np

pytestmark = pytest.mark.gpu

SHAPES = [(1, 8, 64), (33, 1000, 64), (64, 136, 128), (65, 520, 192), (193, 384, 320), (257, 777, 448), (385, 2064, 1024)]


@pytest.mark.parametrize("epilogue", ["store", "add", "swiglu"])
@pytest.mark.parametrize("m,n,k", SHAPES)
def test_every_tile_type_gives_the_same_bits(m, n, k, epilogue):
    """One K step, odd and even numbers of K steps, ragged rows and columns; K is too short here to be cut in parts."""
    from paper_2603_13289_amd import binding as rc
    g = torch.Generator(device="cuda")
    g.manual_seed(m * 31 + n)
    a, w, u = (torch.empty(s, dtype=torch.bfloat16, device="cuda").normal_(generator=g) for s in ((m, k), (n, k), (n, k)))
    c0 = torch.empty((m, n), dtype=torch.float32, device="cuda").normal_(generator=g)
    prod = to_np(a).astype(np.float64) @ to_np(w).astype(np.float64).T
    epi, td, want, tol = {
        "store": (rc.RC_GEMM_STORE, torch.float32, prod, 2e-6 * np.sqrt(k)),
        "add": (rc.RC_GEMM_ADD, torch.float32, to_np(c0) + prod, 2e-6 * np.sqrt(k)),
        # result rounded to bf16 once (2^-9), __expf and the division on top
        "swiglu": (rc.RC_GEMM_SWIGLU, torch.bfloat16,
                   prod / (1 + np.exp(-prod)) * (to_np(a).astype(np.float64) @ to_np(u).astype(np.float64).T), 4e-3),
    }[epilogue]
    ws = rc.alloc_workspace(rc.rc_gemm_workspace_bytes())
    # a workspace allows K parts to the partition that 5 and 6 fix for themselves: they join without one
    for work, tiles in ((None, (5, 6, 8, 9, 10, 11, 12, 13)), (ws, (8, 9, 10, 11, 12, 13))):
        first = None
        for tile in tiles:
            c = c0.clone().to(td)
            rc.rc_tune_set(rc.RC_TUNE_GEMM_TILE, tile)
            try:
                rc.rc_gemm_rows_fused(rc.RC_BF16, epi, a, w, u if epilogue == "swiglu" else None, c, m, n, k, work)
            finally:
                rc.rc_tune_set(rc.RC_TUNE_GEMM_TILE, 0)
            assert rel_err(to_np(c), want) <= tol, tile
            first = c if first is None else first
            assert torch.equal(c, first), tile


CUT = [(100, 4096, 4096, "store"), (193, 4096, 14336, "add"), (65, 777, 8192, "store"), (1100, 4100, 8192, "add"),
       (200, 1000, 4096, "swiglu"), (1639, 4096, 14336, "store"), (5120, 4096, 4096, "add")]


@pytest.mark.parametrize("m,n,k,epilogue", CUT)
def test_every_tile_type_gives_the_same_bits_in_k_parts(m, n, k, epilogue):
    """Products whose K range is cut: all tiles in the same parts (193 rows: with two types that do not fit the workspace
    and stand back) and, the last one, whole tiles with a cut rest."""
    from paper_2603_13289_amd import binding as rc
    cus = torch.cuda.get_device_properties(0).multi_processor_count
    g = torch.Generator(device="cuda")
    g.manual_seed(m * 31 + n)
    a, w, u = (torch.empty(s, dtype=torch.bfloat16, device="cuda").normal_(generator=g) for s in ((m, k), (n, k), (n, k)))
    c0 = torch.empty((m, n), dtype=torch.float32, device="cuda").normal_(generator=g)
    prod = a.double() @ w.double().t()
    epi, td, want, tol = {
        "store": lambda: (rc.RC_GEMM_STORE, torch.float32, prod, 2e-6 * np.sqrt(k)),
        "add": lambda: (rc.RC_GEMM_ADD, torch.float32, c0.double() + prod, 2e-6 * np.sqrt(k)),
        # result rounded to bf16 once (2^-9), __expf and the division on top
        "swiglu": lambda: (rc.RC_GEMM_SWIGLU, torch.bfloat16, prod * torch.sigmoid(prod) * (a.double() @ u.double().t()), 4e-3),
    }[epilogue]()
    ws = rc.alloc_workspace(rc.rc_gemm_workspace_bytes())
    wide = [rc.rc_gemm_plan_check(m, n, k, epilogue == "swiglu", 8, cus, parts) for parts in (True, False)]
    assert wide[0][1] > wide[1][1]          # K is cut: more workgroups than tiles
    first = None
    for tile in (0, 8, 9, 10, 11, 12, 13):
        assert rc.rc_gemm_plan_check(m, n, k, epilogue == "swiglu", tile, cus, True)[0] == 0, tile
        c = c0.clone().to(td)
        rc.rc_tune_set(rc.RC_TUNE_GEMM_TILE, tile)
        try:
            rc.rc_gemm_rows_fused(rc.RC_BF16, epi, a, w, u if epilogue == "swiglu" else None, c, m, n, k, ws)
        finally:
            rc.rc_tune_set(rc.RC_TUNE_GEMM_TILE, 0)
        assert float((c.double() - want).abs().max() / want.abs().max()) <= tol, tile
        first = c if first is None else first
        assert torch.equal(c, first), tile
