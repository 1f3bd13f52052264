"""Few-row products in workgroups of 32 columns: a row gets the bits it gets in a product of four rows, which takes workgroups of 16."""
from types import SimpleNamespace

import numpy as np
import pytest
import torch

from tests.harness import rel_err, to_np

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("epilogue", ["store", "add"])
@pytest.mark.parametrize("n,k,rows", [(5120, 5120, (5, 16, 17, 32)), (6144, 4096, (12, 15, 31)), (7168, 8192, (5, 20)),
                                      (8160, 4352, (7, 25)), (8192, 4096, (24, 32)), (10272, 4096, (29,))])
def test_rows_in_company_have_the_bits_of_four_rows(n, k, rows, epilogue):
    from paper_2603_13289_amd import binding as rc
    g = torch.Generator(device="cuda")
    g.manual_seed(n + k)
    a, w = (torch.empty(s, dtype=torch.bfloat16, device="cuda").normal_(generator=g) for s in ((max(rows), k), (n, k)))
    c0 = torch.empty((max(rows), n), dtype=torch.float32, device="cuda").normal_(generator=g)
    epi = rc.RC_GEMM_STORE if epilogue == "store" else rc.RC_GEMM_ADD
    ws = rc.alloc_workspace(rc.rc_gemm_workspace_bytes())

    def product(first, m):
        c = c0[first:first + m].clone()
        rc.rc_gemm_rows_fused(rc.RC_BF16, epi, a[first:first + m].contiguous(), w, None, c, m, n, k, ws)
        return c

    few = torch.cat([product(r, min(4, max(rows) - r)) for r in range(0, max(rows), 4)])
    want = a.double() @ w.double().t() + (c0.double() if epilogue == "add" else 0)
    assert float((few.double() - want).abs().max() / want.abs().max()) <= 2e-6 * np.sqrt(k)
    for m in rows:
        assert torch.equal(product(0, m), few[:m]), m


@pytest.mark.parametrize("n", [12, 17, 32])
def test_rotated_and_scattered_rows(n):
    """q|k|v of 6144 columns in a decoding step: the first layer's rows in the cache, bit for bit, and the second layer's: with O the identity, no
    feed-forward sum and KV ranges in one piece its inputs are the embeddings and the first layer's attention, which shows every rotated query."""
    from paper_2603_13289_amd import binding as rc
    g = torch.Generator(device="cuda")
    g.manual_seed(n)
    d, ffn, nq, nkv, page = 4096, 256, 32, 8, 16
    rnd = lambda *s: torch.empty(s, dtype=torch.bfloat16, device="cuda").normal_(0.0, 0.02, generator=g)
    ones = torch.ones(d, dtype=torch.bfloat16, device="cuda")
    sh = SimpleNamespace(n_layers=2, d_model=d, n_q_heads=nq, n_kv_heads=nkv, head_dim=128, d_ffn=ffn, vocab=256, rope_base=1e6,
                         rms_eps=1e-5, dtype="bf16")
    layers = [dict(wq=rnd(nq * 128, d), wk=rnd(nkv * 128, d), wv=rnd(nkv * 128, d), wo=torch.eye(d, dtype=torch.bfloat16, device="cuda"),
                   w_gate=rnd(ffn, d), w_up=rnd(ffn, d), w_down=torch.zeros((d, ffn), dtype=torch.bfloat16, device="cuda"), g_attn=ones,
                   g_ffn=ones) for _ in range(2)]
    model = rc.Model(sh, layers, ones, rnd(256, d))
    rows = [1 + 7 * b for b in range(n)]
    need = max(rows) // page + 1
    table = torch.randperm(n * need, generator=g, device="cuda").to(torch.int32).view(n, need).contiguous()
    k, v = (torch.empty((2, n * need, nkv, page, 128), dtype=torch.bfloat16, device="cuda").normal_(generator=g) for _ in range(2))
    x = torch.empty((n, d), dtype=torch.bfloat16, device="cuda").normal_(generator=g)

    def step(groups):
        kk, vv, pre = k.clone(), v.clone(), torch.zeros_like(k)
        cache = rc.PagedKV.from_pools(list(kk.unbind(0)), list(vv.unbind(0)), table, rc.RC_BF16)
        keys = rc.PagedKV.from_pools(list(pre.unbind(0)), list(vv.unbind(0)), table, rc.RC_BF16)
        logits = torch.zeros((n, 256), dtype=torch.float32, device="cuda")
        for lo in range(0, n, groups):
            reqs = [rc.DecodeReq(x[b], rows[b], b, None, None) for b in range(lo, min(lo + groups, n))]
            out = torch.zeros((len(reqs), 256), dtype=torch.float32, device="cuda")
            rc.rc_decode_step(model, reqs, cache, out, rc.alloc_workspace(rc.rc_decode_workspace_bytes(model, reqs)), k_pre=keys)
            logits[lo:lo + len(reqs)] = out
        torch.cuda.synchronize()
        return kk, vv, pre, logits

    rc.rc_tune_set(rc.RC_TUNE_ATTN_CHUNK_TILES, 1000)
    try:
        together, four = step(n), step(4)
    finally:
        rc.rc_tune_set(rc.RC_TUNE_ATTN_CHUNK_TILES, 0)
    for a, b in zip(together[:3], four[:3]):
        assert torch.equal(a, b)
    assert not torch.equal(together[0][0], k[0]) and not torch.equal(together[0][1], k[1])
    assert rel_err(to_np(together[3]), to_np(four[3])) <= 2e-2
