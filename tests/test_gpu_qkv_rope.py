"""The q|k|v product with rotary and scatter in its epilogue against the product, then the scatter stage: the same bits, for every tile
type, with K in parts and without, at the edges of tiles and heads."""
from types import SimpleNamespace

import numpy as np
import pytest
import torch

pytestmark = pytest.mark.gpu

# rows; model width; heads; page; forced tile type (0: by shape)
CASES = [(33, 512, 8, 2, 0, 0), (100, 4096, 32, 8, 16, 0), (257, 5120, 40, 8, 16, 0), (1025, 4096, 32, 8, 0, 0), (1639, 4096, 32, 8, 16, 0),
         (2500, 4096, 32, 8, 0, 0), (5120, 1024, 32, 8, 16, 0), (300, 1024, 7, 1, 3, 0)]
CASES += [(m, 640, 6, 2, 16, t) for m in (40, 197) for t in (5, 6, 7, 8, 9, 10, 11, 12, 13)]
# 256x256 tiles, some of them cut along K, and a thin last tile row: all three ends of the product in one launch (test_gemm_plan.py)
THIN = [(2817, 4096, 32, 8, 16, 0), (3073, 4096, 32, 8, 0, 0), (2305, 5120, 40, 8, 16, 0)]
CASES += THIN


@pytest.mark.parametrize("m,d,nq,nkv,page,tile", CASES)
def test_product_and_scatter(m, d, nq, nkv, page, tile):
    from paper_2603_13289_amd import binding as rc
    g = torch.Generator(device="cuda")
    g.manual_seed(m + d + tile)
    sh = SimpleNamespace(n_layers=1, d_model=d, n_q_heads=nq, n_kv_heads=nkv, head_dim=128, d_ffn=512, vocab=256, rope_base=1e4,
                         rms_eps=1e-5, dtype="bf16")
    rnd = lambda *s: torch.empty(s, dtype=torch.bfloat16, device="cuda").normal_(0.0, 0.02, generator=g)
    ones = torch.ones(d, dtype=torch.bfloat16, device="cuda")
    wq, wk, wv = rnd(nq * 128, d), rnd(nkv * 128, d), rnd(nkv * 128, d)
    model = rc.Model(sh, [dict(wq=wq, wk=wk, wv=wv, wo=rnd(d, nq * 128), w_gate=rnd(512, d), w_up=rnd(512, d), w_down=rnd(d, 512),
                               g_attn=ones, g_ffn=ones)], ones, rnd(256, d))
    x = (torch.randint(0, 2, (m, d), generator=g, device="cuda") * 2 - 1).to(torch.bfloat16)   # rows of rms 1
    size = page or m
    need = -(-m // size)
    table = torch.randperm(need + 2, generator=g, device="cuda")[:need].to(torch.int32).view(1, need).contiguous()

    def pools():
        k = torch.zeros((1, need + 2, nkv, size, 128), dtype=torch.bfloat16, device="cuda")
        return k, torch.zeros_like(k)

    k1, v1 = pools()
    pre, _ = pools()
    cache = rc.PagedKV.from_pools([k1[0]], [v1[0]], table, rc.RC_BF16)
    record = rc.PagedKV.from_pools([pre[0]], [v1[0]], table, rc.RC_BF16)
    logits = torch.zeros((1, 256), dtype=torch.float32, device="cuda")
    rc.rc_tune_set(rc.RC_TUNE_GEMM_TILE, tile)
    try:
        ws_call = rc.alloc_workspace(rc.rc_prefill_workspace_bytes(model, [m]))
        rc.rc_prefill(model, [x], [0], cache, logits, ws_call, k_pre=record)
        # the same product into floats, then the scatter stage
        r = np.float32(1) / np.sqrt(np.float32(1) + np.float32(1e-5))
        a = (x.float() * float(r)).to(torch.bfloat16)
        n = (nq + 2 * nkv) * 128
        qkv = torch.zeros((m, n), dtype=torch.float32, device="cuda")
        rc.rc_gemm_rows(rc.RC_BF16, a, torch.cat([wq, wk, wv]).contiguous(), qkv, m, n, d, rc.alloc_workspace(rc.rc_gemm_workspace_bytes()))
    finally:
        rc.rc_tune_set(rc.RC_TUNE_GEMM_TILE, 0)
    k2, v2 = pools()
    staged = rc.PagedKV.from_pools([k2[0]], [v2[0]], table, rc.RC_BF16)
    pos = torch.arange(m, dtype=torch.int32, device="cuda")
    q = torch.zeros((m, nq * 128), dtype=torch.bfloat16, device="cuda")
    ws = rc.alloc_workspace(rc.rc_rope_scatter_workspace_bytes(m, staged.layer(0)))
    rc.rc_rope_scatter(qkv, pos, m, nq, 1e4, staged.layer(0), 0, q, ws)
    torch.cuda.synchronize()
    assert float(k2.float().abs().sum()) > 0
    assert torch.equal(k1, k2) and torch.equal(v1, v2)
    want = qkv[:, nq * 128:(nq + nkv) * 128].to(torch.bfloat16).view(m, nkv, 128)
    assert torch.equal(record.read("k", 0, 0, m).view(m, nkv, 128), want)
    # the rotated queries of the one layer are still in the call's workspace, at a multiple of 256 bytes
    held, q = ws_call.view(torch.int16), q.view(torch.int16).flatten()
    at = (held[:held.numel() // 128 * 128].view(-1, 128) == q[:128]).all(1).nonzero().flatten().tolist()
    assert any(torch.equal(held[128 * i:128 * i + q.numel()], q) for i in at)
