"""The decode attention kernel (one live row per request) against the 32-row tile kernel: a row of a decoding step gets the same
bits as the same row computed together with the one behind it, whatever the cache looks like."""
from types import SimpleNamespace

import pytest
import torch

from tests.harness import rel_err, to_np

pytestmark = pytest.mark.gpu

D, FFN, LAYERS, NKV, DH = 512, 512, 3, 2, 128
# positions at the edges of 64-key tiles and 16-key pages, one tile, an odd and an even number of tiles
POSITIONS = [0, 1, 15, 31, 62, 63, 64, 127, 190, 300, 448, 1021]


def _model(rc, g, group):
    sh = SimpleNamespace(n_layers=LAYERS, d_model=D, n_q_heads=NKV * group, n_kv_heads=NKV, head_dim=DH, d_ffn=FFN, vocab=256,
                         rope_base=1e4, rms_eps=1e-5, dtype="bf16")
    nq, nkv = sh.n_q_heads * DH, NKV * DH
    rnd = lambda *s: torch.empty(s, dtype=torch.bfloat16, device="cuda").normal_(0.0, 0.05, generator=g)
    ones = torch.ones(D, dtype=torch.bfloat16, device="cuda")
    layers = [dict(wq=rnd(nq, D), wk=rnd(nkv, D), wv=rnd(nkv, D), wo=rnd(D, nq), w_gate=rnd(FFN, D), w_up=rnd(FFN, D), w_down=rnd(D, FFN),
                   g_attn=ones, g_ffn=ones) for _ in range(LAYERS)]
    return sh, rc.Model(sh, layers, ones, rnd(256, D))


@pytest.mark.parametrize("scores", [False, True])
@pytest.mark.parametrize("ramp", [False, True])   # keys that grow along the sequence: sums are rescaled on the way
@pytest.mark.parametrize("group,page,chunk", [(4, 0, 0), (4, 16, 0), (4, 16, 1), (4, 16, 3), (1, 16, 4), (2, 0, 2), (3, 2, 4), (5, 1, 3),
                                              (6, 24, 3), (7, 16, 1000), (8, 256, 2), (4, 0, 1000)])
def test_row_alone_and_with_another(group, page, chunk, ramp, scores):
    from paper_2603_13289_amd import binding as rc
    g = torch.Generator(device="cuda")
    g.manual_seed(group * 100 + page + chunk)
    sh, model = _model(rc, g, group)
    n = len(POSITIONS)
    size = page or 1024
    need = -(-1024 // size)
    table = torch.randperm(n * need, generator=g, device="cuda").to(torch.int32).view(n, need).contiguous()
    k = torch.empty((LAYERS, n * need, NKV, size, DH), dtype=torch.bfloat16, device="cuda").normal_(0.0, 1.0, generator=g)
    v = torch.empty_like(k).normal_(0.0, 1.0, generator=g)
    if ramp:
        for s in range(n):
            for i in range(need):
                at = torch.arange(i * size, (i + 1) * size, device="cuda").clamp(max=1024)
                k[:, table[s, i].long()] *= (1 + at / 64.0).to(torch.bfloat16)[None, None, :, None]
    x = torch.empty((n, D), dtype=torch.bfloat16, device="cuda").normal_(generator=g)

    def cache():
        kk, vv = k.clone(), v.clone()
        return kk, vv, rc.PagedKV.from_pools(list(kk.unbind(0)), list(vv.unbind(0)), table, rc.RC_BF16)

    rc.rc_tune_set(rc.RC_TUNE_ATTN_CHUNK_TILES, chunk if chunk else 1000)   # the same KV chunks for both
    try:
        k1, v1, c1 = cache()
        s_inf = [torch.zeros(p + 1, dtype=torch.float32, device="cuda") for p in POSITIONS]
        reqs = [rc.DecodeReq(x[b], p, b, None, s_inf[b] if scores else None) for b, p in enumerate(POSITIONS)]
        logits = torch.zeros((n, 256), dtype=torch.float32, device="cuda")
        rc.rc_decode_step(model, reqs, c1, logits, rc.alloc_workspace(rc.rc_decode_workspace_bytes(model, reqs)))
        k2, v2, c2 = cache()
        pairs = [rc.Request(torch.stack([x[b], x[b]]), None, dst_seq=b, n_cached=p) for b, p in enumerate(POSITIONS)]
        plan = rc.Plan(0, 1, 1, [0] * n)
        rc.rc_reuse(model, pairs, plan, None, c2, torch.zeros_like(logits), None, None,
                    rc.alloc_workspace(rc.rc_reuse_workspace_bytes(model, pairs, plan)))
        torch.cuda.synchronize()
    finally:
        rc.rc_tune_set(rc.RC_TUNE_ATTN_CHUNK_TILES, 0)
    for b, p in enumerate(POSITIONS):
        for l in range(LAYERS):
            for which in ("k", "v"):
                one, two = (c.read(which, l, b, 1, start=p) for c in (c1, c2))
                if ramp:   # the tile kernel rescales both rows when either grows: other powers of two, rounded P
                    assert rel_err(to_np(one), to_np(two)) <= 2e-2, (p, l, which)
                else:
                    assert torch.equal(one, two), (p, l, which)
        if scores:   # weights of every head and layer add up to one
            assert abs(float(s_inf[b].double().sum()) - LAYERS * sh.n_q_heads) <= 1e-4 * LAYERS * sh.n_q_heads


@pytest.mark.parametrize("group,chunk", [(4, 1), (4, 3), (8, 2), (1, 4)])
def test_influence_added_by_the_merge(group, chunk):
    """One model layer; KV ranges in one piece (a launch of its own adds the weights up) and in chunks (the merge does)."""
    from paper_2603_13289_amd import binding as rc
    g = torch.Generator(device="cuda")
    g.manual_seed(group + chunk)
    sh, model = _model(rc, g, group)
    n = len(POSITIONS)
    table = torch.randperm(n * 64, generator=g, device="cuda").to(torch.int32).view(n, 64).contiguous()
    k, v = (torch.empty((LAYERS, n * 64, NKV, 16, DH), dtype=torch.bfloat16, device="cuda").normal_(generator=g) for _ in range(2))
    x = torch.empty((n, D), dtype=torch.bfloat16, device="cuda").normal_(generator=g)
    got = []
    for c in (1000, chunk):
        kk, vv = k.clone(), v.clone()
        cache = rc.PagedKV.from_pools(list(kk.unbind(0)), list(vv.unbind(0)), table, rc.RC_BF16)
        s_inf = [torch.full((p + 1,), 0.5, dtype=torch.float32, device="cuda") for p in POSITIONS]
        # every third request keeps no influence vector
        reqs = [rc.DecodeReq(x[b], p, b, None, s_inf[b] if b % 3 else None) for b, p in enumerate(POSITIONS)]
        rc.rc_tune_set(rc.RC_TUNE_ATTN_CHUNK_TILES, c)
        try:
            rc.rc_decode_step(model, reqs, cache, torch.zeros((n, 256), dtype=torch.float32, device="cuda"),
                              rc.alloc_workspace(rc.rc_decode_workspace_bytes(model, reqs)))
        finally:
            rc.rc_tune_set(rc.RC_TUNE_ATTN_CHUNK_TILES, 0)
        torch.cuda.synchronize()
        got.append(s_inf)
    for b in range(n):
        if b % 3 == 0:
            assert float((got[1][b] - 0.5).abs().max()) == 0
            continue
        # the layers behind the first see attention outputs rounded to bf16 from other partial sums
        assert rel_err(to_np(got[1][b]), to_np(got[0][b])) <= 1e-2, POSITIONS[b]


@pytest.mark.parametrize("scores", [False, True])
def test_more_blocks_than_the_lds_table_holds(scores):
    """Pages of one slot, a range in one piece: 2049 and more blocks are looked up in memory, fewer are kept in LDS, the same bits."""
    from paper_2603_13289_amd import binding as rc
    g = torch.Generator(device="cuda")
    g.manual_seed(2048)
    sh, model = _model(rc, g, 4)
    positions, size = [2047, 2048, 2300, 40], 2304
    n = len(positions)
    k, v = (torch.empty((LAYERS, n, NKV, size, DH), dtype=torch.bfloat16, device="cuda").normal_(generator=g) for _ in range(2))
    x = torch.empty((n, D), dtype=torch.bfloat16, device="cuda").normal_(generator=g)
    outs = []
    for page in (16, 1):
        table = torch.randperm(n * size // page, generator=g, device="cuda").to(torch.int32).view(n, size // page).contiguous()
        pools = [torch.empty((LAYERS, n * size // page, NKV, page, DH), dtype=torch.bfloat16, device="cuda") for _ in range(2)]
        for pool, rows in zip(pools, (k, v)):
            pool[:, table.flatten().long()] = rows.view(LAYERS, n, NKV, size // page, page, DH).transpose(2, 3).reshape(LAYERS, -1, NKV, page, DH)
        cache = rc.PagedKV.from_pools(list(pools[0].unbind(0)), list(pools[1].unbind(0)), table, rc.RC_BF16)
        s_inf = [torch.zeros(p + 1, dtype=torch.float32, device="cuda") for p in positions]
        reqs = [rc.DecodeReq(x[b], p, b, None, s_inf[b] if scores else None) for b, p in enumerate(positions)]
        logits = torch.zeros((n, 256), dtype=torch.float32, device="cuda")
        rc.rc_tune_set(rc.RC_TUNE_ATTN_CHUNK_TILES, 1000)
        try:
            rc.rc_decode_step(model, reqs, cache, logits, rc.alloc_workspace(rc.rc_decode_workspace_bytes(model, reqs)))
        finally:
            rc.rc_tune_set(rc.RC_TUNE_ATTN_CHUNK_TILES, 0)
        torch.cuda.synchronize()
        outs.append([logits] + s_inf + [cache.read(w, l, b, 1, start=p) for w in ("k", "v") for l in range(LAYERS) for b, p in enumerate(positions)])
    assert bool(torch.isfinite(outs[0][0]).all())
    for one, two in zip(*outs):
        assert torch.equal(one, two)
