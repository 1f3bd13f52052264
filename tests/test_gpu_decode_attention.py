"""One query row per sequence: the decode attention kernel and the few-row products around it, through rc_decode_step
on a one-layer model whose logits are almost only attention (tiny residual input, zero MLP output), against torch in float32."""
import random
from types import SimpleNamespace

import numpy as np
import pytest
import torch

from tests.harness import TOL, rel_err, to_np

pytestmark = pytest.mark.gpu

# around a 16-key block, a wavefront's 32-key step, a round of four of them; then past the length from which ranges are split
SHORT = [0, 1, 15, 16, 31, 32, 63, 64, 127, 130]
LONG = [5, 700, 1023, 1024, 1500, 2111]


def _rot(x, pos, base):
    half = x.shape[-1] // 2
    t = pos * base ** (-torch.arange(half, dtype=torch.float64) / half)
    c, s = t.cos(), t.sin()
    a, b = x[..., :half], x[..., half:]
    return torch.cat([a * c - b * s, b * c + a * s], -1)


@pytest.mark.parametrize("group,page,rows,track", [
    (4, 0, SHORT, True), (4, 16, LONG, True), (4, 16, LONG, False), (1, 8, SHORT, False), (5, 24, LONG, True),
    (8, 64, LONG, False), (3, 16, SHORT * 2, True), (9, 16, SHORT, False)])
def test_decode_step_matches_float_reference(group, page, rows, track):
    from paper_2603_13289_amd import binding as rc
    g = torch.Generator().manual_seed(7 * group + page)
    hkv, dh, d, f, vocab, n = 2, 128, 512, 256, 272, len(rows)
    sh = SimpleNamespace(n_layers=1, d_model=d, n_q_heads=hkv * group, n_kv_heads=hkv, head_dim=dh, d_ffn=f, vocab=vocab,
                         rope_base=1e4, rms_eps=1e-5, dtype="bf16")
    normal = lambda *s, std=0.05: (torch.randn(s, generator=g) * std).bfloat16()
    w = dict(wq=normal(hkv * group * dh, d), wk=normal(hkv * dh, d), wv=normal(hkv * dh, d), wo=normal(d, hkv * group * dh),
             w_gate=normal(f, d), w_up=normal(f, d), w_down=torch.zeros(d, f).bfloat16(), g_attn=normal(d, std=1.0),
             g_ffn=normal(d, std=1.0))
    g_final, w_lm, x = normal(d, std=1.0), normal(vocab, d), normal(n, d, std=0.01)
    model = rc.Model(sh, [{k: v.cuda() for k, v in w.items()}], g_final.cuda(), w_lm.cuda())
    k_all = [normal(hkv, r + 1, dh, std=1.0) for r in rows]
    v_all = [normal(hkv, r + 1, dh, std=1.0) for r in rows]
    size = page or max(rows) + 1
    need = [-(-(r + 1) // size) for r in rows]
    ids = list(range(sum(need)))
    random.Random(3).shuffle(ids)
    k, v = (torch.full((1, len(ids), hkv, size, dh), float("nan")).bfloat16() for _ in range(2))
    table, at = [], 0
    for b in range(n):
        mine = ids[at:at + need[b]]
        at += need[b]
        table.append(mine + [-1] * (max(need) - need[b]))
        for i, blk in enumerate(mine):
            m = min(size, rows[b] + 1 - i * size)
            k[0, blk, :, :m], v[0, blk, :, :m] = k_all[b][:, i * size:i * size + m], v_all[b][:, i * size:i * size + m]
    k, v = k.cuda(), v.cuda()
    cache = rc.PagedKV.from_pools(list(k.unbind(0)), list(v.unbind(0)), torch.tensor(table, dtype=torch.int32, device="cuda"), rc.RC_BF16)
    s_inf = [torch.zeros(r + 1, dtype=torch.float32, device="cuda") for r in rows]
    xd = x.cuda()
    reqs = [rc.DecodeReq(xd[b], r, b, None, s_inf[b] if track and group <= 8 else None) for b, r in enumerate(rows)]
    out = torch.zeros((n, vocab), dtype=torch.float32, device="cuda")
    rc.rc_decode_step(model, reqs, cache, out, rc.alloc_workspace(rc.rc_decode_workspace_bytes(model, reqs)))
    torch.cuda.synchronize()
    wd = {i: t.double() for i, t in w.items()}
    norm = lambda t, gain: t / (t.square().mean(-1, keepdim=True) + 1e-5).sqrt() * gain.double()
    for b, r in enumerate(rows):
        a = norm(x[b].double(), w["g_attn"])
        q = _rot((wd["wq"] @ a).view(hkv, group, dh), r, 1e4)
        kk, vv = k_all[b].double(), v_all[b].double()
        kk[:, r], vv[:, r] = _rot((wd["wk"] @ a).view(hkv, dh), r, 1e4), (wd["wv"] @ a).view(hkv, dh)
        p = torch.softmax(torch.matmul(q, kk.transpose(1, 2).contiguous()) / dh ** 0.5, -1)
        h = x[b].double() + wd["wo"] @ torch.matmul(p, vv).reshape(-1)
        want = w_lm.double() @ norm(h, g_final)
        assert rel_err(to_np(cache.read("k", 0, b, 1, start=r))[:, :], kk[:, r].numpy()[None]) <= TOL["bf16"]
        assert rel_err(to_np(cache.read("v", 0, b, 1, start=r))[:, :], vv[:, r].numpy()[None]) <= TOL["bf16"]
        assert rel_err(to_np(out[b]), want.numpy()) <= TOL["bf16"], f"sequence {b}, {r} cached rows"
        if track and group <= 8:
            assert rel_err(to_np(s_inf[b]), p.sum((0, 1)).numpy()) <= TOL["bf16"], f"influence {b}, {r} cached rows"
    model.close()
