"""Decoding steps of few rows: whatever number of sequences shares a step (norm inside the products or in a launch of its own, one or
two row tiles, rotary and scatter in the epilogue), a sequence gets the same bits."""
from types import SimpleNamespace

import pytest
import torch

pytestmark = pytest.mark.gpu

N, NKV, DH, VOCAB = 20, 2, 128, 272


# model widths: two K steps a wavefront, an odd number, two full register sets, the widest row normalised inside, one beyond it
@pytest.mark.parametrize("d", [512, 1280, 4096, 5120, 5376])
@pytest.mark.parametrize("group,page", [(1, 0), (4, 16), (5, 3)])
def test_rows_do_not_depend_on_company(d, group, page):
    from paper_2603_13289_amd import binding as rc
    g = torch.Generator(device="cuda")
    g.manual_seed(d + group)
    sh = SimpleNamespace(n_layers=2, d_model=d, n_q_heads=NKV * group, n_kv_heads=NKV, head_dim=DH, d_ffn=512, vocab=VOCAB,
                         rope_base=1e4, rms_eps=1e-5, dtype="bf16")
    nq, nkv = sh.n_q_heads * DH, NKV * DH
    rnd = lambda *s: torch.empty(s, dtype=torch.bfloat16, device="cuda").normal_(0.0, 0.02, generator=g)
    gain = lambda: (1 + rnd(d)).contiguous()
    layers = [dict(wq=rnd(nq, d), wk=rnd(nkv, d), wv=rnd(nkv, d), wo=rnd(d, nq), w_gate=rnd(512, d), w_up=rnd(512, d), w_down=rnd(d, 512),
                   g_attn=gain(), g_ffn=gain()) for _ in range(2)]
    model = rc.Model(sh, layers, gain(), rnd(VOCAB, d))
    pos = [(37 * b) % 130 for b in range(N)]
    size = page or 160
    need = -(-160 // size)
    table = torch.randperm(N * need, generator=g, device="cuda").to(torch.int32).view(N, need).contiguous()
    k0, v0 = (torch.empty((2, N * need, NKV, size, DH), dtype=torch.bfloat16, device="cuda").normal_(generator=g) for _ in range(2))
    x = torch.empty((N, d), dtype=torch.bfloat16, device="cuda").normal_(generator=g)

    def run(m):
        k, v, pre = k0.clone(), v0.clone(), torch.zeros_like(k0)
        cache = rc.PagedKV.from_pools(list(k.unbind(0)), list(v.unbind(0)), table, rc.RC_BF16)
        kp = rc.PagedKV.from_pools(list(pre.unbind(0)), list(v.unbind(0)), table, rc.RC_BF16)
        logits = torch.zeros((N, VOCAB), dtype=torch.float32, device="cuda")
        for b in range(0, N, m):
            reqs = [rc.DecodeReq(x[i], pos[i], i, None, None) for i in range(b, min(b + m, N))]
            rc.rc_decode_step(model, reqs, cache, logits[b:], rc.alloc_workspace(rc.rc_decode_workspace_bytes(model, reqs)), k_pre=kp)
        torch.cuda.synchronize()
        return k, v, pre, logits

    rc.rc_tune_set(rc.RC_TUNE_ATTN_CHUNK_TILES, 1000)   # attention in one piece: its chunks may depend on the company
    try:
        want = run(6)   # norms in launches of their own, one row tile
        assert float(want[3].abs().max()) > 0
        # the first layer's keys and values against 64 bits: operands rounded to bf16 once, the result once
        h = x[7].double()
        a = (h / torch.sqrt((h * h).mean() + 1e-5) * layers[0]["g_attn"].double()).to(torch.bfloat16).double()
        key = (layers[0]["wk"].double() @ a).view(NKV, 2, 64)
        ang = pos[7] * 1e4 ** (-torch.arange(64, device="cuda").double() / 64)
        key = torch.cat([key[:, 0] * ang.cos() - key[:, 1] * ang.sin(), key[:, 1] * ang.cos() + key[:, 0] * ang.sin()], 1)
        got = want[0][0, table[7, pos[7] // size].long(), :, pos[7] % size].double()
        assert float((got - key).norm() / key.norm()) <= 2.0 ** -8
        for m in (1, 2, 3, 4, 5, 16, 17, N):
            for name, a, b in zip(("k", "v", "k_pre", "logits"), run(m), want):
                assert torch.equal(a, b), (m, name)
    finally:
        rc.rc_tune_set(rc.RC_TUNE_ATTN_CHUNK_TILES, 0)
