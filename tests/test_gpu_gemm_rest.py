"""K parts of a down projection added up by the next layer's norm, or by a launch of their own (hidden states kept at that layer): the
same rows in the same order, hence the same bits."""
from types import SimpleNamespace

import pytest
import torch

pytestmark = pytest.mark.gpu


# model widths of one to six 1024-element passes, whole and ragged; rows that cut all tiles, some tiles (1639) and leave a thin row;
# every width of a tile (192 columns change places in blocks of 64, the others of 128)
@pytest.mark.parametrize("d,rows,tile", [(512, 40, 0), (1152, 100, 0), (2048, 257, 0), (4096, 70, 0), (4096, 1025, 0), (4096, 1639, 0),
                                         (5120, 300, 0), (5376, 65, 0)] + [(1152, 100, t) for t in range(7, 14)])
def test_norm_adds_the_parts(d, rows, tile):
    from paper_2603_13289_amd import binding as rc
    g = torch.Generator(device="cuda")
    g.manual_seed(d + rows)
    f = 14336 if d == 4096 else 3072
    sh = SimpleNamespace(n_layers=2, d_model=d, n_q_heads=4, n_kv_heads=2, head_dim=128, d_ffn=f, vocab=256, rope_base=1e4,
                         rms_eps=1e-5, dtype="bf16")
    rnd = lambda *s: torch.empty(s, dtype=torch.bfloat16, device="cuda").normal_(0.0, 0.02, generator=g)
    layers = [dict(wq=rnd(512, d), wk=rnd(256, d), wv=rnd(256, d), wo=rnd(d, 512), w_gate=rnd(f, d), w_up=rnd(f, d), w_down=rnd(d, f),
                   g_attn=(1 + rnd(d)).contiguous(), g_ffn=(1 + rnd(d)).contiguous()) for _ in range(2)]
    model = rc.Model(sh, layers, (1 + rnd(d)).contiguous(), rnd(256, d))
    x = torch.empty((rows, d), dtype=torch.bfloat16, device="cuda").normal_(generator=g)
    table = torch.zeros((1, 1), dtype=torch.int32, device="cuda")

    def run(keep):
        k = torch.zeros((2, 1, 2, rows, 128), dtype=torch.bfloat16, device="cuda")
        v = torch.zeros_like(k)
        cache = rc.PagedKV.from_pools(list(k.unbind(0)), list(v.unbind(0)), table, rc.RC_BF16)
        logits = torch.zeros((1, 256), dtype=torch.float32, device="cuda")
        h = [torch.zeros_like(x)] if keep else None
        ws = rc.alloc_workspace(rc.rc_prefill_workspace_bytes(model, [rows]))
        rc.rc_prefill(model, [x], [0], cache, logits, ws, capture_layer=1 if keep else -1, h_capture=h)
        torch.cuda.synchronize()
        return k, v, logits, h

    rc.rc_tune_set(rc.RC_TUNE_GEMM_TILE, tile)
    try:
        k1, v1, logits1, _ = run(False)
        k2, v2, logits2, h = run(True)
    finally:
        rc.rc_tune_set(rc.RC_TUNE_GEMM_TILE, 0)
    for a, b in ((k1, k2), (v1, v2), (logits1, logits2)):
        assert torch.equal(a, b)
    # the second layer's values against 64 bits, from the kept rows (bf16): operands rounded twice, the result once
    hd = h[0].double()
    a = hd / torch.sqrt((hd * hd).mean(1, keepdim=True) + 1e-5) * layers[1]["g_attn"].double()
    want = (a @ layers[1]["wv"].double().t()).view(rows, 2, 128)
    got = v1[1, 0].transpose(0, 1).double()
    assert float((got - want).norm() / want.norm()) <= 2.0 ** -7
