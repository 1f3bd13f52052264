"""Float q|k|v product with rotary and scatter: rows of a launch with more workgroups than the chip holds at once, which finds their place in the
cache behind the product, get the bits of rows of a small launch, which finds it ahead."""
from types import SimpleNamespace

import pytest
import torch

from tests.harness import rel_err, to_np

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("d,nq,dh,reqs,tokens", [(256, 4, 64, 9, 128), (256, 4, 64, 16, 127), (512, 8, 64, 5, 112), (264, 2, 128, 17, 65)])
def test_rows_in_company_and_alone(d, nq, dh, reqs, tokens):
    from paper_2603_13289_amd import binding as rc
    g = torch.Generator(device="cuda")
    g.manual_seed(d + reqs)
    nkv, ffn, layers, page = nq // 2, 64, 2, 16
    assert (nq + 2 * nkv) * dh // 32 * -(-reqs * tokens // 16) > 1024 >= (nq + 2 * nkv) * dh // 32 * -(-tokens // 16)
    rnd = lambda *s: torch.empty(s, device="cuda").normal_(0.0, 0.05, generator=g)
    ones = torch.ones(d, device="cuda")
    sh = SimpleNamespace(n_layers=layers, d_model=d, n_q_heads=nq, n_kv_heads=nkv, head_dim=dh, d_ffn=ffn, vocab=64, rope_base=1e4,
                         rms_eps=1e-5, dtype="f32")
    model = rc.Model(sh, [dict(wq=rnd(nq * dh, d), wk=rnd(nkv * dh, d), wv=rnd(nkv * dh, d), wo=rnd(d, nq * dh), w_gate=rnd(ffn, d),
                               w_up=rnd(ffn, d), w_down=rnd(d, ffn), g_attn=ones, g_ffn=ones) for _ in range(layers)], ones, rnd(64, d))
    need = -(-tokens // page)
    table = torch.randperm(reqs * need, generator=g, device="cuda").to(torch.int32).view(reqs, need).contiguous()
    x = [torch.empty((tokens, d), device="cuda").normal_(generator=g) for _ in range(reqs)]
    runs = []
    for group in (reqs, 1):
        k, v, pre = (torch.zeros((layers, reqs * need, nkv, page, dh), device="cuda") for _ in range(3))
        cache = rc.PagedKV.from_pools(list(k.unbind(0)), list(v.unbind(0)), table, rc.RC_F32)
        keys = rc.PagedKV.from_pools(list(pre.unbind(0)), list(v.unbind(0)), table, rc.RC_F32)
        logits = torch.zeros((reqs, 64), device="cuda")
        for lo in range(0, reqs, group):
            seqs = list(range(lo, min(lo + group, reqs)))
            out = torch.zeros((len(seqs), 64), device="cuda")
            rc.rc_prefill(model, [x[b] for b in seqs], seqs, cache, out,
                          rc.alloc_workspace(rc.rc_prefill_workspace_bytes(model, [tokens] * len(seqs))), k_pre=keys)
            logits[seqs] = out
        torch.cuda.synchronize()
        runs.append((k, v, pre, logits))
    for a, b in zip(runs[0][:3], runs[1][:3]):
        assert torch.equal(a[0], b[0])   # the first layer: the others stand behind products whose kernels go by the rows
        assert bool(a[0].abs().sum() > 0) and rel_err(to_np(a[1]), to_np(b[1])) <= 2e-5
    assert rel_err(to_np(runs[0][3]), to_np(runs[1][3])) <= 2e-5
