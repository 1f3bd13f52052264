"""The tile attention kernel reads a contiguous cache and caches of any page size: the same bits, whatever the layout, for key counts at
the edges of its 64-key tiles and of its main loop (four tiles), and the values of a plain attention."""
import pytest
import torch

from tests.harness import rel_err, to_np

pytestmark = pytest.mark.gpu

NKV, DH = 2, 128
PAGES = [0, 1, 8, 16, 24, 32, 48, 256]


@pytest.mark.parametrize("group", [1, 3, 4, 5, 7, 8])
@pytest.mark.parametrize("keys", [5, 64, 65, 192, 255, 256, 257, 320, 385, 448, 1000])
def test_page_sizes_give_the_same_bits(group, keys):
    from paper_2603_13289_amd import binding as rc
    g = torch.Generator(device="cuda")
    g.manual_seed(100 * group + keys)
    nq = NKV * group
    k, v = (torch.empty((keys, NKV, DH), dtype=torch.bfloat16, device="cuda").normal_(generator=g) for _ in range(2))
    # a whole tile of late rows, and one of rows spread over the sequence
    late = torch.arange(max(keys - 33, 0), keys)
    pos = torch.cat([torch.linspace(0, keys - 1, min(keys, 32)).int().unique(), late]).sort().values.to(torch.int32)
    n = len(pos)
    q = torch.empty((n, nq, DH), dtype=torch.bfloat16, device="cuda").normal_(generator=g)
    outs = []
    for page in PAGES:
        size = page or keys
        need = -(-keys // size)
        table = torch.randperm(need + 2, generator=g, device="cuda").to(torch.int32)[:need].view(1, need).contiguous()
        pools = []
        for x in (k, v):   # slots that hold no key are not numbers: they must not be used
            pool = torch.full(((need + 2) if page else 1, NKV, size, DH), float("nan"), dtype=torch.bfloat16, device="cuda")
            for i in range(need):
                rows = x[i * size:(i + 1) * size]
                pool[table[0, i] if page else 0, :, :len(rows)] = rows.transpose(0, 1)
            pools.append(pool)
        if not page:
            table = torch.zeros((1, 1), dtype=torch.int32, device="cuda")
        cache = rc.PagedKV.from_pools([pools[0]], [pools[1]], table, rc.RC_BF16)
        out = torch.zeros((n, nq, DH), dtype=torch.bfloat16, device="cuda")
        rc.rc_sparse_attention(q, pos.cuda(), n, nq, cache.layer(0), 0, out, None)
        torch.cuda.synchronize()
        outs.append(out)
    for page, out in zip(PAGES[1:], outs[1:]):
        assert torch.equal(outs[0], out), page
    kf, vf = (x.float().cpu().repeat_interleave(group, 1) for x in (k, v))
    s = torch.einsum("nhd,khd->hnk", q.float().cpu(), kf) / DH ** 0.5
    s = s.masked_fill(torch.arange(keys)[None, None] > pos[None, :, None], float("-inf"))
    want = torch.einsum("hnk,khd->nhd", s.softmax(-1), vf)
    assert rel_err(to_np(outs[0]), want.numpy()) <= 1e-2   # weights and outputs rounded to bf16, as in the stage test
