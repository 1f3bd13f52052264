"""The attention kernels read a contiguous cache and caches of any page size: the same bits, whatever the layout, for key counts at the
edges of their key tiles and main loops (bf16: 64 keys, four tiles; float: 16 keys, 8 x 2 or 4 x 2 blocks), and the values of a plain
attention."""
import pytest
import torch

from tests.harness import rel_err, to_np

pytestmark = pytest.mark.gpu

NKV = 2
PAGES = [0, 1, 8, 16, 24, 32, 48, 256]


@pytest.mark.parametrize("group", [1, 3, 4, 5, 7, 8])
@pytest.mark.parametrize("keys", [5, 64, 65, 192, 255, 256, 257, 320, 385, 448, 1000])
def test_page_sizes_give_the_same_bits(group, keys):
    _same_bits(group, keys, 128, torch.bfloat16, 1e-2)   # weights and outputs rounded to bf16, as in the stage test


@pytest.mark.parametrize("group", [1, 4, 5, 8])
@pytest.mark.parametrize("keys", [1601, 2048])   # more than 24 key tiles: late rows in chunks of four tiles, merged
def test_page_sizes_give_the_same_bits_in_chunks(group, keys):
    _same_bits(group, keys, 128, torch.bfloat16, 1e-2, workspace=True)


@pytest.mark.parametrize("dh", [64, 128])
@pytest.mark.parametrize("keys", [5, 16, 17, 64, 65, 128, 129, 256, 257, 300, 1000])
def test_page_sizes_give_the_same_bits_f32(dh, keys):
    _same_bits(2, keys, dh, torch.float32, 2e-5)   # as in the stage test


def _same_bits(group, keys, DH, td, tol, workspace=False):
    from paper_2603_13289_amd import binding as rc
    g = torch.Generator(device="cuda")
    g.manual_seed(100 * group + keys)
    nq = NKV * group
    k, v = (torch.empty((keys, NKV, DH), dtype=td, device="cuda").normal_(generator=g) for _ in range(2))
    # a whole tile of late rows, and one of rows spread over the sequence
    late = torch.arange(max(keys - 33, 0), keys)
    pos = torch.cat([torch.linspace(0, keys - 1, min(keys, 32)).int().unique(), late]).sort().values.to(torch.int32)
    n = len(pos)
    q = torch.empty((n, nq, DH), dtype=td, device="cuda").normal_(generator=g)
    outs = []
    for page in PAGES:
        size = page or keys
        need = -(-keys // size)
        table = torch.randperm(need + 2, generator=g, device="cuda").to(torch.int32)[:need].view(1, need).contiguous()
        pools = []
        for x in (k, v):   # slots that hold no key are not numbers: they must not be used
            pool = torch.full(((need + 2) if page else 1, NKV, size, DH), float("nan"), dtype=td, device="cuda")
            for i in range(need):
                rows = x[i * size:(i + 1) * size]
                pool[table[0, i] if page else 0, :, :len(rows)] = rows.transpose(0, 1)
            pools.append(pool)
        if not page:
            table = torch.zeros((1, 1), dtype=torch.int32, device="cuda")
        cache = rc.PagedKV.from_pools([pools[0]], [pools[1]], table, rc.RC_BF16 if td == torch.bfloat16 else rc.RC_F32)
        out = torch.zeros((n, nq, DH), dtype=td, device="cuda")
        ws = rc.alloc_workspace(rc.rc_sparse_attention_workspace_bytes(n, nq, cache.layer(0))) if workspace else None
        rc.rc_sparse_attention(q, pos.cuda(), n, nq, cache.layer(0), 0, out, ws)
        torch.cuda.synchronize()
        outs.append(out)
    for page, out in zip(PAGES[1:], outs[1:]):
        assert torch.equal(outs[0], out), page
    kf, vf = (x.double().cpu().repeat_interleave(group, 1) for x in (k, v))
    s = torch.einsum("nhd,khd->hnk", q.double().cpu(), kf) / DH ** 0.5
    s = s.masked_fill(torch.arange(keys)[None, None] > pos[None, :, None], float("-inf"))
    want = torch.einsum("hnk,khd->nhd", s.softmax(-1), vf)
    assert rel_err(to_np(outs[0]), want.numpy()) <= tol
