"""Tile attention of a key range that is no multiple of the 64-key tile: an infinite value of its last key reaches the last row as it is."""
import pytest
import torch

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("bad", [float("inf"), float("-inf")])
@pytest.mark.parametrize("page", [0, 16, 24])
@pytest.mark.parametrize("keys,workspace", [(1, False), (5, False), (65, False), (100, False), (255, False), (1000, False), (2000, True)])
@pytest.mark.parametrize("group", [1, 4, 5, 8])
def test_last_row_sees_the_infinity(group, keys, workspace, page, bad):
    from paper_2603_13289_amd import binding as rc
    g = torch.Generator(device="cuda")
    g.manual_seed(keys + group)
    nkv, dh, size = 2, 128, page or keys
    need = -(-keys // size)
    # slots behind the last key hold another infinity
    k, v = (torch.empty((need * size, nkv, dh), dtype=torch.bfloat16, device="cuda").normal_(generator=g) for _ in range(2))
    v[keys:] = -bad
    table = torch.randperm(need, generator=g, device="cuda").to(torch.int32).view(1, need).contiguous()
    pos = torch.tensor(sorted({keys // 2, keys - 1}), dtype=torch.int32, device="cuda")
    n = len(pos)
    q = torch.empty((n, nkv * group, dh), dtype=torch.bfloat16, device="cuda").normal_(generator=g)
    outs = []
    for value in (bad, 0.0):
        v[keys - 1, 1, 7] = value
        pools = [torch.empty((need, nkv, size, dh), dtype=torch.bfloat16, device="cuda") for _ in range(2)]
        for x, pool in zip((k, v), pools):
            pool[table[0].long()] = x.view(need, size, nkv, dh).transpose(1, 2)
        cache = rc.PagedKV.from_pools([pools[0]], [pools[1]], table, rc.RC_BF16)
        ws = rc.alloc_workspace(rc.rc_sparse_attention_workspace_bytes(n, nkv * group, cache.layer(0))) if workspace else None
        out = torch.zeros((n, nkv * group, dh), dtype=torch.bfloat16, device="cuda")
        rc.rc_sparse_attention(q, pos, n, nkv * group, cache.layer(0), 0, out, ws)
        torch.cuda.synchronize()
        outs.append(out[-1])
    assert bool((outs[0][group:, 7] == bad).all())
    outs[0][group:, 7] = outs[1][group:, 7]
    assert torch.equal(outs[0], outs[1]) and bool(torch.isfinite(outs[0]).all())
