"""rc_sparse_attention takes its positions from device memory: one that lies outside the cache counts as the cache's last one, and the
rows beside it are not touched by it."""
import pytest
import torch

pytestmark = pytest.mark.gpu

NKV = 2


def _rows(nkv, group, DH, td, page, capacity, workspace, outside, n):
    """Outputs with the given positions outside the cache behind n - len(outside) valid ones, and with the cache's last position instead."""
    from paper_2603_13289_amd import binding as rc
    g = torch.Generator(device="cuda")
    g.manual_seed(capacity + page)
    size = page or capacity
    need = capacity // size
    pools = [torch.empty((need, nkv, size, DH), dtype=td, device="cuda").normal_(generator=g) for _ in range(2)]
    table = torch.randperm(need, generator=g, device="cuda").to(torch.int32).view(1, need).contiguous()
    cache = rc.PagedKV.from_pools([pools[0]], [pools[1]], table, rc.RC_BF16 if td == torch.bfloat16 else rc.RC_F32)
    q = torch.empty((n, nkv * group, DH), dtype=td, device="cuda").normal_(generator=g)
    inside = torch.linspace(0, capacity - 1, n - len(outside)).int()
    outs = []
    for late in (outside, [capacity - 1] * len(outside)):
        pos = torch.cat([inside, torch.tensor(late, dtype=torch.int32)]).cuda()
        ws = None
        if workspace:   # partial results that nobody wrote are not numbers
            ws = rc.alloc_workspace(rc.rc_sparse_attention_workspace_bytes(n, nkv * group, cache.layer(0)))
            ws.fill_(255)
        out = torch.zeros((n, nkv * group, DH), dtype=td, device="cuda")
        rc.rc_sparse_attention(q, pos, n, nkv * group, cache.layer(0), 0, out, ws)
        torch.cuda.synchronize()
        outs.append(out)
    return outs


@pytest.mark.parametrize("page,capacity", [(0, 1024), (0, 1000), (16, 1008), (24, 1008), (16, 2000)])
@pytest.mark.parametrize("n", [32, 40])
def test_kernel_and_merge_agree_on_the_key_range(page, capacity, n):
    """16 key tiles fit, the positions ask for more than the 24 from which on a range is cut into chunks; 2000 keys are cut anyway."""
    got, want = _rows(NKV, 4, 128, torch.bfloat16, page, capacity, True, [capacity + 900, 2 * capacity], n)
    assert torch.equal(got[:n - 2], want[:n - 2])


@pytest.mark.parametrize("page,capacity", [(0, 1024), (0, 1000), (16, 1008), (24, 1008), (16, 2000), (0, 5)])
@pytest.mark.parametrize("group,DH,td", [(1, 128, torch.bfloat16), (4, 128, torch.bfloat16), (5, 128, torch.bfloat16), (8, 128, torch.bfloat16),
                                         (16, 128, torch.bfloat16), (2, 64, torch.float32), (2, 128, torch.float32)])
@pytest.mark.parametrize("workspace", [False, True])
def test_a_row_outside_counts_as_the_last_one(page, capacity, group, DH, td, workspace):
    if workspace and td == torch.float32:
        pytest.skip("only the bf16 kernel splits ranges")
    for n, outside in ((40, [capacity, capacity + 900, 2 * capacity]), (1, [capacity + 17])):
        got, want = _rows(NKV, group, DH, td, page, capacity, workspace, outside, n)
        assert torch.equal(got, want), n
