"""Float attention: sixteen rows of a group share their key blocks, but a row reads no value behind its own position."""
import numpy as np
import pytest
import torch

from tests.harness import to_np

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("bad", [np.nan, np.inf])
@pytest.mark.parametrize("pos", [list(range(40)), [0, 3, 4, 30, 31, 32, 33, 70, 71, 90, 120, 121, 122, 127, 128, 140, 141]])
@pytest.mark.parametrize("dh,page", [(64, 0), (128, 0), (64, 16)])
def test_values_behind_a_row_do_not_reach_it(dh, page, pos, bad):
    from paper_2603_13289_amd import binding as rc
    hq, hkv, t = 4, 2, 144
    g = np.random.default_rng(dh + len(pos))
    q, k, v = (g.standard_normal(s, dtype=np.float32) for s in ((len(pos), hq, dh), (t, hkv, dh), (t, hkv, dh)))
    for j in (5, 20, 32, 121):                   # not finite in one element; key 32 in all of them
        v[j, j % hkv, 7 if j != 32 else slice(None)] = bad
    v[122, :, 9] = -bad
    k[133, :, 3] = np.nan
    pools = rc.PagedKV(1, 9, 16, hkv, dh, rc.RC_F32, [[8, 3, 0, 7, 1, 2, 6, 5, 4]]) if page else \
        rc.PagedKV.contiguous(1, 1, t, hkv, dh, rc.RC_F32)
    pools.write("k", 0, 0, torch.from_numpy(k).cuda())
    pools.write("v", 0, 0, torch.from_numpy(v).cuda())
    out = torch.zeros((len(pos), hq, dh), dtype=torch.float32, device="cuda")
    rc.rc_sparse_attention(torch.from_numpy(q).cuda(), torch.tensor(pos, dtype=torch.int32, device="cuda"), len(pos), hq,
                           pools.layer(0), 0, out, None)
    got = to_np(out)
    for r, p in enumerate(pos):
        for h in range(hq):
            kk, vv = (x[:p + 1, h // (hq // hkv)].astype(np.float64) for x in (k, v))
            s = kk @ q[r, h].astype(np.float64) / np.sqrt(dh)
            w = np.exp(s - s.max())
            with np.errstate(invalid="ignore"):
                want = (w[:, None] * vv).sum(0) / w.sum()
            fin = np.isfinite(want)
            assert np.array_equal(np.isnan(got[r, h]), np.isnan(want)), (p, h)
            assert np.array_equal(got[r, h][~fin & ~np.isnan(want)], want[~fin & ~np.isnan(want)]), (p, h)
            # sums of at most 144 terms of order one in 32 bits
            assert np.abs(got[r, h][fin] - want[fin]).max(initial=0.) <= 2e-5, (p, h)
