"""The bias and the commit at the edges of their grids: rows whose chunks do not
fill a workgroup, one and eight chunks a thread, a partial last chunk, planes whose
columns straddle workgroups, paths longer than one group of 16 rows.  Both move or
expand bits, so everything is exact."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("batch,N", [(1, 1), (3, 65), (5, 255), (41, 509), (64, 512), (9, 1023)])
@pytest.mark.parametrize("dtype", ["bfloat16", "float32"])
def test_bias_shapes(batch, N, dtype):
    import paper_2608_20375_amd as G
    print("bias", batch, N, dtype, flush=True)
    g = np.random.default_rng(N)
    W = (N + 63) // 64
    ctx = G.Context(batch, 4, 64, 4, N)
    mask = torch.from_numpy(g.integers(-2**63, 2**63, (batch, N, W), dtype=np.int64)).cuda()
    n = torch.from_numpy(g.integers(0, N + 1, batch).astype(np.int32)).cuda()
    n[0] = N
    ld = (N + 7) // 8 * 8 + 8
    bias = torch.full((batch, N, ld), 7.0, dtype=getattr(torch, dtype), device="cuda")
    ctx.mask_to_bias(n, mask, bias)
    j = torch.arange(N, device="cuda")
    on = j[None, :] < n[:, None]
    seen = ((mask[:, :, j >> 6] >> (j & 63)) & 1) == 1
    seen = seen & on[:, :, None] & on[:, None, :]
    want = torch.full_like(bias, 7.0)
    want[:, :, :N] = torch.where(seen, 0.0, float("-inf"))
    assert torch.equal(bias, want)
    ctx.close()


@pytest.mark.parametrize("planes,batch,L,N,width", [(1, 1, 1, 1, 8), (7, 3, 16, 33, 8),
                                                    (5, 2, 33, 100, 72), (3, 4, 17, 64, 1024),
                                                    (2, 2, 64, 65, 2504)])
@pytest.mark.parametrize("in_place", [False, True])
def test_commit_shapes(planes, batch, L, N, width, in_place):
    import paper_2608_20375_amd as G
    print("commit", planes, batch, L, N, width, in_place, flush=True)
    g = np.random.default_rng(width + L)
    ctx = G.Context(batch, L, 64, 4, N)
    src = torch.from_numpy(g.integers(-9, 9, (planes, batch, N, width)).astype(np.int16)).cuda()
    most = min(L, N)
    acc = g.integers(0, most + 1, batch).astype(np.int32)
    acc[0] = most
    nodes = np.full((batch, L), -1, np.int32)
    for b in range(batch):
        nodes[b, :acc[b]] = np.sort(g.choice(N, acc[b], replace=False))
    rows = max(L, N)
    dst = src if in_place else torch.zeros(planes, batch, rows, width, dtype=torch.int16,
                                           device="cuda")
    if in_place and N < L:
        pytest.skip("in place needs L rows")
    want = dst.clone()
    for b in range(batch):
        want[:, b, :acc[b]] = src[:, b, torch.from_numpy(nodes[b, :acc[b]]).long().cuda()]
    ctx.commit_accepted(torch.from_numpy(acc).cuda(), torch.from_numpy(nodes).cuda(), src, dst)
    assert torch.equal(dst, want)
    assert ctx.device_status() == 0
    ctx.close()
