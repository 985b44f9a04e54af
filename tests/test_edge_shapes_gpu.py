"""The edge stage over its dispatch: one to four column tiles, one wave a block and a
wave per parent tile, score dims that fill their k-slots and that are padded (by
whole groups of four and by single entries).  Edge scores against float64 (fp32
products of m terms of order one: 1e-5 relative, floor 1e-6, the parity tests'
bound), and the same sequences in a call of few blocks and of many give the same
bits: a tile's arithmetic does not depend on how the tiles are dealt out."""
import math

import numpy as np
import pytest

torch = pytest.importorskip("torch")

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("K", [1, 16, 17, 32, 33, 64])
@pytest.mark.parametrize("m", [1, 3, 16, 20, 32, 47, 59, 64])
@pytest.mark.parametrize("center", [0, 1])
def test_edge_shapes(K, m, center):
    import paper_2608_20375_amd as G
    print("edges K", K, "m", m, "center", center, flush=True)
    many, few, L, V, E = 129, 3, 8, 300, 12      # 1032 blocks: one wave each
    g = torch.Generator(device="cuda").manual_seed(K * 100 + m)
    rnd = lambda *s: torch.randn(*s, device="cuda", generator=g)
    ctx = G.Context(many, L, V, K, 32)
    emb, gp, gc, u = rnd(V, E) * 0.3, rnd(E, m) * 0.3, rnd(E, m) * 0.3, rnd(L, m) * 0.1
    beta = float(np.float32(0.2))
    ctx.set_scorer(emb, gp, gc, u, 1.5, beta, center)
    ctx.set_fusion(False)
    x = (rnd(many, L, V) * 2).to(torch.bfloat16)
    root = torch.randint(0, V, (many,), device="cuda", generator=g).to(torch.int32)
    fixed = torch.full((many,), 32, dtype=torch.int32, device="cuda")
    a = ctx.build_tree(x, root, root, fixed_budget=fixed, edges=True)
    b = ctx.build_tree(x[:few].contiguous(), root[:few].clone(), root[:few].clone(),
                       fixed_budget=fixed[:few].clone(), edges=True)
    # (rows of one vector a lane have one block shape in the logits pass, 24 or 1032)
    assert torch.equal(a.topk_ids[:few], b.topk_ids)
    assert torch.equal(a.topk_logq[:few], b.topk_logq)
    assert torch.equal(a.edge_scores[:few], b.edge_scores)
    D = torch.float64
    P, C, ud = emb.to(D) @ gp.to(D), emb.to(D) @ gc.to(D), u.to(D)
    ids = a.topk_ids.long()
    for l in range(L):
        prev = root.long()[:, None] if l == 0 else ids[:, l - 1]
        right = (C[ids[:, l]] + ud[l]).transpose(1, 2).contiguous()
        f = 1.5 / math.sqrt(m) * torch.matmul(P[prev] + ud[l], right)
        if center:
            f = f - f.mean(-1, keepdim=True)
        want = a.topk_logq[:, l].to(D)[:, None, :] + beta * f
        got = a.edge_scores[:, l, :want.shape[1]].to(D)
        assert (got - want).abs().le(1e-6 + 1e-5 * want.abs()).all(), l
    assert ctx.device_status() == 0
    ctx.close()
