"""The logits pass at the edges of its block shapes: rows that just fit one tile
a wave and that just do not, four- and eight-wave blocks, rows split over blocks,
misaligned rows, rows of equal logits, whose candidates overflow the block's list,
and rows masked with large negative values.  Against float64 sums and a sort by
(logit descending, id ascending).

Tolerances: ids exact.  log q, lse and the entropy are fp64 sums of fp32
exponentials (2^-22 relative each) rounded to fp32; 1e-5 relative with a floor of
1e-6 is the bound of the parity tests."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")

pytestmark = pytest.mark.gpu

SHAPES = [
    # batch, L, V, K, kind
    (1, 1, 5, 5, "normal"),             # no vector at all: only loose elements
    (1, 3, 16384, 4, "normal"),         # 8 waves, exactly one tile a wave
    (1, 3, 16391, 13, "normal"),        # one vector fewer or the same, misaligned
    (2, 3, 16400, 64, "normal"),        # two vectors more: the streaming kernel
    (1, 2, 18433, 33, "normal"),        # the ninth tile
    (1, 64, 98312, 8, "normal"),        # 64 rows above the split line: 4 blocks a row
    (5, 13, 98312, 8, "normal"),        # one row more: not split
    (5, 13, 147473, 16, "normal"),      # 65 rows just past their line: 3 blocks a row
    (8, 16, 196625, 40, "normal"),      # 128 rows just past it: 2 blocks
    (10, 17, 294929, 8, "normal"),      # 170 rows just past it: 3 blocks, two a CU
    (9, 19, 294929, 8, "normal"),       # 171 rows: not split
    (257, 1, 196625, 64, "normal"),     # 257 rows: 3 blocks of four waves
    (31, 11, 196625, 8, "ordered"),     # 341 rows: the same
    (18, 19, 196625, 8, "normal"),      # 342 rows: not split
    (18, 19, 393233, 16, "normal"),     # 342 rows: 2 blocks
    (1, 4, 98304, 8, "normal"),         # at the line: not split
    (1, 3, 98311, 32, "normal"),        # split, misaligned, last split short
    (1, 1, 151937, 64, "normal"),       # the most splits a row of this size takes
    (1, 5, 300007, 64, "normal"),       # 32 blocks a row at most
    (16, 16, 8192, 16, "normal"),       # 256 rows: 8 waves
    (32, 16, 8192, 16, "normal"),       # 512 rows of one tile a wave: 4 waves
    (32, 16, 8200, 16, "normal"),       # 512 rows of more: 8 waves
    (1, 3, 2048, 40, "normal"),         # one vector a lane: 4 waves
    (1, 3, 2049, 40, "normal"),         # more: 8 waves
    (27, 19, 8201, 16, "normal"),       # 513 rows: 4 waves, just past one tile a wave
    (27, 19, 8191, 40, "normal"),       # 513 rows: 4 waves, at most one tile a wave
    (1, 2, 16000, 16, "equal"),         # one value: 16000 candidates tie
    (1, 2, 40000, 64, "equal"),
    (27, 19, 9000, 5, "equal"),
    (1, 2, 120000, 48, "equal"),        # split: every partial list is a tie
    (257, 1, 196625, 40, "equal"),
    (1, 3, 20011, 64, "levels"),        # four values only
    (1, 3, 120011, 17, "levels"),
    (65, 1, 147473, 24, "levels"),
    (1, 3, 16384, 4, "ordered"),        # the largest logits in one wave's share, most
    (2, 3, 8000, 64, "ordered"),        # of them in a few lanes: one tile a wave
    (27, 19, 8191, 40, "ordered"),
    (1, 3, 33000, 16, "ordered"),       # streamed: candidates of 128, 256 groups of lanes
    (1, 3, 33000, 17, "ordered"),
    (27, 19, 9000, 64, "ordered"),
    (1, 3, 151936, 64, "ordered"),      # split: one partial list holds the row's best
    (32, 1, 131080, 16, "normal"),      # split: the last split has a wave without a tile
    (1, 2, 100, 16, "normal"),          # fewer lanes with elements than candidates
    (1, 2, 1000, 64, "normal"),
]


def draw(kind, rows, V, seed):
    g = np.random.default_rng(seed)
    if kind == "equal":
        x = np.full((rows, V), -1.5, np.float32)
    elif kind == "ordered":   # words by frequency
        x = 2 * g.standard_normal((rows, V), dtype=np.float32) - np.log(np.arange(V) + 10.0)
    elif kind == "levels":
        x = g.integers(-2, 2, (rows, V)).astype(np.float32)
    else:
        x = g.standard_normal((rows, V), dtype=np.float32) * 3
    return torch.from_numpy(x.astype(np.float32)).to(torch.bfloat16)


def check_rows(G, ctx, x, K, out):
    """Candidates and statistics of the rows x [rows, V] against float64 and a stable sort."""
    rows = x.shape[0]
    d = x.double()
    lse = torch.logsumexp(d, -1)
    lp = d - lse[:, None]
    # stable: equal logits keep ascending ids
    want = torch.sort(x.float(), dim=-1, descending=True, stable=True).indices[:, :K]
    assert torch.equal(out.topk_ids.view(rows, K).long(), want)
    # float64 reference, copied to the host
    for got, ref in ((out.topk_logq.view(rows, K), lp.gather(-1, want)),
                     (out.row_lse.view(rows), lse),
                     (out.row_maxprob.view(rows), lp.max(-1).values.exp()),
                     (out.row_entropy.view(rows), -(lp.exp() * lp).sum(-1))):
        ref = ref.cpu().numpy()
        err = np.abs(got.double().cpu().numpy() - ref)
        assert (err <= 1e-6 + 1e-5 * np.abs(ref)).all()
    assert ctx.device_status() == 0


def context(G, batch, L, V, K):
    ctx = G.Context(batch, L, V, K, 8)
    emb = torch.zeros(V, 4, device="cuda")
    g = torch.zeros(4, 4, device="cuda")
    ctx.set_scorer(emb, g, g)
    return ctx


@pytest.mark.parametrize("batch,L,V,K,kind", SHAPES)
@pytest.mark.parametrize("static", [False, True])
def test_logits_shapes(batch, L, V, K, kind, static):
    import paper_2608_20375_amd as G
    print("batch", batch, "L", L, "V", V, "K", K, kind, static, flush=True)
    rows = batch * L
    x = draw(kind, rows, V, 77 + V + K).cuda()
    ctx = context(G, batch, L, V, K)
    zeros = torch.zeros(batch, dtype=torch.int32, device="cuda")
    out = ctx.build_tree(x.view(batch, L, V), zeros, zeros, fixed_budget=zeros + 1,
                         static_scratch=static)
    check_rows(G, ctx, x, K, out)
    ctx.close()


MASKED = [
    # batch, L, V, K
    (1, 3, 16384, 13),       # one tile a wave, 8 waves
    (27, 19, 8191, 40),      # one tile a wave, 4 waves
    (2, 3, 16400, 64),       # streamed, 8 waves
    (27, 19, 9001, 8),       # streamed, 4 waves
    (1, 3, 98311, 32),       # split, a tile a wave
    (32, 1, 131080, 16),     # split, streamed; the last split has a wave without a tile
    (257, 1, 196625, 24),    # split in three, 4 waves
]


@pytest.mark.parametrize("batch,L,V,K", MASKED)
@pytest.mark.parametrize("allowed", ["one", "few", "all but one of K"])
@pytest.mark.parametrize("mask", [-1e30, -1e32])
def test_masked_rows(batch, L, V, K, allowed, mask):
    """Constrained decoding: fewer than K words are allowed and the others hold a large
    negative finite logit, so masked words in id order fill the list."""
    import paper_2608_20375_amd as G
    print("masked", batch, L, V, K, allowed, mask, flush=True)
    rows = batch * L
    n = {"one": 1, "few": 3}.get(allowed, K - 1)
    g = np.random.default_rng(V + n)
    x = np.full((rows, V), mask, np.float32)
    for r in range(rows):
        # the allowed words spread, or at the row's ends, or together
        ids = (g.choice(V, n, replace=False), np.r_[V - 1, np.arange(n - 1)],
               V // 2 + np.arange(n))[r % 3]
        x[r, ids] = g.standard_normal(n) * 3
    x = torch.from_numpy(x).to(torch.bfloat16).cuda()
    ctx = context(G, batch, L, V, K)
    zeros = torch.zeros(batch, dtype=torch.int32, device="cuda")
    out = ctx.build_tree(x.view(batch, L, V), zeros, zeros, fixed_budget=zeros + 8)
    check_rows(G, ctx, x, K, out)
    assert (out.n_nodes == 8).all()
    ctx.close()
