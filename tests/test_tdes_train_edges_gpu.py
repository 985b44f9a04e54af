"""The training step where its blocks end: fewer rows than a contraction block, one
row past it, one and several batches of steps, more blocks of the most rows than CUs,
K at and past one tile of children, m that fills its tiles and that does not, groups
or pairs alone.  Against the oracle with the bounds of test_tdes_train_gpu (the
weighted child sums are sums of terms the oracle's error scale counts one by one)."""
import os
import sys

import numpy as np
import pytest

sys.path.insert(0, os.path.dirname(os.path.abspath(__file__)))
import test_tdes_train_gpu as TT  # noqa: E402
from oracle import tdes_train as T  # noqa: E402

torch = pytest.importorskip("torch")

pytestmark = pytest.mark.gpu

SHAPES = [
    # V, E, m, L, K, G, P
    (300, 128, 32, 3, 16, 1, 0),
    (300, 64, 16, 3, 4, 0, 1),
    (300, 32, 64, 3, 17, 15, 1),          # EB = 2: four row groups a block
    (300, 64, 50, 5, 15, 17, 8),          # EB = 4: two
    (300, 128, 31, 5, 16, 16, 9),
    (2000, 128, 32, 16, 13, 130, 2047),
    (2000, 64, 33, 12, 2, 3000, 1),
    (2000, 32, 8, 4, 2, 66000, 300),      # 347 blocks of 384 rows
]


@pytest.mark.parametrize("shape", SHAPES, ids=lambda s: "V%d_E%d_m%d_L%d_K%d_G%d_P%d" % s)
def test_step_edges(shape):
    V, E, m, L, K, G, P = shape
    TT._say("tdes step edges", shape)
    GR, w, sc, tr, tr_gpu, theta, tt = TT._setup(*shape)
    hg, ho = TT._hyper(GR)
    z = np.zeros_like(theta)
    got = TT._gpu_step(tt, torch.from_numpy(sc["emb"]).cuda(), tr_gpu, theta, z, z, 1, hg)
    ref = T.train_step(theta.astype(np.float64), z, z, 1, sc["emb"], tr, ho, E, m, L)
    np.testing.assert_allclose(got["loss"], np.array(ref["loss"]), rtol=2e-5, atol=1e-9)
    bound = 1e-4 * ref["abs_grad"] + 1e-12
    assert (np.abs(got["grad"] - ref["grad"]) <= bound).all()
    assert tt.device_status() == 0
    tt.close()


@pytest.mark.parametrize("E,m", [(32, 16), (64, 16), (128, 16), (128, 32)])
@pytest.mark.parametrize("G,K", [(1 << 12, 16), (1 << 19, 2)])
def test_gradient_error_does_not_grow_with_the_batch(E, m, G, K):
    """G copies of one group, G a power of two: every row adds the same term, exactly
    1 / G of the one that a batch of the group alone has, so the weight gradients differ
    from that batch's only by the roundings of the sum.  They all point one way, and a
    sum may take at most the ones the step promises: chains of 24 rows, 16 of them, then
    fp64 over the blocks: 40 u, u = 2^-24."""
    TT._say("tdes copies of a group", E, m, G, K)
    V, L = 500, 4
    GR, w, sc, tr, tr_gpu, theta, tt = TT._setup(V, E, m, L, K, 1, 0)
    tt.close()
    hg, _ = TT._hyper(GR, lambda_bce=0.0)
    z = np.zeros_like(theta)
    emb = torch.from_numpy(sc["emb"]).cuda()
    grads = []
    for n in (1, G):
        tt = GR.TdesTrainer(V, E, m, L, K, n, 1)
        copies = {k: v.expand(n, *v.shape[1:]).contiguous() for k, v in tr_gpu.items()
                  if k != "pairs"}
        grad = TT._gpu_step(tt, emb, copies, theta, z, z, 1, hg)["grad"]
        grads.append(grad[:2 * E * m].astype(np.float64))
        assert tt.device_status() == 0
        tt.close()
    assert np.abs(grads[0]).max() > 1e-6
    assert (np.abs(grads[1] - grads[0]) <= 40 * 2.0 ** -24 * np.abs(grads[0])).all()
