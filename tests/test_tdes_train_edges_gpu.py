"""The training step where its blocks end: fewer rows than a contraction block, one
row past it, one and several batches of steps, more rows than a block's token slots,
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
    (2000, 32, 8, 4, 2, 66000, 300),      # 520 rows a block: two rounds of tokens
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
    # 260 rows a wave at the largest shape: still under 2e-5 of the error scale
    bound = 1e-4 * ref["abs_grad"] + 1e-12
    assert (np.abs(got["grad"] - ref["grad"]) <= bound).all()
    assert tt.device_status() == 0
    tt.close()
