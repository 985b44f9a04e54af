"""The binding's short check of a call's tensors against its full one: a tensor that
the short check takes gives the same pointer, and everything else goes to the full
check, which raises what it raised or accepts what it accepted.  On the CPU a tensor
stands in for one on the GPU (is_cuda is all the short check asks of the device)."""
import pytest

torch = pytest.importorskip("torch")

import paper_2608_20375_amd as G  # noqa: E402


class OnGpu(torch.Tensor):
    """A CPU tensor that says it is on the GPU."""
    is_cuda = True


def gpu(*shape, dtype=torch.int32):
    return torch.zeros(*shape, dtype=dtype).as_subclass(OnGpu)


def test_plain_takes_exact_tensors_only():
    t = gpu(3, 4)
    assert G._plain(None, torch.int32, (3, 4)) is None
    assert G._plain(t, torch.int32, (3, 4)) == t.data_ptr()
    for bad in (gpu(4, 3), gpu(12), gpu(3, 4, 1), gpu(4, 4), gpu(3, 4, dtype=torch.int64),
                gpu(4, 3).t(), gpu(3, 8)[:, :4], torch.zeros(3, 4, dtype=torch.int32), [0] * 12, 7):
        assert G._plain(bad, torch.int32, (3, 4)) == -1


def context():
    ctx = G.Context.__new__(G.Context)
    ctx.dims = G.Dims(4, 6, 100, 5, 70, 4)
    return ctx


class Out:
    batch, sizes = 4, (6, 5, 70)


def args(B=3, **kw):
    a = dict(logits=gpu(B, 6, 100, dtype=torch.bfloat16), root_token=gpu(B), base_pos=gpu(B),
             prefix_len=gpu(B), hist=gpu(B, dtype=torch.float32), fixed_budget=gpu(B),
             hidden=gpu(B, 6, 16, dtype=torch.bfloat16), out=Out())
    a.update(kw)
    return a


def test_round_takes_the_forms_of_the_full_check():
    a = args()
    r = context()._round_plain(**a)
    assert (r.batch, r.hidden_dim) == (3, 16)
    for f in ("logits", "root_token", "base_pos", "prefix_len", "hist", "fixed_budget", "hidden"):
        assert getattr(r, f) == a[f].data_ptr()
    a = args(hidden=None, hist=None, prefix_len=None, fixed_budget=None)
    r = context()._round_plain(**a)
    assert r.hidden is None and r.hidden_dim == 0 and r.hist is None
    for dt in (torch.int16, torch.uint16):
        assert context()._round_plain(**args(logits=gpu(3, 6, 100, dtype=dt))) is not None


class Small:
    batch, sizes = 2, (6, 5, 70)


class Other:
    batch, sizes = 4, (6, 5, 71)


@pytest.mark.parametrize("change", [
    dict(out=None), dict(out=Small()), dict(out=Other()), dict(root_token=None),
    dict(base_pos=None), dict(logits=gpu(3, 6, 101, dtype=torch.bfloat16)),
    dict(logits=gpu(3, 6, 100, dtype=torch.float32)), dict(logits=gpu(3, 600)),
    dict(logits=None), dict(root_token=gpu(4)), dict(hist=gpu(3)),
    dict(prefix_len=gpu(3, dtype=torch.int64)), dict(fixed_budget=gpu(3, 1)),
    dict(hidden=gpu(3, 5, 16, dtype=torch.bfloat16)), dict(hidden=gpu(3, 6, 16)),
    dict(hidden=gpu(3, 96, dtype=torch.bfloat16)), dict(base_pos=torch.zeros(3, dtype=torch.int32)),
    dict(logits=gpu(3, 100, 6, dtype=torch.bfloat16).transpose(1, 2))])
def test_round_leaves_the_rest_to_the_full_check(change):
    assert context()._round_plain(**args(**change)) is None
