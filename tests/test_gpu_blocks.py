"""The compositing kernels' 64-pixel wave blocks: every block shape a tile can
give, the dropping of list entries that reach no pixel of a block, and values
that are not finite."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")

from oracle import raster as R  # noqa: E402
from paper_2602_12314_amd import scenes  # noqa: E402
from tests.gpu_helpers import AMBIGUOUS, rel_err, to_np  # noqa: E402

pytestmark = pytest.mark.gpu

GRADS = ("means", "log_scales", "quats", "opacity_logits", "queries")


def _scene(d, n, seed, spread):
    """Gaussians of every aspect: log-scales spread over several orders of
    magnitude, so needles, dots and sheets larger than the image all occur."""
    rng = np.random.default_rng(seed)
    sp = scenes.custom_spec("blocks", n, [scenes.pinhole(75, 53, 60.0)], d=d)
    s = scenes.make_scene(sp, seed=seed, with_target=False)
    s.log_scales[:] = rng.uniform(-3.5 - spread, -2.0 + 0.5 * spread, size=s.log_scales.shape)
    s.opacity_logits[:] = rng.uniform(-7.0, 5.0, size=n)  # some never reach 1/255, some clamp at 0.99
    return s


def _run(s, tile, dQ=None, queries=None):
    from paper_2602_12314_amd import ops
    g = ops.Gaussians.from_numpy(s)
    if queries is not None:
        g.queries = queries
    r = ops.Renderer(s.cams, s.n, s.spec.d, tile=tile)
    Q, T = r.forward(g)
    return r, g, Q, T, (None if dQ is None else r.backward(g, dQ))


@pytest.mark.parametrize("d", [16, 32])
@pytest.mark.parametrize("spread", [0.5, 3.0])
def test_dropped_entries_match_oracle(d, spread):
    s = _scene(d, 700, 5, spread)
    f = R.render_forward(R.Gaussians.of(s), s.cams)
    ok = f["margin"] >= AMBIGUOUS
    assert ok.mean() > 0.98
    dQ = np.random.default_rng(1).standard_normal(f["Q"].shape)
    dQ[~ok] = 0.0
    ref = R.render_backward(R.Gaussians.of(s), s.cams, dQ)
    _, _, Q, T, gr = _run(s, (16, 16), torch.as_tensor(dQ, dtype=torch.float32, device="cuda"))
    assert rel_err(to_np(Q)[ok], f["Q"][ok]) <= 1e-4
    assert rel_err(to_np(T)[ok], f["T_final"][ok]) <= 1e-4
    for name in GRADS:
        assert rel_err(to_np(getattr(gr, name)), ref[name]) <= 1e-4, name


@pytest.mark.parametrize("tile", [(8, 8), (64, 1), (1, 64), (2, 32), (4, 64), (64, 4), (128, 2), (32, 8)])
def test_block_shapes(tile):
    s = _scene(16, 500, 9, 2.0)
    n = int(s.cams[0, 0] * s.cams[0, 1])
    dQ = torch.as_tensor(np.random.default_rng(2).standard_normal((n, 16)), dtype=torch.float32, device="cuda")
    _, _, Q0, T0, g0 = _run(s, (16, 16), dQ)
    _, _, Q1, T1, g1 = _run(s, tile, dQ)
    assert torch.equal(Q0, Q1) and torch.equal(T0, T1)
    # float32 sums in another order: each is within the gradients' bar of 1e-4
    # of the float64 value, so two of them are within twice that
    for name in GRADS:
        assert rel_err(to_np(getattr(g1, name)), to_np(getattr(g0, name))) <= 2e-4, name


@pytest.mark.parametrize("d", [16, 32])
@pytest.mark.parametrize("value", [float("inf"), float("nan")])
def test_values_that_are_not_finite_stay_with_their_pairs(d, value):
    s = _scene(d, 400, 3, 0.5)
    n = int(s.cams[0, 0] * s.cams[0, 1])
    q = torch.as_tensor(s.queries, device="cuda")
    _, _, Q0, _, _ = _run(s, (16, 16))
    # which pixels a Gaussian is blended into: its query alone set to one
    who = int(np.argmax(s.opacity_logits + 0.5 * s.log_scales.sum(1)))
    one = torch.zeros_like(q)
    one[who] = 1.0
    touched = _run(s, (16, 16), queries=one)[2].abs().sum(1) > 0
    assert 0 < int(touched.sum()) < n
    bad = q.clone()
    bad[who, 3] = value
    Q1 = _run(s, (16, 16), queries=bad)[2]
    assert torch.equal(~torch.isfinite(Q1).all(1), touched)
    assert torch.equal(Q1[~touched], Q0[~touched])
    # an upstream gradient that is not finite at one pixel
    pix = int(torch.nonzero(touched)[0])
    dQ = torch.as_tensor(np.random.default_rng(4).standard_normal((n, d)), dtype=torch.float32, device="cuda")
    zero = dQ.clone()
    zero[pix] = 0.0
    dbad = dQ.clone()
    dbad[pix, 1] = value
    only = torch.zeros_like(dQ)
    only[pix] = 1.0
    blended = _run(s, (16, 16), only)[4].queries.abs().sum(1) > 0
    g0, g1 = _run(s, (16, 16), zero)[4], _run(s, (16, 16), dbad)[4]
    assert torch.equal(~torch.isfinite(g1.queries).all(1), blended)
    for name in GRADS:
        a, b = getattr(g1, name)[~blended], getattr(g0, name)[~blended]
        assert bool(torch.isfinite(a).all()) and rel_err(to_np(a), to_np(b)) <= 2e-4, name


@pytest.mark.parametrize("n", [1, 63, 64, 65, 4095, 4096, 4097])
def test_depth_order_around_the_small_sort(n):
    """Both sides of the size from which the records are sorted by radix passes:
    the binning (tests of whole scenes check it entry by entry) and with it Q
    against the oracle, with equal depths among the records."""
    s = _scene(16, n, 11, 0.0)
    s.means[:, 2] = np.round(s.means[:, 2] * 16) / 16  # ties: by index
    s.means[n // 3:n // 2, 2] = -1.0                   # culled
    s.log_scales[:] -= 1.0
    f = R.render_forward(R.Gaussians.of(s), s.cams)
    ok = f["margin"] >= AMBIGUOUS
    _, _, Q, T, _ = _run(s, (16, 16))
    assert rel_err(to_np(T)[ok], f["T_final"][ok]) <= 1e-4
    assert rel_err(to_np(Q)[ok], f["Q"][ok]) <= 1e-4


@pytest.mark.parametrize("d", [16, 32])
@pytest.mark.parametrize("n", [1, 63, 257, 4097])
def test_each_backward_starts_from_cleared_sums(n, d):
    """A backward after another of the same forward, whose upstream gradient left
    values that are not finite in every sum it reached."""
    s = _scene(d, n, 13, 0.5)
    px = int(s.cams[0, 0] * s.cams[0, 1])
    dQ = torch.as_tensor(np.random.default_rng(6).standard_normal((px, d)), dtype=torch.float32, device="cuda")
    r, g, _, _, first = _run(s, (16, 16), dQ)
    first = {name: to_np(getattr(first, name)).copy() for name in GRADS}
    r.backward(g, torch.full_like(dQ, float("nan")))
    again = r.backward(g, dQ)
    # the same sums in another order of arrival: both within the gradients' bar
    for name in GRADS:
        a = to_np(getattr(again, name))
        assert np.isfinite(a).all() and rel_err(a, first[name]) <= 2e-4, name
