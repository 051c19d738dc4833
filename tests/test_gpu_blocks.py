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


def _run_rgbd(s, col, dQ=None, d_rgb=None, d_depth=None, queries=None, tile=(16, 16)):
    """(Q, rgb, depth, T) and, with upstream gradients, the gradients by name."""
    from paper_2602_12314_amd import ops
    g = ops.Gaussians.from_numpy(s)
    if queries is not None:
        g.queries = queries
    r = ops.Renderer(s.cams, s.n, s.spec.d, tile=tile)
    maps = r.forward_rgbd(g, col)
    if dQ is None:
        return maps, None
    out, d_colors = r.backward_rgbd(g, col, dQ, d_rgb, d_depth)
    return maps, dict({name: getattr(out, name) for name in GRADS}, colors=d_colors)


def _upstream(n, d, seed, ok=None):
    rng = np.random.default_rng(seed)
    out = [rng.standard_normal(shape).astype(np.float32) for shape in ((n, d), (n, 3), (n,))]
    if ok is not None:
        for a in out:
            a[~ok] = 0.0
    return out


def _backward(s, queries, colors, up, rgbd):
    """Gradients by name for these queries and colours (numpy float32)."""
    dev = lambda a: torch.as_tensor(a, device="cuda")
    if rgbd:
        return {k: to_np(v) for k, v in
                _run_rgbd(s, dev(colors), *(dev(a) for a in up), queries=dev(queries))[1].items()}
    gr = _run(s, (16, 16), dev(up[0]), queries=dev(queries))[4]
    return {k: to_np(getattr(gr, k)) for k in GRADS}


def _oracle_backward(s, queries, colors, up, rgbd):
    g = R.Gaussians.of(s)
    d = s.spec.d
    g.queries = np.ascontiguousarray(np.concatenate([queries, colors], axis=1) if rgbd else queries)
    dmap = np.concatenate(up[:2], axis=1) if rgbd else up[0]
    ref = R.render_backward(g, s.cams, dmap.astype(np.float64), dZ=up[2].astype(np.float64) if rgbd else None)
    out = {k: ref[k] for k in GRADS}
    if rgbd:
        out["queries"], out["colors"] = ref["queries"][:, :d], ref["queries"][:, d:]
    return out


@pytest.mark.parametrize("rgbd", [False, True])
@pytest.mark.parametrize("d", [16, 32])
@pytest.mark.parametrize("value", [1e4, 1e30])
def test_culled_first_gaussian_takes_no_part(d, value, rgbd):
    """A few entries per block, so that most batches of the backward are not
    full, and a Gaussian 0 that no view sees with a large finite query and
    colour: the others' gradients are the oracle's."""
    s = _scene(d, 60, 21, 0.5)
    s.means[0, 2] = -1.0
    f = R.render_forward(R.Gaussians.of(s), s.cams)
    ok = f["margin"] >= AMBIGUOUS
    up = _upstream(ok.size, d, 22, ok)
    q = s.queries.astype(np.float32)
    col = np.random.default_rng(23).uniform(0.0, 1.0, (s.n, 3)).astype(np.float32)
    q[0], col[0] = value, value
    ref = _oracle_backward(s, q, col, up, rgbd)
    got = _backward(s, q, col, up, rgbd)
    for name in ref:
        assert np.isfinite(got[name]).all(), name
        assert rel_err(got[name], ref[name]) <= 1e-4, name


@pytest.mark.parametrize("rgbd", [False, True])
@pytest.mark.parametrize("d", [16, 32])
@pytest.mark.parametrize("value", [1e4, 1e6, 1e30])
def test_large_values_stay_with_their_pixels(d, value, rgbd):
    """Small Gaussians, many to a block but seldom two on one pixel, a twentieth
    of them with queries and colours ``value`` times the others': Gaussians
    that share no pixel with those have the oracle's gradients."""
    s = _scene(d, 900, 31, 0.0)
    rng = np.random.default_rng(32)
    s.log_scales[:] = rng.uniform(-4.5, -3.5, size=s.log_scales.shape)
    s.opacity_logits[:] = rng.uniform(-1.0, 4.0, size=s.n)
    f = R.render_forward(R.Gaussians.of(s), s.cams)
    ok = f["margin"] >= AMBIGUOUS
    up = _upstream(ok.size, d, 33, ok)
    loud = rng.random(s.n) < 0.05
    mark = np.zeros((s.n, d), np.float32)
    mark[loud] = 1.0
    touched = to_np(_run(s, (16, 16), queries=torch.as_tensor(mark, device="cuda"))[2]).any(axis=1)
    on = np.zeros((ok.size, d), np.float32)
    on[touched] = 1.0
    zero = [on, np.zeros((ok.size, 3), np.float32), np.zeros(ok.size, np.float32)]
    quiet = ~_backward(s, s.queries.astype(np.float32), None, zero, False)["queries"].any(axis=1)
    assert 0.3 * s.n < quiet.sum() < s.n - loud.sum()
    q = s.queries.astype(np.float32)
    col = rng.uniform(0.0, 1.0, (s.n, 3)).astype(np.float32)
    q[loud] *= np.float32(value)
    col[loud] *= np.float32(value)
    ref = _oracle_backward(s, q, col, up, rgbd)
    got = _backward(s, q, col, up, rgbd)
    for name in ref:
        assert np.isfinite(got[name][quiet]).all(), name
        assert rel_err(got[name][quiet], ref[name][quiet]) <= 1e-4, name


@pytest.mark.parametrize("rgbd", [False, True])
@pytest.mark.parametrize("d", [16, 32])
def test_common_offset_of_the_queries(d, rgbd):
    """Opaque pixels and queries (and colours) of unit spread around 1000: the
    gradient of alpha is a difference of dot products that share the offset's.
    Rounded each on its own they would lose 1000 x 2^-24 x a few = 2e-4 of it;
    taken relative to a common query they keep the gradients' bar."""
    s = _scene(d, 700, 41, 0.5)
    s.log_scales[:] += 0.5
    s.opacity_logits[:] = np.random.default_rng(42).uniform(0.0, 4.0, size=s.n)
    f = R.render_forward(R.Gaussians.of(s), s.cams)
    ok = (f["margin"] >= AMBIGUOUS) & (f["T_final"] < 1e-2)
    assert ok.mean() > 0.5
    up = _upstream(ok.size, d, 43, ok)
    q = (1000.0 + s.queries).astype(np.float32)
    col = (1000.0 + np.random.default_rng(44).standard_normal((s.n, 3))).astype(np.float32)
    ref = _oracle_backward(s, q, col, up, rgbd)
    got = _backward(s, q, col, up, rgbd)
    for name in ref:
        assert rel_err(got[name], ref[name]) <= 1e-4, name


@pytest.mark.parametrize("d", [16, 32])
@pytest.mark.parametrize("value", [float("inf"), float("nan")])
def test_rgbd_values_that_are_not_finite_stay_with_their_pairs(d, value):
    s = _scene(d, 400, 3, 0.5)
    n = int(s.cams[0, 0] * s.cams[0, 1])
    col = torch.as_tensor(np.random.default_rng(51).uniform(0.0, 1.0, (s.n, 3)), dtype=torch.float32, device="cuda")
    (Q0, rgb0, z0, _), _ = _run_rgbd(s, col)
    who = int(np.argmax(s.opacity_logits + 0.5 * s.log_scales.sum(1)))
    one = torch.zeros((s.n, d), device="cuda")
    one[who] = 1.0
    touched = _run(s, (16, 16), queries=one)[2].abs().sum(1) > 0
    assert 0 < int(touched.sum()) < n
    bad = col.clone()
    bad[who, 1] = value
    (Q1, rgb1, z1, _), _ = _run_rgbd(s, bad)
    assert torch.equal(Q1, Q0) and torch.equal(z1, z0)
    assert torch.equal(~torch.isfinite(rgb1).all(1), touched)
    assert torch.equal(rgb1[~touched], rgb0[~touched])
    # an upstream gradient of colour or depth that is not finite at one pixel
    pix = int(torch.nonzero(touched)[0])
    up = [torch.as_tensor(a, device="cuda") for a in _upstream(n, d, 52)]
    only = torch.zeros((n, d), device="cuda")
    only[pix] = 1.0
    blended = _run(s, (16, 16), only)[4].queries.abs().sum(1) > 0
    zero = [a.clone() for a in up]
    for a in zero:
        a[pix] = 0.0
    g0 = _run_rgbd(s, col, *zero)[1]
    for which in (1, 2):
        dbad = [a.clone() for a in up]
        if which == 1:
            dbad[1][pix, 2] = value
        else:
            dbad[2][pix] = value
        g1 = _run_rgbd(s, col, *dbad)[1]
        if which == 1:
            assert torch.equal(~torch.isfinite(g1["colors"]).all(1), blended)
        else:  # the depth's gradient reaches the means alone
            assert bool((~torch.isfinite(g1["means"]).all(1))[blended].all())
        for name in g0:
            a, b = g1[name][~blended], g0[name][~blended]
            assert bool(torch.isfinite(a).all()) and rel_err(to_np(a), to_np(b)) <= 2e-4, (which, name)


@pytest.mark.parametrize("n", [1, 257, 4097])
def test_each_rgbd_backward_starts_from_cleared_sums(n):
    s = _scene(16, n, 13, 0.5)
    px = int(s.cams[0, 0] * s.cams[0, 1])
    col = torch.as_tensor(np.random.default_rng(61).uniform(0.0, 1.0, (n, 3)), dtype=torch.float32, device="cuda")
    up = [torch.as_tensor(a, device="cuda") for a in _upstream(px, 16, 62)]
    from paper_2602_12314_amd import ops
    g = ops.Gaussians.from_numpy(s)
    r = ops.Renderer(s.cams, s.n, 16)
    r.forward_rgbd(g, col)

    def grads(up):
        out, dc = r.backward_rgbd(g, col, *up)
        return dict({name: to_np(getattr(out, name)).copy() for name in GRADS}, colors=to_np(dc).copy())

    first = grads(up)
    grads([torch.full_like(a, float("nan")) for a in up])
    again = grads(up)
    for name in first:
        assert np.isfinite(again[name]).all() and rel_err(again[name], first[name]) <= 2e-4, name


@pytest.mark.parametrize("tile", [(8, 8), (64, 1), (1, 64), (64, 4), (128, 2)])
def test_rgbd_block_shapes(tile):
    s = _scene(32, 500, 9, 2.0)
    n = int(s.cams[0, 0] * s.cams[0, 1])
    col = torch.as_tensor(np.random.default_rng(71).uniform(0.0, 1.0, (s.n, 3)), dtype=torch.float32, device="cuda")
    up = [torch.as_tensor(a, device="cuda") for a in _upstream(n, 32, 72)]
    m0, g0 = _run_rgbd(s, col, *up)
    m1, g1 = _run_rgbd(s, col, *up, tile=tile)
    for a, b in zip(m0, m1):
        assert torch.equal(a, b)
    for name in g0:  # both within the gradients' bar of the float64 value
        assert rel_err(to_np(g1[name]), to_np(g0[name])) <= 2e-4, name
