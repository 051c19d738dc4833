"""GPU parity of the dictionary decode and feature loss (Eq. 5-6) against the
FP64 oracle, through the C ABI.

Bars: FP32 path within 1e-4 relative per output tensor (F, loss, dQ, dK, dV);
BF16 path: minimum per-pixel cosine of F >= 0.999 and relative gradient error
<= 1e-2 per tensor.  Shapes cover ragged pixel counts (not a multiple of the
32-pixel block), atom counts that need padding, both query widths and the
full 640x480 workload.
"""
import numpy as np
import pytest

torch = pytest.importorskip("torch")

from oracle import decode_oracle as DO  # noqa: E402
from tests.gpu_helpers import rel_err, say, to_np  # noqa: E402

pytestmark = pytest.mark.gpu

BARS = {"fp32": dict(grad=1e-4, cos=None, F=1e-4), "bf16": dict(grad=1e-2, cos=0.999, F=None),
        "fp8": dict(grad=1e-2, cos=0.999, F=None)}

# FP8: V in OCP E4M3 (3 mantissa bits) with a scale per atom, the softmax
# weights as two E4M3 terms, so F carries V's rounding.  The per-pixel cosine of
# F meets 0.999 everywhere; dQ meets 1e-2 at the logit spread of rendered query
# maps (test_fp8_meets_bars_at_rendered_query_scale) but not with the unit
# Gaussian queries of these shapes, whose sharper softmax puts F close to a few
# rows of V whose rounding is then not averaged out (1.0-1.9e-2; the strict xfail
# below).  At M = 1, dS should vanish exactly but the FP8 F and the BF16
# backward disagree by the E4M3 rounding of V, so dK misses there too.
FP8_MISSES = {"dQ"}


def _inputs(seed, n, d, M, D, qscale=1.0):
    rng = np.random.default_rng(seed)
    Q = (qscale * rng.standard_normal((n, d))).astype(np.float32)
    K = rng.standard_normal((M, d)).astype(np.float32)
    V = rng.standard_normal((M, D)).astype(np.float32)
    T = rng.standard_normal((n, D))
    T = (T / np.linalg.norm(T, axis=1, keepdims=True)).astype(np.float32)
    K0 = (K + 0.01 * rng.standard_normal(K.shape)).astype(np.float32)
    return Q, K, V, T, K0


def _cuda(*arrs):
    return [torch.as_tensor(a, device="cuda") for a in arrs]


def _decoder(prec, n, d, M, D, ctx=None):
    from paper_2602_12314_amd import ops
    return ops.Decoder(prec, n, d, M, D, ctx=ctx)


def _cos(a, b):
    a = np.asarray(a, np.float64)
    b = np.asarray(b, np.float64)
    return (a * b).sum(1) / (np.linalg.norm(a, axis=1) * np.linalg.norm(b, axis=1))


def _min_cos(a, b):
    return float(_cos(a, b).min())


# (n, d, M, D).  M = 150 pads to 192 atoms: six 32-atom tiles (two waves hold
# an odd number), three 64-atom E4M3 chunks, and D = 384 gives three D tiles
# per wave.
SHAPES = [(1000, 16, 64, 128), (777, 32, 100, 256), (4096, 16, 256, 512), (333, 32, 512, 768),
          (200, 16, 1, 128), (96, 32, 1024, 1024), (515, 16, 150, 384)]


@pytest.mark.parametrize("prec", ["fp32", "bf16", "fp8"])
@pytest.mark.parametrize("shape", SHAPES)
def test_forward_F(prec, shape):
    n, d, M, D = shape
    say(f"[decode F] {prec} n={n} d={d} M={M} D={D}")
    Q, K, V, _, _ = _inputs(1, n, d, M, D)
    dec = _decoder(prec, n, d, M, D)
    F = to_np(dec.forward(*_cuda(Q, K, V)))
    ref = DO.decode_forward(Q, K, V)[0]
    if BARS[prec]["F"]:
        e = rel_err(F, ref)
        say(f"  rel err {e:.3e}")
        assert e < BARS[prec]["F"]
    else:
        c = _cos(F, ref)
        say(f"  cos min {c.min():.6f} p1 {np.percentile(c, 1):.6f} mean {c.mean():.6f}")
        assert c.min() >= BARS[prec]["cos"]
        if prec == "fp8":
            # the kernel implements the documented E4M3 rounding
            from tests.fp8_model import fp8_forward
            cm = _cos(F, fp8_forward(Q, K, V))
            assert np.percentile(cm, 0.1) >= 1 - 1e-5, cm.min()


@pytest.mark.parametrize("prec", ["fp32", "bf16", "fp8"])
@pytest.mark.parametrize("shape", SHAPES)
def test_loss_and_grads(prec, shape):
    n, d, M, D = shape
    say(f"[decode loss] {prec} n={n} d={d} M={M} D={D}")
    Q, K, V, T, K0 = _inputs(2, n, d, M, D)
    dec = _decoder(prec, n, d, M, D)
    row_cos = torch.empty(n, device="cuda")
    loss, dQ, dK, dV = dec.loss_and_grads(*_cuda(Q, K, V, T, K0), 0.1, row_cos=row_cos)
    ref = DO.loss_and_grads(Q, K, V, T, K0, 0.1)
    bar = BARS[prec]["grad"]
    el = abs(float(loss) - ref["loss"]) / abs(ref["loss"])
    say(f"  loss {float(loss):.7f} ref {ref['loss']:.7f} rel {el:.2e}")
    assert el < bar
    assert np.abs(to_np(row_cos) - ref["cos"]).max() < {"fp32": 1e-5, "bf16": 5e-3, "fp8": 2e-2}[prec]
    for name, t in (("dQ", dQ), ("dK", dK), ("dV", dV)):
        e = rel_err(to_np(t), ref[name])
        say(f"  {name} rel err {e:.3e}")
        if prec == "fp8" and (name in FP8_MISSES or (M == 1 and name == "dK")):
            assert e < 2.5 * bar, name  # reported; the bar itself is the xfail test below
            continue
        assert e < bar, name


def _fp8_bars(n, d, M, D, qscale, seed=2):
    Q, K, V, T, K0 = _inputs(seed, n, d, M, D, qscale=qscale)
    dec = _decoder("fp8", n, d, M, D)
    F = to_np(dec.forward(*_cuda(Q, K, V)))
    loss, dQ, dK, dV = dec.loss_and_grads(*_cuda(Q, K, V, T, K0), 0.1)
    ref = DO.loss_and_grads(Q, K, V, T, K0, 0.1)
    c = _min_cos(F, ref["F"])
    errs = {k: rel_err(to_np(t), ref[k]) for k, t in (("dQ", dQ), ("dK", dK), ("dV", dV))}
    say(f"  min cos {c:.6f} " + " ".join(f"{k} {v:.3e}" for k, v in errs.items()))
    assert c >= 0.999
    for k, v in errs.items():
        assert v < 1e-2, k


@pytest.mark.parametrize("shape", [(4096, 32, 1024, 1024), (3000, 32, 512, 768)])
def test_fp8_meets_bars_at_rendered_query_scale(shape):
    """The benchmark spec bars (minimum per-pixel cosine of F >= 0.999, every
    gradient within 1e-2) for the E4M3 decode at the logit spread of rendered
    query maps: the queries of the 1200x680 keyframe of the 2M-Gaussian map
    (a blend of N(0, 1) queries) have a per-component spread of 0.56."""
    n, d, M, D = shape
    say(f"[decode fp8 bars, q spread 0.56] n={n} d={d} M={M} D={D}")
    _fp8_bars(n, d, M, D, qscale=0.56)


@pytest.mark.xfail(strict=True, reason="with unit Gaussian queries the softmax is sharper and F sits "
                   "close to a few rows of V, whose E4M3 rounding (3 mantissa bits) is not averaged out: "
                   "dQ reaches 1.0-1.6e-2 (the cosine and dK, dV still meet their bars)")
@pytest.mark.parametrize("shape", [SHAPES[2], SHAPES[5]])
def test_fp8_meets_bars_with_unit_queries(shape):
    n, d, M, D = shape
    say(f"[decode fp8 bars, unit queries] n={n} d={d} M={M} D={D}")
    _fp8_bars(n, d, M, D, qscale=1.0)


# 64-pixel x 8-wave workgroups (the context option "decode_shape": 1): D = 256 (one D tile
# per wave), 512 (two), 768 (three) and 1024 (four, at d = 32 and d = 16, the latter with
# 300 atoms: padded atom tiles and an odd count of 64-atom E4M3 chunks), in BF16 and E4M3.
WIDE_SHAPES = [(777, 32, 100, 256), (4096, 16, 256, 512), (333, 32, 512, 768), (1000, 32, 1000, 1024),
               (2048, 16, 300, 1024)]


@pytest.mark.parametrize("prec", ["bf16", "fp8"])
@pytest.mark.parametrize("shape", WIDE_SHAPES)
def test_wide_decode_shape(prec, shape):
    from paper_2602_12314_amd import _lib
    n, d, M, D = shape
    say(f"[decode px64] {prec} n={n} d={d} M={M} D={D}")
    Q, K, V, T, K0 = _inputs(3, n, d, M, D)
    ctx = _lib.Context(options={"decode_shape": "px64"})
    dec = _decoder(prec, n, d, M, D, ctx=ctx)
    F = to_np(dec.forward(*_cuda(Q, K, V)))
    loss, dQ, dK, dV = dec.loss_and_grads(*_cuda(Q, K, V, T, K0), 0.1)
    dQb, dKb, dVb = dec.backward(*_cuda(Q, K, V, T.astype(np.float32) * 0.01))
    ref = DO.loss_and_grads(Q, K, V, T, K0, 0.1)
    c = _cos(F, ref["F"])
    say(f"  cos min {c.min():.6f} mean {c.mean():.6f}")
    assert c.min() >= 0.999
    assert abs(float(loss) - ref["loss"]) / abs(ref["loss"]) < 1e-2
    for name, t in (("dQ", dQ), ("dK", dK), ("dV", dV)):
        e = rel_err(to_np(t), ref[name])
        say(f"  {name} rel err {e:.3e}")
        assert e < (2.5e-2 if prec == "fp8" and name == "dQ" else 1e-2), name
    refb = dict(zip(("dQ", "dK", "dV"), DO.decode_backward(Q, K, V, T.astype(np.float64) * 0.01)))
    for name, t in (("dQ", dQb), ("dK", dKb), ("dV", dVb)):
        e = rel_err(to_np(t), refb[name])
        say(f"  given dF: {name} rel err {e:.3e}")
        assert e < (5e-2 if prec == "fp8" else 1e-2), name


@pytest.mark.parametrize("prec", ["fp32", "bf16"])
def test_backward_given_dF(prec):
    n, d, M, D = 1500, 32, 192, 384
    say(f"[decode adjoint] {prec}")
    Q, K, V, _, _ = _inputs(3, n, d, M, D)
    dF = np.random.default_rng(4).standard_normal((n, D)).astype(np.float32)
    dec = _decoder(prec, n, d, M, D)
    dQ, dK, dV = dec.backward(*_cuda(Q, K, V, dF))
    rQ, rK, rV = DO.decode_backward(Q, K, V, dF)
    bar = BARS[prec]["grad"]
    for name, t, r in (("dQ", dQ, rQ), ("dK", dK, rK), ("dV", dV, rV)):
        e = rel_err(to_np(t), r)
        say(f"  {name} rel err {e:.3e}")
        assert e < bar, name


@pytest.mark.parametrize("prec", ["fp32", "bf16"])
def test_stage2_without_dQ(prec):
    """Stage II (Alg. 1): the call without dQ returns the same loss, dK and dV
    bit for bit, and iterating it with a gradient step lowers the loss."""
    from paper_2602_12314_amd import ops
    n, d, M, D = 6 * 700, 16, 256, 512   # six small views stacked
    say(f"[stage2] {prec} n={n}")
    Q, K, V, T, K0 = _inputs(5, n, d, M, D)
    dec = _decoder(prec, n, d, M, D)
    q, k, v, t, k0 = _cuda(Q, K, V, T, K0)
    l1, dQ1, dK1, dV1 = dec.loss_and_grads(q, k, v, t, k0, 0.1)
    l0, dQ0, dK0, dV0 = dec.loss_and_grads(q, k, v, t, k0, 0.1, want_dQ=False)
    assert dQ0 is None
    for a, b in ((l0, l1), (dK0, dK1), (dV0, dV1)):
        assert torch.equal(a, b)
    kk, vv = k.clone(), v.clone()

    def sgd(dK, dV, lr=1.0):  # stable: the trust-region curvature is 2 lambda = 0.2
        kk.sub_(lr * dK)
        vv.sub_(lr * dV)

    losses = to_np(ops.stage2(dec, q, kk, vv, t, k0, 0.1, iters=5, step=sgd))
    say(f"  losses {losses}")
    assert losses.shape == (5,) and losses[-1] < losses[0]
    ref = DO.loss_and_grads(Q, K, V, T, K0, 0.1)
    assert abs(float(losses[0]) - ref["loss"]) / ref["loss"] < BARS[prec]["grad"]


def test_one_hot_row_returns_value_row():
    rng = np.random.default_rng(5)
    d, M, D = 16, 64, 128
    basis, _ = np.linalg.qr(rng.standard_normal((d, d)))
    K = np.zeros((M, d), np.float32)
    K[:d] = 3.0 * basis
    K[d:] = -3.0 * basis[0]
    V = rng.standard_normal((M, D)).astype(np.float32)
    js = np.arange(d)
    Q = (40.0 * K[js]).astype(np.float32)  # logit gap 40*9/4 = 90: exp(-90) is below float32 resolution
    say("[decode one-hot] fp32")
    F = to_np(_decoder("fp32", d, d, M, D).forward(*_cuda(Q, K, V)))
    np.testing.assert_allclose(F, V[js], rtol=0, atol=1e-6 * np.abs(V).max())


def test_empty_pixels_gives_trust_region_only():
    d, M, D = 16, 64, 128
    _, K, V, _, K0 = _inputs(6, 1, d, M, D)
    say("[decode n=0]")
    dec = _decoder("bf16", 0, d, M, D)
    Q = torch.zeros((0, d), device="cuda")
    T = torch.zeros((0, D), device="cuda")
    loss, dQ, dK, dV = dec.loss_and_grads(Q, *_cuda(K, V), T, *_cuda(K0), 0.1)
    np.testing.assert_allclose(float(loss), 0.1 * ((K.astype(np.float64) - K0) ** 2).sum(), rtol=1e-5)
    np.testing.assert_allclose(to_np(dK), 0.2 * (K - K0), rtol=1e-5, atol=1e-7)
    assert np.all(to_np(dV) == 0)


@pytest.mark.parametrize("prec", ["fp32", "bf16"])
def test_full_640x480_workload(prec):
    # The 640x480 workload's decode sizes (n=307200, d=16, M=256, D=512), with a
    # Voronoi target; the oracle runs at full size.
    from paper_2602_12314_amd import scenes
    sp = scenes.spec(1)
    s = scenes.make_scene(sp, seed=11)
    rng = np.random.default_rng(12)
    Q = rng.standard_normal((sp.n_pixels, sp.d)).astype(np.float32)
    say(f"[decode full 640x480] {prec}")
    dec = _decoder(prec, sp.n_pixels, sp.d, sp.M, sp.D)
    loss, dQ, dK, dV = dec.loss_and_grads(*_cuda(Q, s.K, s.V, s.target, s.K0), sp.lambda_tr)
    ref = DO.loss_and_grads(Q, s.K, s.V, s.target, s.K0, sp.lambda_tr)
    bar = BARS[prec]["grad"]
    assert abs(float(loss) - ref["loss"]) / ref["loss"] < bar
    for name, t in (("dQ", dQ), ("dK", dK), ("dV", dV)):
        e = rel_err(to_np(t), ref[name])
        say(f"  {name} rel err {e:.3e}")
        assert e < bar, name
    F = to_np(dec.forward(*_cuda(Q, s.K, s.V)))
    if prec == "fp32":
        assert rel_err(F, ref["F"]) < 1e-4
    else:
        c = _min_cos(F, ref["F"])
        say(f"  min cos {c:.6f}")
        assert c >= 0.999


@pytest.mark.parametrize("prec", ["fp32", "bf16"])
def test_overlap_on_a_second_stream_is_bit_identical(prec):
    """lam_decode_loss_overlap: the dictionary gradients on a second stream
    (beside work queued after the call) equal lam_decode_loss bit for bit."""
    n, d, M, D = 5000, 16, 256, 512
    say(f"[overlap] {prec} n={n}")
    Q, K, V, T, K0 = _inputs(8, n, d, M, D)
    dec = _decoder(prec, n, d, M, D)
    q, k, v, t, k0 = _cuda(Q, K, V, T, K0)
    ref = dec.loss_and_grads(q, k, v, t, k0, 0.1)
    torch.cuda.synchronize()
    side = torch.cuda.Stream()
    for _ in range(3):
        out = dec.loss_and_grads(q, k, v, t, k0, 0.1, dict_stream=side)
        busy = torch.randn((2048, 2048), device="cuda") @ torch.randn((2048, 2048), device="cuda")  # work after
        torch.cuda.current_stream().wait_stream(side)
        for a, b in zip(out, ref):
            assert torch.equal(a, b)
        del busy
    # no pixels: only the trust-region term reaches dK, and the loss
    dec0 = _decoder(prec, 0, d, M, D)
    q0, t0 = torch.zeros((0, d), device="cuda"), torch.zeros((0, D), device="cuda")
    l0, _, dK0, dV0 = dec0.loss_and_grads(q0, k, v, t0, k0, 0.1, dict_stream=side)
    torch.cuda.current_stream().wait_stream(side)
    r0 = dec0.loss_and_grads(q0, k, v, t0, k0, 0.1)
    assert torch.equal(l0, r0[0]) and torch.equal(dK0, r0[2]) and torch.equal(dV0, r0[3])
    assert float(dV0.abs().max()) == 0.0


@pytest.mark.parametrize("prec", ["bf16", "fp8"])
def test_paper_dictionary_size_2000(prec):
    """The paper's dictionary size K = 2000 (Sec. IV) with its query width
    d_s = 32 and D = 768: 2000 atoms pad to 2048 (the last 48 masked out of
    the softmax), the largest atom count the library takes; 3000 pixels end
    in a ragged block."""
    n, d, M, D = 3000, 32, 2000, 768
    say(f"[decode K=2000] {prec} n={n} d={d} M={M} D={D}")
    Q, K, V, T, K0 = _inputs(21, n, d, M, D)
    dec = _decoder(prec, n, d, M, D)
    q, k, v, t, k0 = _cuda(Q, K, V, T, K0)
    F = to_np(dec.forward(q, k, v))
    loss, dQ, dK, dV = dec.loss_and_grads(q, k, v, t, k0, 0.1)
    ref = DO.loss_and_grads(Q, K, V, T, K0, 0.1)
    c = _cos(F, ref["F"])
    say(f"  F cos min {c.min():.6f} mean {c.mean():.6f}")
    assert c.min() >= 0.999
    assert abs(float(loss) - ref["loss"]) / abs(ref["loss"]) < 1e-2
    for name, t_ in (("dQ", dQ), ("dK", dK), ("dV", dV)):
        e = rel_err(to_np(t_), ref[name])
        say(f"  {name} rel err {e:.3e}")
        assert e < (2.5e-2 if prec == "fp8" and name == "dQ" else 1e-2), name


@pytest.mark.parametrize("prec", ["bf16", "fp8"])
@pytest.mark.parametrize("n", [256 * 64 - 1, 256 * 64, 256 * 64 + 33])
@pytest.mark.parametrize("M,D", [(100, 512), (70, 768), (2048, 1024), (130, 1024)])
def test_inference_block_choice(prec, n, M, D):
    """Around the pixel count from which inference takes the 64-pixel block by
    itself, on whole and ragged blocks: the rows agree with those of a call too
    small for it.  Both sum the same BF16 products in float32; only the softmax
    normaliser is added up over another number of waves, so the rows differ by
    a few float32 roundings (bound: 16 of 2^-24 relative to the row)."""
    from paper_2602_12314_amd import ops
    g = torch.Generator(device="cuda").manual_seed(n + M)
    Q = torch.randn((n, 32), device="cuda", generator=g)
    K = torch.randn((M, 32), device="cuda", generator=g)
    V = torch.randn((M, D), device="cuda", generator=g)
    F = ops.Decoder(prec, n, 32, M, D).forward(Q, K, V)
    rows = torch.cat([torch.arange(64, device="cuda"), torch.arange(n - 97, n, device="cuda")])
    small = ops.Decoder(prec, rows.numel(), 32, M, D).forward(Q[rows], K, V)
    err = (F[rows] - small).norm(dim=1) / small.norm(dim=1)
    assert float(err.max()) <= 16 * 2.0 ** -24, float(err.max())


@pytest.mark.parametrize("shape", ["px32", "px64"])
@pytest.mark.parametrize("prec,M,D", [("bf16", 100, 512), ("bf16", 500, 768), ("fp8", 130, 1024)])
def test_inference_keeps_to_an_explicit_block_shape(prec, M, D, shape):
    """With the block shape asked for, a row's F is the same bits in a call of
    so many rows that the library's own choice is the 64-pixel block as in a
    call of few; and the two shapes, and that choice, differ by rounding only."""
    from paper_2602_12314_amd import _lib, ops
    n = 256 * 64 + 33
    g = torch.Generator(device="cuda").manual_seed(M)
    Q = torch.randn((n, 32), device="cuda", generator=g)
    K = torch.randn((M, 32), device="cuda", generator=g)
    V = torch.randn((M, D), device="cuda", generator=g)
    rows = torch.cat([torch.arange(64, device="cuda"), torch.arange(n - 97, n, device="cuda")])

    def fwd(opt, q):
        ctx = _lib.Context(options={"decode_shape": opt})
        F = ops.Decoder(prec, q.shape[0], 32, M, D, ctx=ctx).forward(q, K, V)
        torch.cuda.synchronize()
        ctx.close()
        return F

    F = fwd(shape, Q)
    assert torch.equal(F[rows], fwd(shape, Q[rows]))
    assert torch.equal(fwd("auto", Q), fwd("px64", Q)) and _lib.Context().get("decode_shape") == 2
    other = fwd("px64" if shape == "px32" else "px32", Q)
    err = (F - other).norm(dim=1) / other.norm(dim=1)
    assert float(err.max()) <= 16 * 2.0 ** -24
    if M > 128:  # up to 128 atoms no wave of either shape has two tiles to add up: the same bits
        assert float(err.max()) > 0.0
