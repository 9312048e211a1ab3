"""GPU parity of the tensor-level operations (tile grids, both executor
granularities, ragged tilings, structural-zero tiles) against the fp64 oracle."""
import ctypes as C
import math

import numpy as np
import pytest

from gpu_util import TOL, check, quant, relerr
from oracle import definition as D

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def mods():
    from paper_2504_13236_amd import capi, tiled
    return capi, tiled


def rng(seed):
    return np.random.default_rng(seed)


GRANS = [0, 1]     # NNT_GRAN_OP, NNT_GRAN_TILE


def T(tiled, ctx, a, base, dtype, absent=None):
    return tiled.TiledTensor.from_numpy(ctx, np.asarray(a, np.float32), base, dtype, absent)


# ------------------------------------------------------------------ products
@pytest.mark.parametrize("gran", GRANS)
@pytest.mark.parametrize("dtype", ["f32", "bf16"])
def test_gemm_linear_layer_forms(mods, gran, dtype):
    """Y = W X +. b, dX = W^T dY, dW = sum_{s,b} dY X^T on ragged tilings."""
    capi, tiled = mods
    r = rng(1)
    N_d, N_e, N_s, N_b = 200, 136, 72, 3
    W = quant(r.standard_normal((N_d, N_e)) * 0.1, dtype)
    X = quant(r.standard_normal((N_e, N_s, N_b)), dtype)
    b = r.standard_normal(N_d).astype(np.float32)
    dY = quant(r.standard_normal((N_d, N_s, N_b)), dtype)
    with tiled.Context(n_streams=4, granularity=gran) as ctx:
        tW, tX = T(tiled, ctx, W, (64, 48), dtype), T(tiled, ctx, X, (48, 32, 2), dtype)
        tb = T(tiled, ctx, b, (64,), "f32")
        tY = tiled.TiledTensor(ctx, dtype, (N_d, N_s, N_b), (64, 32, 2))
        capi.nnt_gemm(ctx.h, 1.0, 0, tW.h, 0, tX.h, 0.0, tY.h, 1, 0, tb.h)
        check(tY.download(), D.linear_fwd(W, X, b), dtype, "linear fwd")
        tdY = T(tiled, ctx, dY, (64, 32, 2), dtype)
        tdX = tiled.TiledTensor(ctx, dtype, X.shape, (48, 32, 2))
        capi.nnt_gemm(ctx.h, 1.0, 1, tW.h, 0, tdY.h, 0.0, tdX.h, 1, 0, None)
        tdW = tiled.TiledTensor(ctx, "f32", W.shape, (64, 48))
        capi.nnt_gemm(ctx.h, 1.0, 0, tdY.h, 1, tX.h, 0.0, tdW.h, 2, 0, None)
        dXr, dWr, dbr = D.linear_bwd(W, X, dY)
        check(tdX.download(), dXr, dtype, "linear dX")
        check(tdW.download(), dWr, "f32", "linear dW")
        # beta = 1 accumulates on top of the previous result
        capi.nnt_gemm(ctx.h, 0.5, 0, tdY.h, 1, tX.h, 1.0, tdW.h, 2, 0, None)
        check(tdW.download(), 1.5 * dWr, "f32", "linear dW accumulate")
        tdb = tiled.TiledTensor(ctx, "f32", (N_d,), (64,))
        capi.nnt_bias_grad(ctx.h, tdY.h, tdb.h)
        check(tdb.download(), dbr, "f32", "bias grad")
        capi.nnt_bias_add(ctx.h, tb.h, tdY.h)
        check(tdY.download(), D.bias_add(dY, b), dtype, "bias add")
        st = ctx.stats()
        assert st["tasks"] > 0 and (st["tasks"] > 8 if gran else st["tasks"] <= 8)


@pytest.mark.parametrize("gran", GRANS)
@pytest.mark.parametrize("dtype", ["f32", "bf16"])
@pytest.mark.parametrize("tiles", [(64, 40, 2, 3), (32, 24, 1, 1)])
def test_attention_products_with_causal_structure(mods, gran, dtype, tiles):
    """scores, softmax, P V and the four backward products; tiles above the
    diagonal are structural zeros."""
    capi, tiled = mods
    ti, ts, tb, tj = tiles
    r = rng(2)
    h, N_s, N_b, N_h = 64, 100, 2, 3
    Q, K, V, dB = [quant(r.standard_normal((h, N_s, N_b, N_h)), dtype) for _ in range(4)]
    sc = 1.0 / math.sqrt(h)
    with tiled.Context(n_streams=4, granularity=gran) as ctx:
        hb, sb = (ti, ts, tb, tj), (ts, ts, tb, tj)
        absent = tiled.causal_absent(ts, ts, N_s)
        tQ, tK, tV, tdB = [T(tiled, ctx, a, hb, dtype) for a in (Q, K, V, dB)]
        tP = tiled.TiledTensor(ctx, dtype, (N_s, N_s, N_b, N_h), sb, absent)
        tS = tiled.TiledTensor(ctx, "f32", (2, N_s, N_b, N_h), (2, ts, tb, tj))
        capi.nnt_gemm(ctx.h, sc, 1, tK.h, 0, tQ.h, 0.0, tP.h, 1, 2, None)
        capi.nnt_softmax_fwd(ctx.h, tP.h, tS.h, 1.0, 1)
        A = D.attention_scores(K, Q)
        if dtype == "bf16":
            A = quant(A, dtype)           # the device stores the scores in bf16 before the softmax
        Pref, tmax, den = D.softmax_fwd(A, causal=True)
        P = tP.download().astype(np.float64)
        check(P, Pref, dtype, "softmax(K^T Q)")
        np.testing.assert_allclose(P.sum(axis=0), 1.0, atol=2e-2 if dtype == "bf16" else 1e-5)
        stats = tS.download()
        check(stats[0], tmax, dtype, "softmax max")
        tB = tiled.TiledTensor(ctx, dtype, Q.shape, hb)
        capi.nnt_gemm(ctx.h, 1.0, 0, tV.h, 0, tP.h, 0.0, tB.h, 1, 2, None)
        check(tB.download(), D.attention_values(V, P), dtype, "V P")
        # backward from the probabilities the device holds
        tdV = tiled.TiledTensor(ctx, dtype, Q.shape, hb)
        tdP = tiled.TiledTensor(ctx, dtype, (N_s, N_s, N_b, N_h), sb, absent)
        capi.nnt_gemm(ctx.h, 1.0, 0, tdB.h, 1, tP.h, 0.0, tdV.h, 1, 2, None)
        capi.nnt_gemm(ctx.h, 1.0, 1, tV.h, 0, tdB.h, 0.0, tdP.h, 1, 2, None)
        dPdev = tdP.download().astype(np.float64)
        capi.nnt_softmax_bwd(ctx.h, tP.h, tdP.h)
        dA = tdP.download().astype(np.float64)
        check(dA, D.softmax_bwd(P, dPdev), dtype, "softmax bwd")
        tdQ, tdK = tiled.TiledTensor(ctx, dtype, Q.shape, hb), tiled.TiledTensor(ctx, dtype, Q.shape, hb)
        capi.nnt_gemm(ctx.h, sc, 0, tK.h, 0, tdP.h, 0.0, tdQ.h, 1, 2, None)
        capi.nnt_gemm(ctx.h, sc, 0, tQ.h, 1, tdP.h, 0.0, tdK.h, 1, 2, None)
        # the oracle's batched contraction over the last two axes (batch, head), from what the device holds
        check(tdV.download(), D.contract(1.0, "N", dB, "T", P, 0.0, None, 1, 2), dtype, "dV = dB P^T")
        check(tdQ.download(), D.contract(sc, "N", K, "N", dA, 0.0, None, 1, 2), dtype, "dQ = K dA / sqrt(h)")
        check(tdK.download(), D.contract(sc, "N", Q, "T", dA, 0.0, None, 1, 2), dtype, "dK = Q dA^T / sqrt(h)")


@pytest.mark.parametrize("gran", GRANS)
def test_gemm_bf16_tiles_of_400_run_on_the_direct_load_kernel(mods, gran):
    """Linear-layer products on tiles of 400 (GPT-2-XL's tiling: 400 = 256 + 144 rows per macro-tile column,
    12 k-steps of 32 and a short one of 16, sequence tiles 400 + 224): forward with bias, input gradient,
    weight gradient over two contracted axes, against the oracle; in whole-operation launches the profile
    must name the direct-load kernel's ragged variant."""
    capi, tiled = mods
    r = rng(40)
    N_d, N_e, N_s, N_b = 1200, 800, 624, 4
    W = quant(r.standard_normal((N_d, N_e)) * 0.05, "bf16")
    X = quant(r.standard_normal((N_e, N_s, N_b)), "bf16")
    b = r.standard_normal(N_d).astype(np.float32)
    dY = quant(r.standard_normal((N_d, N_s, N_b)), "bf16")
    with tiled.Context(n_streams=2, granularity=gran) as ctx:
        tW, tX = T(tiled, ctx, W, (400, 400), "bf16"), T(tiled, ctx, X, (400, 400, N_b), "bf16")
        tb = T(tiled, ctx, b, (400,), "f32")
        tY = tiled.TiledTensor(ctx, "bf16", (N_d, N_s, N_b), (400, 400, N_b))
        tdY = T(tiled, ctx, dY, (400, 400, N_b), "bf16")
        tdX = tiled.TiledTensor(ctx, "bf16", X.shape, (400, 400, N_b))
        tdW = tiled.TiledTensor(ctx, "f32", W.shape, (400, 400))
        ctx.profile(True)
        capi.nnt_gemm(ctx.h, 1.0, 0, tW.h, 0, tX.h, 0.0, tY.h, 1, 0, tb.h)
        capi.nnt_gemm(ctx.h, 1.0, 1, tW.h, 0, tdY.h, 0.0, tdX.h, 1, 0, None)
        capi.nnt_gemm(ctx.h, 1.0, 0, tdY.h, 1, tX.h, 0.0, tdW.h, 2, 0, None)
        ctx.wait()
        labels = sorted(ctx.profile_read())
        ctx.profile(False)
        check(tY.download(), D.linear_fwd(W, X, b), "bf16", "linear fwd")
        dXr, dWr, _ = D.linear_bwd(W, X, dY)
        check(tdX.download(), dXr, "bf16", "linear dX")
        check(tdW.download(), dWr, "f32", "linear dW")
        if gran == 0:
            products = [l for l in labels if l.startswith("gemm_")]
            assert products and all(l.startswith("gemm_bf16_dl_tall_kernel<") and l.split(">")[0].endswith("true") for l in products), labels


def test_gemm_direct_load_randomized_sweep_over_tile_tables(mods):
    """Seeded random draws of tensor-level products whose tiles are whole macro-tiles and whose contracted
    tiles are multiples of 32 long (several chunks per C tile, including chunks of 32 and 64): the
    table-driven launches of the kernels that load straight into LDS, in every operand orientation and
    both granularities, against the oracle's contraction.  Stops at the first failure."""
    capi, tiled = mods
    r = np.random.default_rng(413236)
    for draw in range(48):
        dtype = ("f32", "bf16")[draw % 2]
        dout = "f32" if dtype == "f32" else ("bf16", "f32")[(draw // 2) % 2]
        unit = 128 if dtype == "f32" else 256
        tm, tn = unit * int(r.integers(1, 3)), unit * int(r.integers(1, 3))
        m, n = tm * int(r.integers(1, 3)), tn * int(r.integers(1, 3))
        tk = 32 * int(r.choice([1, 2, 3, 5, 8]))
        k = tk * int(r.integers(1, 5))
        opA, opB = int(r.integers(2)), int(r.integers(2))
        alpha, beta = ((1.0, 0.0), (0.6, -1.5))[int(r.integers(2))]
        gran = int(r.integers(2))
        A = quant(r.standard_normal((m, k) if opA == 0 else (k, m)), dtype)
        B = quant(r.standard_normal((k, n) if opB == 0 else (n, k)), dtype)
        C0 = quant(r.standard_normal((m, n)), dout)
        ref = D.contract(alpha, "NT"[opA], A, "NT"[opB], B, beta, C0, 1, 0)
        with tiled.Context(n_streams=2, granularity=gran) as ctx:
            tA = T(tiled, ctx, A, (tm, tk) if opA == 0 else (tk, tm), dtype)
            tB = T(tiled, ctx, B, (tk, tn) if opB == 0 else (tn, tk), dtype)
            tC = T(tiled, ctx, C0, (tm, tn), dout)
            capi.nnt_gemm(ctx.h, alpha, opA, tA.h, opB, tB.h, beta, tC.h, 1, 0, None)
            e = relerr(tC.download(), ref)
        assert e <= TOL[dout], ("draw %d: %s->%s op %d%d %dx%dx%d tiles %dx%dx%d alpha %g beta %g gran %d" %
                                (draw, dtype, dout, opA, opB, m, n, k, tm, tn, tk, alpha, beta, gran), e)


def test_gemm_bf16_short_contracted_tiles_randomized_sweep(mods):
    """bf16 tensor-level products whose contracted tiles are multiples of 8 but not of 32 long and often shorter
    than the k-steps a workgroup starts before its loop (8 .. 72, several per C tile, a shorter last one), with
    C tiles that are and are not whole macro-tiles: the table-driven launches of the direct-load kernel's
    ragged variant, whose loading side runs ahead of the multiplying side by whole chunks here.  Every operand
    orientation, both granularities, against the oracle's contraction; stops at the first failure."""
    capi, tiled = mods
    r = np.random.default_rng(250413)
    for draw in range(40):
        dout = ("bf16", "f32")[draw % 2]
        tm, tn = (256, 512, 400, 328)[int(r.integers(4))], (256, 128, 400, 136)[int(r.integers(4))]
        m, n = tm * int(r.integers(1, 3)) + 8 * int(r.integers(0, 20)), tn * int(r.integers(1, 4)) + 8 * int(r.integers(0, 12))
        tk = 8 * int(r.choice([1, 2, 3, 5, 7, 9]))
        k = tk * int(r.integers(2, 6)) + 8 * int(r.integers(0, tk // 8))
        opA, opB = int(r.integers(2)), int(r.integers(2))
        alpha, beta = ((1.0, 0.0), (0.6, -1.5))[int(r.integers(2))]
        gran = int(r.integers(2))
        A = quant(r.standard_normal((m, k) if opA == 0 else (k, m)), "bf16")
        B = quant(r.standard_normal((k, n) if opB == 0 else (n, k)), "bf16")
        C0 = quant(r.standard_normal((m, n)), dout)
        ref = D.contract(alpha, "NT"[opA], A, "NT"[opB], B, beta, C0, 1, 0)
        with tiled.Context(n_streams=2, granularity=gran) as ctx:
            tA = T(tiled, ctx, A, (tm, tk) if opA == 0 else (tk, tm), "bf16")
            tB = T(tiled, ctx, B, (tk, tn) if opB == 0 else (tn, tk), "bf16")
            tC = T(tiled, ctx, C0, (tm, tn), dout)
            capi.nnt_gemm(ctx.h, alpha, opA, tA.h, opB, tB.h, beta, tC.h, 1, 0, None)
            e = relerr(tC.download(), ref)
        assert e <= TOL[dout], ("draw %d: bf16->%s op %d%d %dx%dx%d tiles %dx%dx%d alpha %g beta %g gran %d" %
                                (draw, dout, opA, opB, m, n, k, tm, tn, tk, alpha, beta, gran), e)


def test_gemm_bf16_batched_products_with_ragged_sequence_tiles(mods):
    """Score-shaped and head-row products of an attention layer whose sequence length is not a multiple of its
    tile (1000 = 3 x 256 + 232) and whose head size is not a multiple of a k-step (72): batched launches in which
    macro-tiles end inside their tiles and every chunk ends in a short k-step."""
    capi, tiled = mods
    r = rng(77)
    h, N_s, N_b, N_h, ts = 72, 1000, 2, 8, 256        # 16 x 16 blocks of 256 x 256: enough for the 256 x 128 direct-load shape
    Q, K, V = [quant(r.standard_normal((h, N_s, N_b, N_h)), "bf16") for _ in range(3)]
    with tiled.Context(n_streams=2) as ctx:
        hb, sb = (h, ts, N_b, N_h), (ts, ts, N_b, N_h)
        tQ, tK, tV = [T(tiled, ctx, a, hb, "bf16") for a in (Q, K, V)]
        tA = tiled.TiledTensor(ctx, "bf16", (N_s, N_s, N_b, N_h), sb)
        capi.nnt_gemm(ctx.h, 0.25, 1, tK.h, 0, tQ.h, 0.0, tA.h, 1, 2, None)
        Adev = tA.download().astype(np.float64)
        check(Adev, D.contract(0.25, "T", K, "N", Q, 0.0, None, 1, 2), "bf16", "K^T Q")
        tB = tiled.TiledTensor(ctx, "bf16", Q.shape, hb)
        capi.nnt_gemm(ctx.h, 1.0, 0, tV.h, 0, tA.h, 0.0, tB.h, 1, 2, None)
        check(tB.download(), D.contract(1.0, "N", V, "N", Adev, 0.0, None, 1, 2), "bf16", "V A")
        tD = tiled.TiledTensor(ctx, "bf16", Q.shape, hb)
        capi.nnt_gemm(ctx.h, 1.0, 0, tV.h, 1, tA.h, 0.0, tD.h, 1, 2, None)
        check(tD.download(), D.contract(1.0, "N", V, "T", Adev, 0.0, None, 1, 2), "bf16", "V A^T")


@pytest.mark.parametrize("causal", [1, 0])
@pytest.mark.parametrize("dtype", ["f32", "bf16"])
@pytest.mark.parametrize("shape,base", [((1024, 64, 2, 2), (512, 32, 2, 1)),      # two key tiles: four bf16 columns per wavefront
                                        ((1000, 48, 1, 2), (400, 24, 1, 2)),      # tiles of 400 + 400 + 200: two columns per wavefront
                                        ((256, 40, 3, 1), (256, 20, 2, 1)),       # one key tile
                                        ((200, 30, 2, 1), (64, 15, 1, 1)),        # odd query tiles: one column per wavefront
                                        ((96, 7, 1, 1), (40, 7, 1, 1))])
def test_softmax_tensor_forward_backward(mods, shape, base, dtype, causal):
    """SoftMax over the key axis of a tiled score tensor, in place, and its adjoint: probabilities, the
    fp32 column statistics (maximum, sum of shifted exponentials) and dA against the oracle, for tilings
    that take one, two and four columns per wavefront."""
    capi, tiled = mods
    r = rng(sum(shape) + causal)
    A = quant(3.0 * r.standard_normal(shape), dtype)
    dPn = quant(r.standard_normal(shape), dtype)
    scale = 0.37
    Pref, tmax, den = D.softmax_fwd(scale * A, causal=bool(causal))
    with tiled.Context(n_streams=2) as ctx:
        tA = T(tiled, ctx, A, base, dtype)
        tS = tiled.TiledTensor(ctx, "f32", (2,) + shape[1:], (2,) + base[1:])
        capi.nnt_softmax_fwd(ctx.h, tA.h, tS.h, scale, causal)
        P = tA.download().astype(np.float64)
        check(P, Pref, dtype, "probabilities")
        if causal:
            k = np.arange(shape[0])[:, None]
            q = np.arange(shape[1])[None, :]
            assert np.all(P[(k > q)] == 0.0), "masked probabilities must be exactly 0"
        stats = tS.download()
        check(stats[0], tmax, "f32", "column maximum")
        check(stats[1], den, "f32", "sum of shifted exponentials")
        tdP = T(tiled, ctx, dPn, base, dtype)
        capi.nnt_softmax_bwd(ctx.h, tA.h, tdP.h)
        check(tdP.download(), D.softmax_bwd(P, dPn), dtype, "softmax adjoint")


@pytest.mark.parametrize("dtype,dout", [("f32", "f32"), ("bf16", "f32"), ("bf16", "bf16")])
@pytest.mark.parametrize("form", ["dW", "dX", "fwd"])
def test_gemm_long_contraction_few_tiles(mods, dtype, dout, form):
    """Few output tiles and a long contraction: the product is cut into k-slices
    that are summed in a second kernel (with alpha, beta and the bias)."""
    capi, tiled = mods
    r = rng(11)
    if form == "dW":       # C[d, e] = sum_{s, b} dY[d, s, b] X[e, s, b]; contraction 4 x 96 x 3 in ragged chunks
        A = quant(r.standard_normal((200, 4 * 96, 3)), dtype)
        B = quant(r.standard_normal((136, 4 * 96, 3)), dtype)
        ta, tb, tc = (64, 100, 2), (48, 100, 2), (64, 48)
        ops, ncon, cshape = (0, 1), 2, (200, 136)
        ref = D.contract(1.0, "N", A, "T", B, 0.0, None, 2, 0)
    elif form == "dX":     # C[e, t] = sum_d W[d, e] dY[d, t]
        A = quant(r.standard_normal((1500, 136)) * 0.1, dtype)
        B = quant(r.standard_normal((1500, 300)), dtype)
        ta, tb, tc = (400, 48), (400, 128), (48, 128)
        ops, ncon, cshape = (1, 0), 1, (136, 300)
        ref = D.contract(1.0, "T", A, "N", B, 0.0, None, 1, 0)
    else:                  # C[d, t] = sum_e W[d, e] X[e, t] + b[d]
        A = quant(r.standard_normal((136, 1500)) * 0.1, dtype)
        B = quant(r.standard_normal((1500, 300)), dtype)
        ta, tb, tc = (48, 400), (400, 128), (48, 128)
        ops, ncon, cshape = (0, 0), 1, (136, 300)
        ref = D.contract(1.0, "N", A, "N", B, 0.0, None, 1, 0)
    bias = r.standard_normal(cshape[0]).astype(np.float32)
    C0 = quant(r.standard_normal(cshape), dout)
    with tiled.Context(n_streams=2) as ctx:
        tA, tB = T(tiled, ctx, A, ta, dtype), T(tiled, ctx, B, tb, dtype)
        tC = T(tiled, ctx, C0, tc, dout)
        tbias = T(tiled, ctx, bias, tc[:1], "f32")
        capi.nnt_gemm(ctx.h, 0.5, ops[0], tA.h, ops[1], tB.h, -2.0, tC.h, ncon, 0, tbias.h)
        want = 0.5 * ref - 2.0 * C0 + bias.reshape(-1, 1)
        e = relerr(tC.download(), want)
        assert e <= (2e-2 if dout == "bf16" else 1e-5), (form, e)
        # same call again: the scratch tiles are reused, the result accumulates through beta
        capi.nnt_gemm(ctx.h, 0.5, ops[0], tA.h, ops[1], tB.h, 1.0, tC.h, ncon, 0, None)
        e = relerr(tC.download(), want + 0.5 * ref)
        assert e <= TOL[dout], (form, e)


@pytest.mark.parametrize("gran", GRANS)
@pytest.mark.parametrize("dtype", ["f32", "bf16"])
@pytest.mark.parametrize("shape", ["ragged", "direct-load", "k-slices"])
def test_gemm_with_a_residual_input(mods, gran, dtype, shape):
    """Y = alpha W X +. b + beta R with R a second tensor of Y's geometry (the residual connection of a
    block folded into the product): general kernels on ragged tiles, the direct-load kernels on whole
    macro-tiles, and a product whose contraction is cut into k-slices (the sum kernel adds R)."""
    capi, tiled = mods
    r = rng(77)
    if shape == "ragged":
        m, n, k, tw, tx, ty = 200, 150, 136, (64, 48), (48, 40), (64, 40)
    elif shape == "direct-load":
        m, n, k, tw, tx, ty = 512, 512, 192, (256, 64), (64, 256), (256, 256)
    else:
        m, n, k, tw, tx, ty = 256, 256, 4096, (256, 1024), (1024, 256), (256, 256)
    W = quant(r.standard_normal((m, k)) * 0.1, dtype)
    X = quant(r.standard_normal((k, n)), dtype)
    b = r.standard_normal(m).astype(np.float32)
    R = quant(r.standard_normal((m, n)), dtype)
    Y0 = quant(r.standard_normal((m, n)), dtype)                      # must not enter the result
    want = D.contract(0.5, "N", W, "N", X, -1.5, R, 1, 0) + b.reshape(-1, 1)
    with tiled.Context(n_streams=2, granularity=gran) as ctx:
        tW, tX, tR, tY = T(tiled, ctx, W, tw, dtype), T(tiled, ctx, X, tx, dtype), T(tiled, ctx, R, ty, dtype), T(tiled, ctx, Y0, ty, dtype)
        tb = T(tiled, ctx, b, ty[:1], "f32")
        capi.nnt_gemm_res(ctx.h, 0.5, 0, tW.h, 0, tX.h, -1.5, tY.h, 1, 0, tb.h, tR.h)
        check(tY.download(), want, dtype, "W X + b + beta R")
        np.testing.assert_array_equal(tR.download(), np.asarray(R, np.float32))     # the residual input is only read
        # R = NULL and R = C are the plain product with beta on C
        capi.nnt_gemm_res(ctx.h, 0.5, 0, tW.h, 0, tX.h, 1.0, tR.h, 1, 0, None, tR.h)
        check(tR.download(), D.contract(0.5, "N", W, "N", X, 1.0, R, 1, 0), dtype, "R = C")
        other = tiled.TiledTensor(ctx, dtype, (m, n), (ty[0] // 2, ty[1]))
        with pytest.raises(capi.NntError):
            capi.nnt_gemm_res(ctx.h, 1.0, 0, tW.h, 0, tX.h, 1.0, tY.h, 1, 0, None, other.h)   # tiled differently


@pytest.mark.parametrize("gran", GRANS)
@pytest.mark.parametrize("dtype", ["f32", "bf16"])
@pytest.mark.parametrize("variant", [0, 1])
@pytest.mark.parametrize("shape", ["ragged", "direct-load", "long-k"])
def test_gemm_with_the_activation_on_its_way_out(mods, gran, dtype, variant, shape):
    """H = W X +. b and G = gelu(H) from one launch, and dH = (W^T dY) * gelu'(H) from one launch (the MLP of
    section 3 without activation passes of their own): general kernels on ragged tiles, the direct-load
    kernels on whole macro-tiles, and a long contraction that a plain product would cut into k-slices."""
    capi, tiled = mods
    r = rng(91 + variant)
    if shape == "ragged":
        m, n, k, tw, tx, ty = 200, 150, 136, (64, 48), (48, 40), (64, 40)
    elif shape == "direct-load":
        m, n, k, tw, tx, ty = 512, 768, 192, (256, 64), (64, 256), (256, 256)
    else:
        m, n, k, tw, tx, ty = 256, 256, 4096, (256, 1024), (1024, 256), (256, 256)
    name = ("tanh", "erf")[variant]
    W = quant(r.standard_normal((m, k)) / np.sqrt(k), dtype)
    X = quant(r.standard_normal((k, n)) * 1.5, dtype)
    b = r.standard_normal(m).astype(np.float32) * 0.5
    H = D.contract(1.0, "N", W, "N", X, 0.0, None, 1, 0) + b.reshape(-1, 1)
    junk = quant(r.standard_normal((m, n)), dtype)
    with tiled.Context(n_streams=2, granularity=gran) as ctx:
        tW, tX = T(tiled, ctx, W, tw, dtype), T(tiled, ctx, X, tx, dtype)
        tH, tG = T(tiled, ctx, junk, ty, dtype), T(tiled, ctx, junk, ty, dtype)
        tb = T(tiled, ctx, b, ty[:1], "f32")
        capi.nnt_gemm_gelu(ctx.h, 1.0, 0, tW.h, 0, tX.h, tH.h, 1, tb.h, variant, tG.h)
        Hd = tH.download()
        check(Hd, H, dtype, "H = W X + b")
        check(tG.download(), D.gelu(H, name), dtype, "G = gelu(H)")
        # the same G as the activation pass over the stored H gives
        tG2 = T(tiled, ctx, junk, ty, dtype)
        capi.nnt_gelu(ctx.h, variant, tH.h, tG2.h)
        np.testing.assert_array_equal(tG.download(), tG2.download())
        # adjoint: dX3-shaped product W^T dY (k x n here: contraction over m) times gelu' of a tensor of its shape
        dY = quant(r.standard_normal((m, n)), dtype)
        Z = quant(r.standard_normal((k, n)) * 1.5, dtype)
        tk = (tw[1], tx[1])
        tdY, tZ, tdZ = T(tiled, ctx, dY, ty, dtype), T(tiled, ctx, Z, tk, dtype), T(tiled, ctx, quant(r.standard_normal((k, n)), dtype), tk, dtype)
        capi.nnt_gemm_gelu_bwd(ctx.h, 0.5, 1, tW.h, 0, tdY.h, tdZ.h, 1, variant, tZ.h)
        want = D.contract(0.5, "T", W, "N", dY, 0.0, None, 1, 0) * D.gelu_grad(np.asarray(Z, np.float64), name)
        check(tdZ.download(), want, dtype, "dZ = (W^T dY) gelu'(Z)")
        np.testing.assert_array_equal(tZ.download(), np.asarray(Z, np.float32))      # only read
        with pytest.raises(capi.NntError):
            capi.nnt_gemm_gelu(ctx.h, 1.0, 0, tW.h, 0, tX.h, tH.h, 1, tb.h, variant, tH.h)      # G must not be C
        with pytest.raises(capi.NntError):
            capi.nnt_gemm_gelu_bwd(ctx.h, 1.0, 1, tW.h, 0, tdY.h, tdZ.h, 1, 7, tZ.h)            # unknown variant


@pytest.mark.parametrize("gran", GRANS)
@pytest.mark.parametrize("n", [128, 256])
@pytest.mark.parametrize("tm", [64, 128, 192])
@pytest.mark.parametrize("k", [32, 64])
def test_activation_gradient_behind_a_short_contraction(mods, k, tm, n, gran):
    """dH = (W^T dY) * gelu'(H) where the contraction is a head size long (a narrow MLP): products for which the plain form takes
    the kernel that holds the whole contraction in LDS, whose macro-tiles of 64 rows the activation kernels do not all have.
    Every tile of the result, on tiles that are whole numbers of 64 rows but not of 128."""
    capi, tiled = mods
    r = rng(k + tm + n)
    m = 3 * tm
    W, dY = r.standard_normal((k, m)).astype(np.float32), r.standard_normal((k, 2 * n)).astype(np.float32)
    Z = (1.5 * r.standard_normal((m, 2 * n))).astype(np.float32)
    with tiled.Context(n_streams=2, granularity=gran) as ctx:
        tW, tdY, tZ = T(tiled, ctx, W, (k, tm), "f32"), T(tiled, ctx, dY, (k, n), "f32"), T(tiled, ctx, Z, (tm, n), "f32")
        tdZ = T(tiled, ctx, np.full((m, 2 * n), 7.0), (tm, n), "f32")
        capi.nnt_gemm_gelu_bwd(ctx.h, 1.0, 1, tW.h, 0, tdY.h, tdZ.h, 1, 0, tZ.h)
        check(tdZ.download(), D.contract(1.0, "T", W, "N", dY, 0.0, None, 1, 0) * D.gelu_grad(Z.astype(np.float64), "tanh"), "f32", "dZ")


@pytest.mark.parametrize("din", ["bf16", "f32"])
@pytest.mark.parametrize("form", ["NN", "TN", "NT", "TT"])
@pytest.mark.parametrize("m,n,k,tm,tn,tk", [
    (1333, 1027, 777, 500, 257, 300),       # every extent odd, tiles of C crossed along both axes
    (1281, 513, 1025, 1281, 513, 1025),     # one element beyond the macro-tiles and the k-steps, one tile
    (2051, 1030, 1999, 1024, 515, 1000),    # k-slices
    (300, 3100, 129, 100, 300, 50),         # tiles narrower than a macro-tile along m: operands read as they are
    (1537, 4611, 515, 300, 2305, 257),      # many macro-tiles
    (2816, 2560, 523, 300, 300, 300),       # whole macro-tiles, odd contraction
])
def test_products_of_odd_sizes(mods, m, n, k, tm, tn, tk, form, din):
    """Operands that are laid out afresh: fp32 and bf16 results, bias, beta and residual input, twice in a row with other values in
    the operands (what the first call laid out must not be seen again), and tile by tile as the comparison.  Operands hold
    small multiples of 1/16, so fp32 results are exact up to the sums' rounding."""
    capi, tiled = mods
    r = rng(m + n + k)
    opA, opB = ("NT".index(c) for c in form)
    with tiled.Context(n_streams=2) as ctx:
        ash, abase = ((m, k), (tm, tk)) if opA == 0 else ((k, m), (tk, tm))
        bsh, bbase = ((k, n), (tk, tn)) if opB == 0 else ((n, k), (tn, tk))
        draw = lambda shape: r.integers(-32, 33, shape).astype(np.float32) / 16
        A, B, bias = draw(ash), draw(bsh), draw((m,))
        tA, tB, tbias = T(tiled, ctx, A, abase, din), T(tiled, ctx, B, bbase, din), T(tiled, ctx, bias, (tm,), "f32")
        for dt in ("f32", "bf16") if din == "bf16" else ("f32",):
            C0, R = draw((m, n)), draw((m, n))
            tC, tR, tD = (T(tiled, ctx, x, (tm, tn), dt) for x in (C0, R, C0))
            for _ in range(2):
                A, B = draw(ash), draw(bsh)
                tA.upload(A)
                tB.upload(B)
                want = (A.T if opA else A).astype(np.float64) @ (B.T if opB else B).astype(np.float64)
                capi.nnt_gemm(ctx.h, 1.0, opA, tA.h, opB, tB.h, 0.0, tC.h, 1, 0, tbias.h)
                check(tC.download(), want + bias[:, None], dt, form + " + bias")
                capi.nnt_gemm(ctx.h, 0.5, opA, tA.h, opB, tB.h, 2.0, tD.h, 1, 0, None)
                C0 = 0.5 * want + 2.0 * C0
                check(tD.download(), C0, dt, form + " + beta C")
                C0 = tD.download().astype(np.float64)
                capi.nnt_gemm_res(ctx.h, 1.0, opA, tA.h, opB, tB.h, 1.0, tC.h, 1, 0, tbias.h, tR.h)
                check(tC.download(), want + bias[:, None] + R, dt, form + " + bias + R")
        ctx.set_granularity(1)
        capi.nnt_gemm(ctx.h, 1.0, opA, tA.h, opB, tB.h, 0.0, tD.h, 1, 0, None)
        check(tD.download(), want, dt, form + ", tile by tile")


@pytest.mark.parametrize("form", ["NN", "TN", "NT"])
@pytest.mark.parametrize("din,m,n,k,tile,kernel,cut", [
    ("bf16", 1537, 4611, 515, 300, "gemm_bf16_span_wide_kernel<float", False), ("bf16", 1501, 1503, 3001, 300, "gemm_bf16_span_tall_kernel<float", True),
    ("bf16", 4097, 4099, 1033, 1024, "gemm_bf16_span", None),
    ("f32", 4001, 4099, 2049, 1024, "gemm_f32_span_kernel<%s, 2, 2>", True), ("f32", 1051, 1033, 5001, 400, "gemm_f32_span_kernel<%s, 1, 2>", True),
    ("f32", 1501, 1503, 3001, 300, "gemm_f32_span_kernel<%s, 1, 1>", True),
])
def test_forms_of_products_that_lay_their_operands_out_afresh(mods, din, m, n, k, tile, kernel, cut, form):
    """The kernel that runs, by its record, in the three operand orders; with and without k-slices."""
    capi, tiled = mods
    r = rng(m + n + k)
    opA, opB = ("NT".index(c) for c in form)
    draw = lambda shape: r.integers(-32, 33, shape).astype(np.float32) / 16
    with tiled.Context(n_streams=1) as ctx:
        A, B = draw((k, m) if opA else (m, k)), draw((n, k) if opB else (k, n))
        tA, tB, tC = T(tiled, ctx, A, (tile, tile), din), T(tiled, ctx, B, (tile, tile), din), tiled.TiledTensor(ctx, "f32", (m, n), (tile, tile))
        ctx.profile(True)
        capi.nnt_gemm(ctx.h, 1.0, opA, tA.h, opB, tB.h, 0.0, tC.h, 1, 0, None)
        labels = list(ctx.profile_read())
        ctx.profile(False)
        order = {"NN": "false, true", "TN": "true, true", "NT": "false, false"}[form]
        assert any((kernel % order if "%" in kernel else kernel) in x and order in x for x in labels), labels
        assert cut is None or ("splitk_reduce" in labels) == cut, labels
        check(tC.download(), (A.T if opA else A).astype(np.float64) @ (B.T if opB else B).astype(np.float64), "f32", form)


@pytest.mark.parametrize("din", ["bf16", "f32"])
@pytest.mark.parametrize("case", ["forward", "weights", "narrow"])
def test_operands_laid_out_afresh_of_several_axes_and_of_narrow_tiles(mods, din, case):
    """Lines that belong to two axes, ragged along both, free (a layer's forward pass, with bias and residual) and contracted (its weight
    gradient), and tiles narrower than a vector along the contiguous axis."""
    capi, tiled = mods
    r = rng(83)
    draw = lambda shape: r.integers(-32, 33, shape).astype(np.float32) / 16
    m, n, s, b = 2001, 1333, 517, 4
    base = lambda x: (300, 200, 3) if len(x) == 3 else (300, 300)
    with tiled.Context(n_streams=1) as ctx:
        if case == "forward":
            W, X, R, bias = draw((m, n)), draw((n, s, b)), draw((m, s, b)), draw((m,))
            ts = [T(tiled, ctx, W, base(W.shape), din), T(tiled, ctx, X, base(X.shape), din), T(tiled, ctx, bias, (300,), "f32"), T(tiled, ctx, R, base(R.shape), din)]
            tY = tiled.TiledTensor(ctx, din, (m, s, b), base((m, s, b)))
            call = lambda: capi.nnt_gemm_res(ctx.h, 1.0, 0, ts[0].h, 0, ts[1].h, 1.0, tY.h, 1, 0, ts[2].h, ts[3].h)
            want = np.einsum("mn,nsb->msb", W.astype(np.float64), X.astype(np.float64), optimize=True) + bias[:, None, None] + R
        elif case == "weights":
            dY, X = draw((m, s, b)), draw((n, s, b))
            ts = [T(tiled, ctx, dY, base(dY.shape), din), T(tiled, ctx, X, base(X.shape), din)]
            tY = tiled.TiledTensor(ctx, "f32", (m, n), (300, 300))
            call = lambda: capi.nnt_gemm(ctx.h, 1.0, 0, ts[0].h, 1, ts[1].h, 0.0, tY.h, 2, 0, None)
            want = dY.reshape(m, -1).astype(np.float64) @ X.reshape(n, -1).T.astype(np.float64)
        else:
            m, n, k = 3201, 2803, 1501
            A, B = draw((k, m)), draw((k, n))
            ts = [T(tiled, ctx, A, (3, 700), din), T(tiled, ctx, B, (3, 700), din)]
            tY = tiled.TiledTensor(ctx, "f32", (m, n), (700, 700))
            call = lambda: capi.nnt_gemm(ctx.h, 1.0, 1, ts[0].h, 0, ts[1].h, 0.0, tY.h, 1, 0, None)
            want = A.T.astype(np.float64) @ B.astype(np.float64)
        ctx.profile(True)
        call()
        labels = list(ctx.profile_read())
        ctx.profile(False)
        assert any("_span_" in x for x in labels), labels
        check(tY.download(), want, din if case == "forward" else "f32", case)


@pytest.mark.parametrize("m,n,k,tile,din,bound", [
    (3778, 896, 4736, 300, "f32", 2.4e-7),       # a move every 128 k: 2.1e-7; every 256 k 2.6e-7 to 2.9e-7
    (2688, 3072, 2145, 400, "f32", 2.4e-7),
    (2001, 1333, 2068, 500, "bf16", 1.7e-7),     # 128 x 128 macro-tiles, a move every 512 k: 1.3e-7; one chain 2.7e-7
    (4065, 1211, 2832, 512, "bf16", 2.2e-7),     # 256 x 128 macro-tiles in as many slices as the operands as they are take: 1.8e-7; one chain 3.2e-7
])
def test_products_of_odd_sizes_are_as_exact_as_before(mods, m, n, k, tile, din, bound):
    """fp32 results of operands that are laid out afresh, 2-norm.  A chain of c additions in random order is off by about a * sqrt(c / 2) of its sum,
    so that halving it takes 0.7 of that; the bounds lie between what the chains are and what twice as long ones give."""
    capi, tiled = mods
    r = rng(m + n + k)
    with tiled.Context(n_streams=2) as ctx:
        A, B = quant(r.standard_normal((m, k)), din), quant(r.standard_normal((k, n)), din)
        tA, tB, tC = T(tiled, ctx, A, (tile, tile), din), T(tiled, ctx, B, (tile, tile), din), tiled.TiledTensor(ctx, "f32", (m, n), (tile, tile))
        ctx.profile(True)
        capi.nnt_gemm(ctx.h, 1.0, 0, tA.h, 0, tB.h, 0.0, tC.h, 1, 0, None)
        labels = list(ctx.profile_read())
        ctx.profile(False)
        assert any("_span_" in x for x in labels), labels
        want = A.astype(np.float64) @ B.astype(np.float64)
        e = float(np.linalg.norm(tC.download() - want) / np.linalg.norm(want))
        assert e <= bound, e


@pytest.mark.parametrize("m,n,k,tile,opA,opB,din,afresh", [
    (1258, 1208, 686, 256, 0, 0, "f32", False), (1437, 1032, 903, 512, 0, 1, "f32", False), (1538, 359, 469, 1024, 0, 0, "f32", False),
    (1111, 999, 777, 300, 0, 0, "f32", False), (3778, 896, 4736, 300, 0, 0, "f32", True),
    (1605, 862, 1061, 300, 1, 0, "bf16", False), (4630, 1735, 810, 256, 1, 0, "bf16", False), (3204, 3811, 808, 400, 0, 1, "bf16", True),
    (2001, 2068, 1333, 500, 0, 0, "bf16", True), (1333, 2068, 2001, 500, 1, 0, "bf16", True),
])
def test_which_products_of_odd_sizes_are_laid_out_afresh(mods, m, n, k, tile, opA, opB, din, afresh):
    """Products on which the copy was measured to lose (by 3 to 40 %) and to win."""
    capi, tiled = mods
    with tiled.Context(n_streams=1) as ctx:
        z = lambda shape, dt: tiled.TiledTensor.zeros(ctx, shape, tuple(min(x, tile) for x in shape), dt)
        tA, tB, tC = z((k, m) if opA else (m, k), din), z((n, k) if opB else (k, n), din), z((m, n), "f32")
        ctx.profile(True)
        capi.nnt_gemm(ctx.h, 1.0, opA, tA.h, opB, tB.h, 0.0, tC.h, 1, 0, None)
        labels = list(ctx.profile_read())
        ctx.profile(False)
        assert any("_span_" in x for x in labels) == afresh, labels


def test_device_memory_of_the_library_is_reported(mods):
    """nnt_ctx_stats: tile-pointer tables and plan tables count as table bytes, the fp32 workspace of a
    product cut into k-slices as workspace bytes; both shrink again when the tensors go."""
    capi, tiled = mods
    with tiled.Context(n_streams=1) as ctx:
        base = ctx.stats()
        assert base["device_table_bytes"] == 0 and base["device_workspace_bytes"] == 0
        A = tiled.TiledTensor(ctx, "f32", (256, 8192), (256, 2048))          # dW-like: few output tiles, long contraction
        B = tiled.TiledTensor(ctx, "f32", (256, 8192), (256, 2048))
        Cc = tiled.TiledTensor(ctx, "f32", (256, 256), (256, 256))
        for t in (A, B):
            for k in range(len(t.tile_index)):
                t.tile_view(k).normal_()
        one = ctx.stats()
        assert one["device_table_bytes"] == (4 + 4 + 1) * 8                   # one pointer per tile
        capi.nnt_gemm(ctx.h, 1.0, 0, A.h, 1, B.h, 0.0, Cc.h, 1, 0, None)
        ctx.wait()
        two = ctx.stats()
        assert two["plans"] == 1 and two["device_table_bytes"] > one["device_table_bytes"]
        assert two["device_workspace_bytes"] >= 2 * 128 * 128 * 4             # at least two slices of one macro-tile
        assert two["device_workspace_bytes"] <= 2 << 30
        assert relerr(Cc.download(), D.matmul2d(1.0, "N", A.download(), "T", B.download(), 0.0, None)) <= 1e-5
        Cc.close()                                                            # drops the plan and its workspace
        three = ctx.stats()
        assert three["plans"] == 0 and three["device_workspace_bytes"] == 0 and three["device_table_bytes"] == 8 * 8


def test_gemm_rejects_mismatched_tilings(mods):
    capi, tiled = mods
    with tiled.Context(n_streams=1) as ctx:
        A = tiled.TiledTensor(ctx, "f32", (8, 6), (4, 3))
        B = tiled.TiledTensor(ctx, "f32", (6, 5), (2, 5))       # contracted axis tiled 3 vs 2
        Cc = tiled.TiledTensor(ctx, "f32", (8, 5), (4, 5))
        assert capi.nnt_gemm.raw(ctx.h, 1.0, 0, A.h, 0, B.h, 0.0, Cc.h, 1, 0, None) == capi.NNT_EINVAL
        assert b"contracted" in capi.nnt_last_error(ctx.h)
        B2 = tiled.TiledTensor(ctx, "bf16", (6, 5), (3, 5))
        assert capi.nnt_gemm.raw(ctx.h, 1.0, 0, A.h, 0, B2.h, 0.0, Cc.h, 1, 0, None) == capi.NNT_EDTYPE
        # the context stays usable after an argument error
        B3 = tiled.TiledTensor.from_numpy(ctx, np.ones((6, 5), np.float32), (3, 5))
        A.upload(np.ones((8, 6), np.float32))
        capi.nnt_gemm(ctx.h, 1.0, 0, A.h, 0, B3.h, 0.0, Cc.h, 1, 0, None)
        assert np.all(Cc.download() == 6.0)


# ------------------------------------------------------------------ memory-bound operations
@pytest.mark.parametrize("gran", GRANS)
@pytest.mark.parametrize("dtype", ["f32", "bf16"])
@pytest.mark.parametrize("shape,base", [((768, 40, 3), (256, 16, 3)), ((100, 37, 2), (48, 10, 1)), ((1600, 12, 2), (400, 12, 2)),
                                        # long tokens, shared by the wavefronts of a workgroup: register-cached and looping forms
                                        ((8192, 5, 2), (1024, 5, 1)), ((2560, 7, 1), (512, 7, 1)), ((20000, 3, 1), (5000, 3, 1)),
                                        # odd extents: a last tile of one element, tiles shorter than a vector, tokens shared by wavefronts, the longest
                                        # (4096 vectors) and the next
                                        ((2001, 9, 2), (500, 4, 2)), ((13, 7, 2), (5, 7, 1)), ((3001, 33, 1), (1024, 33, 1)), ((9001, 5, 1), (9001, 5, 1)),
                                        ((16381, 3, 1), (16381, 3, 1)), ((33001, 2, 1), (33001, 2, 1))])
def test_layernorm_tensor(mods, gran, dtype, shape, base):
    capi, tiled = mods
    r = rng(3)
    X = quant(r.standard_normal(shape) * 1.5 + 0.3, dtype)
    dY = quant(r.standard_normal(shape), dtype)
    dR = quant(r.standard_normal(shape), dtype)
    gamma = (1 + 0.1 * r.standard_normal(shape[0])).astype(np.float32)
    beta = (0.1 * r.standard_normal(shape[0])).astype(np.float32)
    Yref, mean, rstd = D.layernorm_fwd(X, gamma, beta, 1e-5)
    dXref, dgref, dbref = D.layernorm_bwd(X, gamma, mean, rstd, dY)
    with tiled.Context(n_streams=4, granularity=gran) as ctx:
        tX, tdY, tdR = [T(tiled, ctx, a, base, dtype) for a in (X, dY, dR)]
        tg, tb = T(tiled, ctx, gamma, base[:1], "f32"), T(tiled, ctx, beta, base[:1], "f32")
        tY = tiled.TiledTensor(ctx, dtype, shape, base)
        tS = tiled.TiledTensor(ctx, "f32", (2,) + shape[1:], (2,) + base[1:])
        capi.nnt_layernorm_fwd(ctx.h, tX.h, tg.h, tb.h, 1e-5, tY.h, tS.h)
        check(tY.download(), Yref, dtype, "ln fwd")
        s = tS.download()
        check(s[0], mean, "f32", "ln mean")
        check(s[1], rstd, "f32", "ln rstd")
        tdX = tiled.TiledTensor(ctx, dtype, shape, base)
        tdg, tdb = tiled.TiledTensor(ctx, "f32", shape[:1], base[:1]), tiled.TiledTensor(ctx, "f32", shape[:1], base[:1])
        capi.nnt_layernorm_bwd(ctx.h, tX.h, tS.h, tg.h, tdY.h, tdR.h, tdX.h, tdg.h, tdb.h)
        e = relerr(tdX.download(), dXref + dR)
        assert e <= TOL[dtype], e
        check(tdg.download(), dgref, "f32", "ln dgamma")
        check(tdb.download(), dbref, "f32", "ln dbeta")
        capi.nnt_layernorm_bwd(ctx.h, tX.h, tS.h, tg.h, tdY.h, None, tdX.h, tdg.h, tdb.h)
        e = relerr(tdX.download(), dXref)
        assert e <= TOL[dtype], e


@pytest.mark.parametrize("dtype", ["f32", "bf16"])
@pytest.mark.parametrize("shape,base", [((128, 1, 1), (32, 1, 1)), ((520, 9, 1), (520, 4, 1)), ((1000, 67, 9), (400, 32, 2)), ((4096, 19, 2), (1024, 19, 2)),
                                        ((4104, 3, 3), (4104, 3, 3)), ((8192, 5, 2), (8192, 5, 1)), ((8200, 3, 1), (8200, 3, 1)), ((16384, 3, 1), (4096, 3, 1)), ((16392, 2, 1), (16392, 2, 1)), ((512, 300, 17), (512, 300, 17)),
                                        ((63, 5, 2), (63, 5, 2)), ((777, 130, 3), (300, 100, 3)), ((4095, 3, 1), (4095, 3, 1)), ((4097, 3, 1), (4097, 3, 1)),
                                        ((96, 1025, 1), (96, 1025, 1)), ((320, 513, 2), (64, 513, 2)), ((1200, 1025, 1), (48, 500, 1)), ((2001, 21, 2), (500, 9, 2)), ((13, 40, 2), (5, 7, 1)), ((8191, 5, 2), (1000, 5, 2))])
def test_layernorm_backward_in_one_pass(mods, dtype, shape, base):
    """One to eight wavefronts per token, fewer and more tokens than groups of wavefronts, ragged tiles, scalar forms, and the
    longest tokens of either form (4096, 8192 in fp32, twice that in bf16) and the next.  The input gradient in place of the
    upstream one, twice in a row with other operations on the second stream: the partial sums of the two streams lie apart."""
    capi, tiled = mods
    r = rng(23)
    X, dY, dR = [quant(r.standard_normal(shape), dtype) for _ in range(3)]
    gamma = (1 + 0.1 * r.standard_normal(shape[0])).astype(np.float32)
    _, mean, rstd = D.layernorm_fwd(X, gamma, 0 * gamma, 1e-5)
    dXref, dgref, dbref = D.layernorm_bwd(X, gamma, mean, rstd, dY)
    with tiled.Context(n_streams=2) as ctx:
        tX, tR, tg = T(tiled, ctx, X, base, dtype), T(tiled, ctx, dR, base, dtype), T(tiled, ctx, gamma, base[:1], "f32")
        tS = tiled.TiledTensor.from_numpy(ctx, np.stack([mean, rstd]).astype(np.float32), (2,) + base[1:])
        runs = []
        for _ in range(2):
            tdY = T(tiled, ctx, dY, base, dtype)
            out = [tiled.TiledTensor(ctx, "f32", shape[:1], base[:1]) for _ in range(3)]
            capi.nnt_bias_grad(ctx.h, tdY.h, out[2].h)
            capi.nnt_layernorm_bwd(ctx.h, tX.h, tS.h, tg.h, tdY.h, tR.h, tdY.h, out[0].h, out[1].h)
            runs.append((tdY, out))
        for tdY, out in runs:
            e = relerr(tdY.download(), dXref + dR)
            assert e <= TOL[dtype], e
            check(out[0].download(), dgref, "f32", "ln dgamma")
            check(out[1].download(), dbref, "f32", "ln dbeta")
            check(out[2].download(), dbref, "f32", "bias grad")


@pytest.mark.parametrize("tokens", [255, 256, 257, 512, 513, 768, 769, 1025])
@pytest.mark.parametrize("dtype,rows,base", [("f32", 2048, 128), ("bf16", 3848, 264), ("f32", 79, 5), ("f32", 593, 66), ("bf16", 8200, 8200), ("f32", 4100, 4100), ("bf16", 8201, 4000)])
def test_layernorm_backward_of_one_to_five_tokens_per_workgroup(mods, dtype, rows, base, tokens):
    """All waves of a workgroup on one token, 256 workgroups: the rounds in which a workgroup has one, two or more tokens left, workgroups without
    one in the last round, whole vectors, odd extents and the longest form.  The last token is full of large values and the input gradient takes
    the place of X: what the others fetch in its stead must not be seen."""
    capi, tiled = mods
    r = rng(43)
    X, dY = [quant(r.standard_normal((rows, tokens)), dtype) for _ in range(2)]
    X[:, -1] *= np.asarray(2.0, X.dtype) ** 100
    gamma = (1 + 0.1 * r.standard_normal(rows)).astype(np.float32)
    _, mean, rstd = D.layernorm_fwd(X.astype(np.float64), gamma, 0 * gamma, 1e-5)
    dXref, dgref, dbref = D.layernorm_bwd(X.astype(np.float64), gamma, mean, rstd, dY.astype(np.float64))
    with tiled.Context(n_streams=2) as ctx:
        tX, tdY, tg = T(tiled, ctx, X, (base, 300), dtype), T(tiled, ctx, dY, (base, 300), dtype), T(tiled, ctx, gamma, (base,), "f32")
        tS = tiled.TiledTensor.from_numpy(ctx, np.stack([mean, rstd]).astype(np.float32), (2, 300))
        out = [tiled.TiledTensor(ctx, "f32", (rows,), (base,)) for _ in range(2)]
        capi.nnt_layernorm_bwd(ctx.h, tX.h, tS.h, tg.h, tdY.h, None, tX.h, out[0].h, out[1].h)
        e = relerr(tX.download(), dXref)
        assert e <= TOL[dtype], e
        check(out[0].download(), dgref, "f32", "ln dgamma")
        check(out[1].download(), dbref, "f32", "ln dbeta")


@pytest.mark.parametrize("rows,base,tokens", [(585, 65, 65536), (1152, 128, 16640), (585, 65, 8192), (585, 65, 8193), (585, 65, 8449), (585, 65, 8705), (1105, 65, 16385), (79, 5, 8705)])
def test_layernorm_backward_sums_over_many_tokens(mods, rows, base, tokens):
    """All waves of a workgroup on one token, 256 workgroups: 65536 tokens are 256 rounds.  Gain and bias gradients in the 2-norm: a chain of m
    additions in random order is off by about 0.29 * 2^-24 * sqrt(m / 2) of its sum, 6.9e-8 for the 32 tokens of a chain, 3.5e-8 for the 8 chains of a
    workgroup, 5e-8 for its row's way through the pairs of 256, 6e-8 for the roundings of the terms: 1.1e-7 together; one chain of 256 is 2.0e-7
    alone.  The numbers of tokens around a move of the sums as well: a token lost or counted twice would be 1e-2."""
    capi, tiled = mods
    r = rng(47)
    X, dY = [r.standard_normal((rows, tokens)).astype(np.float32) for _ in range(2)]
    gamma = (1 + 0.1 * r.standard_normal(rows)).astype(np.float32)
    mean, rstd = [a.astype(np.float32) for a in (X.mean(0, dtype=np.float64), 1 / np.sqrt(X.var(0, dtype=np.float64) + 1e-5))]
    xh = (X - mean.astype(np.float64)) * rstd
    with tiled.Context(n_streams=2) as ctx:
        tX, tdY, tg = T(tiled, ctx, X, (base, tokens), "f32"), T(tiled, ctx, dY, (base, tokens), "f32"), T(tiled, ctx, gamma, (base,), "f32")
        tS = tiled.TiledTensor.from_numpy(ctx, np.stack([mean, rstd]), (2, tokens))
        tdX = tiled.TiledTensor(ctx, "f32", (rows, tokens), (base, tokens))
        out = [tiled.TiledTensor(ctx, "f32", (rows,), (base,)) for _ in range(2)]
        capi.nnt_layernorm_bwd(ctx.h, tX.h, tS.h, tg.h, tdY.h, None, tdX.h, out[0].h, out[1].h)
        for t, ref, what in zip(out, ((dY * xh).sum(1), dY.sum(1, dtype=np.float64)), ("dgamma", "dbeta")):
            e = float(np.linalg.norm(t.download() - ref) / np.linalg.norm(ref))
            assert e <= 2e-7, (what, e)


@pytest.mark.parametrize("dtype,rows,base,tokens", [("bf16", 512, 512, 700), ("bf16", 1024, 512, 700), ("bf16", 768, 256, 4096), ("bf16", 1600, 400, 4100), ("bf16", 2048, 512, 6200),
                                                    ("bf16", 2800, 400, 700), ("bf16", 4096, 1024, 700), ("f32", 200, 200, 700), ("f32", 512, 256, 700), ("f32", 2048, 1024, 700)])
@pytest.mark.parametrize("res", [False, True])
def test_layernorm_backward_in_one_pass_and_in_two_gives_the_same(mods, dtype, rows, base, tokens, res):
    """The input gradient of the one pass is that of the two passes bit for bit where both add a token's sums in the same order.  Two passes run inside a
    capture before the stream's scratch is there; the shared one is, from a bias gradient."""
    capi, tiled = mods
    r = rng(71)
    X, dY, dR = [quant(r.standard_normal((rows, tokens)), dtype) for _ in range(3)]
    gamma = (1 + 0.1 * r.standard_normal(rows)).astype(np.float32)
    _, mean, rstd = D.layernorm_fwd(X, gamma, 0 * gamma, 1e-5)
    with tiled.Context(n_streams=2) as ctx:
        tX, tdY, tR, tg = [T(tiled, ctx, a, (base, 400), dtype) for a in (X, dY, dR)] + [T(tiled, ctx, gamma, (base,), "f32")]
        tS = tiled.TiledTensor.from_numpy(ctx, np.stack([mean, rstd]).astype(np.float32), (2, 400))
        two, one = (tiled.TiledTensor(ctx, dtype, X.shape, (base, 400)) for _ in range(2))
        out = [tiled.TiledTensor(ctx, "f32", (rows,), (base,)) for _ in range(2)]
        capi.nnt_bias_grad(ctx.h, tdY.h, out[0].h)
        call = lambda dX: capi.nnt_layernorm_bwd(ctx.h, tX.h, tS.h, tg.h, tdY.h, tR.h if res else None, dX.h, out[0].h, out[1].h)
        before = ctx.stats()["tasks"]
        g = C.c_void_p()
        capi.nnt_capture_begin(ctx.h)
        call(two)
        capi.nnt_capture_end(ctx.h, C.byref(g))
        assert ctx.stats()["tasks"] - before == 2
        capi.nnt_graph_launch(g)
        want = np.asarray(two.download())
        call(one)
        assert ctx.stats()["tasks"] - before == 3
        assert np.array_equal(np.asarray(one.download()), want)
        capi.nnt_graph_destroy(g)


@pytest.mark.parametrize("dtype,rows,base", [("f32", 1088, 64), ("f32", 2048, 64), ("f32", 2112, 64), ("bf16", 1700, 100), ("bf16", 1920, 64)])
def test_layernorm_backward_of_many_tokens_on_narrow_tiles(mods, dtype, rows, base):
    """Two passes on tiles that fill less than half of a wave: 17 and 32 vectors per lane, the forms that keep the token in registers, and 33."""
    capi, tiled = mods
    r = rng(61)
    X, dY, dR = [quant(r.standard_normal((rows, 1100)), dtype) for _ in range(3)]
    gamma = (1 + 0.1 * r.standard_normal(rows)).astype(np.float32)
    _, mean, rstd = D.layernorm_fwd(X, gamma, 0 * gamma, 1e-5)
    dXref, dgref, dbref = D.layernorm_bwd(X, gamma, mean, rstd, dY)
    with tiled.Context(n_streams=2) as ctx:
        tX, tdY, tR, tg = [T(tiled, ctx, a, (base, 400), dtype) for a in (X, dY, dR)] + [T(tiled, ctx, gamma, (base,), "f32")]
        tS, tdX = tiled.TiledTensor.from_numpy(ctx, np.stack([mean, rstd]).astype(np.float32), (2, 400)), tiled.TiledTensor(ctx, dtype, X.shape, (base, 400))
        out = [tiled.TiledTensor(ctx, "f32", (rows,), (base,)) for _ in range(2)]
        capi.nnt_layernorm_bwd(ctx.h, tX.h, tS.h, tg.h, tdY.h, tR.h, tdX.h, out[0].h, out[1].h)
        e = relerr(tdX.download(), dXref + dR)
        assert e <= TOL[dtype], e
        check(out[0].download(), dgref, "f32", "ln dgamma")
        check(out[1].download(), dbref, "f32", "ln dbeta")


@pytest.mark.parametrize("rows,base,tokens,passes", [(256, 256, 40, 1), (16384, 4096, 40, 2), (256, 32, 40, 1), (256, 32, 1025, 2), (255, 51, 1024, 1), (255, 51, 1025, 2), (255, 85, 1025, 1),
                                                     (449, 50, 257, 2), (449, 50, 256, 1), (399, 50, 257, 1)])
def test_layernorm_backward_counts_the_bytes_it_moves(mods, rows, base, tokens, passes):
    """One pass reads x, dy (and the residual) once and writes dx, two read x and dy twice: that is what the records say."""
    capi, tiled = mods
    with tiled.Context(n_streams=2) as ctx:
        z = lambda shape, b: tiled.TiledTensor.zeros(ctx, shape, b)
        tX, tdY, tR, tdX = (z((rows, tokens), (base, tokens)) for _ in range(4))
        tS, tg, dg, db = z((2, tokens), (2, tokens)), z((rows,), (base,)), z((rows,), (base,)), z((rows,), (base,))
        for res in (None, tR):
            ctx.profile(True)
            capi.nnt_layernorm_bwd(ctx.h, tX.h, tS.h, tg.h, tdY.h, res.h if res else None, tdX.h, dg.h, db.h)
            rec = ctx.profile_read()["layernorm_bwd"]
            ctx.profile(False)
            assert rec["unit"] == "bytes" and rec["tasks"] == passes
            assert rec["work"] == rows * tokens * 4 * ((3 if passes == 1 else 5) + (1 if res else 0))


@pytest.mark.parametrize("dtype", ["f32", "bf16"])
@pytest.mark.parametrize("shape,base", [((8191, 150, 2), (1000, 150, 2)), ((4097, 300, 1), (4097, 300, 1)), ((1025, 700, 1), (513, 700, 1)), ((15, 40, 1), (5, 40, 1))])
def test_layernorm_backward_in_place_of_the_residual(mods, dtype, shape, base):
    """dX is the residual, odd extents: the last vector of a tile is moved back over elements that another lane, or another wavefront of
    the token, adds its own copy of the residual to.  Every element gets it once."""
    capi, tiled = mods
    r = rng(41)
    X, dY, dR = [quant(r.standard_normal(shape), dtype) for _ in range(3)]
    gamma = (1 + 0.1 * r.standard_normal(shape[0])).astype(np.float32)
    _, mean, rstd = D.layernorm_fwd(X, gamma, 0 * gamma, 1e-5)
    dXref, _, _ = D.layernorm_bwd(X, gamma, mean, rstd, dY)
    with tiled.Context(n_streams=2) as ctx:
        tX, tdY, tg = T(tiled, ctx, X, base, dtype), T(tiled, ctx, dY, base, dtype), T(tiled, ctx, gamma, base[:1], "f32")
        tS = tiled.TiledTensor.from_numpy(ctx, np.stack([mean, rstd]).astype(np.float32), (2,) + base[1:])
        tR, apart = T(tiled, ctx, dR, base, dtype), tiled.TiledTensor(ctx, dtype, shape, base)
        out = [tiled.TiledTensor(ctx, "f32", shape[:1], base[:1]) for _ in range(2)]
        capi.nnt_layernorm_bwd(ctx.h, tX.h, tS.h, tg.h, tdY.h, tR.h, apart.h, out[0].h, out[1].h)
        want = apart.download()
        e = relerr(want, dXref + dR)
        assert e <= TOL[dtype], e
        capi.nnt_layernorm_bwd(ctx.h, tX.h, tS.h, tg.h, tdY.h, tR.h, tR.h, out[0].h, out[1].h)
        assert np.array_equal(np.asarray(tR.download()), np.asarray(want))


@pytest.mark.parametrize("dtype", ["f32", "bf16"])
@pytest.mark.parametrize("shape,base", [((1, 1), (1, 1)), ((128, 128), (32, 32)), ((40, 1024), (16, 1000)), ((40, 1025), (16, 1000)), ((777, 31, 5), (300, 7, 2)),
                                        ((3168, 1024), (1056, 512)), ((3176, 1024), (3176, 1024)), ((6344, 1024), (6344, 1024)), ((6352, 1024), (6352, 1024))])
def test_bias_grad_in_one_launch(mods, dtype, shape, base):
    """Both sides of the rule (1024 columns, 13 MB), ragged tiles on every axis, rows that are no whole vectors."""
    capi, tiled = mods
    r = rng(29)
    dY = quant(r.standard_normal(shape), dtype)
    with tiled.Context(n_streams=2) as ctx:
        t, db = T(tiled, ctx, dY, base, dtype), tiled.TiledTensor(ctx, "f32", shape[:1], base[:1])
        capi.nnt_bias_grad(ctx.h, t.h, db.h)
        check(db.download(), np.asarray(dY, np.float64).reshape(shape[0], -1).sum(1), "f32", "bias grad")


@pytest.mark.parametrize("dtype", ["f32", "bf16"])
@pytest.mark.parametrize("rows,base,tokens", [(63, 63, 90), (129, 129, 90), (193, 193, 90), (501, 50, 1200), (501, 50, 1201), (386, 129, 1201), (513, 257, 90), (4111, 257, 1201), (770, 257, 1201),
                                              (602, 201, 1300), (37, 5, 1300), (1499, 1499, 1100), (1500, 600, 1100), (255, 51, 1599), (1823, 65, 1097), (1823, 65, 1098), (200, 25, 1000), (65 * 25, 25, 70), (17 * 25, 25, 256), (17 * 25, 25, 257), (2049, 75, 1300)])
def test_odd_extents_by_vectors_and_by_single_elements(mods, dtype, rows, base, tokens):
    """Both sides of the rules that say whether layer norm and the column sums take odd extents by vectors or element by element."""
    capi, tiled = mods
    r = rng(89)
    X, dY = [quant(r.standard_normal((rows, tokens)), dtype) for _ in range(2)]
    gamma, beta = (1 + 0.1 * r.standard_normal(rows)).astype(np.float32), r.standard_normal(rows).astype(np.float32)
    Yref, mean, rstd = D.layernorm_fwd(X, gamma, beta, 1e-5)
    with tiled.Context(n_streams=2) as ctx:
        tX, tdY = T(tiled, ctx, X, (base, 700), dtype), T(tiled, ctx, dY, (base, 700), dtype)
        tg, tb = T(tiled, ctx, gamma, (base,), "f32"), T(tiled, ctx, beta, (base,), "f32")
        tY, tdX = (tiled.TiledTensor(ctx, dtype, (rows, tokens), (base, 700)) for _ in range(2))
        tS = tiled.TiledTensor(ctx, "f32", (2, tokens), (2, 700))
        db = tiled.TiledTensor(ctx, "f32", (rows,), (base,))
        capi.nnt_layernorm_fwd(ctx.h, tX.h, tg.h, tb.h, 1e-5, tY.h, tS.h)
        capi.nnt_bias_grad(ctx.h, tdY.h, db.h)
        check(tY.download(), Yref, dtype, "ln")
        check(tS.download(), np.stack([mean, rstd]), "f32", "statistics")
        check(db.download(), np.asarray(dY, np.float64).sum(1), "f32", "bias grad")


@pytest.mark.parametrize("shape,base,launches", [((300, 64), (100, 64), 1), ((300, 64), (100, 33), 1), ((300, 64), (100, 30), 2), ((300, 16, 8), (300, 16, 4), 1),
                                                 ((300, 16, 8), (300, 16, 2), 2), ((40, 1024), (40, 1), 2), ((301, 8, 64), (75, 8, 1), 2)])
def test_bias_grad_of_many_tiles_takes_two_launches(mods, shape, base, launches):
    """The one-launch form walks the tiles along the columns one after the other: one or two of them, however few columns they hold."""
    capi, tiled = mods
    r = rng(53)
    dY = r.standard_normal(shape).astype(np.float32)
    with tiled.Context(n_streams=2) as ctx:
        t, db = T(tiled, ctx, dY, base, "f32"), tiled.TiledTensor(ctx, "f32", shape[:1], base[:1])
        before = ctx.stats()["launches"]
        capi.nnt_bias_grad(ctx.h, t.h, db.h)
        assert ctx.stats()["launches"] - before == launches
        check(db.download(), dY.astype(np.float64).reshape(shape[0], -1).sum(1), "f32", "bias grad")


@pytest.mark.parametrize("shape,base", [((768, 6, 2), (256, 6, 2)), ((5000, 3, 1), (2500, 3, 1)), ((101, 5, 1), (37, 5, 1))])
@pytest.mark.parametrize("gran", GRANS)
def test_layernorm_token_with_an_outlier(mods, gran, shape, base):
    """One element of every token lies a thousand standard deviations from the rest (first element, or
    one in the middle): mean and variance must come out at fp32 accuracy, which a one-pass variance
    (difference of two large sums) does not deliver.  Register-cached, long-column and scalar paths."""
    capi, tiled = mods
    r = rng(17)
    X = r.standard_normal(shape)
    X[0, ::2] += 1000.0
    X[shape[0] // 2, 1::2] -= 3000.0
    X = quant(X, "f32")
    gamma = (1 + 0.1 * r.standard_normal(shape[0])).astype(np.float32)
    beta = (0.1 * r.standard_normal(shape[0])).astype(np.float32)
    Yref, mean, rstd = D.layernorm_fwd(X, gamma, beta, 1e-5)
    with tiled.Context(n_streams=1, granularity=gran) as ctx:
        tX = T(tiled, ctx, X, base, "f32")
        tg, tb = T(tiled, ctx, gamma, base[:1], "f32"), T(tiled, ctx, beta, base[:1], "f32")
        tY = tiled.TiledTensor(ctx, "f32", shape, base)
        tS = tiled.TiledTensor(ctx, "f32", (2,) + shape[1:], (2,) + base[1:])
        capi.nnt_layernorm_fwd(ctx.h, tX.h, tg.h, tb.h, 1e-5, tY.h, tS.h)
        s = tS.download()
        check(s[0], mean, "f32", "ln mean")
        assert np.abs(s[1] / rstd - 1.0).max() <= 1e-5, "ln rstd, element-wise relative"
        check(tY.download(), Yref, "f32", "ln fwd")


@pytest.mark.parametrize("gran", GRANS)
@pytest.mark.parametrize("dtype", ["f32", "bf16"])
def test_elementwise_tensor_ops(mods, gran, dtype):
    capi, tiled = mods
    r = rng(4)
    shape, base = (200, 50, 3), (64, 24, 2)
    X, Y = quant(r.standard_normal(shape) * 2, dtype), quant(r.standard_normal(shape), dtype)
    with tiled.Context(n_streams=4, granularity=gran) as ctx:
        tX, tY = T(tiled, ctx, X, base, dtype), T(tiled, ctx, Y, base, dtype)
        capi.nnt_add(ctx.h, 1.0, tX.h, 1.0, tY.h)
        check(tY.download(), X + Y, dtype, "add")
        tG = tiled.TiledTensor(ctx, dtype, shape, base)
        capi.nnt_gelu(ctx.h, 0, tX.h, tG.h)
        check(tG.download(), D.gelu(X), dtype, "gelu")
        tD = T(tiled, ctx, Y, base, dtype)
        capi.nnt_gelu_bwd(ctx.h, 0, tX.h, tD.h, tD.h)            # in place
        check(tD.download(), Y * D.gelu_grad(X), dtype, "gelu bwd in place")
        capi.nnt_fill(ctx.h, -3.0, tG.h)
        assert np.all(tG.download() == -3.0)
        if dtype == "f32":
            tL = tiled.TiledTensor(ctx, "bf16", shape, base)
            capi.nnt_cast(ctx.h, tX.h, tL.h)
            np.testing.assert_array_equal(tL.download(), D.round_to_bf16(X.astype(np.float32)))


@pytest.mark.parametrize("gran", GRANS)
@pytest.mark.parametrize("dtype", ["f32", "bf16"])
@pytest.mark.parametrize("zb,pb", [((64, 16, 2), (32, 16, 2, 2)), ((100, 7, 1), (24, 5, 1, 1)), ((400, 30, 2), (64, 30, 2, 5))])
def test_head_split_merge(mods, gran, dtype, zb, pb):
    capi, tiled = mods
    N_h, h, N_s, N_b = 5, 64, 30, 2
    Z = quant(rng(5).standard_normal((3 * N_h * h, N_s, N_b)), dtype)
    with tiled.Context(n_streams=4, granularity=gran) as ctx:
        tZ = T(tiled, ctx, Z, zb, dtype)
        parts = [tiled.TiledTensor(ctx, dtype, (h, N_s, N_b, N_h), pb) for _ in range(3)]
        arr = capi.ptr_array([p.h.value for p in parts])
        capi.nnt_head_split(ctx.h, tZ.h, 3, arr)
        for got, ref in zip(parts, D.split_heads(Z, N_h, 3)):
            np.testing.assert_array_equal(got.download(), ref.astype(np.float32))
        tZ2 = tiled.TiledTensor(ctx, dtype, Z.shape, zb)
        capi.nnt_head_merge(ctx.h, 3, arr, tZ2.h)
        np.testing.assert_array_equal(tZ2.download(), Z.astype(np.float32))


@pytest.mark.parametrize("gran", GRANS)
@pytest.mark.parametrize("dtype", ["f32", "bf16"])
@pytest.mark.parametrize("geom", [(64, 6, 128, 100, 40, 3, 2, 6),      # h, N_h, row tile, N_s, seq tile, N_b, batch tile, head tile of the scores
                                  (64, 4, 256, 96, 96, 2, 2, 4),
                                  (128, 4, 256, 72, 24, 1, 1, 2),
                                  (16, 8, 32, 50, 50, 2, 1, 8)])
def test_attention_products_on_tensors_with_the_heads_side_by_side(mods, gran, dtype, geom):
    """The six per-head products of the attention layer read Q, K, V and dB straight out of, and write B, dQ, dK,
    dV straight into, tensors [parts * N_h * h, N_s, N_b] (what the linear layers produce and consume): against
    the oracle's head split, batched contraction and head merge.  Scores with causal structure (absent tiles) and
    a head axis tiled coarser than the windows; rows of a result tensor outside the written part keep their values."""
    capi, tiled = mods
    h, N_h, t0, N_s, ts, N_b, tb, tjP = geom
    N_e = h * N_h
    r = rng(sum(geom))
    QKV = quant(r.standard_normal((3 * N_e, N_s, N_b)), dtype)
    dBm = quant(r.standard_normal((N_e, N_s, N_b)), dtype)
    Q, K, V = D.split_heads(QKV, N_h, 3)
    dB = D.split_heads(dBm, N_h, 1)[0]
    sc = 1.0 / math.sqrt(h)
    with tiled.Context(n_streams=4, granularity=gran) as ctx:
        tQKV = T(tiled, ctx, QKV, (t0, ts, tb), dtype)
        tdBm = T(tiled, ctx, dBm, (t0, ts, tb), dtype)
        sb = (ts, ts, tb, tjP)
        absent = tiled.causal_absent(ts, ts, N_s)
        tP = tiled.TiledTensor(ctx, dtype, (N_s, N_s, N_b, N_h), sb, absent)
        tS = tiled.TiledTensor(ctx, "f32", (2, N_s, N_b, N_h), (2, ts, tb, tjP))
        capi.nnt_gemm_heads(ctx.h, sc, 1, tQKV.h, 1, 0, tQKV.h, 0, tP.h, -1, h, N_h)           # K^T Q
        capi.nnt_softmax_fwd(ctx.h, tP.h, tS.h, 1.0, 1)
        A = D.attention_scores(K, Q)
        if dtype == "bf16":
            A = quant(A, dtype)
        Pref, _, _ = D.softmax_fwd(A, causal=True)
        P = tP.download().astype(np.float64)
        check(P, Pref, dtype, "softmax(K^T Q)")
        marker = quant(r.standard_normal((2 * N_e, N_s, N_b)), dtype)
        tBm = T(tiled, ctx, marker, (t0, ts, tb), dtype)                                       # B goes into part 1 of two
        capi.nnt_gemm_heads(ctx.h, 1.0, 0, tQKV.h, 2, 0, tP.h, -1, tBm.h, 1, h, N_h)           # V P
        got = tBm.download()
        check(got[N_e:], D.merge_heads([D.attention_values(V, P)]), dtype, "V P")
        np.testing.assert_array_equal(got[:N_e], marker[:N_e].astype(np.float32))
        tdP = tiled.TiledTensor(ctx, dtype, (N_s, N_s, N_b, N_h), sb, absent)
        tdQKV = tiled.TiledTensor(ctx, dtype, QKV.shape, (t0, ts, tb))
        capi.nnt_gemm_heads(ctx.h, 1.0, 0, tdBm.h, 0, 1, tP.h, -1, tdQKV.h, 2, h, N_h)         # dV = dB P^T
        capi.nnt_gemm_heads(ctx.h, 1.0, 1, tQKV.h, 2, 0, tdBm.h, 0, tdP.h, -1, h, N_h)         # dP = V^T dB
        dPdev = tdP.download().astype(np.float64)
        capi.nnt_softmax_bwd(ctx.h, tP.h, tdP.h)
        dA = tdP.download().astype(np.float64)
        check(dA, D.softmax_bwd(P, dPdev), dtype, "softmax bwd")
        capi.nnt_gemm_heads(ctx.h, sc, 0, tQKV.h, 1, 0, tdP.h, -1, tdQKV.h, 0, h, N_h)         # dQ = K dA
        capi.nnt_gemm_heads(ctx.h, sc, 0, tQKV.h, 0, 1, tdP.h, -1, tdQKV.h, 1, h, N_h)         # dK = Q dA^T
        ref = D.merge_heads([D.contract(sc, "N", K, "N", dA, 0.0, None, 1, 2), D.contract(sc, "N", Q, "T", dA, 0.0, None, 1, 2),
                             D.contract(1.0, "N", dB, "T", P, 0.0, None, 1, 2)])
        got = tdQKV.download()
        for part, name in enumerate(("dQ = K dA / sqrt(h)", "dK = Q dA^T / sqrt(h)", "dV = dB P^T")):
            check(got[part * N_e:(part + 1) * N_e], ref[part * N_e:(part + 1) * N_e], dtype, name)
        # geometry that does not fit is refused and leaves the context usable
        assert capi.nnt_gemm_heads.raw(ctx.h, 1.0, 0, tQKV.h, 3, 0, tP.h, -1, tBm.h, 1, h, N_h) == capi.NNT_EINVAL
        assert capi.nnt_gemm_heads.raw(ctx.h, 1.0, 0, tP.h, -1, 0, tP.h, -1, tP.h, -1, h, N_h) == capi.NNT_EINVAL
        ctx.wait()


@pytest.mark.parametrize("gran", GRANS)
@pytest.mark.parametrize("lowp", [False, True])
def test_adam_tensor(mods, gran, lowp):
    capi, tiled = mods
    r = rng(6)
    shape, base = (300, 130), (128, 64)
    p, g = r.standard_normal(shape).astype(np.float32), r.standard_normal(shape).astype(np.float32)
    with tiled.Context(n_streams=4, granularity=gran) as ctx:
        tp, tg = T(tiled, ctx, p, base, "f32"), T(tiled, ctx, g, base, "f32")
        tm, tv = tiled.TiledTensor.zeros(ctx, shape, base), tiled.TiledTensor.zeros(ctx, shape, base)
        tl = tiled.TiledTensor(ctx, "bf16", shape, base) if lowp else None
        cfg = capi.nnt_adam_cfg(1e-3, 0.9, 0.999, 1e-8, 0.0)
        pr, mr, vr = p.astype(np.float64), 0.0, 0.0
        for step in (1, 2):
            capi.nnt_adam_step(ctx.h, C.byref(cfg), step, tg.h, tp.h, tm.h, tv.h, tl.h if lowp else None)
            pr, mr, vr = D.adam_step(pr, g, mr, vr, step)
        check(tp.download(), pr, "f32", "adam p")
        check(tm.download(), mr, "f32", "adam m")
        check(tv.download(), vr, "f32", "adam v")
        if lowp:
            np.testing.assert_array_equal(tl.download(), D.round_to_bf16(tp.download()))


@pytest.mark.parametrize("gran", GRANS)
@pytest.mark.parametrize("lowp", [False, True])
def test_sgd_tensor(mods, gran, lowp):
    capi, tiled = mods
    r = rng(7)
    shape, base = (300, 130), (128, 64)
    p = r.standard_normal(shape).astype(np.float32)
    with tiled.Context(n_streams=4, granularity=gran) as ctx:
        tp = T(tiled, ctx, p, base, "f32")
        tv = tiled.TiledTensor.zeros(ctx, shape, base)
        tl = tiled.TiledTensor(ctx, "bf16", shape, base) if lowp else None
        cfg = capi.nnt_sgd_cfg(0.05, 0.9, 0.01, 0)
        pr, vr = p.astype(np.float64), 0.0
        for step in (1, 2):
            g = r.standard_normal(shape).astype(np.float32)
            tg = T(tiled, ctx, g, base, "f32")
            capi.nnt_sgd_step(ctx.h, C.byref(cfg), tg.h, tp.h, tv.h, tl.h if lowp else None)
            pr, vr = D.sgd_step(pr, g, vr, 0.05, 0.9, 0.01)
        check(tp.download(), pr, "f32", "sgd p")
        check(tv.download(), vr, "f32", "sgd v")
        if lowp:
            np.testing.assert_array_equal(tl.download(), D.round_to_bf16(tp.download()))


# ------------------------------------------------------------------ executor
def test_executor_orders_dependent_tasks_across_streams(mods):
    """A chain y <- y + x repeated many times on 8 streams must give the serial
    result; independent chains may overlap."""
    capi, tiled = mods
    shape, base = (192, 64), (64, 16)        # 12 tiles: chains of different tensors land on different streams
    x = rng(7).standard_normal(shape).astype(np.float32)
    results = {}
    for name, kw in (("serial", dict(n_streams=1, serial=True)), ("streams8_tiles", dict(n_streams=8, granularity=1)),
                     ("streams8_ops", dict(n_streams=8, granularity=0))):
        with tiled.Context(**kw) as ctx:
            tx = T(tiled, ctx, x, base, "f32")
            ys = [tiled.TiledTensor.zeros(ctx, shape, base) for _ in range(3)]
            for it in range(20):
                for k, ty in enumerate(ys):
                    capi.nnt_add(ctx.h, 1.0 + k, tx.h, 1.0, ty.h)         # RAW + WAW chain per y
                capi.nnt_add(ctx.h, 1.0, ys[0].h, 0.5, ys[1].h)            # cross-chain dependency
            results[name] = [t.download() for t in ys]
            st = ctx.stats()
            if name == "streams8_tiles":
                assert st["event_waits"] > 0 and st["tasks"] == 20 * 4 * 12
    for name in ("streams8_tiles", "streams8_ops"):
        for a, b in zip(results[name], results["serial"]):
            np.testing.assert_array_equal(a, b)


def test_graph_capture_replays_task_flow(mods):
    capi, tiled = mods
    r = rng(8)
    A, B = r.standard_normal((96, 80)).astype(np.float32), r.standard_normal((80, 70)).astype(np.float32)
    with tiled.Context(n_streams=4) as ctx:
        tA, tB = T(tiled, ctx, A, (32, 40), "f32"), T(tiled, ctx, B, (40, 35), "f32")
        tC, tG = tiled.TiledTensor(ctx, "f32", (96, 70), (32, 35)), tiled.TiledTensor(ctx, "f32", (96, 70), (32, 35))

        def flow():
            capi.nnt_gemm(ctx.h, 1.0, 0, tA.h, 0, tB.h, 0.0, tC.h, 1, 0, None)
            capi.nnt_gelu(ctx.h, 0, tC.h, tG.h)
            capi.nnt_add(ctx.h, 1.0, tC.h, 1.0, tG.h)
        flow()                                     # builds the plans
        want = tG.download().copy()
        g = C.c_void_p()
        capi.nnt_capture_begin(ctx.h)
        flow()
        capi.nnt_capture_end(ctx.h, C.byref(g))
        for rep in range(3):
            capi.nnt_fill(ctx.h, 0.0, tG.h)        # eager work between replays
            capi.nnt_graph_launch(g)
            np.testing.assert_array_equal(tG.download(), want)
        capi.nnt_graph_destroy(g)
        ref = A.astype(np.float64) @ B.astype(np.float64)
        check(want, ref + D.gelu(ref), "f32", "captured flow")


def test_graph_capture_behind_other_forms_of_the_operation(mods):
    """Calls inside a capture whose scratch or plan comes from an earlier call that ran another form: column sums in two launches behind
    one in a single launch, a layer norm adjoint with more partial rows than the last one, a product of odd sizes tile by tile that
    ran as a whole before."""
    capi, tiled = mods
    r = rng(31)
    with tiled.Context(n_streams=2) as ctx:
        def norm_case(shape, base):
            X, dY = (r.standard_normal(shape).astype(np.float32) for _ in range(2))
            gamma = (1 + 0.1 * r.standard_normal(shape[0])).astype(np.float32)
            _, mean, rstd = D.layernorm_fwd(X, gamma, 0 * gamma, 1e-5)
            ts = [T(tiled, ctx, X, base, "f32"), tiled.TiledTensor.from_numpy(ctx, np.stack([mean, rstd]).astype(np.float32), (2,) + base[1:]),
                  T(tiled, ctx, gamma, base[:1], "f32"), T(tiled, ctx, dY, base, "f32"), tiled.TiledTensor(ctx, "f32", shape, base)]
            ts += [tiled.TiledTensor(ctx, "f32", shape[:1], base[:1]) for _ in range(2)]
            return ts, D.layernorm_bwd(X, gamma, mean, rstd, dY)

        def norm(ts):
            capi.nnt_layernorm_bwd(ctx.h, ts[0].h, ts[1].h, ts[2].h, ts[3].h, None, ts[4].h, ts[5].h, ts[6].h)

        A, B = (r.integers(-32, 33, s).astype(np.float32) / 16 for s in ((1333, 777), (777, 1027)))
        tA, tB, tC = T(tiled, ctx, A, (500, 300), "bf16"), T(tiled, ctx, B, (300, 257), "bf16"), tiled.TiledTensor(ctx, "f32", (1333, 1027), (500, 257))
        product = lambda: capi.nnt_gemm(ctx.h, 1.0, 0, tA.h, 0, tB.h, 0.0, tC.h, 1, 0, None)
        Y = r.standard_normal((256, 1500)).astype(np.float32)
        small, large = T(tiled, ctx, Y[:, :64], (128, 64), "f32"), T(tiled, ctx, Y, (128, 500), "f32")
        db = tiled.TiledTensor(ctx, "f32", (256,), (128,))
        first, _ = norm_case((2050, 400, 1), (2050, 400, 1))
        last, want = norm_case((8191, 300, 1), (8191, 300, 1))      # 2 x 256 partial rows: 4.2 million elements
        # eager: a product as a whole, sums in one launch, a smaller layer norm
        product()
        capi.nnt_bias_grad(ctx.h, small.h, db.h)
        norm(first)
        g = C.c_void_p()
        capi.nnt_capture_begin(ctx.h)
        ctx.set_granularity(1)
        product()
        ctx.set_granularity(0)
        capi.nnt_bias_grad(ctx.h, large.h, db.h)
        norm(last)
        capi.nnt_capture_end(ctx.h, C.byref(g))
        for rep in range(3):
            for t in (tC, db, last[4], last[5], last[6]):
                capi.nnt_fill(ctx.h, 0.0, t.h)
            capi.nnt_graph_launch(g)
            check(tC.download(), A.astype(np.float64) @ B.astype(np.float64), "f32", "captured product")
            check(db.download(), Y.astype(np.float64).sum(1), "f32", "captured bias gradient")
            for t, ref, what in zip(last[4:], want, ("dX", "dgamma", "dbeta")):
                e = relerr(t.download(), ref)
                assert e <= TOL["f32"], (what, e)
        capi.nnt_graph_destroy(g)


def test_graph_keeps_the_scratch_it_was_captured_with(mods):
    """The partial sums of captured tasks lie in the scratch that the context had then.  An eager call that needs more takes a new
    one; the old one stays until the graph goes (seen by the reported bytes), and the graph replays on it."""
    capi, tiled = mods
    r = rng(37)
    with tiled.Context(n_streams=2) as ctx:
        def case(rows, cols):
            X, dY = (r.standard_normal((rows, cols)).astype(np.float32) for _ in range(2))
            gamma = (1 + 0.1 * r.standard_normal(rows)).astype(np.float32)
            _, mean, rstd = D.layernorm_fwd(X, gamma, 0 * gamma, 1e-5)
            base = (rows, cols)
            ts = [T(tiled, ctx, X, base, "f32"), tiled.TiledTensor.from_numpy(ctx, np.stack([mean, rstd]).astype(np.float32), (2, cols)),
                  T(tiled, ctx, gamma, (rows,), "f32"), T(tiled, ctx, dY, base, "f32"), tiled.TiledTensor(ctx, "f32", base, base)]
            ts += [tiled.TiledTensor(ctx, "f32", (rows,), (rows,)) for _ in range(3)]
            return ts, D.layernorm_bwd(X, gamma, mean, rstd, dY) + (dY.astype(np.float64).sum(1),)

        def run(ts):
            capi.nnt_layernorm_bwd(ctx.h, ts[0].h, ts[1].h, ts[2].h, ts[3].h, None, ts[4].h, ts[5].h, ts[6].h)
            capi.nnt_bias_grad(ctx.h, ts[3].h, ts[7].h)

        held = lambda: ctx.stats()["device_workspace_bytes"]
        small, want = case(512, 1100)             # both scratches at their least, 2^20 floats
        large, _ = case(4096, 1100)               # 2 x 256 partial rows: twice that and more
        wide = tiled.TiledTensor.zeros(ctx, (8192, 17000), (8192, 17000), "bf16")      # 133 partial rows of 8192 in the shared scratch
        wide_db = tiled.TiledTensor(ctx, "f32", (8192,), (8192,))
        run(small)
        first = held()
        assert first == (1 + 2) * 4 * 2 ** 20
        g = C.c_void_p()
        capi.nnt_capture_begin(ctx.h)
        run(small)
        capi.nnt_capture_end(ctx.h, C.byref(g))
        run(large)
        capi.nnt_bias_grad(ctx.h, wide.h, wide_db.h)
        both = held()
        assert both == first + 2 * 2 * 256 * 4096 * 4 + 133 * 8192 * 4
        for rep in range(3):
            for t in small[4:]:
                capi.nnt_fill(ctx.h, 0.0, t.h)
            capi.nnt_graph_launch(g)
            run(large)
            for t, ref, what in zip(small[4:], want, ("dX", "dgamma", "dbeta", "db")):
                e = relerr(t.download(), ref)
                assert e <= TOL["f32"], (rep, what, e)
        capi.nnt_graph_destroy(g)
        assert both - held() == first             # what only the graph still held, and not before


def test_products_of_odd_sizes_share_the_space_of_their_copies(mods):
    """The operands that products lay out afresh lie in one space per context, a part per stream as large as the largest of them needs, for as long as
    one of the products lives.  A graph captured before the space grew replays on the space it was captured with."""
    capi, tiled = mods
    r = rng(59)
    up = lambda x, q: (x + q - 1) // q * q
    part = lambda m, n, k: (up(m, 256) + up(n, 256)) * up(k, 64) * 2
    sizes = [(2001, 1333, 2068, 500), (1333, 2068, 2001, 500), (2001, 2068, 1333, 500), (2509, 2523, 3643, 300)]
    with tiled.Context(n_streams=2) as ctx:
        held = lambda: ctx.stats()["device_workspace_bytes"]
        cases = []
        for m, n, k, t in sizes:
            A, B = (r.integers(-32, 33, s).astype(np.float32) / 16 for s in ((m, k), (k, n)))
            cases.append((T(tiled, ctx, A, (t, t), "bf16"), T(tiled, ctx, B, (t, t), "bf16"), tiled.TiledTensor(ctx, "bf16", (m, n), (t, t)),
                          A.astype(np.float64) @ B.astype(np.float64)))
        run = lambda c: capi.nnt_gemm(ctx.h, 1.0, 0, c[0].h, 0, c[1].h, 0.0, c[2].h, 1, 0, None)
        ctx.profile(True)
        for i in range(3):
            run(cases[i])
            assert held() == 2 * max(part(*s[:3]) for s in sizes[:i + 1])
        assert all("_span_" in x for x in ctx.profile_read())
        ctx.profile(False)
        before = held()
        g = C.c_void_p()
        capi.nnt_capture_begin(ctx.h)
        for c in cases[:3]:
            run(c)
        capi.nnt_capture_end(ctx.h, C.byref(g))
        run(cases[3])
        assert held() == before + 2 * part(*sizes[3][:3])
        for _ in range(3):
            for c in cases[:3]:
                capi.nnt_fill(ctx.h, 0.0, c[2].h)
            capi.nnt_graph_launch(g)
            run(cases[3])
            for c in cases:
                check(c[2].download(), c[3], "bf16", "shared space")
        capi.nnt_graph_destroy(g)
        assert held() == 2 * part(*sizes[3][:3])
        for c in cases:
            run(c)
        for c in cases:
            check(c[2].download(), c[3], "bf16", "shared space, grown")
        for c in cases[1:]:
            for x in c[:3]:
                x.close()
        assert held() == 2 * part(*sizes[3][:3])
        for x in cases[0][:3]:
            x.close()
        assert held() == 0


@pytest.mark.parametrize("n_streams", [1, 4])
def test_per_task_timing_records(mods, n_streams):
    """nnt_profile_*: every task is bracketed by timing events; the records come back aggregated per
    operation label."""
    capi, tiled = mods
    r = rng(21)
    X = r.standard_normal((256, 64, 2)).astype(np.float32)
    with tiled.Context(n_streams=n_streams) as ctx:
        tX = T(tiled, ctx, X, (128, 32, 2), "f32")
        tY = T(tiled, ctx, X, (128, 32, 2), "f32")
        tG = tiled.TiledTensor(ctx, "f32", X.shape, (128, 32, 2))
        ctx.profile(True)
        for _ in range(3):
            capi.nnt_add(ctx.h, 1.0, tX.h, 1.0, tY.h)
        capi.nnt_gelu(ctx.h, capi.NNT_GELU_TANH, tY.h, tG.h)
        ctx.wait()
        capi.nnt_add(ctx.h, 1.0, tX.h, 1.0, tY.h)
        rec = ctx.profile_read()
        ctx.profile(False)
        assert set(rec) == {"add", "gelu"}
        assert rec["add"]["tasks"] == 4 and rec["add"]["launches"] == 4 and rec["gelu"]["tasks"] == 1
        assert all(0.0 < e["ms"] < 50.0 for e in rec.values())
        assert rec["add"]["unit"] == "bytes" and rec["add"]["work"] == 4 * 3 * X.size * 4
        check(tY.download(), 5.0 * X, "f32", "sum")
        # a second round reuses the events of the first
        ctx.profile(True)
        capi.nnt_gelu(ctx.h, capi.NNT_GELU_TANH, tY.h, tG.h)
        rec = ctx.profile_read()
        ctx.profile(False)
        assert set(rec) == {"gelu"} and rec["gelu"]["tasks"] == 1 and rec["gelu"]["ms"] > 0.0


# N_d, N_e, N_s, N_b, tile: few macro-tiles and a long contraction (k-slices), tiles that end inside a macro-tile, token
# counts that are no multiple of a k-step or of a vector, one macro-tile of each shape, and enough of them for the largest
RAGGED_LINEAR = [(128, 4096, 20, 3, 1024), (64, 64, 7, 1, 64), (200, 132, 84, 5, 128), (96, 48, 333, 3, 40), (1100, 260, 333, 3, 512),
                 (2052, 36, 513, 4, 4096), (2048, 2048, 129, 8, 1024), (130, 70, 77, 2, 50)]


@pytest.mark.parametrize("dtype", ["f32", "bf16"])
@pytest.mark.parametrize("case", RAGGED_LINEAR, ids=lambda c: "x".join(map(str, c)))
def test_linear_layers_of_any_size(mods, case, dtype):
    """A linear layer's three products on sizes where the plan changes shape (macro-tiles, k-slices, direct-load kernels and
    their ragged forms, register-staged ones) against the oracle; the tolerances are those of the storage types."""
    capi, tiled = mods
    N_d, N_e, N_s, N_b, t = case
    r = rng(sum(case))
    W, X = quant(r.standard_normal((N_d, N_e)) * 0.05, dtype), quant(r.standard_normal((N_e, N_s, N_b)), dtype)
    b, dY = r.standard_normal(N_d).astype(np.float32), quant(r.standard_normal((N_d, N_s, N_b)), dtype)
    with tiled.Context(n_streams=2) as ctx:
        tW, tX, tdY = T(tiled, ctx, W, (t, t), dtype), T(tiled, ctx, X, (t, t, N_b), dtype), T(tiled, ctx, dY, (t, t, N_b), dtype)
        tb = T(tiled, ctx, b, (t,), "f32")
        tY, tdX = tiled.TiledTensor(ctx, dtype, dY.shape, (t, t, N_b)), tiled.TiledTensor(ctx, dtype, X.shape, (t, t, N_b))
        tdW = tiled.TiledTensor(ctx, "f32", W.shape, (t, t))
        capi.nnt_gemm(ctx.h, 1.0, 0, tW.h, 0, tX.h, 0.0, tY.h, 1, 0, tb.h)
        capi.nnt_gemm(ctx.h, 1.0, 1, tW.h, 0, tdY.h, 0.0, tdX.h, 1, 0, None)
        capi.nnt_gemm(ctx.h, 1.0, 0, tdY.h, 1, tX.h, 0.0, tdW.h, 2, 0, None)
        check(tY.download(), D.linear_fwd(W, X, b), dtype, "linear fwd")
        dXr, dWr, _ = D.linear_bwd(W, X, dY)
        check(tdX.download(), dXr, dtype, "linear dX")
        check(tdW.download(), dWr, "f32", "linear dW")


@pytest.mark.parametrize("opA,opB", [(0, 0), (0, 1), (1, 0), (1, 1)])
@pytest.mark.parametrize("m,n,k", [(128, 231, 6514), (126, 77, 3001), (500, 300, 2050), (1030, 1027, 1101), (128, 384, 6528)])
def test_long_contractions_of_odd_extents(mods, m, n, k, opA, opB):
    """fp32 products whose contraction is several times the 256 after which the partial sums leave the matrix accumulators, on
    operands that only the register-staged kernels take (the last: the direct-load ones): few macro-tiles whose slices are
    longer than that, and many without slices.  In the 2-norm: a chain of 256 additions in random order is off by about
    0.29 * 2^-24 * sqrt(256 / 2) of its sum, 2e-7, and so are the k / 256 chains together; 2e-6 leaves room for both roundings of
    the slice sums and for chains twice as long.  One wrong register of the sixteen of a block would be 1e-2."""
    capi, tiled = mods
    r = rng(m + n + k)
    A = r.standard_normal((m, k) if opA == 0 else (k, m)).astype(np.float32)
    B = r.standard_normal((k, n) if opB == 0 else (n, k)).astype(np.float32)
    ref = (A if opA == 0 else A.T).astype(np.float64) @ (B if opB == 0 else B.T).astype(np.float64)
    with tiled.Context(n_streams=2) as ctx:
        tA, tB = T(tiled, ctx, A, A.shape, "f32"), T(tiled, ctx, B, B.shape, "f32")
        tC = tiled.TiledTensor(ctx, "f32", (m, n), (m, n))
        capi.nnt_gemm(ctx.h, 1.0, opA, tA.h, opB, tB.h, 0.0, tC.h, 1, 0, None)
        got = tC.download().astype(np.float64)
    e = np.linalg.norm(got - ref) / np.linalg.norm(ref)
    assert e <= 2e-6, e


# head size, positions, tile, batch members: more than 128 rows on ragged tiles (whole vectors, and tiles that are none), and
# products of which only the tiles of whole vectors qualify for the direct-load kernels, few enough for one launch and too many
RAGGED_BATCHED = [(160, 264, 136, 3), (192, 330, 300, 2), (64, 261, 128, 8), (128, 261, 128, 4), (64, 1301, 128, 24)]


@pytest.mark.parametrize("gran", GRANS)
@pytest.mark.parametrize("dtype", ["f32", "bf16"])
@pytest.mark.parametrize("h,S,t,bat", RAGGED_BATCHED, ids=lambda c: str(c))
def test_batched_products_on_ragged_tiles(mods, h, S, t, bat, dtype, gran):
    """The attention layer's products with batch axes (scores K^T Q, V P, and the adjoint's Q P^T) where plans choose between
    shapes and between one launch and two, against the oracle's contraction."""
    capi, tiled = mods
    r = rng(h + S)
    Q, K, P = (quant(r.standard_normal(s), dtype) for s in ((h, S, bat), (h, S, bat), (S, S, bat)))
    with tiled.Context(n_streams=2, granularity=gran) as ctx:
        tQ, tK, tP = T(tiled, ctx, Q, (h, t, bat), dtype), T(tiled, ctx, K, (h, t, bat), dtype), T(tiled, ctx, P, (t, t, bat), dtype)
        tS, tO, tR = (tiled.TiledTensor(ctx, dtype, s, b) for s, b in (((S, S, bat), (t, t, bat)), ((h, S, bat), (h, t, bat)), ((h, S, bat), (h, t, bat))))
        capi.nnt_gemm(ctx.h, 0.125, 1, tK.h, 0, tQ.h, 0.0, tS.h, 1, 1, None)
        capi.nnt_gemm(ctx.h, 1.0, 0, tK.h, 0, tP.h, 0.0, tO.h, 1, 1, None)
        capi.nnt_gemm(ctx.h, 1.0, 0, tQ.h, 1, tP.h, 0.0, tR.h, 1, 1, None)
        check(tS.download(), D.contract(0.125, "T", K, "N", Q, 0.0, None, 1, 1), dtype, "K^T Q")
        check(tO.download(), D.contract(1.0, "N", K, "N", P, 0.0, None, 1, 1), dtype, "V P")
        check(tR.download(), D.contract(1.0, "N", Q, "T", P, 0.0, None, 1, 1), dtype, "Q P^T")
