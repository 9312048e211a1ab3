"""The work that a user of this framework has it do, as cases that can be timed and compared: training steps of whole
GPT-2 blocks and of a language model made of them, and the single layers that such a program calls by themselves
(linear layers, the MLP, fused attention, layer normalisation, the tied head with its loss).

A case is a dict of plain values.  `listed()` gives the fixed ones, `draw(rng)` one more of the same ranges, `prepare`
what a program holds before the call, `run` one pass through the public entry points, `work` what a pass cannot do
without, `tolerance` how far two correct implementations may differ, `exact` the same outputs in 64 bits by plain torch.

Arrays are handled with their axes reversed (first axis of the tiled tensor last, contiguous): an activation
[N_e, N_s, N_b] is a torch tensor of shape (N_b, N_s, N_e).  Outputs are whole tensors in the framework's layout, the
tiles one after the other, each padded with zeros to 256 bytes.
"""
from __future__ import annotations

import itertools
import math

import torch

KINDS = ("block", "linear", "mlp", "attention", "layernorm", "head", "model")
ADAM = dict(lr=1e-3, beta1=0.9, beta2=0.999, eps=1e-8, weight_decay=0.0)
ADAM_STEP = 100                     # a step in the middle of a training run: the moments are not zero
LN_EPS = 1e-5


# ------------------------------------------------------------------------------------------------- the cases
def listed():
    return [
        # the smallest training step (64 tokens, 2 sequences, tiles of 32): some seventy launches of next to no work
        _block("block_tiny_f32", "f32", 2, 64, 64, 2, 32, False, True),
        # one GPT-2-small block in fp32, the configuration that the benchmark quotes; scores stored, as in the paper
        _block("block_small_f32", "f32", 12, 64, 1024, 8, 256, False, False),
        # one GPT-2-medium block in bf16 with the fused attention and the optimiser step: ordinary mixed-precision training
        _block("block_medium_bf16", "bf16", 16, 64, 1024, 16, 512, True, True),
        # one GPT-2-XL block in bf16: 25 heads, tiles of 400 that leave ragged edges everywhere, scores stored
        _block("block_xl_ragged_bf16", "bf16", 25, 64, 1024, 8, 400, False, False),
        # the MLP of a 50B-class block (8192 wide), forward and backward: the largest products there are
        dict(name="mlp_wide_bf16", kind="mlp", dtype="bf16", N_e=8192, N_m=32768, N_s=1024, N_b=4, tile=1024),
        # linear layers of odd sizes (an adapter or an odd vocabulary slice), where no extent is a multiple of a vector
        dict(name="linear_odd_f32", kind="linear", dtype="f32", N_e=777, N_d=1111, N_s=333, N_b=3, tile=300),
        dict(name="linear_odd_bf16", kind="linear", dtype="bf16", N_e=1333, N_d=2001, N_s=517, N_b=4, tile=500),
        # fused attention, forward and backward: long sequences with head size 128 in bf16 ...
        dict(name="attention_long_bf16", kind="attention", dtype="bf16", h=128, N_h=16, N_s=4096, N_b=2, tile=1024, tile_s=1024, causal=True),
        # ... and short ragged ones in fp32 with the tiles of GPT-2 small
        dict(name="attention_ragged_f32", kind="attention", dtype="f32", h=64, N_h=12, N_s=1000, N_b=3, tile=256, tile_s=256, causal=True),
        # layer normalisation of long tokens with the residual gradient: bound by memory
        dict(name="layernorm_wide_bf16", kind="layernorm", dtype="bf16", N_e=8192, N_s=1024, N_b=4, tile=1024),
        # the tied head and its loss over GPT-2's (padded) vocabulary: logits, loss, both gradients
        dict(name="head_loss_bf16", kind="head", dtype="bf16", N_e=1024, N_v=50304, N_s=1024, N_b=4, tile=512, tile_v=8192),
        # a whole training iteration of a small language model: lookup, four blocks, final norm, head, loss, backward, Adam
        dict(name="model_f32", kind="model", dtype="f32", N_h=12, h=64, N_s=1024, N_b=2, tile=256, blocks=4, N_v=50304, tile_v=8192, fused=True),
    ]


def _block(name, dtype, N_h, h, N_s, N_b, tile, fused, adam):
    return dict(name=name, kind="block", dtype=dtype, N_h=N_h, h=h, N_s=N_s, N_b=N_b, tile=tile, fused=fused, adam=adam)


#: the dearest listed case: no drawn one costs more
MOST_FLOPS, MOST_BYTES = 1.3e13, 8e9


def draw(rng):
    while True:
        c = _draw(rng)
        w = work(c)
        if w["flops"] <= MOST_FLOPS and w["bytes"] <= MOST_BYTES:
            return c


def _log(rng, lo, hi):
    """An integer between lo and hi, spread evenly over its logarithm: round sizes and odd ones alike."""
    n = int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))
    step = rng.choice((1, 8, 64))
    return max(lo, min(hi, (n + step // 2) // step * step))


def _draw(rng):
    kind, dtype = rng.choice(KINDS), rng.choice(("f32", "bf16"))
    tokens = dict(N_s=_log(rng, 64, 1024), N_b=rng.randint(1, 8))
    tile = rng.choice((256, 300, 400, 512, 1024))
    if kind == "block":
        h = rng.choice((64, 64, 128))
        return dict(kind=kind, dtype=dtype, N_h=_log(rng, 2, 24), h=h, tile=rng.choice((64, 128, 256, 400, 512)), fused=rng.random() < 0.5,
                    adam=rng.random() < 0.5, **tokens)
    if kind == "linear":
        return dict(kind=kind, dtype=dtype, N_e=_log(rng, 128, 8192), N_d=_log(rng, 128, 8192), tile=tile, **tokens)
    if kind == "mlp":
        e = _log(rng, 128, 8192 if dtype == "bf16" else 2048)
        return dict(kind=kind, dtype=dtype, N_e=e, N_m=4 * e, tile=tile, **tokens)
    if kind == "attention":
        h, N_h = rng.choice((64, 128)), _log(rng, 1, 32)
        per = rng.choice([n for n in (1, 2, 4, 8) if N_h % n == 0])            # heads in a row tile
        return dict(kind=kind, dtype=dtype, h=h, N_h=N_h, N_s=_log(rng, 64, 4096), N_b=rng.randint(1, 4), tile=per * h,
                    tile_s=rng.choice((128, 256, 300, 512, 1024)), causal=rng.random() < 0.75)
    if kind == "layernorm":
        return dict(kind=kind, dtype=dtype, N_e=_log(rng, 128, 8192), tile=tile, **tokens)
    if kind == "head":
        return dict(kind=kind, dtype=dtype, N_e=_log(rng, 128, 2048), N_v=_log(rng, 1000, 50304), tile=tile, tile_v=rng.choice((1024, 4096, 8192)), **tokens)
    return dict(kind=kind, dtype="f32", N_h=_log(rng, 2, 12), h=64, tile=rng.choice((128, 256)), blocks=rng.randint(1, 4), N_v=_log(rng, 1000, 50304),
                tile_v=rng.choice((4096, 8192)), fused=rng.random() < 0.75, **tokens)


# ------------------------------------------------------------------------------------------------- inputs
class _Inputs:
    """The inputs of a case, drawn one after the other from the seed: the same for prepare() and exact()."""

    def __init__(self, seed, dtype):
        self.g = torch.Generator(device="cuda")
        self.g.manual_seed(int(seed) + 250413236)
        self.dtype = dtype

    def normal(self, *shape, std=1.0, mean=0.0):
        return torch.randn(*shape, generator=self.g, device="cuda", dtype=torch.float32).mul_(std).add_(mean)

    def act(self, *shape, std=1.0):
        a = self.normal(*shape, std=std)
        return a.bfloat16() if self.dtype == "bf16" else a

    def second_moment(self, *shape, std):
        return torch.rand(*shape, generator=self.g, device="cuda", dtype=torch.float32).add_(0.5).mul_(std * std)

    def ints(self, n, *shape):
        return torch.randint(0, n, shape, generator=self.g, device="cuda", dtype=torch.int32)


def _low(a, dtype):
    """A fp32 parameter as the products read it."""
    return a.bfloat16() if dtype == "bf16" else a


def _weights_of_block(i, e, m):
    """The twelve parameters (reversed axes: W [rows, cols] as (cols, rows))."""
    return dict(W_qkv=i.normal(e, 3 * e, std=0.02), W_o=i.normal(e, e, std=0.02), W_1=i.normal(e, m, std=0.02), W_2=i.normal(m, e, std=0.02),
                b_qkv=i.normal(3 * e, std=0.02), b_o=i.normal(e, std=0.02), b_1=i.normal(m, std=0.02), b_2=i.normal(e, std=0.02),
                gamma1=i.normal(e, std=0.02, mean=1.0), beta1=i.normal(e, std=0.02),
                gamma2=i.normal(e, std=0.02, mean=1.0), beta2=i.normal(e, std=0.02))


def _moments(i, params, std):
    return ({k: i.normal(*p.shape, std=0.3 * std) for k, p in params.items()},
            {k: i.second_moment(*p.shape, std=std) for k, p in params.items()})


def _inputs(c, seed):
    i = _Inputs(seed, c["dtype"])
    kind, S, B = c["kind"], c["N_s"], c["N_b"]
    d = {}
    if kind == "block":
        e = c["N_h"] * c["h"]
        d.update(params=_weights_of_block(i, e, 4 * e), X=i.act(B, S, e), dOut=i.act(B, S, e))
        if c["adam"]:
            d["m"], d["v"] = _moments(i, d["params"], 0.5 * math.sqrt(S * B))
    elif kind == "linear":
        e, n = c["N_e"], c["N_d"]
        d.update(W=i.act(e, n, std=0.02), b=i.normal(n, std=0.02), X=i.act(B, S, e), dY=i.act(B, S, n))
    elif kind == "mlp":
        e, m = c["N_e"], c["N_m"]
        d.update(W_1=i.act(e, m, std=0.02), W_2=i.act(m, e, std=0.02), b_1=i.normal(m, std=0.02), b_2=i.normal(e, std=0.02),
                 X=i.act(B, S, e), R=i.act(B, S, e), dY=i.act(B, S, e))
    elif kind == "attention":
        e = c["N_h"] * c["h"]
        d.update(QKV=i.act(B, S, 3 * e), dB=i.act(B, S, e))
    elif kind == "layernorm":
        e = c["N_e"]
        d.update(X=i.act(B, S, e), gamma=i.normal(e, std=0.02, mean=1.0), beta=i.normal(e, std=0.02), dY=i.act(B, S, e), dR=i.act(B, S, e))
    elif kind == "head":
        d.update(W=i.act(c["N_v"], c["N_e"], std=0.02), X=i.act(B, S, c["N_e"]), labels=i.ints(c["N_v"], B, S))
    else:
        e = c["N_h"] * c["h"]
        d["blocks"] = []
        for _ in range(c["blocks"]):
            p = _weights_of_block(i, e, 4 * e)
            d["blocks"].append((p,) + _moments(i, p, 1.0))
        top = dict(wte=i.normal(c["N_v"], e, std=0.02), wpe=i.normal(S, e, std=0.01), gamma=i.normal(e, std=0.02, mean=1.0), beta=i.normal(e, std=0.02))
        d["top"] = (top,) + _moments(i, top, 1.0)
        d.update(tokens=i.ints(c["N_v"], B, S), labels=i.ints(c["N_v"], B, S))
    return d


# ------------------------------------------------------------------------------------------------- the program's state
_ctx = None


def _context():
    """One executor for the whole program, with the benchmark's two streams."""
    global _ctx
    if _ctx is None:
        from paper_2504_13236_amd import tiled
        _ctx = tiled.Context(n_streams=2)
    return _ctx


class _State:
    """Tensors, handles and outputs of one case; given back when the program drops it."""

    def __init__(self, case):
        self.case, self.ctx, self.tensors, self.handles = case, _context(), [], []

    def tensor(self, dtype, shape, base, a=None):
        """A tiled tensor (axes in the framework's order), zero or filled with `a` (axes reversed)."""
        from paper_2504_13236_amd import tiled
        t = tiled.TiledTensor(self.ctx, dtype, shape, base)
        self.tensors.append(t)
        _fill(t, a)
        return t

    def __del__(self):
        try:
            for h in reversed(self.handles):
                h.close()
            for t in self.tensors:
                t.close()
        except Exception:       # the interpreter is ending
            pass


def _fill(t, a=None):
    t.buf.zero_()
    if a is not None:
        for k, idx in enumerate(t.tile_index):
            t.tile_view(k).copy_(a[tuple(reversed(t.slices(idx)))].reshape(-1))


def _whole(t):
    return t.buf.view(torch.float32 if t.esize == 4 else torch.bfloat16)


def _tiles_of_block(c):
    e = c["N_h"] * c["h"]
    t = c["tile"]
    return dict(e=min(e, t), m=min(4 * e, t), s=min(c["N_s"], t), b=c["N_b"], j=c["N_h"], i=c["h"] if c["fused"] else min(c["h"], t))


def _make_block(s, c, params, moments, adam):
    from paper_2504_13236_amd import tiled
    e = c["N_h"] * c["h"]
    blk = tiled.Gpt2Block(s.ctx, e, c["N_h"], 4 * e, c["N_s"], c["N_b"], _tiles_of_block(c), dtype=c["dtype"], eps=LN_EPS, adam=adam, fused_attention=c["fused"])
    s.handles.append(blk)
    s.tensors += [t for t in blk.slots if t is not None]
    for k, a in params.items():
        _fill(blk.param(k), a)
        if adam:
            _fill(blk.moment(k, "m"), moments[0][k])
            _fill(blk.moment(k, "v"), moments[1][k])
    return blk


def prepare(case, seed):
    from paper_2504_13236_amd import capi, tiled
    c, d = case, _inputs(case, seed)
    s = _State(case)
    kind, S, B = c["kind"], c["N_s"], c["N_b"]
    ts = min(S, c.get("tile_s", c["tile"]))
    dt, t = c["dtype"], c["tile"]

    def act(n, a=None, base=t):
        return s.tensor(dt, (n, S, B), (min(n, base), ts, B), a)

    if kind == "block":
        e = c["N_h"] * c["h"]
        s.blk = _make_block(s, c, d["params"], (d.get("m"), d.get("v")), c["adam"])
        torch.cuda.synchronize()
        capi.nnt_gpt2_block_sync_lowp(s.blk.h)
        s.X, s.dOut, s.Out, s.dX = act(e, d["X"]), act(e, d["dOut"]), act(e), act(e)
        s.out = dict(Out=_whole(s.Out), dX=_whole(s.dX))
        for k in d["params"]:
            s.out["d" + k] = _whole(s.blk.grad(k))
            if c["adam"]:
                s.out["new_" + k], s.out["m_" + k], s.out["v_" + k] = _whole(s.blk.param(k)), _whole(s.blk.moment(k, "m")), _whole(s.blk.moment(k, "v"))
    elif kind == "linear":
        e, n = c["N_e"], c["N_d"]
        tw = (min(n, t), min(e, t))
        s.W, s.b = s.tensor(dt, (n, e), tw, d["W"]), s.tensor("f32", (n,), tw[:1], d["b"])
        s.X, s.dY, s.Y, s.dX = act(e, d["X"]), act(n, d["dY"]), act(n), act(e)
        s.dW, s.db = s.tensor("f32", (n, e), tw), s.tensor("f32", (n,), tw[:1])
        s.out = dict(Y=_whole(s.Y), dX=_whole(s.dX), dW=_whole(s.dW), db=_whole(s.db))
    elif kind == "mlp":
        e, m = c["N_e"], c["N_m"]
        t1, t2 = (min(m, t), min(e, t)), (min(e, t), min(m, t))
        s.W1, s.W2 = s.tensor(dt, (m, e), t1, d["W_1"]), s.tensor(dt, (e, m), t2, d["W_2"])
        s.b1, s.b2 = s.tensor("f32", (m,), t1[:1], d["b_1"]), s.tensor("f32", (e,), t2[:1], d["b_2"])
        s.X, s.R, s.dY = act(e, d["X"]), act(e, d["R"]), act(e, d["dY"])
        s.H, s.G, s.dH, s.Y, s.dX = act(m), act(m), act(m), act(e), act(e)
        s.dW1, s.dW2 = s.tensor("f32", (m, e), t1), s.tensor("f32", (e, m), t2)
        s.db1, s.db2 = s.tensor("f32", (m,), t1[:1]), s.tensor("f32", (e,), t2[:1])
        s.out = dict(Y=_whole(s.Y), dX=_whole(s.dX), dW_1=_whole(s.dW1), dW_2=_whole(s.dW2), db_1=_whole(s.db1), db_2=_whole(s.db2))
    elif kind == "attention":
        e = c["N_h"] * c["h"]
        s.QKV, s.dB, s.B, s.dQKV = act(3 * e, d["QKV"]), act(e, d["dB"]), act(e), act(3 * e)
        s.stats = s.tensor("f32", (2, S, B, c["N_h"]), (2, ts, B, c["N_h"]))
        s.out = dict(B=_whole(s.B), dQKV=_whole(s.dQKV), stats=_whole(s.stats))
    elif kind == "layernorm":
        e = c["N_e"]
        te = (min(e, t),)
        s.X, s.dY, s.dR, s.Y, s.dX = act(e, d["X"]), act(e, d["dY"]), act(e, d["dR"]), act(e), act(e)
        s.gamma, s.beta, s.dgamma, s.dbeta = (s.tensor("f32", (e,), te, d.get(k)) for k in ("gamma", "beta", "-", "-"))
        s.stats = s.tensor("f32", (2, S, B), (2, ts, B))
        s.out = dict(Y=_whole(s.Y), dX=_whole(s.dX), dgamma=_whole(s.dgamma), dbeta=_whole(s.dbeta))
    elif kind == "head":
        e, v = c["N_e"], c["N_v"]
        tw = (min(e, t), min(v, c["tile_v"]))
        s.W, s.X, s.dX, s.dW = s.tensor(dt, (e, v), tw, d["W"]), act(e, d["X"]), act(e), s.tensor("f32", (e, v), tw)
        s.L, s.stats = act(v, base=c["tile_v"]), s.tensor("f32", (2, S, B), (2, ts, B))
        s.labels = d["labels"]
        s.losses, s.loss = torch.zeros(S * B, device="cuda"), torch.zeros(1, device="cuda")
        s.out = dict(losses=s.losses, loss=s.loss, dL=_whole(s.L), dX=_whole(s.dX), dW=_whole(s.dW))
    else:
        blks = [_make_block(s, c, p, (m, v), True) for p, m, v in d["blocks"]]
        s.model = tiled.Gpt2Model(s.ctx, blks, c["N_v"], c["tile_v"])
        s.handles.append(s.model)
        s.tensors += [x for x in s.model.slots if x is not None] + s.model.stack.acts + s.model.stack.dacts
        for x in s.model.stack.acts + s.model.stack.dacts + [s.model.logits]:
            _fill(x)
        top, m, v = d["top"]
        s.out = dict(loss=s.model.loss, col_loss=s.model.col_loss, dlogits=_whole(s.model.logits), last=_whole(s.model.stack.acts[-1]))
        for k in top:
            g = getattr(s.model, k)
            _fill(g["p"], top[k])
            _fill(g["m"], m[k])
            _fill(g["v"], v[k])
            s.out["d" + k], s.out["new_" + k] = _whole(g["g"]), _whole(g["p"])
        for n, b in enumerate(blks):
            for k in ("W_qkv", "W_o", "W_1", "W_2", "b_1", "gamma1"):
                s.out["d%s_%d" % (k, n)], s.out["new_%s_%d" % (k, n)] = _whole(b.grad(k)), _whole(b.param(k))
        torch.cuda.synchronize()
        capi.nnt_gpt2_model_sync_lowp(s.model.h)
        s.model.tokens.copy_(d["tokens"].reshape(-1))
        s.model.labels.copy_(d["labels"].reshape(-1))
    torch.cuda.synchronize()
    s.ctx.wait()
    return s


def run(s):
    from paper_2504_13236_amd import capi
    c, h = s.case, s.ctx.h
    kind = c["kind"]
    N, T = capi.NNT_OP_N, capi.NNT_OP_T
    if kind == "block":
        s.blk.forward(s.X, s.Out)
        s.blk.backward(s.dOut, s.dX)
        if c["adam"]:
            s.blk.adam(ADAM_STEP, **ADAM)
    elif kind == "linear":
        capi.nnt_gemm(h, 1.0, N, s.W.h, N, s.X.h, 0.0, s.Y.h, 1, 0, s.b.h)
        capi.nnt_gemm(h, 1.0, N, s.dY.h, T, s.X.h, 0.0, s.dW.h, 2, 0, None)
        capi.nnt_bias_grad(h, s.dY.h, s.db.h)
        capi.nnt_gemm(h, 1.0, T, s.W.h, N, s.dY.h, 0.0, s.dX.h, 1, 0, None)
    elif kind == "mlp":
        g = capi.NNT_GELU_TANH
        capi.nnt_gemm_gelu(h, 1.0, N, s.W1.h, N, s.X.h, s.H.h, 1, s.b1.h, g, s.G.h)
        capi.nnt_gemm_res(h, 1.0, N, s.W2.h, N, s.G.h, 1.0, s.Y.h, 1, 0, s.b2.h, s.R.h)
        capi.nnt_gemm(h, 1.0, N, s.dY.h, T, s.G.h, 0.0, s.dW2.h, 2, 0, None)
        capi.nnt_bias_grad(h, s.dY.h, s.db2.h)
        capi.nnt_gemm_gelu_bwd(h, 1.0, T, s.W2.h, N, s.dY.h, s.dH.h, 1, g, s.H.h)
        capi.nnt_gemm(h, 1.0, N, s.dH.h, T, s.X.h, 0.0, s.dW1.h, 2, 0, None)
        capi.nnt_bias_grad(h, s.dH.h, s.db1.h)
        capi.nnt_gemm(h, 1.0, T, s.W1.h, N, s.dH.h, 0.0, s.dX.h, 1, 0, None)
    elif kind == "attention":
        scale, causal = 1.0 / math.sqrt(c["h"]), 1 if c["causal"] else 0
        capi.nnt_attention_fwd_heads(h, s.QKV.h, scale, causal, s.B.h, s.stats.h, c["N_h"])
        capi.nnt_attention_bwd_heads(h, s.QKV.h, s.B.h, s.stats.h, s.dB.h, scale, causal, s.dQKV.h, c["N_h"])
    elif kind == "layernorm":
        capi.nnt_layernorm_fwd(h, s.X.h, s.gamma.h, s.beta.h, LN_EPS, s.Y.h, s.stats.h)
        capi.nnt_layernorm_bwd(h, s.X.h, s.stats.h, s.gamma.h, s.dY.h, s.dR.h, s.dX.h, s.dgamma.h, s.dbeta.h)
    elif kind == "head":
        capi.nnt_gemm(h, 1.0, T, s.W.h, N, s.X.h, 0.0, s.L.h, 1, 0, None)
        capi.nnt_cross_entropy(h, s.L.h, s.labels.data_ptr(), s.stats.h, s.losses.data_ptr(), s.loss.data_ptr())
        capi.nnt_gemm(h, 1.0, N, s.W.h, N, s.L.h, 0.0, s.dX.h, 1, 0, None)
        capi.nnt_gemm(h, 1.0, N, s.X.h, T, s.L.h, 0.0, s.dW.h, 2, 0, None)
    else:
        s.model.forward()
        s.model.backward()
        s.model.adam(ADAM_STEP, **ADAM)
    return s.out


# ------------------------------------------------------------------------------------------------- what a pass needs
def _pairs(S, causal):
    return S * (S + 1) // 2 if causal else S * S


def _block_work(c, w, adam):
    """(flops, bytes of the parameters and what happens to them) of one block's forward and backward pass."""
    e, T = c["N_h"] * c["h"], c["N_s"] * c["N_b"]
    flops = 3.0 * (2.0 * T * 12 * e * e + 4.0 * _pairs(c["N_s"], True) * e * c["N_b"])
    n = 12 * e * e + 13 * e
    # the weights as the products read them and the gradients; Adam reads p, m, v and writes them (and the bf16 copies)
    return flops, n * (w + 4) + (n * 24 + (12 * e * e * 2 if w == 2 else 0) if adam else 0)


def work(case):
    c = case
    w = 2 if c["dtype"] == "bf16" else 4
    kind, S, B = c["kind"], c["N_s"], c["N_b"]
    T = S * B
    if kind == "block":
        flops, byts = _block_work(c, w, c["adam"])
        return dict(flops=flops, bytes=byts + 4 * T * c["N_h"] * c["h"] * w)
    if kind == "linear":
        e, n = c["N_e"], c["N_d"]
        return dict(flops=6.0 * T * e * n, bytes=e * n * (w + 4) + 8 * n + 2 * T * (e + n) * w)
    if kind == "mlp":
        e, m = c["N_e"], c["N_m"]
        return dict(flops=12.0 * T * e * m, bytes=2 * e * m * (w + 4) + 8 * (e + m) + 5 * T * e * w)
    if kind == "attention":
        e = c["N_h"] * c["h"]
        return dict(flops=12.0 * _pairs(S, c["causal"]) * e * B, bytes=8 * T * e * w + 8 * T * c["N_h"])
    if kind == "layernorm":
        return dict(flops=20.0 * T * c["N_e"], bytes=5 * T * c["N_e"] * w + 16 * c["N_e"])
    if kind == "head":
        e, v = c["N_e"], c["N_v"]
        return dict(flops=6.0 * T * e * v, bytes=e * v * (w + 4) + 2 * T * e * w + T * v * w + 8 * T)
    flops, byts = _block_work(c, w, True)
    e, v = c["N_h"] * c["h"], c["N_v"]
    return dict(flops=c["blocks"] * flops + 6.0 * T * e * v, bytes=c["blocks"] * byts + 32 * e * (v + S) + T * v * w + 12 * T)


def tolerance(case):
    # about four times the distance from the 64-bit results measured at the listed cases and some drawn ones: 32-bit sums 0.2 to
    # 1.7e-6; bf16 layers 1.7 to 2.9e-3 (one or two roundings of every result), a whole bf16 block up to 5.4e-3
    if case["dtype"] == "f32":
        return {"rel": 1e-5, "max": 4e-4}
    return {"rel": 2e-2, "max": 0.5} if case["kind"] == "block" else {"rel": 1e-2, "max": 0.4}


# ------------------------------------------------------------------------------------------------- the same in 64 bits
def _pack(a, base, esize):
    """`a` (axes reversed) as the framework lays it out: tile after tile, first axis fastest, padded to 256 bytes."""
    shape = tuple(reversed(a.shape))
    grid = [-(-n // b) for n, b in zip(shape, base)]
    step, parts = 256 // esize, []
    for idx in itertools.product(*[range(g) for g in reversed(grid)]):
        cut = tuple(slice(i * b, min(n, (i + 1) * b)) for i, b, n in zip(idx, reversed(base), a.shape))
        t = a[cut].reshape(-1)
        parts.append(torch.nn.functional.pad(t, (0, -t.numel() % step)))
    return torch.cat(parts)


def _ln(x, gamma, beta):
    mean = x.mean(-1, keepdim=True)
    xc = x - mean
    rstd = 1.0 / torch.sqrt((xc * xc).mean(-1, keepdim=True) + LN_EPS)
    xh = xc * rstd
    return xh * gamma + beta, (xh, rstd)


def _ln_bwd(saved, gamma, dy):
    xh, rstd = saved
    g = dy * gamma
    dx = rstd * (g - g.mean(-1, keepdim=True) - xh * (g * xh).mean(-1, keepdim=True))
    return dx, (dy * xh).sum((0, 1)), dy.sum((0, 1))


_C = math.sqrt(2.0 / math.pi)


def _gelu(x):
    return 0.5 * x * (1.0 + torch.tanh(_C * (x + 0.044715 * x ** 3)))


def _gelu_bwd(x, dy):
    t = torch.tanh(_C * (x + 0.044715 * x ** 3))
    return dy * (0.5 * (1.0 + t) + 0.5 * x * (1.0 - t * t) * _C * (1.0 + 3 * 0.044715 * x * x))


def _linear_bwd(W, X, dY):
    """dX, dW, db for Y = X W + b, W as (in, out)."""
    e, n = W.shape
    return dY @ W.t(), X.reshape(-1, e).t() @ dY.reshape(-1, n), dY.reshape(-1, n).sum(0)


def _heads(x, N_h):
    B, S, e = x.shape
    return x.reshape(B, S, N_h, e // N_h).permute(0, 2, 1, 3)


def _unheads(x):
    B, H, S, h = x.shape
    return x.permute(0, 2, 1, 3).reshape(B, S, H * h)


def _attention(QKV, N_h, causal):
    """B, its statistics and what the adjoint needs; one sequence at a time."""
    e = QKV.shape[-1] // 3
    S = QKV.shape[1]
    sc = 1.0 / math.sqrt(e // N_h)
    hidden = torch.ones(S, S, dtype=torch.bool, device=QKV.device).triu(1) if causal else None
    out, top, den = [], [], []
    for z in QKV.split(1):
        q, k, v = (_heads(p, N_h) for p in z.split(e, -1))
        a = (q @ k.transpose(-1, -2)) * sc
        if causal:
            a.masked_fill_(hidden, -math.inf)
        m = a.amax(-1, keepdim=True)
        a = (a - m).exp_()
        s = a.sum(-1, keepdim=True)
        out.append(_unheads((a / s) @ v))
        top.append(m[..., 0])
        den.append(s[..., 0])
    return torch.cat(out), torch.cat(top), torch.cat(den)


def _attention_bwd(QKV, dB, N_h, causal):
    e = QKV.shape[-1] // 3
    S = QKV.shape[1]
    sc = 1.0 / math.sqrt(e // N_h)
    hidden = torch.ones(S, S, dtype=torch.bool, device=QKV.device).triu(1) if causal else None
    out = []
    for z, d in zip(QKV.split(1), dB.split(1)):
        q, k, v = (_heads(p, N_h) for p in z.split(e, -1))
        d = _heads(d, N_h)
        a = (q @ k.transpose(-1, -2)) * sc
        if causal:
            a.masked_fill_(hidden, -math.inf)
        p = torch.softmax(a, -1)
        dv = p.transpose(-1, -2) @ d
        dp = d @ v.transpose(-1, -2)
        da = p * (dp - (p * dp).sum(-1, keepdim=True)) * sc
        out.append(torch.cat([_unheads(da @ k), _unheads(da.transpose(-1, -2) @ q), _unheads(dv)], -1))
    return torch.cat(out)


def _block_params(params, dtype):
    return {k: (_low(p, dtype) if k.startswith("W") else p).double() for k, p in params.items()}


def _block_forward(p, X, N_h):
    X1, ln1 = _ln(X, p["gamma1"], p["beta1"])
    QKV = X1 @ p["W_qkv"] + p["b_qkv"]
    Bm = _attention(QKV, N_h, True)[0]
    X2 = X + Bm @ p["W_o"] + p["b_o"]
    X3, ln2 = _ln(X2, p["gamma2"], p["beta2"])
    H = X3 @ p["W_1"] + p["b_1"]
    G = _gelu(H)
    return X2 + G @ p["W_2"] + p["b_2"], (X1, ln1, QKV, Bm, X3, ln2, H, G)


def _block_backward(p, saved, dOut, N_h):
    X1, ln1, QKV, Bm, X3, ln2, H, G = saved
    g = {}
    dG, g["W_2"], g["b_2"] = _linear_bwd(p["W_2"], G, dOut)
    dX3, g["W_1"], g["b_1"] = _linear_bwd(p["W_1"], X3, _gelu_bwd(H, dG))
    dX2, g["gamma2"], g["beta2"] = _ln_bwd(ln2, p["gamma2"], dX3)
    dX2 = dX2 + dOut
    dBm, g["W_o"], g["b_o"] = _linear_bwd(p["W_o"], Bm, dX2)
    dX1, g["W_qkv"], g["b_qkv"] = _linear_bwd(p["W_qkv"], X1, _attention_bwd(QKV, dBm, N_h, True))
    dX, g["gamma1"], g["beta1"] = _ln_bwd(ln1, p["gamma1"], dX1)
    return dX + dX2, g


def _adam(p, g, m, v):
    a = ADAM
    m = a["beta1"] * m.double() + (1 - a["beta1"]) * g
    v = a["beta2"] * v.double() + (1 - a["beta2"]) * g * g
    mh, vh = m / (1 - a["beta1"] ** ADAM_STEP), v / (1 - a["beta2"] ** ADAM_STEP)
    return p.double() - a["lr"] * mh / (vh.sqrt() + a["eps"]), m, v


def _loss(L, labels):
    """Per-position losses and dL/dlogits."""
    top = L.amax(-1, keepdim=True)
    p = (L - top).exp_()
    s = p.sum(-1, keepdim=True)
    at = labels.long().unsqueeze(-1)
    losses = -(L.gather(-1, at) - top - s.log())[..., 0]
    p /= s
    p.scatter_add_(-1, at, torch.full(at.shape, -1.0, dtype=p.dtype, device=p.device))
    return losses, p


def exact(case, seed):
    c, d = case, _inputs(case, seed)
    kind, S, B, dt, t = c["kind"], c["N_s"], c["N_b"], c["dtype"], c["tile"]
    w = 2 if dt == "bf16" else 4
    ts = min(S, c.get("tile_s", t))

    def act(a, base=t):
        return _pack(a, (min(a.shape[-1], base), ts, B), w)

    def mat(a, b0=t, b1=t):
        return _pack(a, (min(a.shape[1], b0), min(a.shape[0], b1)), 4)

    def vec(a):
        return _pack(a, (min(a.shape[0], t),), 4)

    def param(k, a):
        """A parameter of a block (or its gradient or moment): the rows of W_qkv are cut like the embedding axis."""
        e = c["N_h"] * c["h"]
        te, tm = min(e, t), min(4 * e, t)
        b0, b1 = dict(W_1=(tm, te), W_2=(te, tm), b_1=(tm, 0)).get(k, (te, te))
        return _pack(a, (b0,) if a.dim() == 1 else (b0, b1), 4)

    if kind == "block":
        p = _block_params(d["params"], dt)
        Out, saved = _block_forward(p, d["X"].double(), c["N_h"])
        dX, g = _block_backward(p, saved, d["dOut"].double(), c["N_h"])
        out = dict(Out=act(Out), dX=act(dX))
        for k in g:
            out["d" + k] = param(k, g[k])
            if c["adam"]:
                q, m, v = _adam(d["params"][k], g[k], d["m"][k], d["v"][k])
                out["new_" + k], out["m_" + k], out["v_" + k] = param(k, q), param(k, m), param(k, v)
        return out
    if kind == "linear":
        W, X, dY = d["W"].double(), d["X"].double(), d["dY"].double()
        dX, dW, db = _linear_bwd(W, X, dY)
        return dict(Y=act(X @ W + d["b"].double()), dX=act(dX), dW=mat(dW), db=vec(db))
    if kind == "mlp":
        W1, W2, X, dY = d["W_1"].double(), d["W_2"].double(), d["X"].double(), d["dY"].double()
        H = X @ W1 + d["b_1"].double()
        G = _gelu(H)
        dG, dW2, db2 = _linear_bwd(W2, G, dY)
        dX, dW1, db1 = _linear_bwd(W1, X, _gelu_bwd(H, dG))
        return dict(Y=act(G @ W2 + d["b_2"].double() + d["R"].double()), dX=act(dX), dW_1=mat(dW1), dW_2=mat(dW2), db_1=vec(db1), db_2=vec(db2))
    if kind == "attention":
        QKV, N_h = d["QKV"].double(), c["N_h"]
        out, top, den = _attention(QKV, N_h, c["causal"])
        dQKV = _attention_bwd(QKV, d["dB"].double(), N_h, c["causal"])
        stats = torch.stack([top, den], -1).permute(1, 0, 2, 3)            # (N_h, N_b, N_s, 2)
        return dict(B=act(out), dQKV=act(dQKV), stats=_pack(stats, (2, ts, B, N_h), 4))
    if kind == "layernorm":
        gamma = d["gamma"].double()
        Y, saved = _ln(d["X"].double(), gamma, d["beta"].double())
        dX, dg, db = _ln_bwd(saved, gamma, d["dY"].double())
        return dict(Y=act(Y), dX=act(dX + d["dR"].double()), dgamma=vec(dg), dbeta=vec(db))
    if kind == "head":
        W, X = d["W"].double(), d["X"].double()
        losses, dL = _loss(X @ W.t(), d["labels"])
        dW = dL.reshape(-1, c["N_v"]).t() @ X.reshape(-1, c["N_e"])
        return dict(losses=losses.reshape(-1), loss=losses.sum().reshape(1), dL=act(dL, c["tile_v"]), dX=act(dL @ W), dW=mat(dW, t, c["tile_v"]))
    top, tm, tv = d["top"]
    q = {k: a.double() for k, a in top.items()}
    tok = d["tokens"].long()
    x = q["wte"][tok] + q["wpe"][:S].unsqueeze(0)
    ps = [_block_params(p, dt) for p, _, _ in d["blocks"]]
    saved = []
    for p in ps:
        x, sv = _block_forward(p, x, c["N_h"])
        saved.append(sv)
    last = x
    xf, ln = _ln(x, q["gamma"], q["beta"])
    losses, dL = _loss(xf @ q["wte"].t(), d["labels"])
    g = dict(wte=dL.reshape(-1, c["N_v"]).t() @ xf.reshape(-1, xf.shape[-1]))
    out = dict(loss=losses.sum().reshape(1), col_loss=losses.reshape(-1), dlogits=act(dL, c["tile_v"]), last=act(last))
    dx, g["gamma"], g["beta"] = _ln_bwd(ln, q["gamma"], dL @ q["wte"])
    for n in reversed(range(len(ps))):
        dx, gb = _block_backward(ps[n], saved[n], dx, c["N_h"])
        p, m, v = d["blocks"][n]
        for k in ("W_qkv", "W_o", "W_1", "W_2", "b_1", "gamma1"):
            out["d%s_%d" % (k, n)], out["new_%s_%d" % (k, n)] = param(k, gb[k]), param(k, _adam(p[k], gb[k], m[k], v[k])[0])
    g["wte"].index_add_(0, tok.reshape(-1), dx.reshape(-1, dx.shape[-1]))
    g["wpe"] = dx.sum(0)
    for k in top:
        new = _adam(top[k], g[k], tm[k], tv[k])[0]
        if k == "wte":
            out["dwte"], out["new_wte"] = mat(g[k], t, c["tile_v"]), mat(new, t, c["tile_v"])
        elif k == "wpe":
            out["dwpe"], out["new_wpe"] = mat(g[k], t, t), mat(new, t, t)
        else:
            out["d" + k], out["new_" + k] = vec(g[k]), vec(new)
    return out
