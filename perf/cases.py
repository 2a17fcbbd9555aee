"""The measured work of this library: what a program that builds deep-learning primitives on it
asks of it, through the public entry points of ``paper_2104_05755_amd``.

Each case is a dict with a ``family`` (which of the builders below makes it) and its sizes and
options.  ``listed()`` names twelve; ``draw(rng)`` gives more of the same families over their whole
ranges.  A state (``prepare``) holds device tensors and dispatched handles, as a program keeps them;
``run`` issues one pass on torch's current stream and returns every output; ``exact`` is the same
computation in float64 by plain torch (tensors that the path stores in bf16 between two calls are
rounded there too, since that rounding is part of what the calls are asked for).

All 2D blocks are column-major: a torch tensor ``[cols][rows]`` is a rows x cols block.
"""
from __future__ import annotations

import math

import torch
import torch.nn.functional as F

import paper_2104_05755_amd as tpp

_DT = {"f32": torch.float32, "bf16": torch.bfloat16}
_CODE = {"f32": tpp.TPP_DT_F32, "bf16": tpp.TPP_DT_BF16}
_SIZE = {"f32": 4, "bf16": 2}
BLK = 64   # the block edge of the blocked layouts


def listed():
    return [
        # One BRGEMM call as an HPC code or a small layer issues it: launch latency.
        dict(name="single_f32", family="single", m=64, n=64, k=64, count=16, kind="stride",
             dtype="f32", c_type="f32", act="none", beta=0),
        # A fully-connected layer in fp32, the precision that most of the paper's runs use.
        dict(name="fc_f32", family="fc", tokens=2048, c_in=1024, k_out=1024, layout="blocked",
             dtype="f32", c_type="f32", act="relu", residual=False),
        # The same layer in bf16: an ordinary layer of an MLP (DLRM, GNN), a small grid.
        dict(name="fc_bf16", family="fc", tokens=2048, c_in=1024, k_out=1024, layout="blocked",
             dtype="bf16", c_type="bf16", act="relu", residual=False),
        # A layer whose sizes are no multiple of anything: a classifier head of 1000 outputs on an
        # odd number of features and tokens, plain (unblocked) operands, a residual in C.
        dict(name="fc_ragged_bf16", family="fc", tokens=1533, c_in=777, k_out=1000,
             layout="plain", dtype="bf16", c_type="bf16", act="gelu_tanh", residual=True),
        # The transformer MLP block of BERT-Large, forward: the headline workload.
        dict(name="mlp_forward", family="mlp_fwd", tokens=8192, hidden=1024, inter=4096),
        # The same block trained: the forward call that keeps its pre-activation, then dZ, dW2, db2,
        # dX, dW1, db1.
        dict(name="mlp_backward", family="mlp_bwd", tokens=8192, hidden=1024, inter=4096),
        # A ResNet-50 3x3 convolution as offset-based BRGEMMs, and the batchnorm statistics of its
        # output.
        dict(name="conv_bn", family="conv", images=28, h=56, w=56, c=64, k=64),
        # Address-based BRGEMMs over block lists: block-sparse products, the largest call.
        dict(name="gathered", family="gathered", n_out=4096, pool=8192, m=128, n=128, k=64,
             min_len=8, max_len=64, c_type="f32"),
        # DLRM's sparse embedding lookups.
        dict(name="embedding", family="embedding", rows=1_000_000, dim=128, bags=16384,
             min_pool=1, max_pool=64, w_type="f32", out_type="f32"),
        # Layer normalization of a transformer's tokens: a Reduce and two matrix equations.
        dict(name="layernorm", family="layernorm", features=1024, tokens=8192, dtype="bf16"),
        # Softmax of attention scores: two Reduces and two matrix equations.
        dict(name="softmax", family="softmax", keys=512, columns=32768, dtype="bf16"),
        # A transpose of a tensor with odd extents (activations whose token count is no multiple of
        # anything); the aligned sizes come up in the drawn cases.
        dict(name="transpose_odd", family="transform", kind="transpose", m=4097, n=2049,
             dtype="f32", alpha=1, G=1),
    ]


# ---- draws -----------------------------------------------------------------------------------
def _logint(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def _mult(rng, lo, hi, step):
    """A size from lo to hi: half the time a multiple of step, else any integer."""
    v = _logint(rng, lo, hi)
    return min(hi, max(step, -(-v // step) * step)) if rng.random() < 0.5 else v


def draw(rng):
    family = rng.choice(["single", "fc", "fc", "mlp_fwd", "mlp_bwd", "conv", "gathered",
                         "embedding", "layernorm", "softmax", "transform"])
    if family == "single":
        dtype = rng.choice(["f32", "bf16"])
        return dict(family=family, m=_mult(rng, 8, 128, 16), n=_mult(rng, 8, 128, 16),
                    k=_mult(rng, 8, 128, 16), count=_logint(rng, 1, 64),
                    kind=rng.choice(["stride", "offset", "address"]), dtype=dtype,
                    c_type=rng.choice(["f32", dtype]), act=rng.choice(["none", "relu", "gelu_tanh"]),
                    beta=rng.choice([0, 0, 1]))
    if family == "fc":
        layout = rng.choice(["blocked", "plain"])
        dtype = rng.choice(["f32", "bf16"])
        if layout == "blocked":
            size = lambda lo, hi: BLK * _logint(rng, lo // BLK, hi // BLK)
        else:
            size = lambda lo, hi: _mult(rng, lo, hi, 64)
        return dict(family=family, tokens=size(128, 4096), c_in=size(128, 2048),
                    k_out=size(128, 2048), layout=layout, dtype=dtype, c_type=dtype,
                    act=rng.choice(["none", "relu", "gelu_tanh"]),
                    residual=rng.choice([False, False, True]))
    if family in ("mlp_fwd", "mlp_bwd"):
        hidden = BLK * _logint(rng, 4, 16)
        return dict(family=family, tokens=BLK * _logint(rng, 4, 128), hidden=hidden,
                    inter=hidden * rng.choice([2, 4]))
    if family == "conv":
        hw = rng.choice([7, 14, 28, 56])
        return dict(family=family, images=_logint(rng, 4, 28), h=hw, w=hw,
                    c=rng.choice([16, 32, 64]), k=rng.choice([32, 64, 128]))
    if family == "gathered":
        edge = rng.choice([32, 64, 128])
        return dict(family=family, n_out=_logint(rng, 256, 4096), pool=_logint(rng, 256, 8192),
                    m=edge, n=edge, k=rng.choice([32, 64]), min_len=_logint(rng, 1, 8),
                    max_len=_logint(rng, 9, 64), c_type=rng.choice(["f32", "bf16"]))
    if family == "embedding":
        w_type = rng.choice(["f32", "bf16"])
        return dict(family=family, rows=_logint(rng, 10_000, 1_000_000),
                    dim=rng.choice([16, 32, 64, 100, 128, 256]), bags=_logint(rng, 256, 16384),
                    min_pool=1, max_pool=_logint(rng, 2, 64), w_type=w_type,
                    out_type=rng.choice(["f32", w_type]))
    if family == "layernorm":
        return dict(family=family, features=_mult(rng, 128, 4096, 64),
                    tokens=_logint(rng, 64, 8192) // 4 + 1, dtype=rng.choice(["f32", "bf16"]))
    if family == "softmax":
        return dict(family=family, keys=_mult(rng, 32, 1024, 32),
                    columns=_logint(rng, 256, 16384), dtype=rng.choice(["f32", "bf16"]))
    kind = rng.choice(["transpose", "vnni", "vnni_t"])
    big = rng.random() < 0.5
    return dict(family="transform", kind=kind, m=_mult(rng, 256, 4096, 64) if big else 64,
                n=_mult(rng, 256, 4096, 64) if big else 64, dtype=rng.choice(["f32", "bf16"]),
                alpha=1 if kind == "transpose" else 2, G=1 if big else _logint(rng, 16, 1024))


# ---- inputs ----------------------------------------------------------------------------------
class _Draws:
    def __init__(self, seed):
        self.g = torch.Generator(device="cuda")
        self.g.manual_seed(seed)

    def normal(self, shape, std, dtype, mean=0.0):
        x = torch.randn(shape, generator=self.g, device="cuda") * std + mean
        return x.to(dtype)

    def uniform(self, shape, dtype):
        return (torch.rand(shape, generator=self.g, device="cuda") * 2 - 1).to(dtype)

    def ints(self, lo, hi, shape):   # lo .. hi inclusive
        return torch.randint(lo, hi + 1, shape, generator=self.g, device="cuda")


def _empty(shape, dtype):
    return torch.empty(shape, dtype=dtype, device="cuda")


def _grid(**kw):
    return tpp.tpp_grid_strided(**kw)   # steps left out are 0


def _flags(act, bias=False, extra=()):
    return ([] if act == "none" else [act]) + (["bias"] if bias else []) + list(extra)


def _brgemm(h, grid, a, b, c, count, bias=None, aux=None):
    """One batched stride-kind call on the current stream (arguments as the C entry point)."""
    G = grid.gm * grid.gn
    s = tpp.current_stream()
    if aux is None:
        tpp.tpp_brgemm_execute_batched(h, grid, G, None, None, None, None, a, b, c, bias, count,
                                       None, None, None, None, None, s)
    else:
        tpp.tpp_brgemm_execute_batched_aux(h, grid, G, None, None, None, None, a, b, c, aux, bias,
                                           count, None, None, None, None, None, s)


def _act64(z, act):
    if act == "relu":
        return F.relu(z)
    return F.gelu(z, approximate="tanh") if act == "gelu_tanh" else z


# ---- single: one call of the single-call API ----------------------------------------------------
def _single_prepare(c, seed):
    r = _Draws(seed)
    m, n, k, cnt, dt = c["m"], c["n"], c["k"], c["count"], _DT[c["dtype"]]
    a, b = r.uniform((cnt, k, m), dt), r.uniform((cnt, n, k), dt)
    st = dict(case=c, a=a, b=b, c=_empty((n, m), _DT[c["c_type"]]),
              c0=r.uniform((n, m), _DT[c["c_type"]]))
    # lists name the blocks in a shuffled order
    st["perm"] = torch.randperm(cnt, generator=r.g, device="cuda")
    if c["kind"] == "offset":
        st["la"], st["lb"] = st["perm"] * (m * k), st["perm"] * (k * n)
    elif c["kind"] == "address":
        es = _SIZE[c["dtype"]]
        st["la"] = st["perm"] * (m * k * es) + a.data_ptr()
        st["lb"] = st["perm"] * (k * n * es) + b.data_ptr()
    st["h"] = tpp.tpp_brgemm_dispatch(tpp.make_desc(
        m, n, k, m, k, m, c["dtype"], c["c_type"], float(c["beta"]), c["kind"], m * k, k * n,
        _flags(c["act"])))
    return st


def _single_run(st):
    c, s = st["case"], tpp.current_stream()
    if c["beta"]:
        st["c"].copy_(st["c0"])
    if c["kind"] == "stride":
        tpp.tpp_brgemm_execute_stride(st["h"], st["a"], st["b"], st["c"], None, c["count"], s)
    elif c["kind"] == "offset":
        tpp.tpp_brgemm_execute_offset(st["h"], st["a"], st["b"], st["la"], st["lb"], st["c"], None,
                                      c["count"], s)
    else:
        tpp.tpp_brgemm_execute_address(st["h"], st["la"], st["lb"], st["c"], None, c["count"], s)
    return st["c"]


def _single_exact(c, seed):
    st = _single_prepare(c, seed)
    a = st["a"].double().permute(0, 2, 1)                       # [cnt][m][k]
    b = st["b"].double().permute(0, 2, 1)                       # [cnt][k][n]
    z = a.permute(1, 0, 2).reshape(c["m"], -1) @ b.reshape(-1, c["n"])
    z = z.t() + c["beta"] * st["c0"].double()
    return _act64(z, c["act"])


def _single_work(c):
    e, m, n, k = _SIZE[c["dtype"]], c["m"], c["n"], c["k"]
    return dict(bytes=c["count"] * (m * k + k * n) * e + m * n * _SIZE[c["c_type"]] *
                (2 if c["beta"] else 1), flops=2 * m * n * k * c["count"])


# ---- fc: a fully-connected layer, blocked (Alg. 6) or plain ---------------------------------------
def _fc_dims(c):
    if c["layout"] == "blocked":
        return (c["tokens"] // BLK, c["c_in"] // BLK, c["k_out"] // BLK, BLK, BLK, BLK)
    return 1, 1, 1, c["tokens"], c["c_in"], c["k_out"]


def _fc_prepare(c, seed):
    r = _Draws(seed)
    nb, cb, kb, bn, bc, bk = _fc_dims(c)
    dt, ct = _DT[c["dtype"]], _DT[c["c_type"]]
    st = dict(case=c, x=r.uniform((nb, cb, bn, bc), dt),
              w=r.uniform((kb, cb, bc, bk), torch.float32).mul_(c["c_in"] ** -0.5).to(dt),
              bias=r.uniform((c["k_out"],), torch.float32), out=_empty((nb, kb, bn, bk), ct),
              res=r.uniform((nb, kb, bn, bk), ct), cb=cb)
    st["grid"] = _grid(gm=kb, gn=nb, a_step_m=cb * bc * bk, b_step_n=cb * bn * bc,
                       c_step_m=bn * bk, c_step_n=kb * bn * bk, bias_step_m=bk)
    st["h"] = tpp.tpp_brgemm_dispatch(tpp.make_desc(
        bk, bn, bc, bk, bc, bk, c["dtype"], c["c_type"], 1.0 if c["residual"] else 0.0, "stride",
        bc * bk, bn * bc, _flags(c["act"], bias=True)))
    return st


def _fc_run(st):
    if st["case"]["residual"]:
        st["out"].copy_(st["res"])
    _brgemm(st["h"], st["grid"], st["w"], st["x"], st["out"], st["cb"], st["bias"])
    return st["out"]


def _fc_exact(c, seed):
    st = _fc_prepare(c, seed)
    z = _mm_blocked(st["w"], st["x"]) + st["bias"].double().reshape(1, -1, 1, st["w"].shape[3])
    if c["residual"]:
        z = z + st["res"].double()
    return _act64(z, c["act"])


def _mm_blocked(w, x):
    """[Nb][Kb][bn][bk] = X[Nb][Cb][bn][bc] times W[Kb][Cb][bc][bk], in float64."""
    nb, cb, bn, bc = x.shape
    kb, _, _, bk = w.shape
    xd = x.double().permute(0, 2, 1, 3).reshape(nb * bn, cb * bc)
    wd = w.double().permute(1, 2, 0, 3).reshape(cb * bc, kb * bk)
    return (xd @ wd).reshape(nb, bn, kb, bk).permute(0, 2, 1, 3).contiguous()


def _fc_work(c):
    e, t, i, o = _SIZE[c["dtype"]], c["tokens"], c["c_in"], c["k_out"]
    return dict(bytes=(t * i + i * o) * e + o * 4 +
                t * o * _SIZE[c["c_type"]] * (2 if c["residual"] else 1), flops=2 * t * i * o)


# ---- mlp_fwd: the transformer MLP, two fused layers ------------------------------------------------
def _mlp_inputs(c, seed):
    r = _Draws(seed)
    nb, hb, ib = c["tokens"] // BLK, c["hidden"] // BLK, c["inter"] // BLK
    b16 = torch.bfloat16
    st = dict(case=c, x=r.normal((nb, hb, BLK, BLK), 1.0, b16),
              w1=r.normal((ib, hb, BLK, BLK), 0.02, b16), b1=r.normal((c["inter"],), 0.02,
                                                                      torch.float32),
              w2=r.normal((hb, ib, BLK, BLK), 0.02, b16), b2=r.normal((c["hidden"],), 0.02,
                                                                      torch.float32),
              h=_empty((nb, ib, BLK, BLK), b16), dims=(nb, hb, ib))
    return r, st


def _desc64(stride_a, stride_b, flags, c_type="bf16"):
    return tpp.tpp_brgemm_dispatch(tpp.make_desc(BLK, BLK, BLK, BLK, BLK, BLK, "bf16", c_type, 0.0,
                                                 "stride", stride_a, stride_b, flags))


_B2 = BLK * BLK


def _mlp_fwd_prepare(c, seed):
    _, st = _mlp_inputs(c, seed)
    nb, hb, ib = st["dims"]
    st["y"] = _empty((nb, hb, BLK, BLK), torch.bfloat16)
    st["h1"] = _desc64(_B2, _B2, ["bias", "gelu_tanh"])
    st["h2"] = _desc64(_B2, _B2, ["bias"])
    st["g1"] = _grid(gm=ib, gn=nb, a_step_m=hb * _B2, b_step_n=hb * _B2, c_step_m=_B2,
                     c_step_n=ib * _B2, bias_step_m=BLK)
    st["g2"] = _grid(gm=hb, gn=nb, a_step_m=ib * _B2, b_step_n=ib * _B2, c_step_m=_B2,
                     c_step_n=hb * _B2, bias_step_m=BLK)
    return st


def _mlp_fwd_run(st):
    _, hb, ib = st["dims"]
    _brgemm(st["h1"], st["g1"], st["w1"], st["x"], st["h"], hb, st["b1"])
    _brgemm(st["h2"], st["g2"], st["w2"], st["h"], st["y"], ib, st["b2"])
    return dict(h=st["h"], y=st["y"])


def _mlp_fwd_exact(c, seed):
    _, st = _mlp_inputs(c, seed)
    z = _mm_blocked(st["w1"], st["x"]) + st["b1"].double().reshape(1, -1, 1, BLK)
    h = F.gelu(z, approximate="tanh")
    y = _mm_blocked(st["w2"], h.to(torch.bfloat16)) + st["b2"].double().reshape(1, -1, 1, BLK)
    return dict(h=h, y=y)


def _mlp_fwd_work(c):
    t, h, i = c["tokens"], c["hidden"], c["inter"]
    return dict(bytes=2 * (2 * t * h + t * i + 2 * h * i) + 4 * (h + i), flops=4 * t * h * i)


# ---- mlp_bwd: the transformer MLP trained ---------------------------------------------------------
def _mlp_bwd_prepare(c, seed):
    r, st = _mlp_inputs(c, seed)
    nb, hb, ib = st["dims"]
    b16, f32 = torch.bfloat16, torch.float32
    st["dy"] = r.normal((nb, hb, BLK, BLK), 1.0, b16)
    for name, shape, dt in (("z", (nb, ib, BLK, BLK), b16), ("dz", (nb, ib, BLK, BLK), b16),
                            ("dx", (nb, hb, BLK, BLK), b16), ("dw1", (ib, hb, BLK, BLK), f32),
                            ("dw2", (hb, ib, BLK, BLK), f32), ("p1", (ib * _B2,), f32),
                            ("p2", (hb * _B2,), f32), ("db1", (c["inter"],), f32),
                            ("db2", (c["hidden"],), f32)):
        st[name] = _empty(shape, dt)
    st["hf"] = _desc64(_B2, _B2, ["bias", "gelu_tanh", "save_preact"])
    st["hdz"] = _desc64(ib * _B2, _B2, ["gelu_tanh_inv", "a_trans"])
    st["hdw2"] = _desc64(hb * _B2, ib * _B2, ["b_trans"], "f32")
    st["hdx"] = _desc64(hb * _B2, _B2, ["a_trans"])
    st["hdw1"] = _desc64(ib * _B2, hb * _B2, ["b_trans"], "f32")
    st["gf"] = _grid(gm=ib, gn=nb, a_step_m=hb * _B2, b_step_n=hb * _B2, c_step_m=_B2,
                     c_step_n=ib * _B2, bias_step_m=BLK)
    st["gdz"] = _grid(gm=ib, gn=nb, a_step_m=_B2, b_step_n=hb * _B2, c_step_m=_B2,
                      c_step_n=ib * _B2)
    st["gdw2"] = _grid(gm=hb, gn=ib, a_step_m=_B2, b_step_n=_B2, c_step_m=ib * _B2, c_step_n=_B2)
    st["gdx"] = _grid(gm=hb, gn=nb, a_step_m=_B2, b_step_n=ib * _B2, c_step_m=_B2,
                      c_step_n=hb * _B2)
    st["gdw1"] = _grid(gm=ib, gn=hb, a_step_m=_B2, b_step_n=_B2, c_step_m=hb * _B2, c_step_n=_B2)
    return st


def _bias_grad(src, fb, nb, part, db):
    """Sum over the token blocks, then over the tokens of each 64 x 64 block."""
    s, fl = tpp.current_stream(), tpp.TPP_RED_BY_COLS | tpp.TPP_RED_X
    tpp.tpp_reduce_batched(fb * _B2, nb, fb * _B2, tpp.TPP_DT_BF16, src, 1, 0, tpp.TPP_RED_SUM, fl,
                           part, None, 0, s)
    tpp.tpp_reduce_batched(BLK, BLK, BLK, tpp.TPP_DT_F32, part, fb, _B2, tpp.TPP_RED_SUM, fl, db,
                           None, BLK, s)


_BWD_OUT = ("z", "h", "dz", "dx", "dw1", "dw2", "db1", "db2")


def _mlp_bwd_run(st):
    nb, hb, ib = st["dims"]
    _brgemm(st["hf"], st["gf"], st["w1"], st["x"], st["h"], hb, st["b1"], st["z"])
    _brgemm(st["hdz"], st["gdz"], st["w2"], st["dy"], st["dz"], hb, None, st["z"])
    _brgemm(st["hdw2"], st["gdw2"], st["dy"], st["h"], st["dw2"], nb)
    _bias_grad(st["dy"], hb, nb, st["p2"], st["db2"])
    _brgemm(st["hdx"], st["gdx"], st["w1"], st["dz"], st["dx"], ib)
    _brgemm(st["hdw1"], st["gdw1"], st["dz"], st["x"], st["dw1"], nb)
    _bias_grad(st["dz"], ib, nb, st["p1"], st["db1"])
    return {k: st[k] for k in _BWD_OUT}


def _mlp_bwd_exact(c, seed):
    st = _mlp_bwd_prepare(c, seed)
    b16 = torch.bfloat16
    z = _mm_blocked(st["w1"], st["x"]) + st["b1"].double().reshape(1, -1, 1, BLK)
    h = F.gelu(z, approximate="tanh")
    zb = z.to(b16).double().requires_grad_(True)
    with torch.enable_grad():
        F.gelu(zb, approximate="tanh").backward(torch.ones_like(zb))
    tr = lambda w: w.permute(1, 0, 3, 2).contiguous()     # the transposed matrix, blocked
    dz = _mm_blocked(tr(st["w2"]), st["dy"]) * zb.grad
    dzb, hb16 = dz.to(b16), h.to(b16)
    dx = _mm_blocked(tr(st["w1"]), dzb)
    # dW[fb][cb][bc][bf] = sum over tokens of d[nb][fb][bn][bf] * s[nb][cb][bn][bc]
    dw = lambda d, s: _mm_blocked(d.permute(1, 0, 2, 3), s.permute(1, 0, 3, 2)) \
        .permute(1, 0, 2, 3).contiguous()
    red = lambda d: d.double().sum(dim=(0, 2)).reshape(-1)
    return dict(z=z, h=h, dz=dz, dx=dx, dw1=dw(dzb, st["x"]), dw2=dw(st["dy"], hb16),
                db1=red(dzb), db2=red(st["dy"]))


def _mlp_bwd_work(c):
    t, h, i = c["tokens"], c["hidden"], c["inter"]
    # read x, dy, w1, w2, b1; write z, h, dz, dx, dw1, dw2, db1, db2
    return dict(bytes=2 * (2 * t * h + 2 * h * i) + 4 * i + 2 * (3 * t * i + t * h) +
                4 * (2 * h * i + h + i), flops=10 * t * h * i)


# ---- conv: 3x3, stride 1, pad 1, and the batchnorm statistics of its output -------------------------
def _conv_prepare(c, seed):
    r = _Draws(seed)
    im, h, w, ci, k = c["images"], c["h"], c["w"], c["c"], c["k"]
    x = torch.zeros((im, h + 2, w + 2, ci), dtype=torch.bfloat16, device="cuda")
    x[:, 1:h + 1, 1:w + 1] = r.normal((im, h, w, ci), 0.5, torch.bfloat16).relu_()
    i64 = lambda v: torch.tensor(v, dtype=torch.int64, device="cuda")
    img = torch.arange(im, device="cuda").reshape(-1, 1)
    row = torch.arange(h, device="cuda").reshape(1, -1)
    st = dict(case=c, x=x, wt=r.normal((3, 3, ci, k), 0.1, torch.bfloat16),
              out=_empty((im, h, w, k), torch.bfloat16), s=_empty((k,), torch.float32),
              s2=_empty((k,), torch.float32),
              offs_a=i64([(r_ * 3 + s) * ci * k for r_ in range(3) for s in range(3)]),
              offs_b=i64([(r_ * (w + 2) + s) * ci for r_ in range(3) for s in range(3)]),
              a_off=torch.zeros(im * h, dtype=torch.int64, device="cuda"),
              b_off=((img * (h + 2) + row) * ((w + 2) * ci)).reshape(-1).contiguous(),
              c_off=((img * h + row) * (w * k)).reshape(-1).contiguous())
    st["hd"] = tpp.tpp_brgemm_dispatch(tpp.make_desc(k, w, ci, k, ci, k, "bf16", "bf16", 0.0,
                                                     "offset", 0, 0, ["relu"]))
    return st


def _conv_run(st):
    c, s = st["case"], tpp.current_stream()
    G = c["images"] * c["h"]
    tpp.tpp_brgemm_execute_batched(st["hd"], None, G, st["a_off"], st["b_off"], st["c_off"], None,
                                   st["wt"], st["x"], st["out"], None, 9, st["offs_a"],
                                   st["offs_b"], None, None, None, s)
    tpp.tpp_reduce(c["k"], G * c["w"], c["k"], tpp.TPP_DT_BF16, st["out"], tpp.TPP_RED_SUM,
                   tpp.TPP_RED_BY_COLS | tpp.TPP_RED_X | tpp.TPP_RED_X2, st["s"], st["s2"], s)
    return dict(out=st["out"], s=st["s"], s2=st["s2"])


def _conv_exact(c, seed):
    st = _conv_prepare(c, seed)
    h, w, k = c["h"], c["w"], c["k"]
    x, wt = st["x"].double(), st["wt"].double()
    z = torch.zeros((c["images"], h, w, k), dtype=torch.float64, device="cuda")
    for r in range(3):
        for s in range(3):
            z += x[:, r:r + h, s:s + w].reshape(-1, c["c"]).matmul(wt[r, s]).reshape(z.shape)
    z = F.relu(z)
    o = z.to(torch.bfloat16).double()
    return dict(out=z, s=o.sum(dim=(0, 1, 2)), s2=o.square().sum(dim=(0, 1, 2)))


def _conv_work(c):
    im, h, w, ci, k = c["images"], c["h"], c["w"], c["c"], c["k"]
    return dict(bytes=2 * (im * (h + 2) * (w + 2) * ci + 9 * ci * k + im * h * w * k) + 8 * k,
                flops=18 * im * h * w * ci * k)


# ---- gathered: address-based BRGEMMs over random block lists ---------------------------------------
def _gathered_prepare(c, seed):
    r = _Draws(seed)
    m, n, k, g = c["m"], c["n"], c["k"], c["n_out"]
    ap = r.uniform((c["pool"], k, m), torch.bfloat16)
    bp = r.uniform((c["pool"], n, k), torch.bfloat16)
    lens = r.ints(c["min_len"], c["max_len"], (g,))
    begin = torch.zeros(g + 1, dtype=torch.int64, device="cuda")
    begin[1:] = torch.cumsum(lens, 0)
    pairs = int(begin[-1])
    ia, ib = r.ints(0, c["pool"] - 1, (pairs,)), r.ints(0, c["pool"] - 1, (pairs,))
    st = dict(case=c, ap=ap, bp=bp, ia=ia, ib=ib, begin=begin,
              out=_empty((g, n, m), _DT[c["c_type"]]),
              c_off=torch.arange(g, dtype=torch.int64, device="cuda") * (m * n),
              pa=ia * (m * k * 2) + ap.data_ptr(), pb=ib * (k * n * 2) + bp.data_ptr())
    st["h"] = tpp.tpp_brgemm_dispatch(tpp.make_desc(m, n, k, m, k, m, "bf16", c["c_type"], 0.0,
                                                    "address"))
    return st


def _gathered_run(st):
    c = st["case"]
    tpp.tpp_brgemm_execute_batched(st["h"], None, c["n_out"], None, None, st["c_off"], None, None,
                                   None, st["out"], None, 0, None, None, st["begin"], st["pa"],
                                   st["pb"], tpp.current_stream())
    return st["out"]


def _gathered_exact(c, seed):
    st = _gathered_prepare(c, seed)
    m, n, k, g = c["m"], c["n"], c["k"], c["n_out"]
    out = torch.empty((g, n, m), dtype=torch.float64, device="cuda")
    begin = st["begin"].tolist()
    for i in range(g):
        lo, hi = begin[i], begin[i + 1]
        a = st["ap"][st["ia"][lo:hi]].double().reshape(-1, m)                   # [len*k][m]
        b = st["bp"][st["ib"][lo:hi]].double().permute(1, 0, 2).reshape(n, -1)  # [n][len*k]
        out[i] = b @ a
    return out


def _gathered_work(c):
    pairs = c["n_out"] * (c["min_len"] + c["max_len"]) / 2
    seen = c["pool"] * (1 - (1 - 1 / c["pool"]) ** pairs)   # blocks listed at least once
    m, n, k = c["m"], c["n"], c["k"]
    return dict(bytes=2 * seen * (m * k + k * n) + 16 * pairs + 16 * c["n_out"] +
                c["n_out"] * m * n * _SIZE[c["c_type"]], flops=2 * m * n * k * pairs)


# ---- embedding: sparse lookups ---------------------------------------------------------------------
def _embedding_prepare(c, seed):
    r = _Draws(seed)
    w = r.uniform((c["rows"], c["dim"]), _DT[c["w_type"]])
    lens = r.ints(c["min_pool"], c["max_pool"], (c["bags"],))
    begin = torch.zeros(c["bags"] + 1, dtype=torch.int64, device="cuda")
    begin[1:] = torch.cumsum(lens, 0)
    idx = r.ints(0, c["rows"] - 1, (int(begin[-1]),))
    return dict(case=c, w=w, begin=begin, idx=idx,
                out=_empty((c["bags"], c["dim"]), _DT[c["out_type"]]))


def _embedding_run(st):
    c = st["case"]
    tpp.tpp_embedding_bag(c["rows"], c["dim"], _CODE[c["w_type"]], st["w"], c["dim"], c["bags"],
                          st["begin"], st["idx"], _CODE[c["out_type"]], st["out"], c["dim"],
                          tpp.current_stream())
    return st["out"]


def _embedding_exact(c, seed):
    st = _embedding_prepare(c, seed)
    bag = torch.repeat_interleave(torch.arange(c["bags"], device="cuda"), st["begin"].diff())
    out = torch.zeros((c["bags"], c["dim"]), dtype=torch.float64, device="cuda")
    return out.index_add_(0, bag, st["w"][st["idx"]].double())


def _embedding_work(c):
    looks = c["bags"] * (c["min_pool"] + c["max_pool"]) / 2
    seen = c["rows"] * (1 - (1 - 1 / c["rows"]) ** looks)   # rows listed at least once
    return dict(bytes=seen * c["dim"] * _SIZE[c["w_type"]] + 8 * looks + 8 * c["bags"] +
                c["bags"] * c["dim"] * _SIZE[c["out_type"]], flops=looks * c["dim"])


# ---- layernorm: a Reduce by rows and two matrix equations --------------------------------------------
# rs = rcp(sqrt(s2 / F - (s / F)^2 + eps)), then y = (x - s / F) * rs * gamma + beta
_RS = [("leaf", 0), ("leaf", 1), ("mul", 0, 1), ("leaf", 2), ("leaf", 1), ("mul", 3, 4),
       ("square", 5), ("sub", 2, 6), ("leaf", 3), ("add", 7, 8), ("sqrt", 9), ("rcp", 10)]
_NORM = [("leaf", 0), ("leaf", 1), ("leaf", 2), ("mul", 1, 2), ("sub", 0, 3), ("leaf", 3),
         ("mul", 4, 5), ("leaf", 4), ("leaf", 5), ("muladd", 6, 7, 8)]
_EPS = 1e-5


def _layernorm_prepare(c, seed):
    r = _Draws(seed)
    f, t, dt, f32 = c["features"], c["tokens"], _DT[c["dtype"]], torch.float32
    return dict(case=c, x=r.normal((t, f), 1.0, dt, 0.5), gamma=r.normal((f,), 0.1, f32, 1.0),
                beta=r.normal((f,), 0.1, f32), inv_f=torch.full((1,), 1.0 / f, device="cuda"),
                eps=torch.full((1,), _EPS, device="cuda"), s=_empty((t,), f32), s2=_empty((t,), f32),
                rs=_empty((t,), f32), y=_empty((t, f), dt))


def _layernorm_run(st):
    c, s = st["case"], tpp.current_stream()
    f, t, dt, f32 = c["features"], c["tokens"], _CODE[c["dtype"]], tpp.TPP_DT_F32
    tpp.tpp_reduce(f, t, f, dt, st["x"], tpp.TPP_RED_SUM,
                   tpp.TPP_RED_BY_ROWS | tpp.TPP_RED_X | tpp.TPP_RED_X2, st["s"], st["s2"], s)
    tpp.tpp_equation_execute(_RS, 11, 1, t, [(st["s2"], 1, f32, "none"),
                                             (st["inv_f"], 1, f32, "scalar"),
                                             (st["s"], 1, f32, "none"),
                                             (st["eps"], 1, f32, "scalar")], st["rs"], 1, f32, s)
    tpp.tpp_equation_execute(_NORM, 9, f, t, [(st["x"], f, dt, "none"), (st["s"], 1, f32, "row"),
                                              (st["inv_f"], 1, f32, "scalar"),
                                              (st["rs"], 1, f32, "row"),
                                              (st["gamma"], 1, f32, "col"),
                                              (st["beta"], 1, f32, "col")], st["y"], f, dt, s)
    return dict(s=st["s"], s2=st["s2"], rs=st["rs"], y=st["y"])


def _layernorm_exact(c, seed):
    st = _layernorm_prepare(c, seed)
    x, f = st["x"].double(), c["features"]
    s, s2 = x.sum(1), x.square().sum(1)
    mu = s / f
    rs = 1.0 / torch.sqrt(s2 / f - mu * mu + _EPS)
    y = (x - mu[:, None]) * rs[:, None] * st["gamma"].double() + st["beta"].double()
    return dict(s=s, s2=s2, rs=rs, y=y)


def _layernorm_work(c):
    f, t = c["features"], c["tokens"]
    return dict(bytes=2 * f * t * _SIZE[c["dtype"]] + 12 * t + 8 * f, flops=9 * f * t)


# ---- softmax: Reduce MAX, exp equation, Reduce SUM, scaling equation -----------------------------------
def _softmax_prepare(c, seed):
    r = _Draws(seed)
    k, n, dt, f32 = c["keys"], c["columns"], _DT[c["dtype"]], torch.float32
    return dict(case=c, x=r.normal((n, k), 2.0, dt), mx=_empty((n,), f32), xe=_empty((n, k), f32),
                s=_empty((n,), f32), y=_empty((n, k), dt))


def _softmax_run(st):
    c, s = st["case"], tpp.current_stream()
    k, n, dt, f32 = c["keys"], c["columns"], _CODE[c["dtype"]], tpp.TPP_DT_F32
    fl = tpp.TPP_RED_BY_ROWS | tpp.TPP_RED_X
    tpp.tpp_reduce(k, n, k, dt, st["x"], tpp.TPP_RED_MAX, fl, st["mx"], None, s)
    tpp.tpp_equation_execute([("leaf", 0), ("leaf", 1), ("sub", 0, 1), ("exp", 2)], 3, k, n,
                             [(st["x"], k, dt, "none"), (st["mx"], 1, f32, "row")], st["xe"], k,
                             f32, s)
    tpp.tpp_reduce(k, n, k, f32, st["xe"], tpp.TPP_RED_SUM, fl, st["s"], None, s)
    tpp.tpp_equation_execute([("leaf", 0), ("leaf", 1), ("rcp", 1), ("mul", 0, 2)], 3, k, n,
                             [(st["xe"], k, f32, "none"), (st["s"], 1, f32, "row")], st["y"], k,
                             dt, s)
    return dict(mx=st["mx"], xe=st["xe"], s=st["s"], y=st["y"])


def _softmax_exact(c, seed):
    x = _softmax_prepare(c, seed)["x"].double()
    mx = x.amax(1)
    xe = torch.exp(x - mx[:, None])
    s = xe.sum(1)
    return dict(mx=mx, xe=xe, s=s, y=xe / s[:, None])


def _softmax_work(c):
    e, n = c["keys"] * c["columns"], c["columns"]
    # x read, xe (fp32) and y written, the per-column statistics written
    return dict(bytes=e * (2 * _SIZE[c["dtype"]] + 4) + 8 * n, flops=5 * e)


# ---- transform: transposes and VNNI formatting ---------------------------------------------------------
_TR = {"transpose": tpp.TPP_TR_TRANSPOSE, "vnni": tpp.TPP_TR_VNNI,
       "vnni_t": tpp.TPP_TR_VNNI_TO_VNNI_T}


def _transform_dims(c):
    """(ld_in, entries of a block in, ld_out, entries of a block out)."""
    m, n, al = c["m"], c["n"], c["alpha"]
    if c["kind"] == "transpose":
        return m, m * n, n, m * n
    if c["kind"] == "vnni":
        return m, m * n, m * al, -(-n // al) * al * m
    return m * al, -(-n // al) * al * m, n * al, -(-m // al) * al * n


def _transform_prepare(c, seed):
    _, size_in, _, size_out = _transform_dims(c)
    dt = _DT[c["dtype"]]
    return dict(case=c, x=_Draws(seed).normal((c["G"], size_in), 1.0, dt),
                y=_empty((c["G"], size_out), dt))


def _transform_run(st):
    c = st["case"]
    ld_in, size_in, ld_out, size_out = _transform_dims(c)
    tpp.tpp_transform_batched(_TR[c["kind"]], c["m"], c["n"], ld_in, ld_out, _CODE[c["dtype"]],
                              c["alpha"], st["x"], size_in, st["y"], size_out, c["G"],
                              tpp.current_stream())
    return st["y"]


def _transform_exact(c, seed):
    x = _transform_prepare(c, seed)["x"].double()
    m, n, al, g = c["m"], c["n"], c["alpha"], c["G"]
    if c["kind"] == "vnni_t":
        nat = x.reshape(g, -1, m, al).permute(0, 1, 3, 2).reshape(g, -1, m)[:, :n]
    else:
        nat = x.reshape(g, n, m)                      # [n][m]: column-major m x n
    if c["kind"] == "vnni":
        src, rows, cols = nat, m, n
    else:
        src, rows, cols = nat.permute(0, 2, 1), n, m  # the n x m transpose, [m][n]
    if c["kind"] != "transpose":
        src = F.pad(src, (0, 0, 0, -cols % al))
        src = src.reshape(g, -1, al, rows).permute(0, 1, 3, 2)
    return src.reshape(g, -1).contiguous()


def _transform_work(c):
    _, size_in, _, size_out = _transform_dims(c)
    return dict(bytes=c["G"] * (size_in + size_out) * _SIZE[c["dtype"]], flops=0)


# ---- the interface --------------------------------------------------------------------------------------
_FAMILIES = {
    "single": (_single_prepare, _single_run, _single_exact, _single_work),
    "fc": (_fc_prepare, _fc_run, _fc_exact, _fc_work),
    "mlp_fwd": (_mlp_fwd_prepare, _mlp_fwd_run, _mlp_fwd_exact, _mlp_fwd_work),
    "mlp_bwd": (_mlp_bwd_prepare, _mlp_bwd_run, _mlp_bwd_exact, _mlp_bwd_work),
    "conv": (_conv_prepare, _conv_run, _conv_exact, _conv_work),
    "gathered": (_gathered_prepare, _gathered_run, _gathered_exact, _gathered_work),
    "embedding": (_embedding_prepare, _embedding_run, _embedding_exact, _embedding_work),
    "layernorm": (_layernorm_prepare, _layernorm_run, _layernorm_exact, _layernorm_work),
    "softmax": (_softmax_prepare, _softmax_run, _softmax_exact, _softmax_work),
    "transform": (_transform_prepare, _transform_run, _transform_exact, _transform_work),
}


def prepare(case, seed):
    return _FAMILIES[case["family"]][0](case, seed)


def run(state):
    return _FAMILIES[state["case"]["family"]][1](state)


def exact(case, seed):
    return _FAMILIES[case["family"]][2](case, seed)


def work(case):
    return _FAMILIES[case["family"]][3](case)


def tolerance(case):
    """Moved entries are the same bits.  Outputs all in fp32 (from fp32 or exactly widened bf16
    inputs): fp32 sums in any order.  Outputs in bf16: one rounding to 8 bits, about 1.7e-3 of the
    result in the 2-norm, and in a chain the flips it causes downstream."""
    if case["family"] == "transform":
        return "exact"
    stored = {"single": "c_type", "fc": "c_type", "gathered": "c_type", "embedding": "out_type",
              "layernorm": "dtype", "softmax": "dtype"}.get(case["family"])
    return {"rel": 1e-5} if stored and case[stored] == "f32" else {"rel": 7e-3}
