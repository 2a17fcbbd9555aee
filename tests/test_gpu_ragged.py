"""GPU parity, bit-exact: bf16 blocks whose m or k is no multiple of 8, on small-integer data
(every product and partial sum an integer below 2^24, so any summation order gives the same
fp32 value and the same rounding).  The whole C buffer is compared, so a row window that passed its
block, or a padded row stored, shows."""
from __future__ import annotations

import sys

import numpy as np
import pytest
import torch

import workloads as wk
from helpers import run_oracle
from test_gpu_exact import assert_bits_equal, run_gpu

pytestmark = pytest.mark.gpu

# (m, n, k): one element past and short of a chunk, of the 64-row and 64-k tile edges, and of the
# larger tiles; the smallest that has windows (8) and the element-load instance below it (7)
SHAPES = [(7, 9, 13), (9, 7, 5), (8, 1, 9), (9, 3, 8), (15, 65, 63), (63, 5, 65), (65, 64, 71),
          (71, 130, 127), (100, 33, 129), (129, 131, 77), (257, 260, 70)]


def grid_case(m, n, k, count, kind, c_type, beta, flags, gm, gn, pad, seed):
    """gm x gn instances over padded blocks, all operands small integers."""
    rng = np.random.default_rng(seed)
    lda, ldb, ldc = m + pad, k + pad, m + pad
    ab, bb, cb = lda * k, ldb * n, ldc * n
    ints = lambda size, r: rng.integers(-r, r + 1, size=size).astype(np.float32)
    c = ints(gm * gn * cb, 8)
    arrays = dict(a=wk.bf16_bits(ints(gm * count * ab, 3)), b=wk.bf16_bits(ints(gn * count * bb, 3)),
                  c=c if c_type == "f32" else wk.bf16_bits(c), bias=ints(gm * m, 8))
    assert count * k * 9 + 16 < 1 << 24
    call = wk.Call(m, n, k, lda, ldb, ldc, "bf16", c_type, beta, kind, flags=set(flags), G=gm * gn,
                   grid=dict(gm=gm, gn=gn, a_step_m=count * ab, b_step_n=count * bb, c_step_m=cb,
                             c_step_n=gm * cb, bias_step_m=m),
                   count=count, a="a", b="b", c="c", bias="bias" if "bias" in flags else None)
    if kind == "stride":
        call.stride_a, call.stride_b = ab, bb
    else:
        call.offs_a = (rng.permutation(count) * ab).astype(np.int64)
        call.offs_b = (rng.permutation(count) * bb).astype(np.int64)
    return wk.Workload("ragged", arrays, [call])


@pytest.mark.parametrize("kid", [None, 0, 1, 2])
@pytest.mark.parametrize("m,n,k", SHAPES)
def test_ragged_grid_bit_exact(m, n, k, kid, monkeypatch):
    if kid is not None:
        monkeypatch.setenv("TPP_FORCE_KERNEL", str(kid))
    for i, (kind, c_type, beta, flags, gm, gn, pad) in enumerate([
            ("stride", "bf16", 0.0, ("bias", "relu"), 3, 2, 0),
            ("offset", "f32", 1.0, ("relu",), 2, 3, 1),
            ("stride", "bf16", 1.0, ("bias",), 1, 1, 5)]):
        wl = grid_case(m, n, k, 3, kind, c_type, beta, flags, gm, gn, pad, m * 100 + k + i)
        print(f"ragged {m}x{n}x{k} {kind} {c_type} kernel {kid}", flush=True)
        sys.stdout.flush()
        got, names = run_gpu(wl)
        generic = m < 8 or k < 8
        assert ("vec_kernel" in names[0]) != generic, names
        assert_bits_equal(got["c"], run_oracle(wl)[0], f"{names[0]} {m}x{n}x{k}")


@pytest.mark.parametrize("m,n,k", [(17, 33, 65), (64, 40, 24), (100, 9, 136)])
def test_pointer_lists_at_any_alignment(m, n, k):
    wl = wk.small_case(np.random.default_rng(m), m, n, k, 5, "address", "bf16", "f32", 0.0, set(),
                       pad=1, integer=True)
    print(f"address {m}x{n}x{k}", flush=True)
    got, names = run_gpu(wl)
    ref = run_oracle(wl)[0]
    # the padding rows of C keep the NaN they were filled with on both sides
    assert_bits_equal(got["c"], ref, names[0])


def test_ragged_aux_steps_match_elementwise():
    """SAVE_PREACT and RELU_INV on a ragged m: aux has C's layout, the last chunk row by row."""
    wl = grid_case(27, 19, 45, 2, "stride", "bf16", 0.0, ("bias", "relu", "save_preact"), 3, 2, 1, 5)
    call = wl.calls[0]
    call.aux = "z"
    wl.arrays["z"] = np.full_like(wl.arrays["c"], 0x7FC0)
    plain = wk.Workload("plain", wl.arrays, [wk.Call(**dict(call.__dict__, flags={"bias"}, aux=None))])
    print("ragged save_preact", flush=True)
    got, names = run_gpu(wl)
    z = run_oracle(plain)[0]
    stored = np.zeros(z.shape, bool)
    for g in range(call.G):
        gi, gj = g % 3, g // 3
        base = gi * call.grid["c_step_m"] + gj * call.grid["c_step_n"]
        for c in range(call.n):
            stored[base + c * call.ldc: base + c * call.ldc + call.m] = True
    assert_bits_equal(got["z"][stored], z[stored], names[0])
    assert (got["z"][~stored] == 0x7FC0).all()
    inv = wk.Call(**dict(call.__dict__, flags={"relu_inv"}, bias=None))
    wl2 = wk.Workload("inv", dict(wl.arrays, z=z), [inv])
    nobias = wk.Call(**dict(call.__dict__, flags=set(), aux=None, bias=None))
    v = run_oracle(wk.Workload("v", wl.arrays, [nobias]))[0]
    got2, _ = run_gpu(wl2)
    want = np.where(wk.bf16_values(z) > 0, v, 0).astype(np.uint16)
    assert_bits_equal(got2["c"][stored], want[stored], "relu_inv")
