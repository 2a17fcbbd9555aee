"""GPU parity, bit-exact: bf16 blocks whose m or k is no multiple of 8 and fp32 blocks of any size, on small-integer data
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


def grid_case(m, n, k, count, kind, c_type, beta, flags, gm, gn, pad, seed, ab_type="bf16"):
    """gm x gn instances over padded blocks, all operands small integers."""
    rng = np.random.default_rng(seed)
    lda, ldb, ldc = m + pad, k + pad, m + pad
    ab, bb, cb = lda * k, ldb * n, ldc * n
    ints = lambda size, r: rng.integers(-r, r + 1, size=size).astype(np.float32)
    c = ints(gm * gn * cb, 8)
    conv = wk.bf16_bits if ab_type == "bf16" else lambda v: v
    arrays = dict(a=conv(ints(gm * count * ab, 3)), b=conv(ints(gn * count * bb, 3)),
                  c=c if c_type == "f32" else wk.bf16_bits(c), bias=ints(gm * m, 8))
    assert count * k * 9 + 16 < 1 << 24
    call = wk.Call(m, n, k, lda, ldb, ldc, ab_type, c_type, beta, kind, flags=set(flags), G=gm * gn,
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


@pytest.mark.parametrize("kid", [None, 0, 1, 2])
@pytest.mark.parametrize("k", [8, 24, 40, 56, 72, 120, 136, 9, 31, 73])
def test_partial_stages_of_k_bit_exact(k, kid, monkeypatch):
    """Every block ends with a partial stage (most have no other): the operands are masked on their way
    to LDS, one or two stages after their loads."""
    if kid is not None:
        monkeypatch.setenv("TPP_FORCE_KERNEL", str(kid))
    for m, count in ((64, 1), (72, 2), (60, 5)):
        wl = grid_case(m, 70, k, count, "stride", "f32", 0.0, (), 2, 2, 0, k + m)
        print(f"partial stages {m}x70x{k} count {count} kernel {kid}", flush=True)
        got, names = run_gpu(wl)
        assert "vec_kernel" in names[0], names
        assert_bits_equal(got["c"], run_oracle(wl)[0], names[0])


@pytest.mark.parametrize("m,n,k", [(17, 33, 65), (64, 40, 24), (100, 9, 136)])
def test_pointer_lists_at_any_alignment(m, n, k):
    wl = wk.small_case(np.random.default_rng(m), m, n, k, 5, "address", "bf16", "f32", 0.0, set(),
                       pad=1, integer=True)
    print(f"address {m}x{n}x{k}", flush=True)
    got, names = run_gpu(wl)
    ref = run_oracle(wl)[0]
    # the padding rows of C keep the NaN they were filled with on both sides
    assert_bits_equal(got["c"], ref, names[0])


@pytest.mark.parametrize("ab_type,c_type,k", [("bf16", "bf16", 45), ("bf16", "f32", 45), ("f32", "f32", 45),
                                              ("f32", "bf16", 45), ("f32", "f32", 20)])
def test_ragged_aux_steps_match_elementwise(ab_type, c_type, k):
    """SAVE_PREACT and RELU_INV on a ragged m: aux has C's layout, the last chunk row by row."""
    wl = grid_case(27, 19, k, 2, "stride", c_type, 0.0, ("bias", "relu", "save_preact"), 3, 2, 1, 5, ab_type)
    call = wl.calls[0]
    call.aux = "z"
    gap = np.float32(-77) if c_type == "f32" else np.uint16(0x7FC0)
    wl.arrays["z"] = np.full_like(wl.arrays["c"], gap)
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
    assert (got["z"][~stored] == gap).all()
    inv = wk.Call(**dict(call.__dict__, flags={"relu_inv"}, bias=None))
    wl2 = wk.Workload("inv", dict(wl.arrays, z=z), [inv])
    nobias = wk.Call(**dict(call.__dict__, flags=set(), aux=None, bias=None))
    v = run_oracle(wk.Workload("v", wl.arrays, [nobias]))[0]
    got2, _ = run_gpu(wl2)
    z32 = wk.bf16_values(z) if c_type == "bf16" else z
    want = np.where(z32 > 0, v, 0).astype(v.dtype)
    assert_bits_equal(got2["c"][stored], want[stored], "relu_inv")


# fp32: windows of 4 rows and 4 k, 64-k stages shared by two groups of waves, split stage lists
F32_SHAPES = [(3, 9, 5), (4, 4, 4), (5, 1, 7), (7, 65, 63), (63, 5, 65), (65, 64, 71), (68, 130, 32),
              (100, 33, 129), (130, 66, 200)]


@pytest.mark.parametrize("split", [None, 1, 3])
@pytest.mark.parametrize("m,n,k", F32_SHAPES)
def test_fp32_grid_bit_exact(m, n, k, split, monkeypatch):
    if split is not None:
        monkeypatch.setenv("TPP_SPLIT", str(split))
    for i, (kind, c_type, beta, flags, gm, gn, pad) in enumerate([
            ("stride", "f32", 0.0, ("bias", "relu"), 3, 2, 0),
            ("offset", "bf16", 1.0, ("bias",), 2, 3, 1),
            ("stride", "f32", 1.0, (), 1, 1, 5)]):
        wl = grid_case(m, n, k, 3, kind, c_type, beta, flags, gm, gn, pad, m * 100 + k + i, "f32")
        print(f"fp32 {m}x{n}x{k} {kind} {c_type} split {split}", flush=True)
        got, names = run_gpu(wl)
        assert ("kernel<true>" in names[0]) == (m >= 4 and k >= 4), names
        assert_bits_equal(got["c"], run_oracle(wl)[0], f"{names[0]} {m}x{n}x{k}")


@pytest.mark.parametrize("k", [4, 8, 9, 16, 17, 24, 31, 32, 36, 64, 65, 96, 100])
@pytest.mark.parametrize("kind", ["stride", "offset", "address"])
def test_fp32_steps_of_two_pairs_in_a_stage(kind, k):
    """An odd number of 32-k steps per block: a stage may hold the last step of one pair and the first
    of the next, and the last stage a single step; one to four groups of 8 k per step."""
    for count in (1, 2, 3, 8, 67):
        for split in (None, "3"):
            wl = wk.small_case(np.random.default_rng(k + count), 68, 70, k, count, kind, "f32", "f32", 0.0,
                               {"bias"}, pad=1 if count == 3 else 0, integer=True)
            print(f"fp32 {kind} k {k} count {count} split {split}", flush=True)
            with pytest.MonkeyPatch.context() as mp:
                if split:
                    mp.setenv("TPP_SPLIT", split)
                got, names = run_gpu(wl)
            assert ("paired" in names[0]) == ((k + 31) // 32 % 2 == 1), names
            assert_bits_equal(got["c"], run_oracle(wl)[0], f"{names[0]} {kind} {k} x {count}")


@pytest.mark.parametrize("count", [1, 5, 64, 65, 130])
@pytest.mark.parametrize("kind", ["offset", "address"])
def test_fp32_lists_past_64_pairs(kind, count):
    # the entries of 64 pairs are held in lanes and refilled
    wl = wk.small_case(np.random.default_rng(count), 36, 20, 24, count, kind, "f32", "f32", 1.0,
                       {"bias"}, pad=1, integer=True)
    print(f"fp32 {kind} of {count}", flush=True)
    got, names = run_gpu(wl)
    assert_bits_equal(got["c"], run_oracle(wl)[0], names[0])


def test_fp32_split_call_under_capture():
    """A split call captured on a stream that has no work buffer yet."""
    from paper_2104_05755_amd import torch_io
    wl = grid_case(64, 64, 64, 8, "stride", "f32", 0.0, (), 1, 1, 0, 3, "f32")
    dev = torch_io.upload(wl)
    dc = torch_io.prepare(wl.calls[0], dev)
    assert "split_finish" in torch_io.describe(dc)
    s, g = torch.cuda.Stream(), torch.cuda.CUDAGraph()
    print("capture", flush=True)
    torch.cuda.synchronize()
    with torch.cuda.graph(g, stream=s):
        torch_io.launch(dc, s.cuda_stream)
    ref = run_oracle(wl)[0]
    for _ in range(3):
        dev["c"].fill_(float("nan"))
        torch.cuda.synchronize()
        g.replay()
        torch.cuda.synchronize()
        assert_bits_equal(torch_io.to_host(dev["c"], wl.arrays["c"]), ref, "replay")


def test_fp32_instances_past_2_pow_23():
    """More instances than 512 threads each fit a grid (the element kernel takes them)."""
    import paper_2104_05755_amd as tpp
    G, e, blocks = 2 ** 23 + 5, 16, 61
    g = torch.Generator(device="cuda")
    g.manual_seed(3)
    a, b = (torch.randint(-4, 5, (blocks, e), generator=g, device="cuda").float() for _ in range(2))
    c = torch.full((G * e,), float("nan"), device="cuda")
    i = torch.arange(G, dtype=torch.int64, device="cuda")
    h = tpp.tpp_brgemm_dispatch(tpp.make_desc(4, 4, 4, 4, 4, 4, "f32", "f32", 0.0, "stride", 0, 0, []))
    a_off, b_off, c_off = i % blocks * e, i % (blocks - 1) * e, i * e
    print(f"fp32 4x4x4 x {G}", flush=True)
    tpp.tpp_brgemm_execute_batched(h, None, G, a_off, b_off, c_off, None, a, b, c, None, 1, None, None,
                                   None, None, None, tpp.current_stream())
    torch.cuda.synchronize()
    # blocks are column-major: a[k][row], b[col][k], c[col][row]; elementwise products, exact
    at, bt = a.view(blocks, 1, 4, 4), b.view(blocks, 4, 4, 1)
    for s in range(0, G, 1 << 20):
        j = i[s:s + (1 << 20)]
        want = (at[j % blocks] * bt[j % (blocks - 1)]).sum(dim=2)
        assert torch.equal(c[s * e:(s + j.numel()) * e].view(-1, 4, 4), want)
