"""GPU Reduce TPP, exact on integer data: every group width of the by-rows kernel (8 to 64 lanes per
column), row tails and bases at any element, the by-columns window of the last rows and its
shared-slot fold, both combine widths, and a call captured on a stream that has no work buffer.  Values are integers of at most 8 in magnitude and sums stay below 2^24, so fp32 sums are
exact in any order and the reference is numpy's integer sum."""
from __future__ import annotations

import numpy as np
import pytest
import torch

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module", autouse=True)
def gpu():
    assert torch.cuda.is_available(), "GPU tests need an MI355X"


def call(x, m, n, ld, op, by, flags="x2", G=1, in_stride=0, stream=None):
    import paper_2104_05755_amd as tpp
    no = m if by == "cols" else n
    ox = torch.full((G * no,), float("nan"), device="cuda")
    ox2 = torch.full((G * no,), float("nan"), device="cuda")
    f = (tpp.TPP_RED_BY_COLS if by == "cols" else tpp.TPP_RED_BY_ROWS)
    f |= (tpp.TPP_RED_X if "x" in flags else 0) | (tpp.TPP_RED_X2 if "2" in flags else 0)
    dt = tpp.TPP_DT_BF16 if x.dtype == torch.bfloat16 else tpp.TPP_DT_F32
    tpp.tpp_reduce_batched(m, n, ld, dt, x, G, in_stride, op, f, ox if "x" in flags else None,
                           ox2 if "2" in flags else None, no, stream or tpp.current_stream())
    return ox, ox2


def check(m, n, pad, shift, dtype, by, G=1):
    import paper_2104_05755_amd as tpp
    rng = np.random.default_rng(m * 31 + n * 7 + pad + shift)
    ld = m + pad
    v = rng.integers(-8, 9, G * n * ld + shift)
    x = torch.from_numpy(v.astype(np.float32)).to(dtype).cuda()[shift:]
    a = v[shift:].reshape(G, n, ld)[:, :, :m]
    axis = 1 if by == "cols" else 2
    print(f"reduce by {by} {m}x{n} G{G} pad {pad} shift {shift} {dtype}", flush=True)
    for op, f in ((tpp.TPP_RED_SUM, np.sum), (tpp.TPP_RED_MAX, np.max)):
        ox, ox2 = call(x, m, n, ld, op, by, G=G, in_stride=n * ld)
        torch.cuda.synchronize()
        assert np.array_equal(ox.cpu().numpy(), f(a, axis=axis).reshape(-1))
        assert np.array_equal(ox2.cpu().numpy(), f(a * a, axis=axis).reshape(-1))
    ox, _ = call(x, m, n, ld, tpp.TPP_RED_SUM, by, flags="x", G=G, in_stride=n * ld)
    _, ox2 = call(x, m, n, ld, tpp.TPP_RED_MIN, by, flags="2", G=G, in_stride=n * ld)
    torch.cuda.synchronize()
    assert np.array_equal(ox.cpu().numpy(), a.sum(axis=axis).reshape(-1))
    assert np.array_equal(ox2.cpu().numpy(), (a * a).min(axis=axis).reshape(-1))


@pytest.mark.parametrize("dtype", [torch.float32, torch.bfloat16])
@pytest.mark.parametrize("m", [1, 3, 7, 8, 9, 31, 33, 64, 65, 127, 129, 255, 257, 511, 513, 1030])
def test_rows_group_widths_and_tails(m, dtype):
    # 4096 columns: one round per wavefront; 70000 short columns: two or four
    check(m, 4096, 0, 0, dtype, "rows")
    check(m, 4099, 1, 1, dtype, "rows")
    if m <= 65:
        check(m, 70001, 0, 3, dtype, "rows")


@pytest.mark.parametrize("dtype", [torch.float32, torch.bfloat16])
@pytest.mark.parametrize("m", [1, 3, 8, 9, 20, 63, 65, 130, 511, 513, 1001])
def test_cols_windows_and_combine_widths(m, dtype):
    for n in (1, 5, 70, 2000):
        check(m, n, n % 3, m % 2, dtype, "cols")


@pytest.mark.parametrize("dtype", [torch.float32, torch.bfloat16])
@pytest.mark.parametrize("m,n,G", [(17, 9, 40), (3, 32, 7), (16, 8, 5), (65, 8, 3), (100000, 10, 1), (9000, 1, 1),
                                   (2100, 3, 2), (4096, 64, 1), (1030, 130, 1), (257, 3000, 1), (300, 2001, 2)])
def test_cols_plans(m, n, G, dtype):
    # one wavefront per small block, more row vectors than 64 for few columns, one pass in place of
    # two ranges, row blocks of 16 and 8 vectors for an uneven number of rows
    check(m, n, 0, 0, dtype, "cols", G=G)
    check(m, n, 1, 1, dtype, "cols", G=G)


def test_batched_blocks_at_any_alignment():
    check(61, 67, 2, 1, torch.bfloat16, "cols", G=9)
    check(61, 67, 2, 1, torch.float32, "rows", G=9)


@pytest.mark.parametrize("by,m,n", [("cols", 64, 40000), ("rows", 60000, 5)])
def test_capture_without_a_work_buffer(by, m, n):
    """A shape that folds partial results, captured on a stream that has no work buffer.  Replays
    see the inputs of their time."""
    import paper_2104_05755_amd as tpp
    s = torch.cuda.Stream()
    x = torch.zeros(m * n, dtype=torch.bfloat16, device="cuda")
    g = torch.cuda.CUDAGraph()
    print(f"capture by {by} {m}x{n}", flush=True)
    torch.cuda.synchronize()
    with torch.cuda.graph(g, stream=s):
        ox, ox2 = call(x, m, n, m, tpp.TPP_RED_SUM, by, stream=s.cuda_stream)
    for seed in (1, 2, 3):
        v = np.random.default_rng(seed).integers(-4, 5, m * n)
        x.copy_(torch.from_numpy(v.astype(np.float32)))
        torch.cuda.synchronize()
        g.replay()
        torch.cuda.synchronize()
        a = v.reshape(n, m)
        assert np.array_equal(ox.cpu().numpy(), a.sum(axis=0 if by == "cols" else 1))
        assert np.array_equal(ox2.cpu().numpy(), (a * a).sum(axis=0 if by == "cols" else 1))


@pytest.mark.parametrize("by,m,n", [("rows", 2 ** 31 - 1, 1), ("cols", 1, 2 ** 31 - 1),
                                    ("cols", 3, 2 ** 31 - 1), ("cols", 2 ** 31 - 1, 1)])
@pytest.mark.parametrize("captured", [False, True])
def test_extents_at_the_top_of_int32(by, m, n, captured):
    """Row segments, column ranges and windows whose ends pass 2^31 - 1.  x(e) = (e mod 61) - 30: any
    run sums to less than 2^24 in magnitude in whatever order, and every residue comes up in the
    strided part of each thread."""
    import paper_2104_05755_amd as tpp
    total = m * n
    print(f"reduce by {by} {m} x {n} captured {captured}", flush=True)
    x = torch.empty(total, dtype=torch.bfloat16, device="cuda")
    for s in range(0, total, 1 << 27):
        e = torch.arange(s, min(s + (1 << 27), total), dtype=torch.int64, device="cuda")
        x[s:s + e.numel()] = ((e % 61) - 30).to(torch.bfloat16)
    stream = torch.cuda.Stream()
    torch.cuda.synchronize()
    if captured:
        g = torch.cuda.CUDAGraph()
        with torch.cuda.graph(g, stream=stream):
            ox, _ = call(x, m, n, m, tpp.TPP_RED_SUM, by, flags="x", stream=stream.cuda_stream)
            mx, _ = call(x, m, n, m, tpp.TPP_RED_MAX, by, flags="x", stream=stream.cuda_stream)
        g.replay()
    else:
        with torch.cuda.stream(stream):
            ox, _ = call(x, m, n, m, tpp.TPP_RED_SUM, by, flags="x")
            mx, _ = call(x, m, n, m, tpp.TPP_RED_MAX, by, flags="x")
    torch.cuda.synchronize()
    if (m if by == "cols" else n) <= 3:   # few outputs, each over every m-th (or every) element
        step = m if by == "cols" else 1
        for o in range(m if by == "cols" else n):
            count = (total - o + step - 1) // step
            # whole periods of 61 sum to zero (61 is prime: any step walks all residues)
            rest = sum((o + step * i) % 61 - 30 for i in range(count - count % 61, count))
            assert ox[o].item() == rest and mx[o].item() == 30
    else:                                 # one column: a copy
        for s in range(0, total, 1 << 27):
            e = torch.arange(s, min(s + (1 << 27), total), dtype=torch.int64, device="cuda")
            want = ((e % 61) - 30).float()
            assert torch.equal(ox[s:s + e.numel()], want) and torch.equal(mx[s:s + e.numel()], want)


@pytest.mark.parametrize("captured", [False, True])
def test_combine_of_2_pow_28_outputs(captured):
    """A batch whose partial results have so many outputs that 16 per workgroup of the combine pass
    would pass a grid's 2^32 threads.  Every call reads the same block (in_stride 0).  Captured, its
    partials would pass the 4 GiB that captures may take, and it runs with one partial per output."""
    import paper_2104_05755_amd as tpp
    m, n, G = 512, 40, (1 << 19) + 3
    v = np.random.default_rng(5).integers(-8, 9, n * m)
    x = torch.from_numpy(v.astype(np.float32)).to(torch.bfloat16).cuda()
    print(f"reduce by cols {m} x {n}, {G} calls, captured {captured}", flush=True)
    if captured:
        s, g = torch.cuda.Stream(), torch.cuda.CUDAGraph()
        torch.cuda.synchronize()
        with torch.cuda.graph(g, stream=s):
            ox, _ = call(x, m, n, m, tpp.TPP_RED_SUM, "cols", flags="x", G=G, stream=s.cuda_stream)
        g.replay()
    else:
        ox, _ = call(x, m, n, m, tpp.TPP_RED_SUM, "cols", flags="x", G=G)
    torch.cuda.synchronize()
    want = torch.from_numpy(v.reshape(n, m).sum(axis=0).astype(np.float32)).cuda()
    assert bool((ox.view(G, m) == want).all())
