"""Transposes and VNNI reformatting at any alignment and order of tiles: the windows of last, partial
64 x 64 tiles, tiles numbered along the output with a contiguous run per XCD (workgroup counts that
are and are not multiples of 8), 16-byte accesses at entry alignment.  The transforms only move
entries, so the whole output buffer, gaps between rows included, has to equal the oracle's."""
from __future__ import annotations

import numpy as np
import pytest
import torch

import oracle

pytestmark = pytest.mark.gpu

# 64: one tile; 65, 127: windows that start 1 and 63 entries in; 63: entry by entry; 190 x 129 and
# 513 x 65: runs per XCD with a remainder
SIZES = [(64, 64), (65, 64), (64, 71), (65, 65), (127, 127), (63, 200), (200, 63), (190, 129),
         (513, 65), (1, 300), (512, 130)]


@pytest.mark.parametrize("dtype", ["bf16", "f32"])
@pytest.mark.parametrize("kind,alpha", [("transpose", 1), ("vnni", 2), ("vnni", 4), ("vnni_t", 2),
                                        ("vnni_t", 4)])
@pytest.mark.parametrize("m,n", SIZES)
@pytest.mark.parametrize("G,pad,shift", [(1, 0, 0), (3, 1, 1), (9, 5, 3)])
def test_any_alignment_matches_the_oracle(dtype, kind, alpha, m, n, G, pad, shift):
    import paper_2104_05755_amd as tpp
    nt, st = (np.uint32, torch.int32) if dtype == "f32" else (np.uint16, torch.int16)
    si = np.int32 if dtype == "f32" else np.int16
    gm, gn = -(-m // alpha), -(-n // alpha)
    ld_in, rows_in, ld_out, rows_out = {
        "transpose": (m, n, n, m), "vnni": (m, n, m * alpha, gn),
        "vnni_t": (m * alpha, gn, n * alpha, gm)}[kind]
    ld_in, ld_out = ld_in + pad, ld_out + 2 * pad
    s_in, s_out = ld_in * rows_in + pad, ld_out * rows_out + pad
    rng = np.random.default_rng(m * 1000 + n)
    x = rng.integers(0, 2 ** (32 if dtype == "f32" else 16), size=G * s_in, dtype=np.uint64).astype(nt)
    want = np.full(G * s_out, 0xBEEF, dtype=nt)
    view = (lambda a: a.view(np.float32)) if dtype == "f32" else (lambda a: a)
    for g in range(G):
        xi, oi = x[g * s_in:(g + 1) * s_in].copy(), want[g * s_out:(g + 1) * s_out].copy()
        oracle.transform(kind, m, n, ld_in, ld_out, dtype, alpha, view(xi), view(oi))
        want[g * s_out:(g + 1) * s_out] = oi
    xd = torch.zeros(G * s_in + shift, dtype=st, device="cuda")
    xd[shift:] = torch.from_numpy(x.view(si)).cuda()
    od = torch.from_numpy(np.full(G * s_out + shift, 0xBEEF, dtype=nt).view(si)).cuda()
    tpp.tpp_transform_batched({"transpose": 0, "vnni": 1, "vnni_t": 2}[kind], m, n, ld_in, ld_out,
                              tpp.TPP_DT_F32 if dtype == "f32" else tpp.TPP_DT_BF16, alpha,
                              xd[shift:].data_ptr(), s_in, od[shift:].data_ptr(), s_out, G)
    torch.cuda.synchronize()
    got = od.cpu().numpy().view(nt)
    assert (got[:shift] == 0xBEEF).all()
    assert (got[shift:] == want).all()


# whole 128-byte lines: launch order below 32 MiB, in one-tile strips and past 384 MiB, runs per XCD
# in between; a line shared by tiles: runs at any size
@pytest.mark.parametrize("m,n,G,pad", [(1024, 2048, 1, 0), (2048, 2048, 1, 0), (4096, 2176, 1, 0),
                                       (64, 131072, 1, 0), (131072, 64, 1, 0), (10240, 5184, 1, 0),
                                       (1024, 1088, 9, 0), (2048, 2048, 1, 1), (10240, 5184, 1, 1)])
def test_orders_of_tiles(m, n, G, pad):
    import paper_2104_05755_amd as tpp
    print(f"transpose {G} x {m} x {n} pad {pad}", flush=True)
    x = torch.arange(G * n * (m + pad), dtype=torch.int32, device="cuda")
    y = torch.full((G, m, n), -1, dtype=torch.int32, device="cuda")
    tpp.tpp_transform_batched(tpp.TPP_TR_TRANSPOSE, m, n, m + pad, n, tpp.TPP_DT_F32, 1, x,
                              n * (m + pad), y, m * n, G, tpp.current_stream())
    torch.cuda.synchronize()
    assert torch.equal(y, x.view(G, n, m + pad)[:, :, :m].transpose(1, 2))
    # alpha 2: groups of two columns in, groups of two rows out
    if pad == 0:
        y.fill_(-1)
        tpp.tpp_transform_batched(tpp.TPP_TR_VNNI_TO_VNNI_T, m, n, 2 * m, 2 * n, tpp.TPP_DT_F32, 2, x,
                                  n * m, y, m * n, G, tpp.current_stream())
        torch.cuda.synchronize()
        a = x.view(G, n // 2, m // 2, 2, 2)                  # [g][c/2][r/2][r%2][c%2]
        assert torch.equal(y.view(G, m // 2, n // 2, 2, 2), a.permute(0, 2, 1, 4, 3))
