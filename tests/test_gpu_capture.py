"""Calls that fold partial results in device work space, captured into graphs: a graph's replays must
not depend on what its stream's work buffer has become since, nor on calls that use it meanwhile.
Random fp32 sums differ between the split form and the whole one, so bit equality with the eager call
also shows that the captured call is split as the eager one is."""
from __future__ import annotations

import numpy as np
import pytest
import torch

import workloads as wk

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module", autouse=True)
def gpu():
    assert torch.cuda.is_available(), "GPU tests need an MI355X"


class _Brgemm:
    """One tile of fp32: a single pair of k = 4096, or a pointer list, through the single calls."""

    def __init__(self, kind, k, count, seed):
        import paper_2104_05755_amd as tpp
        self.tpp, self.kind, self.count = tpp, kind, count
        g = torch.Generator(device="cuda")
        g.manual_seed(seed)
        self.a = torch.randn(count * 64 * k, generator=g, device="cuda")
        self.b = torch.randn(count * 64 * k, generator=g, device="cuda")
        self.out = torch.zeros(64 * 64, device="cuda")
        st = 64 * k
        self.h = tpp.tpp_brgemm_dispatch(tpp.make_desc(64, 64, k, 64, k, 64, "f32", "f32", 0.0, kind,
                                                       *((st, st) if kind == "stride" else (0, 0)), []))
        at = lambda x: torch.from_numpy(x.data_ptr() + np.arange(count, dtype=np.int64) * st * 4).cuda()
        self.pa, self.pb = at(self.a), at(self.b)

    def __call__(self, stream):
        if self.kind == "stride":
            self.tpp.tpp_brgemm_execute_stride(self.h, self.a, self.b, self.out, None, self.count,
                                               stream.cuda_stream)
        else:
            self.tpp.tpp_brgemm_execute_address(self.h, self.pa, self.pb, self.out, None, self.count,
                                                stream.cuda_stream)


class _Grid:
    """A bf16 layer of few tiles and a long reduction: split by the direct-to-LDS instances."""

    def __init__(self, tokens, c_in, seed):
        from paper_2104_05755_amd import torch_io
        wl = wk.mlp_fc(seed=seed, minibatch=tokens, c_in=c_in, k_out=256)
        self.dev = torch_io.upload(wl)
        self.dc = torch_io.prepare(wl.calls[0], self.dev)
        assert "split_finish" in torch_io.describe(self.dc)
        self.launch, self.out = torch_io.launch, self.dev[wl.calls[0].c].view(torch.bfloat16)

    def __call__(self, stream):
        self.launch(self.dc, stream.cuda_stream)


class _Reduce:
    """Sums over columns or rows that fold partial results."""

    def __init__(self, by, m, n, seed):
        import paper_2104_05755_amd as tpp
        self.tpp, self.shape = tpp, (m, n)
        g = torch.Generator(device="cuda")
        g.manual_seed(seed)
        self.x = torch.randn(m * n, generator=g, device="cuda")
        self.out = torch.zeros(m if by == "cols" else n, device="cuda")
        self.flags = tpp.TPP_RED_X | (tpp.TPP_RED_BY_COLS if by == "cols" else tpp.TPP_RED_BY_ROWS)

    def __call__(self, stream):
        m, n = self.shape
        self.tpp.tpp_reduce(m, n, m, self.tpp.TPP_DT_F32, self.x, self.tpp.TPP_RED_SUM, self.flags,
                            self.out, None, stream.cuda_stream)


# (the captured call, a call of the same family that needs a larger work buffer)
FORMS = {
    "fp32_single_pair": (lambda s: _Brgemm("stride", 4096, 1, s), lambda s: _Brgemm("stride", 4096, 16, s)),
    "fp32_pointer_list": (lambda s: _Brgemm("address", 64, 12, s), lambda s: _Brgemm("address", 64, 200, s)),
    "bf16_grid": (lambda s: _Grid(128, 2048, s), lambda s: _Grid(256, 4096, s)),
    "reduce_cols": (lambda s: _Reduce("cols", 64, 20000, s), lambda s: _Reduce("cols", 512, 90000, s)),
    "reduce_rows": (lambda s: _Reduce("rows", 60000, 3, s), lambda s: _Reduce("rows", 200000, 40, s)),
}


def eager(call, stream):
    call.out.fill_(float("nan"))
    torch.cuda.synchronize()
    call(stream)
    torch.cuda.synchronize()
    return call.out.clone()


def capture(call, stream):
    g = torch.cuda.CUDAGraph()
    torch.cuda.synchronize()
    with torch.cuda.graph(g, stream=stream):
        call(stream)
    torch.cuda.synchronize()
    return g


@pytest.mark.parametrize("warm", [False, True], ids=["cold", "warm"])
@pytest.mark.parametrize("form", sorted(FORMS))
def test_replay_after_the_work_buffer_has_grown(form, warm):
    make, larger = FORMS[form]
    call, big = make(1), larger(2)
    want, big_want = (eager(c, torch.cuda.Stream()) for c in (call, big))
    print(f"capture {form} {'warm' if warm else 'cold'}", flush=True)
    s = torch.cuda.Stream()
    if warm:
        assert torch.equal(eager(call, s), want)
    g = capture(call, s)
    for _ in range(3):
        assert torch.equal(eager(big, s), big_want)   # the first of them grows the stream's buffer
        call.out.fill_(float("nan"))
        torch.cuda.synchronize()
        g.replay()
        torch.cuda.synchronize()
        assert torch.equal(call.out, want), form


@pytest.mark.parametrize("form", sorted(FORMS))
def test_replays_beside_calls_and_other_graphs_of_the_stream(form):
    """Two graphs captured on one stream, replayed on two others while that stream runs eager
    calls of the same family."""
    calls = [FORMS[form][0](seed) for seed in (1, 2, 3)]
    want = [eager(c, torch.cuda.Stream()) for c in calls]
    print(f"capture beside {form}", flush=True)
    s, r0, r1 = (torch.cuda.Stream() for _ in range(3))
    assert torch.equal(eager(calls[2], s), want[2])
    g0, g1 = capture(calls[0], s), capture(calls[1], s)
    for _ in range(20):
        for c in calls:
            c.out.fill_(float("nan"))
        torch.cuda.synchronize()
        for _ in range(10):
            with torch.cuda.stream(r0):
                g0.replay()
            with torch.cuda.stream(r1):
                g1.replay()
            calls[2](s)
        torch.cuda.synchronize()
        for c, w in zip(calls, want):
            assert torch.equal(c.out, w), form
