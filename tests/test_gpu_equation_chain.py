"""GPU parity of equations whose tree is one running value taking a leaf, a row-uniform subtree or
a pair of them per operation (the forms of norms, softmaxes, biases, scalings and residuals), against
the oracle: random trees over every operation and operand order, every broadcast form and datatype,
at rows around a chunk of 8 and a wavefront's 64 chunks, with padded leading dimensions, in place,
and on infinities and NaN.  Small integers keep every value exact (below 2^24), so the comparison
is equality."""
from __future__ import annotations

import numpy as np
import pytest
import torch

import oracle
import workloads as wk
from helpers import values
from test_gpu_equation import gpu_steps, one

pytestmark = pytest.mark.gpu

ROWS = [8, 9, 15, 63, 64, 65, 257, 511, 512, 520, 1025]


class _Tree:
    def __init__(self, rng):
        self.rng, self.nodes, self.specs = rng, [], []

    def add(self, *node):
        self.nodes.append(node)
        return len(self.nodes) - 1

    def leaf(self, kinds):
        bc = str(self.rng.choice(kinds))
        self.specs.append((-2, 2, str(self.rng.choice(["f32", "bf16"])), bc,
                           int(self.rng.integers(0, 4))))
        return self.add("leaf", len(self.specs) - 1)

    def operand(self):
        """A leaf of any form, or a subtree that is the same for all rows."""
        kind = self.rng.integers(0, 3)
        if kind < 2:
            return self.leaf(["none", "col", "row", "scalar"] if kind else ["row", "scalar"])
        a = self.leaf(["row"])
        b = self.leaf(["row", "scalar"])
        return self.add(str(self.rng.choice(["add", "mul", "max"])), a, b)

    def chain(self, steps, last):
        x = self.leaf(["none"])
        for _ in range(steps):
            op = str(self.rng.choice(["add", "sub", "mul", "muladd", "neg", "identity"]))
            if op in ("neg", "identity"):
                x = self.add(op, x)
            elif op == "muladd":
                a, b = self.operand(), self.operand()
                kids = [(x, a, b), (a, x, b), (a, b, x)][int(self.rng.integers(0, 3))]
                x = self.add(op, *kids)
            else:
                a = self.operand()
                x = self.add(op, x, a) if self.rng.integers(0, 2) else self.add(op, a, x)
        return self.add(last, x)


@pytest.mark.parametrize("m", ROWS)
@pytest.mark.parametrize("n", [1, 3, 70])
def test_random_chains_exact(m, n):
    rng = np.random.default_rng(m * 1000 + n)
    for i in range(12):
        t = _Tree(rng)
        root = t.chain(int(rng.integers(0, 5)), str(rng.choice(["identity", "relu", "neg"])))
        out_type = "bf16" if i % 2 else "f32"
        print(f"chain {m}x{n} {out_type} {t.nodes}", flush=True)
        # at most 4 steps of at most x -> 8 x + 8 on values of at most 2: below 2^24
        g, r, got, init = one(t.nodes, root, m, n, t.specs, out_type=out_type,
                              ldo=m + int(rng.integers(0, 3)), seed=i, integer=True)
        assert np.array_equal(g, r)
        ldo = got.size // n
        bits = lambda x: x.view(np.uint32 if x.dtype == np.float32 else np.uint16).reshape(n, ldo)
        assert np.array_equal(bits(got)[:, m:], bits(init)[:, m:])   # gaps untouched


@pytest.mark.parametrize("m,n", [(256, 20000), (64, 70001), (8, 600003), (520, 20003), (33, 130000)])
def test_several_steps_per_wavefront(m, n):
    """Enough columns that a wavefront takes several steps of them, one or more columns each (64 /
    chunks of 8 rows), and loads the full leaves of the next step ahead; the last column tile is
    partial."""
    specs = [(-2, 2, "bf16", "none", 1), (-2, 2, "f32", "row", 0), (-2, 2, "f32", "col", 0),
             (-2, 2, "f32", "none", 0), (-2, 2, "bf16", "row", 0)]
    nodes = [("leaf", 0), ("leaf", 1), ("sub", 0, 1), ("leaf", 2), ("leaf", 3), ("muladd", 2, 3, 4),
             ("leaf", 4), ("mul", 5, 6), ("relu", 7)]
    for out_type in ("f32", "bf16"):
        print(f"chain {m}x{n} {out_type}", flush=True)
        g, r, _, _ = one(nodes, 8, m, n, specs, out_type=out_type, ldo=m + 1, seed=m, integer=True)
        assert np.array_equal(g, r)


@pytest.mark.parametrize("m", [9, 64, 517])
def test_chain_in_place(m):
    # out is the full leaf exactly: the window of a column's last rows re-reads rows that other
    # lanes may have stored already
    n = 37
    rng = np.random.default_rng(m)
    x = rng.integers(-8, 9, m * n).astype(np.float32)
    row = rng.integers(-8, 9, n).astype(np.float32)
    nodes = [("leaf", 0), ("leaf", 1), ("sub", 0, 1), ("leaf", 1), ("mul", 2, 3)]
    st = wk.EquationStep(nodes, 4, m, n, [("x", m, "f32", "none"), ("row", 1, "f32", "row")], "x", m,
                         "f32")
    print(f"in place {m}", flush=True)
    got = gpu_steps([st], dict(x=x, row=row), ["x"])["x"].reshape(n, m)
    want = (x.reshape(n, m) - row[:, None]) * row[:, None]
    assert np.array_equal(got, want)


def test_infinities_nan_and_signed_zeros():
    """x + o, x - o, o - x, x o and muladd give what IEEE arithmetic gives: the forms with 1 and
    -0 in place of an operand keep infinities, NaN and the signs of zeros."""
    special = np.array([0.0, -0.0, 1.0, -1.0, np.inf, -np.inf, np.nan, 1e-38, -3e38], np.float32)
    m, n = special.size, special.size
    x = np.tile(special, n)                       # column c holds every value
    for op, f in (("add", np.add), ("sub", np.subtract), ("mul", np.multiply)):
        for swap in (False, True):
            nodes = [("leaf", 0), ("leaf", 1), (op, 1, 0) if swap else (op, 0, 1)]
            st = wk.EquationStep(nodes, 2, m, n, [("x", m, "f32", "none"), ("row", 1, "f32", "row")],
                                 "out", m, "f32")
            arrays = dict(x=x, row=special, out=np.zeros(m * n, np.float32))
            print(f"special values {op} swap={swap}", flush=True)
            got = gpu_steps([st], arrays, ["out"])["out"].reshape(n, m)
            a, b = x.reshape(n, m), special[:, None]
            with np.errstate(all="ignore"):
                want = f(b, a) if swap else f(a, b)
            assert np.array_equal(got, want, equal_nan=True), op
            live = ~np.isnan(want)
            assert np.array_equal(np.signbit(got[live]), np.signbit(want[live])), op


@pytest.mark.parametrize("m,n", [(1, 70000), (3, 30000), (5, 14000)])
def test_few_contiguous_rows(m, n):
    # more than 65536 elements in fewer than 8 contiguous rows: run as one column
    specs = [(-3, 3, "bf16", "none", 0), (-3, 3, "f32", "scalar", 0)]
    nodes = [("leaf", 0), ("leaf", 1), ("mul", 0, 1), ("leaf", 0), ("add", 2, 3)]
    if m == 1:
        specs += [(-3, 3, "f32", "row", 0), (-3, 3, "f32", "col", 0)]
        nodes += [("leaf", 2), ("sub", 4, 5), ("leaf", 3), ("mul", 6, 7)]
    print(f"few rows {m}x{n}", flush=True)
    g, r, _, _ = one(nodes, len(nodes) - 1, m, n, specs, seed=m, integer=True)
    assert np.array_equal(g, r)


TOP = 2 ** 31 - 1


def _top_case(m, n, nodes, root, leaves, want):
    """out = want(r, c) over an m x n bf16 output with 64 guard entries behind it."""
    import paper_2104_05755_amd as tpp
    total = m * n
    out = torch.full((total + 64,), -1.0, dtype=torch.bfloat16, device="cuda")
    print(f"equation {m} x {n}", flush=True)
    tpp.tpp_equation_execute(nodes, root, m, n, [(x, ld, tpp.TPP_DT_BF16, bc) for x, ld, bc in leaves],
                             out, m, tpp.TPP_DT_BF16, tpp.current_stream())
    torch.cuda.synchronize()
    assert bool((out[total:] == -1).all()), "stored past the output"
    chunk = 1 << 26
    # all of an output of one column or row, the two ends of a larger one
    starts = range(0, total, chunk) if total <= TOP else (0, total - chunk)
    for s in starts:
        e = torch.arange(s, min(s + chunk, total), dtype=torch.int64, device="cuda")
        assert bool((out[s:s + e.numel()].float() == want(e % m, e // m)).all()), s


def test_extents_at_the_top_of_int32():
    """Rows and columns within a chunk of 2^31: the last window and the host's tile counts do not wrap.
    One contiguous row (run as one column by the chain kernel), one column of a tree that is no
    chain, and 8 x (2^31 - 1) over column tiles."""
    def pattern(n):
        x = torch.empty(n, dtype=torch.bfloat16, device="cuda")
        for s in range(0, n, 1 << 26):
            e = torch.arange(s, min(s + (1 << 26), n), dtype=torch.int64, device="cuda")
            x[s:s + e.numel()] = ((e % 61) - 30).to(torch.bfloat16)
        return x
    at = lambda e: ((e % 61) - 30).float()
    x = pattern(TOP)
    two = torch.full((1,), 2.0, dtype=torch.bfloat16, device="cuda")
    scaled = [("leaf", 0), ("leaf", 1), ("mul", 0, 1)]
    _top_case(1, TOP, scaled, 2, [(x, 1, "none"), (two, 1, "scalar")], lambda r, c: 2 * at(c))
    larger = [("leaf", 0), ("leaf", 1), ("max", 0, 1)]
    _top_case(TOP - 2, 1, larger, 2, [(x, TOP - 2, "none"), (two, 1, "scalar")],
              lambda r, c: at(r).clamp(min=2))
    col = torch.arange(8, dtype=torch.float32, device="cuda").to(torch.bfloat16)
    added = [("leaf", 0), ("leaf", 1), ("add", 0, 1)]
    _top_case(8, TOP, added, 2, [(col, 1, "col"), (x, 1, "row")], lambda r, c: r.float() + at(c))
