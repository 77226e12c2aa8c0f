"""GPU parity of the 1-D composition chain at the edges of its staging: rows
that are staged whole and rows just long enough to be windowed, chains whose
cells can be predicted and chains whose cells jump across the row (sec. 3's
lookups lambda_{j+1} = phi^j(lambda_j) over hand-written tables), ranges
shorter than and around a group of 4 and a block of 64 slices, states that
leave the grid, and a non-finite entry at any place of a group.  Every
composition equals the oracle's over the same tables to the bit (the lookup
and the interpolants are specified operation for operation)."""
import sys

import numpy as np
import pytest

from paper_1304_6514_amd import nv
from paper_1304_6514_amd import workloads as W

pytestmark = pytest.mark.gpu

LO, HI = -1.0, 1.0


def say(*a):
    print("[gpu-test]", *a, file=sys.__stderr__, flush=True)


@pytest.fixture(scope="module")
def torch():
    torch = pytest.importorskip("torch")
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    nv.load()
    return torch


@pytest.fixture(scope="module")
def orc():
    import oracle
    oracle.build()
    return oracle


def tables(kind, n_slices, n, interp):
    """(components, n_slices, n) FP64 tables of slice maps on [-1, 1]: "drift"
    moves the state slowly, "wild" is x -> 1 - 2 x^2 (chaotic: no cell follows
    from the ones before), "leave" expands, so the state leaves the grid."""
    x = np.linspace(LO, HI, n)[None, :]
    j = np.arange(n_slices)[:, None]
    if kind == "drift":
        t, d = x + 0.004 * np.cos(3 * x + 0.05 * j), 1 - 0.012 * np.sin(3 * x + 0.05 * j)
    elif kind == "wild":
        t, d = 1 - 1.99 * x * x + 0 * j, -3.98 * x + 0 * j
    else:
        t, d = 1.02 * x + 0 * j, 1.02 + 0 * x + 0 * j
    return np.stack([t, d]) if interp == "hermite_slopes" else t[None]


def compose_both(orc, torch, tab, precision, interp, y0):
    from paper_1304_6514_amd.propagator import Propagator
    C, N, n = tab.shape
    tab = tab.astype(np.float32 if precision == "fp32" else np.float64)
    w = W.Workload("chain", "linear", (0.5,), 0.0, 1.0, N, (n,), (LO,), (HI,), 1, (y0,),
                   precision, interp)
    with Propagator("cuda:0") as p:
        p.build(w)
        for c in range(C):
            p.table_tensor(c).copy_(torch.from_numpy(tab[c]))
        torch.cuda.synchronize()
        r = p.compose(y0)
    g = orc.make_grid((n,), (LO,), (HI,))
    o = orc.compose_tables(g, interp, tab.astype(np.float64), (y0,))
    assert r.status == (nv.NV_OK if o.status == 0 else nv.NV_ERR_NONFINITE)
    assert r.bad_slice == o.bad_slice and r.n_out_of_grid == o.n_out_of_grid
    k = (o.bad_slice if o.status != 0 else N) + 1
    got, exp = r.boundary[:k], o.boundary[:k]
    assert np.array_equal(got.view(np.int64), exp.view(np.int64))
    return o


# the smallest rows, rows on either side of 12 KiB (both components of a slope
# table counted), and a row of several windows
SIZES = [("fp32", "linear", (2, 3, 64, 3071, 3072, 9000)),
         ("fp64", "linear", (2, 1535, 1536, 4001)),
         ("fp32", "hermite", (3, 4, 5, 3071, 3072, 9000)),
         ("fp64", "hermite", (3, 1535, 1536)),
         ("fp32", "hermite_slopes", (2, 1535, 1536, 5000)),
         ("fp64", "hermite_slopes", (2, 767, 768, 2001))]


@pytest.mark.parametrize("kind", ["drift", "wild", "leave"])
@pytest.mark.parametrize("precision,interp,sizes", SIZES,
                         ids=[f"{p}-{i}" for p, i, _ in SIZES])
def test_chain_equals_oracle_across_staging_modes(orc, torch, precision, interp, sizes, kind):
    for n in sizes:
        say("chain", precision, interp, kind, n)
        compose_both(orc, torch, tables(kind, 300, n, interp), precision, interp, 0.3)


@pytest.mark.parametrize("n", [257, 4000])
@pytest.mark.parametrize("n_slices", [1, 2, 3, 4, 5, 11, 12, 13, 63, 64, 65, 67, 128, 131])
def test_chain_equals_oracle_for_any_number_of_slices(orc, torch, n, n_slices):
    say("chain slices", n, n_slices)
    for kind in ("drift", "wild"):
        compose_both(orc, torch, tables(kind, n_slices, n, "hermite"), "fp32", "hermite", -0.4)


@pytest.mark.parametrize("n", [257, 4000])
@pytest.mark.parametrize("bad", [0, 1, 2, 3, 4, 62, 63, 64, 65, 101, 129])
def test_chain_finds_the_slice_with_a_nonfinite_entry(orc, torch, n, bad):
    """One slice's whole row is infinite or NaN: that slice fails, the states
    before it stand, wherever it lies in its group and block."""
    say("chain non-finite", n, bad)
    for value in (np.inf, np.nan):
        for interp in ("linear", "hermite"):
            tab = tables("drift", 130, n, interp)
            tab[0, bad] = value
            o = compose_both(orc, torch, tab, "fp64", interp, 0.1)
            assert o.bad_slice == bad


@pytest.mark.parametrize("precision", ["fp64", "fp32"])
@pytest.mark.parametrize("M", [2, 3, 5, 7, 8, 9])
@pytest.mark.parametrize("case", ["smooth", "zero", "tiny", "huge", "overflow", "nonfinite"])
def test_chebyshev_chain_equals_oracle(orc, torch, M, precision, case):
    """The Lagrange chain (spread quotients up to 8 nodes, one division after
    another above) over hand-written tables: ordinary states, states that are
    exactly zero or a node, states below and above the magnitudes the
    reciprocal quotients serve (taken again by division), a chain that
    overflows, and a non-finite row; 700 slices cross a staged chunk for
    M >= 6."""
    from paper_1304_6514_amd.propagator import Propagator
    N = 700
    dt = np.float32 if precision == "fp32" else np.float64
    w = W.paper_model(N, M, 0.5 / N, precision)
    xs = orc.paper_nodes(M, 0.0, 2.0)
    j = np.arange(N)[:, None]
    tab = 1.0 + 0.7 * np.sin(xs[None] + 0.1 * j)
    y0 = 0.8
    if case == "zero":
        tab[5::7] = 0.0
        tab[8::7] = xs[None]                 # the identity: the state reaches a node
        tab[9::35] = 2.0
    elif case == "tiny":
        tab[40:44] = 1e-37 * (1.0 if precision == "fp32" else 1e-113) * (1.0 + xs)
    elif case == "huge":
        tab[40:43] = 1e37 * (1.0 if precision == "fp32" else 1e113) * (1.0 + xs)
    elif case == "overflow":
        tab[:] = 1e30 * xs[None] * xs[None]
    elif case == "nonfinite":
        tab[650, M - 1] = np.inf
    tab = tab.astype(dt)
    say("chebyshev chain", M, precision, case)
    with Propagator("cuda:0") as p:
        p.build(w)
        p.table_tensor(0).copy_(torch.from_numpy(tab))
        torch.cuda.synchronize()
        r = p.compose((y0,))
    o = orc.paper_compose(M, 0.0, 2.0, tab.astype(np.float64), y0)
    assert r.status == (nv.NV_OK if o.status == 0 else nv.NV_ERR_NONFINITE)
    assert r.bad_slice == o.bad_slice and r.n_out_of_grid == o.n_out_of_grid
    k = (o.bad_slice if o.status != 0 else N) + 1
    got, exp = r.boundary[:k, 0], o.boundary.reshape(-1)[:k]
    fin = np.isfinite(exp)
    assert np.array_equal(np.isfinite(got), fin)
    assert np.array_equal(got[fin].view(np.int64), exp[fin].view(np.int64))
