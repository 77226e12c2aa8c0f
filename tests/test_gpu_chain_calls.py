"""GPU parity of the 1-D composition chain where its lookups meet the grid's ends."""
import sys

import numpy as np
import pytest

from paper_1304_6514_amd import nv
from paper_1304_6514_amd import workloads as W

pytestmark = pytest.mark.gpu


def say(*a):
    print("[gpu-test]", *a, file=sys.__stderr__, flush=True)


@pytest.fixture(scope="module")
def torch():
    torch = pytest.importorskip("torch")
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    nv.load()
    return torch


def compose_both(orc, torch, tab, precision, interp, y0, lo, hi):
    from paper_1304_6514_amd.propagator import Propagator
    C, N, n = tab.shape
    tab = tab.astype(np.float32 if precision == "fp32" else np.float64)
    w = W.Workload("chain", "linear", (0.5,), 0.0, 1.0, N, (n,), (lo,), (hi,), 1, (y0,),
                   precision, interp)
    with Propagator("cuda:0") as p:
        p.build(w)
        for c in range(C):
            p.table_tensor(c).copy_(torch.from_numpy(tab[c]))
        torch.cuda.synchronize()
        r = p.compose(y0)
    o = orc.compose_tables(orc.make_grid((n,), (lo,), (hi,)), interp, tab.astype(np.float64),
                           (y0,))
    # extrapolation far outside a fine grid may overflow: then in the same slice
    assert r.status == (nv.NV_OK if o.status == 0 else nv.NV_ERR_NONFINITE)
    assert r.bad_slice == o.bad_slice and r.n_out_of_grid == o.n_out_of_grid
    k = (o.bad_slice if o.status != 0 else N) + 1
    assert np.array_equal(r.boundary[:k].view(np.int64), o.boundary[:k].view(np.int64))
    return r


@pytest.mark.parametrize("n", [64, 9000])
@pytest.mark.parametrize("precision", ["fp32", "fp64"])
@pytest.mark.parametrize("interp", ["linear", "hermite", "hermite_slopes"])
def test_the_sign_of_a_zero_is_kept(orc, torch, n, precision, interp):
    """A state of -0.0 at a grid that starts at 0, over tables that hold -0.0 there:
    u = -0.0 lies in cell 0 at w = u - 0 = -0.0, and the state stays -0.0."""
    say("sign of zero", n, precision, interp)
    x = np.linspace(0.0, 1.0, n)
    val = np.tile(-0.9 * x if interp != "linear" else 0.9 * x, (100, 1))
    val[:, 0] = -0.0
    tab = np.stack([val, np.full_like(val, 0.9)]) if interp == "hermite_slopes" else val[None]
    r = compose_both(orc, torch, tab, precision, interp, -0.0, 0.0, 1.0)
    if interp == "linear":
        assert np.all(np.signbit(r.boundary))


ENDS = [("fp32", "linear", (2, 3, 64, 5000)), ("fp64", "linear", (2, 700, 3000)),
        ("fp32", "hermite", (3, 4, 5, 64, 5000)), ("fp64", "hermite", (3, 4, 700, 3000)),
        ("fp32", "hermite_slopes", (2, 300, 5000)), ("fp64", "hermite_slopes", (2, 300, 2000))]


@pytest.mark.parametrize("kind", ["lower", "upper", "outside", "crossing", "edge cells"])
@pytest.mark.parametrize("precision,interp,sizes", ENDS, ids=[f"{p}-{i}" for p, i, _ in ENDS])
def test_states_at_the_ends_of_the_grid(orc, torch, precision, interp, sizes, kind):
    """States that rest on either end of the grid or outside it, that leave it and come
    back, and that wander through its first and last cells: clamped cells, counted
    lookups and one-sided slopes, a group at a time, in rows and in windows."""
    N = 333
    j = np.arange(N)[:, None]
    for n in sizes:
        say("ends", precision, interp, n, kind)
        x = np.linspace(-1.0, 1.0, n)[None]
        to = {"lower": -1.0 + 0.0 * j, "upper": 1.0 + 0.0 * j, "outside": 1.3 + 0.1 * np.sin(j),
              "crossing": 0.9 + 0.2 * np.sin(0.04 * j),
              "edge cells": np.where(j % 32 < 16, -1.0, 1.0) * (1.0 - 2.6 / n * (j % 5) / 4.0)}[kind]
        val = to + 1e-3 * (x - np.clip(to, -1.0, 1.0))
        tab = np.stack([val, np.full_like(val, 1e-3)]) if interp == "hermite_slopes" else val[None]
        r = compose_both(orc, torch, tab, precision, interp, 0.3, -1.0, 1.0)
        if kind == "outside" and r.status == nv.NV_OK:
            assert r.n_out_of_grid == N - 1
