"""GPU parity of the affine basis propagator's less usual calls."""
import sys

import numpy as np
import pytest

from oracle import linear_oracle as lo
from paper_1304_6514_amd import nv
from paper_1304_6514_amd.linear import HeatWorkload, LinearPropagator
from test_gpu_linear import check_chain

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


@pytest.mark.parametrize("N", [12, 100])
@pytest.mark.parametrize("boundary", [False, True])
def test_compose_many_in_place(torch, N, boundary):
    """The final states may overwrite the initial ones (a workgroup reads its chains
    before it writes them), also where a chain beyond 1e300, or one that is not finite,
    takes the chains from the blocks' products back to the slices."""
    M = 9
    w = HeatWorkload("in-place", M, 0.01, N, T=0.01 * N)
    rng = np.random.default_rng(5)
    y0 = rng.normal(0.0, 1.0, (300, M))
    for case in ("ordinary", "large", "nan"):
        say("compose_many in place", N, boundary, case)
        if case == "large":
            y0[7] = 1e305
        elif case == "nan":
            y0[211, 3] = np.nan
        with LinearPropagator() as lin:
            lin.build(w)
            G, c = lin.tables()
            y = torch.from_numpy(y0).cuda()
            b = torch.empty((300, N + 1, M), dtype=torch.float64, device="cuda") \
                if boundary else None
            torch.cuda.synchronize()
            st = nv.nv_lin_compose_many(lin.h, y.data_ptr(), 300, y.data_ptr(),
                                        b.data_ptr() if boundary else None)
            assert st == (nv.NV_ERR_NONFINITE if case == "nan" else nv.NV_OK)
            got = y.cpu().numpy()
        for q in (0, 7, 15, 16, 299):
            ref = lo.compose(G, c, y0[q])
            check_chain(G, c, np.concatenate([ref[:-1], got[q:q + 1]]), ref, f"chain {q}")
            if boundary:
                check_chain(G, c, b[q].cpu().numpy(), ref, f"states of chain {q}")


def test_a_forcing_beyond_the_numbers_leaves_the_homogeneous_solves(torch):
    """a(t) = 3e307: h a / dx^2 is finite, beta(t) = pi^2 a(t) cos t - sin t is not.
    The forced solves (c) are not finite; the homogeneous ones (G) have no forcing
    and are the oracle's to the bit."""
    for M in (1, 3, 70):
        w = HeatWorkload("beyond", M, 1e-5 / (M + 1) ** 2, 3, T=6e-5 / (M + 1) ** 2, a0=3e307,
                         a1=0.0)
        say("forcing beyond the numbers", M)
        with LinearPropagator() as lin:
            lin.build(w)
            G, c = lin.tables()
        with np.errstate(all="ignore"):
            Go, co = lo.build_tables(M, w.a0, w.a1, True, w.t0, w.T, w.n_slices, w.dt)
        assert np.all(np.isfinite(Go)) and not np.any(np.isfinite(co))
        assert np.array_equal(G, Go)
        assert not np.any(np.isfinite(c))


def test_more_chains_than_one_launch_by_blocks_holds(torch):
    """2,200,000 chains of 1024 slices with their states (18 GB): over the blocks'
    states this would be 8.8 million workgroups of 512, more than a launch holds;
    the chains run slice by slice, as a few of them alone do through the blocks."""
    w = HeatWorkload("many", 1, 0.01, 1024, T=10.24)
    Q = 2_200_000
    if torch.cuda.mem_get_info()[0] < 24 << 30:
        pytest.skip("needs 24 GB of device memory")
    say("compose_many", Q)
    with LinearPropagator() as lin:
        lin.build(w)
        G, c = lin.tables()
        y0 = torch.linspace(-1.0, 1.0, Q, dtype=torch.float64, device="cuda").reshape(Q, 1)
        st, yT, b = lin.compose_many(y0, want_boundary=True)
        assert st == nv.NV_OK
        for q in (0, 31, 1_100_000, Q - 1):
            got = b[q].cpu().numpy()
            check_chain(G, c, got, lo.compose(G, c, y0[q].cpu().numpy()), f"chain {q}")
            assert np.array_equal(yT[q].cpu().numpy(), got[-1])
        del b
