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


def stated_order(G, c, y0):
    """lambda_{j+1} = c + (((p0 + p1) + (p2 + p3)) + ((p4 + p5) + (p6 + p7))), p_r =
    G_i,r l_r + G_i,r+8 l_r+8 + ... summed left to right from 0."""
    lam, out = np.array(y0), [np.array(y0)]
    for Gj, cj in zip(G, c):
        p = np.zeros((8, len(lam)))
        for k in range(len(lam)):
            p[k % 8] = p[k % 8] + Gj[:, k] * lam[k]
        lam = cj + (((p[0] + p[1]) + (p[2] + p[3])) + ((p[4] + p[5]) + (p[6] + p[7])))
        out.append(lam)
    return np.array(out)


@pytest.mark.parametrize("M,N", [(1, 70), (9, 63), (9, 64), (30, 300), (127, 128)])
def test_the_stated_order_holds_to_the_bit_for_any_number_of_slices(torch, M, N):
    w = HeatWorkload("order", M, 0.0013, N, T=0.0031 * N)
    say("fixed order", M, N)
    y0 = np.random.default_rng(3).normal(0.0, 1.0, M)
    with LinearPropagator() as lin:
        lin.build(w)
        G, c = lin.tables()
        ref = stated_order(G, c, y0)
        lin.fixed_order()
        st, yT, bnd = lin.compose(y0)
        assert st == nv.NV_OK and np.array_equal(bnd, ref) and np.array_equal(yT, ref[-1])
        lin.fixed_order(False)
        st, yT, bnd = lin.compose(y0)
        assert st == nv.NV_OK and (N >= 64 or np.array_equal(bnd, ref))
        check_chain(G, c, bnd, ref, "by blocks")


@pytest.mark.parametrize("N", [72, 100, 130])
@pytest.mark.parametrize("more", [0, 1])
def test_states_on_either_side_of_the_number_of_chains_for_blocks(torch, N, more):
    """The states of as many chains as run through the blocks (12, 24, 32 per compute
    unit by the number of slices), ragged last blocks among them, and of one more."""
    M = 19
    w = HeatWorkload("line", M, 0.0013, N, T=0.0031 * N)
    per_cu = 12 if N < 96 else 24 if N < 128 else 32
    Q = per_cu * torch.cuda.get_device_properties(0).multi_processor_count + more
    say("compose_many states", N, Q)
    y0 = np.random.default_rng(N).normal(0.0, 1.0, (Q, M))
    with LinearPropagator() as lin:
        lin.build(w)
        G, c = lin.tables()
        st, yT, b = lin.compose_many(y0, want_boundary=True)
    assert st == nv.NV_OK and torch.equal(yT, b[:, -1])
    for q in (0, 15, 16, 17, Q // 2, Q - 2, Q - 1):
        check_chain(G, c, b[q].cpu().numpy(), lo.compose(G, c, y0[q]), f"chain {q}")
