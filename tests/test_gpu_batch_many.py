"""GPU parity of batches on either side of the number of problems up to which their
chains run staged (two per compute unit): every problem's states and counts are the
single-problem path's to the bit, whichever way its chain runs."""
import sys

import numpy as np
import pytest

from paper_1304_6514_amd import nv
from paper_1304_6514_amd import workloads as W

pytestmark = pytest.mark.gpu


def problem(i, precision):
    """Ragged small problems of every lookup; y0 inside and outside the grid."""
    kind, n, N = i % 4, 5 + 37 * (i % 7), 1 + (i * 29) % 140
    y0 = -0.9 + 2.0 * ((i * 13) % 100) / 100.0
    if kind == 3:
        return W.Workload(f"p{i}", "vdp", (1.0,), 0.0, 2.0, N, (5 + i % 9, 6 + i % 5),
                          (-3.0, -6.0), (3.0, 6.0), 2, (y0, 0.5), precision, "bilinear")
    rhs, params = (("linear", (0.5,)), ("logistic", ()), ("square", ()))[kind]
    # y' = y^2 from 0.9 blows up before t = 2: such chains meet non-finite entries
    return W.Workload(f"p{i}", rhs, params, 0.0, 2.0, N, (n,), (-1.0,), (1.0,), 2, (y0,),
                      precision, "hermite" if i % 8 < 4 else "linear")


@pytest.mark.parametrize("precision", ["fp32", "fp64"])
@pytest.mark.parametrize("more", [0, 1, 200])
def test_batch_of_many_problems_equals_single_problem_path(precision, more):
    torch = pytest.importorskip("torch")
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    nv.load()
    from paper_1304_6514_amd.propagator import Batch, Propagator
    count = 2 * torch.cuda.get_device_properties(0).multi_processor_count + more
    probs = [problem(i, precision) for i in range(count)]
    print(f"[gpu-test] batch of {count} {precision}", file=sys.__stderr__, flush=True)
    with Batch(probs, precision=precision) as b, Propagator("cuda:0", traj_per_lane=1) as p:
        for _ in range(2):                                # the graph, replayed
            st, yT, infos = b.run()
            bad = 0
            for i in range(0, count, 7):
                w = probs[i]
                p.build(w)
                r = p.compose()
                bad += r.status != nv.NV_OK
                assert infos[i][0] == r.n_out_of_grid, (i, w)
                k = (r.bad_slice if r.status != nv.NV_OK else w.n_slices) + 1
                assert np.array_equal(b.boundary(i)[:k].view(np.int64),
                                      r.boundary[:k].view(np.int64)), (i, w)
                assert np.array_equal(yT[i, :w.dim], r.yT, equal_nan=True), (i, w)
            assert st == nv.NV_ERR_NONFINITE or not bad
