"""The surrogate's composition at each of its workgroup sizes: 4, 8 and 16 chains per
workgroup, chosen by the number of chains against the compute units, each with a
last workgroup that is not full.

Tolerance: the network's output, an FP32 sum of 128 terms of size about 1 fed by
bfloat16 operands that differ from the oracle's by rare flipped roundings, is within
1e-3 of the oracle's; it enters scaled by d (1e-3 at most here) x 0.05: 5e-8 per
slice at most where a rounding flips, far less otherwise; 1e-7 over 8 slices."""
import sys

import numpy as np
import pytest

from oracle import mlp_oracle as mo
from paper_1304_6514_amd import nv
from paper_1304_6514_amd import workloads as W

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("per", [4, 8, 16])
def test_chains_of_every_workgroup_size_match_the_oracle(per):
    torch = pytest.importorskip("torch")
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    nv.load()
    from paper_1304_6514_amd.surrogate import Surrogate
    cu = torch.cuda.get_device_properties(0).multi_processor_count
    Q = {4: 4 * cu - 1, 8: 4 * cu + 1, 16: 8 * cu + 1}[per]
    N, T = 8, 50.0 * 8 / 1024
    p = W.surrogate_init_params(11)
    rng = np.random.default_rng(per)
    y0 = np.column_stack([rng.uniform(-2, 2, Q), rng.uniform(-4, 4, Q)])
    mu = rng.uniform(1, 5, Q)
    print(f"[gpu-test] surrogate chains Q={Q}", file=sys.__stderr__, flush=True)
    with Surrogate("cuda:0", max_batch=1024, correction="step-doubling", coarse_steps=1,
                   out_scale=W.SUR_SD_OUT_SCALE, gate=W.SUR_SD_GATE,
                   loss_scale=W.SUR_SD_LOSS_SCALE) as s:
        s.set_params(p)
        st, final, bnd, info = s.compose(y0, mu, 0.0, T, N, want_boundary=True)
    assert st == nv.NV_OK and info.bad_chain == -1
    final, bnd = final.cpu().numpy(), bnd.cpu().numpy()
    assert np.array_equal(bnd[:, -1], final) and np.array_equal(bnd[:, 0], y0)
    scale = np.array(W.SUR_IN_SCALE, dtype=np.float32).astype(np.float64)
    # a whole workgroup from the middle, and the last chains
    for q in [*range(Q // 32 * 16, Q // 32 * 16 + 16), Q - 3, Q - 2, Q - 1]:
        ref = mo.surrogate_chain(p.astype(np.float64), np.array(W.SUR_IN_SHIFT), scale,
                                 W.SUR_SD_OUT_SCALE, y0[q], mu[q], 0.0, T, N, emulate_bf16=True,
                                 coarse_steps=1, correction="step-doubling", gate=W.SUR_SD_GATE)
        assert np.max(np.abs(bnd[q] - ref)) < 1e-7, q
