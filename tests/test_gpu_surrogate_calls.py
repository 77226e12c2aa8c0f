"""The surrogate's composition of more chains than a workgroup per compute unit, and of
more than one launch, holds."""
import sys

import numpy as np
import pytest

from oracle import mlp_oracle as mo
from paper_1304_6514_amd import nv
from paper_1304_6514_amd import workloads as W

pytestmark = pytest.mark.gpu


def test_more_chains_than_one_launch_holds():
    """120,000,000 chains of one slice: 7.5 million workgroups of 576 threads, more than
    2^32 work-items.  Chains on either side of a launch's end and the last ones are those
    of the same chains in a small run (a chain's operations do not depend on its place)."""
    torch = pytest.importorskip("torch")
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    if torch.cuda.mem_get_info()[0] < 16 << 30:
        pytest.skip("needs 16 GB of device memory")
    nv.load()
    from paper_1304_6514_amd.surrogate import Surrogate
    Q, T = 120_000_000, 50.0 / 1024
    print(f"[gpu-test] surrogate chains Q={Q}", file=sys.__stderr__, flush=True)
    edge = (2 ** 32 - 1) // 576 * 16
    pick = torch.cat([torch.arange(0, 2048), torch.arange(edge - 1024, edge + 1024),
                      torch.arange(Q - 100, Q)]).cuda()
    g = torch.Generator(device="cuda").manual_seed(5)
    y0 = torch.rand((Q, 2), dtype=torch.float64, device="cuda", generator=g) * 4 - 2
    mu = torch.rand(Q, dtype=torch.float64, device="cuda", generator=g) * 4 + 1
    with Surrogate("cuda:0", max_batch=1024, correction="step-doubling", coarse_steps=2,
                   out_scale=W.SUR_SD_OUT_SCALE, gate=W.SUR_SD_GATE,
                   loss_scale=W.SUR_SD_LOSS_SCALE) as s:
        s.set_params(W.surrogate_init_params(11))
        st, final, _, info = s.compose(y0, mu, 0.0, T, 1)
        assert st == nv.NV_OK and info.bad_chain == -1
        got = final[pick].clone()
        del final
        st, ref, _, _ = s.compose(y0[pick].contiguous(), mu[pick].contiguous(), 0.0, T, 1)
        assert st == nv.NV_OK
    assert pick.numel() > 8 * torch.cuda.get_device_properties(0).multi_processor_count
    assert torch.equal(got, ref)


@pytest.mark.parametrize("correction,coarse,per_cu", [
    ("additive", 0, 16), ("additive", 1, 16), ("additive", 16, 16), ("step-doubling", 16, 16),
    ("step-doubling", 1, 64), ("step-doubling", 4, 64), ("step-doubling", 6, 64)])
@pytest.mark.parametrize("more", [0, 1])
def test_many_chains_of_every_form_match_the_oracle(correction, coarse, per_cu, more):
    """Either side of the counts from which 16 chains run by four waves, each with a last
    workgroup that is not full beyond it.

    Tolerance: the network's output, an FP32 sum of 128 terms of size about 1 fed by
    bfloat16 operands that differ from the oracle's by rare flipped roundings, is within
    1e-3 of the oracle's.  Additive: it enters scaled by 1e-3, and the flow over T = 0.1
    at mu <= 5 spreads a difference by less than e^0.5: 3 slices x 1e-6 x 2 = 6e-6.  Step
    doubling: scaled by d (1e-2 at most here) x 0.05: below that."""
    torch = pytest.importorskip("torch")
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    nv.load()
    from paper_1304_6514_amd.surrogate import Surrogate
    Q = per_cu * torch.cuda.get_device_properties(0).multi_processor_count + more
    N, T = 3, 50.0 * 3 / 1024
    print(f"[gpu-test] surrogate chains {correction} {coarse} Q={Q}", file=sys.__stderr__,
          flush=True)
    sd = correction == "step-doubling"
    scale_out = W.SUR_SD_OUT_SCALE if sd else (1e-3, 1e-3)
    kw = dict(gate=W.SUR_SD_GATE, loss_scale=W.SUR_SD_LOSS_SCALE) if sd else {}
    p = W.surrogate_init_params(11)
    rng = np.random.default_rng(Q + coarse)
    y0 = np.column_stack([rng.uniform(-2, 2, Q), rng.uniform(-4, 4, Q)])
    mu = rng.uniform(1, 5, Q)
    with Surrogate("cuda:0", max_batch=1024, correction=correction, coarse_steps=coarse,
                   out_scale=scale_out, **kw) as s:
        s.set_params(p)
        st, final, bnd, info = s.compose(y0, mu, 0.0, T, N, want_boundary=True)
    assert st == nv.NV_OK and info.bad_chain == -1
    final, bnd = final.cpu().numpy(), bnd.cpu().numpy()
    assert np.array_equal(bnd[:, -1], final) and np.array_equal(bnd[:, 0], y0)
    scale = np.array(W.SUR_IN_SCALE, dtype=np.float32).astype(np.float64)
    for q in [*range(Q // 32 * 16, Q // 32 * 16 + 16), Q - 2, Q - 1]:
        ref = mo.surrogate_chain(p.astype(np.float64), np.array(W.SUR_IN_SHIFT), scale,
                                 scale_out, y0[q], mu[q], 0.0, T, N, emulate_bf16=True,
                                 coarse_steps=coarse, correction=correction,
                                 **(dict(gate=W.SUR_SD_GATE) if sd else {}))
        assert np.max(np.abs(bnd[q] - ref)) < 6e-6, q
