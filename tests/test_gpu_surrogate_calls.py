"""The surrogate's composition of more chains than one launch holds."""
import sys

import pytest

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
    with Surrogate("cuda:0", max_batch=1024, correction="step-doubling", coarse_steps=1,
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
