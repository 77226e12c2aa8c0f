"""The gradient sums that the training kernel keeps in registers, over several passes of
32 samples per workgroup: two for some workgroups and one for others, eight for all of
them, and eight with a ninth, half empty, for one.

Tolerances as for single passes (against the oracle that rounds to bfloat16 where the
kernel does: FP32 against FP64 accumulation and the bfloat16 roundings that it flips,
below 2e-3 of any gradient; the loss, a mean of FP32 squares, within 1e-5)."""
import sys

import numpy as np
import pytest

from oracle import mlp_oracle as mo
from paper_1304_6514_amd import nv
from paper_1304_6514_amd import workloads as W

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("weighted", [False, True])
@pytest.mark.parametrize("n", [12304, 65536, 65552])
def test_gradients_over_several_passes(n, weighted):
    torch = pytest.importorskip("torch")
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    nv.load()
    from paper_1304_6514_amd.surrogate import Surrogate
    kw = dict(correction="step-doubling", coarse_steps=1, out_scale=W.SUR_SD_OUT_SCALE,
              gate=W.SUR_SD_GATE, loss_scale=W.SUR_SD_LOSS_SCALE) if weighted else {}
    shift = np.array(W.SUR_IN_SHIFT)
    scale = np.array(W.SUR_IN_SCALE, dtype=np.float32).astype(np.float64)
    p = W.surrogate_init_params(3)
    x, t = W.surrogate_samples(n, seed=n)
    wts = np.random.default_rng(n).uniform(-2.0, 2.0, (2, n)).astype(np.float32)
    print(f"[gpu-test] training passes n={n} weighted={weighted}", file=sys.__stderr__, flush=True)
    with Surrogate("cuda:0", max_batch=n, **kw) as s:
        s.set_params(p)
        loss, g = s.loss_grad(x, np.concatenate([t, wts]) if weighted else t)
    ref, gr = mo.loss_and_grad(p.astype(np.float64), x.T.astype(np.float64),
                               t.T.astype(np.float64), shift, scale, emulate_bf16=True,
                               **(dict(weights=wts.T.astype(np.float64)) if weighted else {}))
    assert abs(loss - ref) <= 1e-5 * ref, (loss, ref)
    gu = mo.unflatten(g)
    for name, _ in mo.SHAPES:
        d = np.linalg.norm(np.asarray(gu[name], np.float64) - gr[name])
        assert d < 2e-3 * np.linalg.norm(gr[name]), (name, d)
