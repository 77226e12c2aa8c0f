"""The training kernel at the edges of its passes: minibatches of one tile (half a
pass of 32 samples), one pass, an odd number of tiles, and more passes than there
are compute units (some workgroups take two passes, the last only half of one), and
on both sides of 8192 samples, where the gradient sums change from rows of a
workspace to the training kernel's registers; with and without per-sample weights.

Tolerances against the oracle that rounds to bfloat16 where the kernel does: what
is left is FP32 against FP64 accumulation (2^-24 per operation, under 1e-5 over
the sums here) and the bfloat16 roundings that those differences flip, at most a
few per ten thousand operands of 2^-9 each: below 2e-3 of any gradient."""
import sys

import numpy as np
import pytest

from oracle import mlp_oracle as mo
from paper_1304_6514_amd import nv
from paper_1304_6514_amd import workloads as W

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def torch():
    torch = pytest.importorskip("torch")
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    nv.load()
    return torch


@pytest.mark.parametrize("weighted", [False, True])
@pytest.mark.parametrize("n", [16, 32, 48, 8176, 8192, 8208])
def test_gradients_at_the_edges_of_a_pass(torch, n, weighted):
    from paper_1304_6514_amd.surrogate import Surrogate
    kw = dict(correction="step-doubling", coarse_steps=1, out_scale=W.SUR_SD_OUT_SCALE,
              gate=W.SUR_SD_GATE, loss_scale=W.SUR_SD_LOSS_SCALE) if weighted else {}
    shift = np.array(W.SUR_IN_SHIFT)
    scale = np.array(W.SUR_IN_SCALE, dtype=np.float32).astype(np.float64)
    p = W.surrogate_init_params(3)
    x, t = W.surrogate_samples(n, seed=n)
    wts = np.random.default_rng(n).uniform(-2.0, 2.0, (2, n)).astype(np.float32)
    print(f"[gpu-test] training pass n={n} weighted={weighted}", file=sys.__stderr__, flush=True)
    with Surrogate("cuda:0", max_batch=n, **kw) as s:
        s.set_params(p)
        loss, g = s.loss_grad(x, np.concatenate([t, wts]) if weighted else t)
        again = s.loss_grad(x, np.concatenate([t, wts]) if weighted else t)
    assert loss == again[0] and np.array_equal(g, again[1])        # a fixed order of sums
    ref, gr = mo.loss_and_grad(p.astype(np.float64), x.T.astype(np.float64),
                               t.T.astype(np.float64), shift, scale, emulate_bf16=True,
                               **(dict(weights=wts.T.astype(np.float64)) if weighted else {}))
    assert abs(loss - ref) <= 1e-5 * ref, (loss, ref)
    gu = mo.unflatten(g)
    for name, _ in mo.SHAPES:
        d = np.linalg.norm(np.asarray(gu[name], np.float64) - gr[name])
        assert d < 2e-3 * np.linalg.norm(gr[name]), (name, d)
