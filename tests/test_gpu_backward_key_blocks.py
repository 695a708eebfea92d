"""The dK/dV kernel with 64 keys a wave (256 per block), which only layers of many
blocks and long query ranges take: 256 heads, so that the plan chooses it, with
query ranges of 24 and 49 stages and of one to six (its stage buffers are four),
contexts that end inside a block, and an infinite key, which the stages that
fill the last round meet too.  Gradients of sampled heads against the fp64 oracle
with the tolerance of test_gpu_backward, whose small layers take 32 keys a wave.
The bounds harness checks the choice."""

import numpy as np
import pytest

from paper_2607_20940_amd.inputs import to_f64

from gpu_common import errors
from test_gpu_backward import GRAD_TOL, BwdRun, _assert_grads, _desc
from test_gpu_infinite_scores import _masked_inputs

pytestmark = pytest.mark.gpu

HEADS = (0, 131, 255)
# (scales, grid): coarse ranges of 24, 54 and 192 queries
SHAPES = {"one_coarse_stage": ([1, 1, 4], (16, 24)), "two_coarse_stages": ([1, 1, 4], (23, 34)),
          "six_coarse_stages": ([1, 2], (24, 32))}
# queries in whole 32-query stages: 48 and 1, 64 and 2, 26 (fills 28)
INFINITE = {"one_coarse_stage": ([1, 1, 1, 4], (16, 32)), "two_coarse_stages": ([1, 1, 4], (32, 32)),
            "stages_26": ([1, 1], (16, 26))}


class _SampledHeads(BwdRun):
    """The oracle's inputs restricted to HEADS (the others are never widened)."""

    def x64(self):
        x = {k: (None if v is None else to_f64(v[:, HEADS], self.dtype)) for k, v in self.x.items()}
        x["q_win"] = x["q_win"] / self.qf
        return x

    def oracle(self, heads=None):
        full, self.desc = self.desc, dict(self.desc, num_heads=len(HEADS))
        go, self.go = self.go, np.ascontiguousarray(self.go[:, HEADS])
        try:
            return super().oracle()
        finally:
            self.desc, self.go = full, go

    def grads(self):
        return {k: (None if v is None else v[:, HEADS]) for k, v in super().grads().items()}


@pytest.mark.parametrize("d, prescaled", [(64, False), (64, True), (128, False), (128, True)])
@pytest.mark.parametrize("name", sorted(SHAPES))
def test_gradients(name, d, prescaled):
    scales, grid = SHAPES[name]
    print(f"[key blocks] {name} d={d} prescaled={prescaled}", flush=True)
    desc = _desc(len(scales), scales, *grid, F=1, S=0, Hh=1, nh=256, d=d, q_prescaled=prescaled)
    r = _SampledHeads(desc, "bf16", 21 + d, 1.0 / np.sqrt(d))
    r.run()
    _assert_grads(r.grads(), r.oracle(), "bf16", name)


@pytest.mark.parametrize("d, prescaled", [(64, False), (128, True)])
@pytest.mark.parametrize("name", sorted(INFINITE))
def test_key_and_value_gradients_with_an_infinite_key(name, d, prescaled):
    scales, grid = INFINITE[name]
    print(f"[key blocks] infinite key {name} d={d} prescaled={prescaled}", flush=True)
    desc = _desc(len(scales), scales, *grid, F=1, S=1, Hh=0, nh=256, d=d, q_prescaled=prescaled)
    r = _SampledHeads(desc, "bf16", 22 + d, 1.0, inputs=lambda run: _masked_inputs(desc, run, "bf16", 22 + d, 5, 6))
    r.run()
    got = r.grads()
    with np.errstate(invalid="ignore"):  # dQ: 0 times the infinite key
        ref = r.oracle()
    for k in ("k_sink", "v_sink", "k_win", "v_win"):
        assert np.isfinite(got[k]).all(), (name, k)
        e = errors(got[k], ref["d" + k])
        assert all(e[t] <= GRAD_TOL["bf16"][t] for t in GRAD_TOL["bf16"]), (name, k, e)
