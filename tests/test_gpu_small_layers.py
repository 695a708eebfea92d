"""Small layers at the edges of the kernels whose waves split the context of a
32-query item: one query more or less than a tile, contexts of one key, of
fewer tiles than waves and of many, in one block or split over two to eight;
forward, log-sum-exp and every gradient against the fp64 oracle.

Tolerances as for the other parity tests (tolerances.py, test_gpu_backward):
fp32 sums of a few thousand terms in any order stay near 1e-6 relative; bf16
outputs and gradients carry the rounding of P and dS, and the log-sum-exp of
fp32 scores from bf16 inputs 1e-3 absolute."""

import numpy as np
import pytest
import torch

import oracle

from gpu_common import assert_close, from_device
from test_gpu_backward import BwdRun, _assert_grads, _desc

pytestmark = pytest.mark.gpu

# (scales, grid, frames, sink, hist, heads): 32 and 33 queries per scale; a
# single query on a context of one key; runs of 31 and 1 tokens; one head on a
# long history (fp32: split over blocks); several heads, no split.
SHAPES = {
    "one_token": ([1], (1, 1), 1, 0, 0, 1),
    "tile_32": ([1], (4, 8), 1, 0, 1, 1),
    "tile_33": ([1, 2], (3, 11), 1, 1, 0, 2),
    "run_31": ([1, 1], (1, 31), 1, 1, 1, 1),
    "long_history": ([1, 2], (5, 7), 1, 1, 40, 1),
    "many_items": ([1, 2, 4], (11, 13), 2, 1, 3, 12),
}


# bf16 layers whose contexts 256 CUs split over (last) blocks per item; at 4x
# the context of the second has fewer tiles than the blocks have waves.
SPLIT = {
    "two_blocks": ([1, 2], (20, 23), 1, 1, 8, 6, 2),
    "four_blocks": ([1, 2, 4], (9, 13), 1, 1, 30, 1, 4),
    "eight_blocks": ([1], (7, 9), 1, 1, 80, 1, 8),
}


def _check(desc, dtype, name):
    nh, d = desc["num_heads"], desc["head_dim"]
    r = BwdRun(desc, dtype, 40 + d, 1.0 / np.sqrt(d))
    r.run()
    x = r.x64()
    ref = oracle.mssa_attention(desc, x["q_win"], x["k_sink"], x["v_sink"], x["k_hist"], x["v_hist"], x["k_win"],
                                x["v_win"])
    assert_close(from_device(r.out, dtype), ref, dtype, name)
    lse = r.lse.cpu().numpy().reshape(nh, -1).astype(np.float64)
    assert np.abs(lse - r.oracle_lse()).max() <= (1e-5 if dtype == "f32" else 1e-3), name
    if name != "one_token":  # a single key: dq and dk are exactly zero, and so is their reference
        _assert_grads(r.grads(), r.oracle(), dtype, name)
    return r


@pytest.mark.parametrize("dtype, prescaled", [("f32", False), ("bf16", False), ("bf16", True)])
@pytest.mark.parametrize("d", [64, 128])
@pytest.mark.parametrize("name", sorted(SHAPES))
def test_small_layer(name, d, dtype, prescaled):
    scales, (h, w), f, s, hist, nh = SHAPES[name]
    print(f"[small] {dtype} prescaled={prescaled} {name} d={d}", flush=True)
    _check(_desc(len(scales), scales, h, w, F=f, S=s, Hh=hist, nh=nh, d=d, q_prescaled=prescaled), dtype, name)


@pytest.mark.parametrize("prescaled", [False, True])
@pytest.mark.parametrize("d", [64, 128])
@pytest.mark.parametrize("name", sorted(SPLIT))
def test_context_split_over_blocks(name, d, prescaled):
    """The records of contexts split over blocks and their merge; that the plan
    does split shows in the workspace it asks for."""
    scales, (h, w), f, s, hist, nh, splits = SPLIT[name]
    print(f"[small] split prescaled={prescaled} {name} d={d}", flush=True)
    desc = _desc(len(scales), scales, h, w, F=f, S=s, Hh=hist, nh=nh, d=d, q_prescaled=prescaled)
    r = _check(desc, "bf16", name)
    if torch.cuda.get_device_properties(0).multi_processor_count == 256:
        a256 = lambda n: (n + 255) // 256 * 256  # noqa: E731
        items = sum(-(-(e - b) // 32) for b, e in zip(r.info["q_begin"], r.info["q_end"])) * nh
        pooled = 2 * sum(a256(n * nh * d * 2) for n in r.info["pooled_tokens"])
        assert r.info["workspace_bytes"] == pooled + a256(items * splits * 32 * (d + 2) * 4)
