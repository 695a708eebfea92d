"""Keys whose scores are -inf for every query (a channel of K at -inf against
queries that are positive there), over whole tiles of the context, at its start
and in its middle, and over whole pieces of it: such keys weigh nothing, and the
output, the log-sum-exp and the gradients of the keys and values are those of
the remaining keys, whichever kernel and schedule a plan takes.  Against the fp64 oracle with the tolerances of the
other parity tests; the number of pieces comes from the given attention
blocks."""

import numpy as np
import pytest

import oracle
from paper_2607_20940_amd.inputs import f32_to_bf16_bits, make_inputs, to_f64
from paper_2607_20940_amd.workloads import input_shapes

from gpu_common import assert_close, errors, from_device, q_prescale
from test_gpu_backward import GRAD_TOL, BwdRun, _desc

pytestmark = pytest.mark.gpu

# (sink frames of 16 x 16 tokens: keys, -inf keys [lo, hi))
HOLES = {"first_tile": (0, 64), "first_tiles": (0, 192), "middle": (128, 320), "ragged": (70, 451)}


def _masked_inputs(desc, run, dtype, seed, lo, hi):
    shapes = input_shapes(desc, run.info["n_q"], run.info["n_sink_tok"], run.info["n_hist_tok"])
    qa = q_prescale(desc) if desc.get("q_prescaled") else 1.0
    x = make_inputs(shapes, seed, 1.0, dtype, q_amplitude=qa)
    q = to_f64(x["q_win"], dtype)
    q[:, :, 0] = np.abs(q[:, :, 0]) + 0.125 * qa
    k = to_f64(x["k_sink"], dtype)
    k[lo:hi, :, 0] = -np.inf
    for name, v in (("q_win", q), ("k_sink", k)):
        v = v.astype(np.float32)
        x[name] = f32_to_bf16_bits(v) if dtype == "bf16" else v
    return x


# blocks 0: the kernel of small layers (fp32: the fp32 kernel); 1: whole items
# on the persistent kernel; 3: pieces that start in the hole and around it; 40:
# pieces of a tile or two, whole pieces in the hole
@pytest.mark.parametrize("dtype, prescaled, blocks",
                         [("f32", False, 0)] + [("bf16", p, b) for p in (False, True) for b in (0, 1, 3, 40)])
@pytest.mark.parametrize("d", [64, 128])
@pytest.mark.parametrize("hole", sorted(HOLES))
def test_forward_with_infinite_scores(hole, d, dtype, prescaled, blocks):
    print(f"[inf] {hole} d={d} {dtype} prescaled={prescaled} blocks={blocks}", flush=True)
    lo, hi = HOLES[hole]
    desc = _desc(2, [1, 2], 16, 16, F=1, S=2, Hh=0, nh=2, d=d, q_prescaled=prescaled)
    r = BwdRun(desc, dtype, 5, 1.0, attention_blocks=blocks,
               inputs=lambda run: _masked_inputs(desc, run, dtype, 5, lo, hi))
    r.forward()
    x = r.x64()
    ref = oracle.mssa_attention(desc, x["q_win"], x["k_sink"], x["v_sink"], x["k_hist"], x["v_hist"], x["k_win"],
                                x["v_win"])
    assert_close(from_device(r.out, dtype), ref, dtype, hole)
    lse = r.lse.cpu().numpy().reshape(2, -1).astype(np.float64)
    assert np.abs(lse - r.oracle_lse()).max() <= (1e-5 if dtype == "f32" else 1e-3), hole


# 64, 192, 256 and 96 queries: whole 64-query stages that do not fill a round
# of the dK/dV kernel's four, that do, and a half
@pytest.mark.parametrize("dtype, prescaled", [("f32", False), ("bf16", False), ("bf16", True)])
@pytest.mark.parametrize("d", [64, 128])
@pytest.mark.parametrize("grid", [(8, 8), (8, 24), (16, 16), (8, 12)])
def test_key_and_value_gradients_with_an_infinite_key(grid, d, dtype, prescaled):
    """A key that weighs nothing has zero dK and dV, and the others' are those
    without it (dQ is not compared: 0 times the infinite key)."""
    print(f"[inf] backward {grid} d={d} {dtype} prescaled={prescaled}", flush=True)
    desc = _desc(1, [1], *grid, F=1, S=1, Hh=0, nh=2, d=d, q_prescaled=prescaled)
    r = BwdRun(desc, dtype, 6, 1.0, inputs=lambda run: _masked_inputs(desc, run, dtype, 6, 5, 6))
    r.run()
    got = r.grads()
    x = r.x64()
    go = to_f64(r.go, dtype)
    sc = oracle.softmax_scale(desc)
    n_sink = x["k_sink"].shape[0]
    ref = {k: np.zeros_like(x[k]) for k in ("k_sink", "v_sink", "k_win", "v_win")}
    for h in range(2):
        k = np.concatenate([x["k_sink"][:, h], x["k_win"][:, h]])
        v = np.concatenate([x["v_sink"][:, h], x["v_win"][:, h]])
        z = sc * (x["q_win"][:, h] @ k.T)
        p = np.exp(z - z.max(axis=1, keepdims=True))
        p /= p.sum(axis=1, keepdims=True)
        dp = go[:, h] @ v.T
        ds = p * (dp - (go[:, h] * (p @ v)).sum(axis=1, keepdims=True))
        dk, dv = sc * (ds.T @ x["q_win"][:, h]), p.T @ go[:, h]
        ref["k_sink"][:, h], ref["k_win"][:, h] = dk[:n_sink], dk[n_sink:]
        ref["v_sink"][:, h], ref["v_win"][:, h] = dv[:n_sink], dv[n_sink:]
    for name, b in ref.items():
        a, tol = got[name], GRAD_TOL[dtype]
        assert np.isfinite(a).all(), (grid, name)
        e = errors(a, b)
        assert all(e[t] <= tol[t] for t in tol), (grid, name, e)
    assert np.abs(got["k_sink"][5]).max() == 0 and np.abs(got["v_sink"][5]).max() == 0
