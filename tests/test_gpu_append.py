"""The cache roll copies frames bit for bit (negative zeros, NaN payloads and
infinities included) into the native and the pooled rings, through wrap-around,
from tensors aligned for the copy kernel and from others."""

import pytest
import torch

from paper_2607_20940_amd import mssa

pytestmark = pytest.mark.gpu


def _bits(shape, seed, dtype, offset):
    """Random bit patterns of `dtype`, `offset` elements past an allocation's
    start."""
    gen = torch.Generator(device="cuda").manual_seed(seed)
    it = torch.int16 if dtype == torch.bfloat16 else torch.int32
    lim = torch.iinfo(it)
    n = 1
    for s in shape:
        n *= s
    raw = torch.randint(lim.min, lim.max, (n + offset,), generator=gen, device="cuda", dtype=it)
    raw[offset] = lim.min  # -0.0
    return raw[offset:].view(dtype).reshape(shape), raw


@pytest.mark.parametrize("offset", [0, 2])
@pytest.mark.parametrize("dtype", ["bf16", "f32"])
@pytest.mark.parametrize("pooled", [False, True])
def test_append_is_a_copy(pooled, dtype, offset):
    gh, gw, F, cap, nh, d = 3, 5, 2, 5, 2, 64
    print(f"[append] pooled={pooled} {dtype} offset={offset}", flush=True)
    desc = dict(num_states=2, scales=[1, 2], grid_h=gh, grid_w=gw, frames_per_state=F, sink_frames=0, hist_frames=0,
                num_heads=nh, head_dim=d, dtype=dtype, flags=mssa.MSSA_PLAN_POOLED_HIST_RING if pooled else 0)
    plan = mssa.mssa_plan_create(desc)
    info = plan.info()
    tdt = torch.bfloat16 if dtype == "bf16" else torch.float32
    it = torch.int16 if dtype == "bf16" else torch.int32
    tok1, tok2 = gh * gw, 2 * 3
    ring = mssa.Ring(cap)
    kr, vr = (torch.zeros((cap * tok1, nh, d), dtype=tdt, device="cuda") for _ in range(2))
    kp, vp = (torch.zeros((cap * tok2, nh, d), dtype=tdt, device="cuda") for _ in range(2))
    ws = torch.zeros(max(256, info["workspace_bytes"]), dtype=torch.uint8, device="cuda")
    want = {}
    for step in range(5):
        (kw, _k), (vw, _v) = (_bits((info["n_q"], nh, d), 10 * step + i, tdt, offset) for i in range(2))
        if pooled:
            if offset == 0:
                mssa.mssa_pool_kv(plan, None, None, kw, vw, ws)
            mssa.mssa_hist_append_ring(plan, kw, vw, ws, kr, vr, [None, kp], [None, vp], ring)
        else:
            mssa.mssa_hist_append(plan, kw, vw, kr, vr, ring)
        torch.cuda.synchronize()
        for f in range(F):
            want[2 * step + f] = (kw[f * tok1:(f + 1) * tok1].clone(), vw[f * tok1:(f + 1) * tok1].clone())
        n = 2 * (step + 1)
        for fr in range(max(0, n - cap), n):
            # frames fill the slots in order and then replace the oldest: frame fr is in slot fr mod cap
            s = fr % cap
            for got, w in ((kr, want[fr][0]), (vr, want[fr][1])):
                assert torch.equal(got[s * tok1:(s + 1) * tok1].view(it), w.view(it)), (step, fr)
        if pooled and offset == 0:
            for f in range(F):
                s = (2 * step + f) % cap
                for got, off in ((kp, info["pooled_k_offset"][1]), (vp, info["pooled_v_offset"][1])):
                    row = nh * d * (2 if dtype == "bf16" else 4)
                    w = ws[off + f * tok2 * row: off + (f + 1) * tok2 * row].view(it)
                    assert torch.equal(got[s * tok2:(s + 1) * tok2].view(it).reshape(-1), w), (step, f)
