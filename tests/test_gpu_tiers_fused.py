"""The tier GEMMs that gather and scatter their own patches, at the edges of
their tiles and of the rule that chooses them: one token, tokens and features
one past a 64-tile, an odd number of K stages (the two halves of the
de-embedding's block), more tiles than CUs, K = 64 .. 256 and 1024 for the
embedding, and sizes that stay with the separate passes (odd patches, odd frame
widths, hidden sizes that are no multiple of 64, a de-embedding of few tokens on
a long hidden size, a wide embedding).  Outputs against the fp64 oracle with the
tolerance of test_gpu_tiers."""

import numpy as np
import pytest
import torch

import oracle
from paper_2607_20940_amd import mssa

from test_gpu_tiers import _bf16, _close, _desc, _f64, _weights

pytestmark = pytest.mark.gpu

# (scales, grid h, grid w, frames, channels, patch, hidden)
CASES = {
    "one_token": ([1], 1, 1, 1, 16, 2, 64),
    "rows_65": ([1], 5, 13, 1, 16, 2, 128),
    "features_72": ([1], 4, 6, 1, 18, 2, 192),
    "k_stages_odd": ([1, 2], 6, 7, 1, 16, 2, 320),
    "many_tiles": ([1, 2], 40, 45, 5, 16, 2, 192),
    "scale_4": ([1, 2, 4], 9, 11, 2, 16, 2, 256),
    "narrow_hidden": ([1, 2], 5, 6, 1, 16, 2, 72),
    "odd_patch": ([1, 2], 5, 7, 1, 16, 1, 128),
    "odd_channels_patch_3": ([1, 2], 4, 5, 1, 8, 3, 64),
    "hidden_past_a_tile": ([1], 3, 5, 2, 16, 2, 200),
    "one_tier_long_hidden": ([1], 14, 15, 1, 16, 2, 4928),
    "one_tier_wide_embedding": ([2], 52, 60, 1, 16, 2, 5184),
}


@pytest.mark.parametrize("name", sorted(CASES))
def test_tiers(name):
    scales, gh, gw, F, C, patch, hidden = CASES[name]
    print(f"[tiers] {name}", flush=True)
    desc = _desc(scales, gh, gw, F=F)
    rng = np.random.default_rng(11)
    plan = mssa.mssa_plan_create(dict(desc, dtype="bf16"))
    tier = mssa.tier_desc(C, patch, hidden)
    nq, frames = plan.info()["n_q"], len(scales) * F
    H, W = gh * patch, gw * patch
    ws = torch.full((max(256, mssa.mssa_tier_workspace_size(plan, tier)),), 0xFF, dtype=torch.uint8, device="cuda")
    lat, lat64 = _bf16(rng, (frames, C, H, W))
    w, b, wd, bd = _weights(rng, plan, desc, C, patch, hidden)
    guard = 3
    tok = torch.full((nq + guard, hidden), float("nan"), dtype=torch.bfloat16, device="cuda")
    mssa.mssa_patch_embed(plan, tier, lat, w, b, ws, tok)
    torch.cuda.synchronize()
    assert torch.isnan(tok[nq:]).all()
    _close(_f64(tok[:nq]), oracle.patch_embed(desc, patch, lat64, wd, bd), name + " embed")

    t_in, t64 = _bf16(rng, (nq, hidden))
    wo, bo, wod, bod = _weights(rng, plan, desc, C, patch, hidden, out=True)
    out = torch.full((frames + 1, C, H, W), float("nan"), dtype=torch.bfloat16, device="cuda")
    mssa.mssa_patch_unembed(plan, tier, t_in, wo, bo, ws, out)
    torch.cuda.synchronize()
    assert torch.isnan(out[frames:]).all()
    _close(_f64(out[:frames]), oracle.patch_unembed(desc, patch, C, t64, wod, bod), name + " unembed")
