"""Workspace of plans that choose between schedules (no GPU needed): the
records a schedule needs never push a plan past the scratch of the entry point
without allocations when another schedule fits, and the forward's workspace
holds nothing but the pooled blocks and those records."""

import pytest

from paper_2607_20940_amd import mssa

SCRATCH = mssa.MSSA_NOALLOC_SCRATCH_BYTES


def _plan(hist, dtype, blocks=0, heads=1, grid=64, flags=0):
    desc = dict(num_states=2, scales=[1, 2], grid_h=grid, grid_w=grid, frames_per_state=1, sink_frames=0,
                hist_frames=hist, num_heads=heads, head_dim=128, dtype=dtype, flags=flags)
    return mssa.mssa_plan_create_ex(desc, blocks)


@pytest.mark.parametrize("dtype", ["bf16", "f32"])
def test_long_history_of_one_head_fits_the_scratch(dtype):
    """One head on a long history: few query items (20 of 256 queries) whose
    pooled history alone takes most of the scratch."""
    eb = 2 if dtype == "bf16" else 4
    for hist in (100, 200, 300, 400, 500):
        pooled = 2 * (hist + 1) * 32 * 32 * 128 * eb
        small = 2 * 20 * 256 * (128 + 2) * 4 if dtype == "bf16" else 0  # records of one range per item
        ws = _plan(hist, dtype).info()["workspace_bytes"]
        assert ws >= pooled
        if pooled + small + 4096 <= SCRATCH:
            assert ws <= SCRATCH, hist
    # away from the limit the records are there: a range per pair of tiles
    assert dtype == "f32" or _plan(100, dtype).info()["workspace_bytes"] > 2 * 101 * 32 * 32 * 128 * eb + small


def test_given_attention_blocks_are_kept():
    """A given number of blocks is the number of ranges, whatever the layer
    (a plan without a backward, whose sums share the records' place)."""
    rec = 2 * 256 * (128 + 2) * 4
    for blocks in (2, 7, 97):
        base = _plan(4, "bf16", 1, grid=32, flags=mssa.MSSA_PLAN_POOLED_HIST_RING).info()["workspace_bytes"]
        ws = _plan(4, "bf16", blocks, grid=32, flags=mssa.MSSA_PLAN_POOLED_HIST_RING).info()["workspace_bytes"]
        assert ws == base + blocks * rec + ((blocks + 1) * 8 + 255) // 256 * 256


def _align(n):
    return (n + 255) // 256 * 256


@pytest.mark.parametrize("scales, heads, d, hist", [([1], 1, 128, 20), ([1, 2], 2, 64, 30), ([1, 1, 2, 4], 3, 128, 9)])
def test_forward_workspace_holds_nothing_of_the_backward(scales, heads, d, hist):
    """One range and no records: the pooled blocks alone, also where the
    backward splits dQ (few query items on a long context)."""
    desc = dict(num_states=len(scales), scales=scales, grid_h=16, grid_w=16, frames_per_state=1, sink_frames=1,
                hist_frames=hist, num_heads=heads, head_dim=d, dtype="bf16")
    info = mssa.mssa_plan_create_ex(desc, 1).info()
    assert info["workspace_bytes"] == 2 * sum(_align(n * heads * d * 2) for n in info["pooled_tokens"])


def _forward_records(scales, grid, frames, hist, heads, d):
    """Bytes of a bf16 plan's records: its workspace without the pooled blocks."""
    desc = dict(num_states=len(scales), scales=scales, grid_h=grid[0], grid_w=grid[1], frames_per_state=frames,
                sink_frames=0, hist_frames=hist, num_heads=heads, head_dim=d, dtype="bf16")
    info = mssa.mssa_plan_create(desc).info()
    return info["workspace_bytes"] - 2 * sum(_align(n * heads * d * 2) for n in info["pooled_tokens"]), info


# Layers of one scale on a 24 x 32 grid, three 256-query items a head: whole
# items where cutting them up would only add records and their merge (300 to
# 510 items of 12 or 24 tiles; a plan assumes 512 CUs without a device).
@pytest.mark.parametrize("d", [64, 128])
@pytest.mark.parametrize("heads, hist", [(100, 0), (150, 0), (170, 0), (170, 1)])
def test_layers_of_many_short_items_stay_whole(heads, hist, d):
    got, info = _forward_records([1], (24, 32), 1, hist, heads, d)
    ranges = 3 * heads
    assert got == _align(2 * ranges * 256 * (d + 2) * 4) + _align((ranges + 1) * 8)


@pytest.mark.parametrize("d", [64, 128])
@pytest.mark.parametrize("scales, grid, hist, heads, splits", [
    ([1, 2], (20, 33), 20, 1, 8), ([1, 2, 4], (15, 18), 14, 2, 4), ([1, 2], (10, 12), 10, 2, 1)])
def test_few_queries_on_a_long_context_split_over_blocks(scales, grid, hist, heads, splits, d):
    got, info = _forward_records(scales, grid, 1, hist, heads, d)
    items = sum(-(-(e - b) // 32) for b, e in zip(info["q_begin"], info["q_end"])) * heads
    assert got == (_align(items * splits * 32 * (d + 2) * 4) if splits > 1 else 0)
