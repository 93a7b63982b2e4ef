"""GPU parity of dense launches whose unit lists are tail-balanced: with few
units per XCD the host cuts the last round's units into pieces of whole key
tiles (partial slots merged by the combine kernel), including Sink/Dummy units
that otherwise write their output directly.  480P-shaped layers with 2-4 heads
(296, 518 and 814 units: all of them are cut on a 256-CU MI355X), full tensors
against the oracle; max-abs 1e-2, mean-abs 1e-3."""
import numpy as np
import pytest

from helpers import assert_close, dev_bf16, out_tensor
from oracle import headcast_oracle as O
from synth import inputs as S

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("types", [(0, 3), (3, 3), (1, 3, 3, 3)])
def test_balanced_tail_480p(hc, types):
    import torch
    types = np.array(types, np.uint8)
    w = S.Workload("bal", 1, len(types), 128, 30, 52, 3, 7, 4, 2, 481, (0, 0, 0, len(types)))
    cur = w.window_blocks - 1
    print(f"balanced tail types={types.tolist()} generate", flush=True)
    q, k, v = S.gen_layer(w, 0, cur)
    ctx = hc.Context(hc.config_from_workload(w), 0)
    ctx.set_head_types(0, types, cur, dev_bf16(k), dev_bf16(v))
    o = out_tensor(w)
    ctx.attention(0, dev_bf16(q), types, o)
    torch.cuda.synchronize()
    print("oracle", flush=True)
    ref = O.routed_attention(types, q, k, v, w.grid_h, w.grid_w, w.frames_per_block,
                             w.spatial_radius)
    assert_close(o.cpu().numpy(), ref, f"balanced tail types={types.tolist()}")


@pytest.mark.parametrize("types", [(0, 3), (3, 3), (1, 3, 3, 3)])
def test_balanced_tail_64_dim_heads(hc, types):
    """64-dim heads: three work groups share a CU, so the runs are cut for 96 slots per
    XCD; the tile loop ends on every remainder modulo its unrolling (L = 2376 = 37 tiles
    and 8 keys, cut into pieces of 12 tiles or more)."""
    import torch
    types = np.array(types, np.uint8)
    w = S.Workload("bal64", 1, len(types), 64, 22, 36, 3, 5, 4, 2, 482, (0, 0, 0, len(types)))
    cur = w.window_blocks - 1
    q, k, v = S.gen_layer(w, 0, cur)
    ctx = hc.Context(hc.config_from_workload(w), 0)
    ctx.set_head_types(0, types, cur, dev_bf16(k), dev_bf16(v))
    o = out_tensor(w)
    ctx.attention(0, dev_bf16(q), types, o)
    torch.cuda.synchronize()
    ref = O.routed_attention(types, q, k, v, w.grid_h, w.grid_w, w.frames_per_block,
                             w.spatial_radius)
    assert_close(o.cpu().numpy(), ref, f"balanced tail, 64-dim, types={types.tolist()}")


@pytest.mark.parametrize("d, L, nv", [(128, 128, 6), (128, 136, 6), (64, 256, 6), (64, 264, 6),
                                      (128, 8, 1)])
def test_uncut_small_windows(hc, d, L, nv):
    """Windows of up to 12 key tiles (24 with 64-dim heads) are one unit per query tile
    that writes its output itself; one tile more goes back to one unit per block."""
    import torch
    types = np.array([3, 0, 1, 3], np.uint8)
    w = S.Workload("uncut", 1, 4, d, 8, L // 8, 1, 7, 1, 1, 483, (1, 1, 0, 2))
    cur = nv - 1
    q, k, v = S.gen_layer(w, 0, cur)
    ctx = hc.Context(hc.config_from_workload(w), 0)
    ctx.set_head_types(0, types, cur, dev_bf16(k), dev_bf16(v))
    ref = O.routed_attention(types, q, k, v, w.grid_h, w.grid_w, w.frames_per_block,
                             w.spatial_radius)
    for call in ("attention", "attention_static"):
        o = out_tensor(w)
        getattr(ctx, call)(0, dev_bf16(q), types, o)
        torch.cuda.synchronize()
        assert_close(o.cpu().numpy(), ref, f"{call} d={d} L={L} nv={nv}")


@pytest.mark.parametrize("types", [(3, 3, 3, 0, 0, 1, 1, 0, 1, 1, 2, 2), (3, 3, 1, 2), (3, 0)])
def test_static_key_ranges_480p(hc, types):
    """The no-allocation call cuts Global windows into as many ranges as end first, not
    at block borders (six for the first table), and its dense partials take the place of
    the Spatial ones, which are merged by then."""
    import torch
    types = np.array(types, np.uint8)
    w = S.Workload("ranges", 1, len(types), 128, 30, 52, 3, 7, 4, 2, 484, (0, 0, 0, len(types)))
    ctx = hc.Context(hc.config_from_workload(w), 0)
    dev = torch.device("cuda:0")
    shape = (w.n_heads, w.window_tokens, w.head_dim)
    ctx.set_head_types(0, types, w.window_blocks - 1, S.device_normal_bf16(shape, 1, dev),
                       S.device_normal_bf16(shape, 2, dev))
    q = S.device_normal_bf16((w.n_heads, w.block_tokens, w.head_dim), 3, dev)
    ref, got = out_tensor(w), out_tensor(w)
    ctx.attention(0, q, types, ref)
    ctx.attention_static(0, q, types, got)
    torch.cuda.synchronize()
    assert_close(got.cpu().numpy(), ref.cpu().numpy().astype(np.float64), f"ranges {types.tolist()}")


@pytest.mark.parametrize("d, grid, frames, nv, n_sd, n_g", [
    (128, (30, 52), 3, 7, 0, 3),    # four ranges of seven blocks, 64 queries per wave
    (128, (30, 52), 3, 2, 8, 4),    # one per block, 32 queries per wave although the list is long
    (128, (23, 40), 3, 5, 4, 4),    # four ranges of five blocks, 32 queries per wave
    (64, (30, 52), 3, 7, 7, 3),     # six ranges of seven blocks
    (64, (30, 52), 3, 1, 0, 4),     # a single block in three ranges
    (64, (20, 22), 1, 7, 0, 16),    # ranges of 12 and 13 tiles, the last one ragged
])
def test_static_choices(hc, d, grid, frames, nv, n_sd, n_g):
    """The no-allocation call against hc_attention where it takes other key ranges or
    another kernel (the counts are the planner's for these shapes)."""
    import torch
    types = np.array([0, 1] * (n_sd // 2) + [1] * (n_sd % 2) + [3] * n_g, np.uint8)
    w = S.Workload("choice", 1, len(types), d, grid[0], grid[1], frames, 7, 4, 2, 485, (0, 0, 0, len(types)))
    ctx = hc.Context(hc.config_from_workload(w), 0)
    dev = torch.device("cuda:0")
    shape = (w.n_heads, nv * w.block_tokens, d)
    ctx.set_head_types(0, types, nv - 1, S.device_normal_bf16(shape, 1, dev), S.device_normal_bf16(shape, 2, dev))
    q = S.device_normal_bf16((w.n_heads, w.block_tokens, d), 3, dev)
    ref, got = out_tensor(w), out_tensor(w)
    ctx.attention(0, q, types, ref)
    ctx.attention_static(0, q, types, got)
    torch.cuda.synchronize()
    assert_close(got.cpu().numpy(), ref.cpu().numpy().astype(np.float64), f"choice d={d} {grid} nv={nv} {n_sd}+{n_g}")
