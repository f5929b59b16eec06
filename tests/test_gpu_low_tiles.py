"""Grouped GEMMs of a handful of tokens on few, wide experts: fewer tiles than XCDs in equal parts, fewer K steps than
copy stages and many, 16- and 32-row tiles, experts without a row, half-width items."""
import pytest
import torch

import test_gpu_tile_handover as handover
from paper_2602_19128_amd import binding as moe

pytestmark = pytest.mark.gpu


# parts: down launches in equal parts, which the rule keeps to ranges of more than 16 column slabs
@pytest.mark.parametrize("rows, H, I, parts", [
    ([1], 64, 64, False), ([2, 0, 1, 0, 0, 3], 128, 320, False), ([1, 1, 0, 1, 1, 1, 1], 1024, 4160, False),
    ([16, 15, 1], 576, 2048, False), ([17, 32, 1, 9], 448, 1024, False), ([12] * 40, 256, 192, False), ([3, 1, 2], 1088, 256, False),
    ([1, 1, 0, 1, 1, 1, 1], 2176, 4160, True), ([16, 15, 1], 2112, 2048, True), ([17, 32, 1, 9], 4096, 1024, True),
    ([5] * 18, 768, 1088, True), ([20, 0, 1] * 10, 640, 1024, True), ([9] * 33, 640, 1024, False), ([1, 1, 0, 1, 1, 1, 1], 2048, 4160, False),
])
def test_low_tiles_of_few_experts(rows, H, I, parts):
    E, T = len(rows), sum(rows)
    cfg = moe.MoEConfig(T, H, I, E, 1, 0, 1, 1, 1, 1, 0, 1.0, 0, 0, 0)
    plan = moe.moe_gemm_plan(cfg, "down")
    assert plan["tile_rows"] <= 32 and plan["wavefronts"] == 4 and plan["whole_ranges"] == (not parts)
    gen = torch.Generator("cuda").manual_seed(H + I)
    ids = torch.repeat_interleave(torch.arange(E), torch.tensor(rows)).cuda()[torch.randperm(T, generator=gen, device="cuda")]
    ids = ids.to(torch.int32).view(T, 1)
    draw = lambda *shape: torch.randn(shape, generator=gen, device="cuda")
    x, w1, w2 = draw(T, H).bfloat16(), (draw(E, 2 * I, H) * H ** -0.5).bfloat16(), (draw(E, H, I) * I ** -0.5).bfloat16()
    offsets, pair, inv, tiles, sched = moe.moe_permute(cfg, ids)
    act, _ = moe.moe_grouped_gemm_swiglu(cfg, x, None, w1, None, pair, tiles, sched)
    y = moe.moe_grouped_gemm_down(cfg, act, None, w2, None, tiles, sched)
    off = offsets.tolist()
    for e in range(E):
        lo, hi = off[e], off[e + 1]
        xe, w = x[pair[lo:hi].long()].double(), w1[e].double().t()
        gu = xe @ w
        ref = torch.nn.functional.silu(gu[:, :I]) * gu[:, I:]
        # one bf16 rounding (2^-9 of the value) of fp32 sums of up to 4160 terms (2^-24 each, of the sum of magnitudes)
        slack = (xe.abs() @ w.abs()).max() ** 2 * 2.0 ** -20 if hi > lo else 0.0
        assert ((act[lo:hi].double() - ref).abs() <= ref.abs() * 2.0 ** -8 + slack).all(), f"gate/up, expert {e}"
        a, w = act[lo:hi].double(), w2[e].double().t()
        ref = a @ w
        assert ((y[lo:hi].double() - ref).abs() <= ref.abs() * 2.0 ** -8 + (a.abs() @ w.abs()) * 2.0 ** -20).all(), f"down, expert {e}"


@pytest.mark.parametrize("which, dtype, rows, H, I", [
    ("gateup", "bf16", [6] * 48, 256, 1408), ("gateup", "bf16", [3, 20] * 20, 192, 1664), ("down", "bf16", [16, 9] * 20, 4096, 192),
    ("down", "fp8", [16, 15] * 20, 4096, 256), ("down", "fp8", [5] * 40, 4096, 128),
])
def test_half_width_items_of_low_tiles(which, dtype, rows, H, I):
    """Wide workgroups of 16- and 32-row tiles whose last round is short (see test_last_round_of_low_tiles)."""
    plan = moe.moe_gemm_plan(handover.config(which, dtype, rows, H, I), which)
    assert plan["tile_rows"] <= 32 and plan["wavefronts"] == 8 and plan["whole_ranges"] and plan["half_items"]
    items = len(rows) * -(-(I if which == "gateup" else H) // plan["columns"]) // 8
    assert 1 <= items % 64 <= 16
    handover.check_gemm(which, dtype, rows, H, I)
