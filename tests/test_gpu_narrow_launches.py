"""Narrow workgroups with the shallow copy rings (launches whose items fill their rounds better that way): every tile
height that has them, ragged and full tiles, one K step and up, ragged last slabs."""
import pytest

import test_gpu_tile_handover as handover
from paper_2602_19128_amd import binding as moe

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("tile_rows, rows", [
    (16, [1, 6, 2, 4] * 24), (32, [9, 5, 32, 1] * 24), (64, [64, 30, 3, 17] * 24), (128, [127, 20, 128, 1, 45] * 12),
])
@pytest.mark.parametrize("which, dtype, H, I", [
    ("gateup", "bf16", 64, 448), ("gateup", "bf16", 448, 448), ("down", "bf16", 768, 64), ("down", "bf16", 832, 320),
    ("down", "fp8", 768, 128), ("down", "fp8", 896, 640),
])
def test_shallow_rings(which, dtype, H, I, tile_rows, rows):
    plan = moe.moe_gemm_plan(handover.config(which, dtype, rows, H, I), which)
    assert plan["tile_rows"] == tile_rows and plan["wavefronts"] == 4
    items = len(rows) * -(-(I if which == "gateup" else H) // plan["columns"])
    deep, shallow = {16: (2, 4), 32: (2, 4), 64: (2, 3), 128: (1, 2)}[tile_rows]          # workgroups a compute unit runs
    assert -(-items // (256 * shallow)) * shallow <= -(-items // (256 * deep)) * deep
    handover.check_gemm(which, dtype, rows, H, I)
