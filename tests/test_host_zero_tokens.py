"""Size queries of a layer without tokens, on both sides of the line between the router's paths."""
import pytest

from paper_2602_19128_amd import binding as moe


@pytest.mark.parametrize("E", [8, 16, 17, 64, 256, 512])
@pytest.mark.parametrize("dtype", [0, 1])
def test_size_queries_of_zero_tokens(E, dtype):
    cfg = moe.MoEConfig(0, 128, 128, E, 4, 0, 1, 1, 1, 1, dtype, 1.0, 0, 0, 0)
    assert moe.moe_route_workspace_size(cfg) >= 0 and moe.moe_workspace_size(cfg) > 0
    assert moe.moe_max_tiles(cfg) == 0 and moe.moe_tile_rows(cfg) == 16
