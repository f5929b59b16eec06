"""Sort-scatter of a handful of pairs: both sides of the line between its two workgroup sizes, dropped ids, a local share."""
import numpy as np
import pytest
import torch

from paper_2602_19128_amd import binding as moe
from paper_2602_19128_amd import synthetic as syn
from parity_util import check_tiles, local_permute

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("T, k, E, lo, n", [(1, 1, 1, 0, 0), (128, 2, 64, 0, 0), (85, 3, 63, 0, 0), (257, 1, 64, 0, 0),
                                            (32, 8, 65, 0, 0), (32, 8, 256, 64, 64), (31, 8, 256, 7, 33)])
def test_permute_few_pairs(T, k, E, lo, n):
    cfg = moe.MoEConfig.from_workload(syn.Workload("few_pairs", T=T, H=128, I=64, E=E, top_k=k, local_offset=lo, local_experts=n))
    rng = np.random.default_rng(T + E)
    ids = rng.integers(0, E, size=(T, k)).astype(np.int32)
    ids[rng.random((T, k)) < 0.3] = lo                       # one expert above the others
    off, sp, inv, tiles, sched = moe.moe_permute(cfg, torch.from_numpy(ids).cuda())
    torch.cuda.synchronize()
    off_r, sp_r, inv_r, kept = local_permute(ids, E, lo, n)
    assert np.array_equal(off.cpu().numpy(), off_r)
    assert np.array_equal(sp.cpu().numpy()[:kept], sp_r)
    assert np.array_equal(inv.cpu().numpy(), inv_r)
    check_tiles(tiles, sched, off_r, moe.moe_tile_rows(cfg))
