"""Routing of 512 tokens and more on the matrix cores: ragged token tiles, expert counts that leave wavefronts or their last
experts without work and that take two tiles, slices of one K step, of an odd number and of many, fp8 slices of one scale
block and of several, element-wise stores of an expert count that is no multiple of 4."""
import numpy as np
import pytest
import torch

from paper_2602_19128_amd import binding as moe
from paper_2602_19128_amd import synthetic as syn
from parity_util import compare_routing, oracle_all

pytestmark = pytest.mark.gpu

GROUPED = dict(scoring="sigmoid", has_bias=True, routed_scale=2.5, group_score_topn=2)

CASES = [
    syn.Workload("whole_tiles", T=512, H=64, I=64, E=256, top_k=8),                       # two slices of one step
    syn.Workload("one_over", T=513, H=192, I=64, E=17, top_k=2),                          # one wavefront with work
    syn.Workload("odd_steps", T=640, H=1344, I=64, E=49, top_k=6),                        # slices of two steps
    syn.Workload("two_expert_tiles", T=700, H=448, I=64, E=300, top_k=4),
    syn.Workload("many_steps", T=4100, H=2112, I=64, E=250, top_k=3),                     # slices of nine steps, the last of three
    syn.Workload("fp8_one_block", T=512, H=128, I=128, E=33, top_k=2, fp8=True),
    syn.Workload("fp8_blocks", T=2000, H=1152, I=128, E=256, top_k=8, n_group=8, topk_group=4, fp8=True, **GROUPED),
    syn.Workload("fp8_deep", T=9000, H=1664, I=128, E=62, top_k=2, fp8=True),             # slices of four blocks, the last of one
    syn.Workload("fp8_two_tiles", T=1025, H=640, I=128, E=384, top_k=4, fp8=True),
]


@pytest.mark.parametrize("wl", CASES, ids=lambda wl: wl.name)
def test_route_many_tokens(wl):
    cpu = syn.make_inputs(wl, seed=4)
    gpu = cpu.to("cuda:0")
    p, ids, w, margin, *_rest, keys = oracle_all(cpu)
    cfg = moe.MoEConfig.from_workload(wl)
    ids_g, w_g = moe.moe_route(cfg, gpu.x, gpu.x_scale, gpu.router_w, gpu.bias)
    again = moe.moe_route(cfg, gpu.x, gpu.x_scale, gpu.router_w, gpu.bias)
    torch.cuda.synchronize()
    compare_routing(ids_g, w_g, ids, w, margin, wl.routed_scale, wl.E, keys)
    np.testing.assert_allclose(w_g.sum(dim=1).cpu().numpy(), wl.routed_scale, rtol=1e-5)
    assert torch.equal(ids_g, again[0]) and torch.equal(w_g, again[1]), "not run-to-run identical"
