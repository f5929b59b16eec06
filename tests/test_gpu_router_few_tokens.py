"""Routing of fewer than 512 tokens on the matrix cores: ragged token and expert tiles, one K step and several per
slice of H, fp8 slices that end on scale blocks, the element-wise stores of an expert count that is no multiple of 4."""
import numpy as np
import pytest
import torch

from paper_2602_19128_amd import binding as moe
from paper_2602_19128_amd import synthetic as syn
from parity_util import compare_routing, oracle_all

pytestmark = pytest.mark.gpu

GROUPED = dict(scoring="sigmoid", has_bias=True, routed_scale=2.5, group_score_topn=2)

CASES = [
    syn.Workload("one_token", T=1, H=128, I=128, E=17, top_k=2, fp8=True),
    syn.Workload("below_a_tile", T=63, H=384, I=128, E=130, top_k=6, fp8=True),
    syn.Workload("above_a_tile", T=65, H=640, I=128, E=256, top_k=8, n_group=8, topk_group=4, fp8=True, **GROUPED),
    syn.Workload("quantised_here", T=70, H=256, I=128, E=64, top_k=6, n_group=4, topk_group=2, fp8=True, quantize_x=True, **GROUPED),
    syn.Workload("eight_slices", T=201, H=512, I=128, E=256, top_k=8, fp8=True),          # slices of half a scale block
    syn.Workload("whole_blocks", T=511, H=384, I=128, E=384, top_k=4, fp8=True),
    syn.Workload("bf16_ragged", T=200, H=1344, I=64, E=49, top_k=6),
    syn.Workload("bf16_most", T=511, H=192, I=64, E=512, top_k=8),
]


@pytest.mark.parametrize("wl", CASES, ids=lambda wl: wl.name)
def test_route_few_tokens(wl):
    cpu = syn.make_inputs(wl, seed=3)
    gpu = cpu.to("cuda:0")
    p, ids, w, margin, *_rest, keys = oracle_all(cpu)
    cfg = moe.MoEConfig.from_workload(wl)
    moe.moe_single_launch(True)
    try:                                                  # not a layer of the single launch, whose router is another one
        assert moe.moe_single_launch_mode(cfg) == moe.SINGLE_LAUNCH_NONE
    finally:
        moe.moe_single_launch(False)
    ids_g, w_g = moe.moe_route(cfg, gpu.x, gpu.x_scale, gpu.router_w, gpu.bias)
    torch.cuda.synchronize()
    compare_routing(ids_g, w_g, ids, w, margin, wl.routed_scale, wl.E, keys)
    np.testing.assert_allclose(w_g.sum(dim=1).cpu().numpy(), wl.routed_scale, rtol=1e-5)


@pytest.mark.parametrize("T, H, I, E", [(201, 512, 128, 256), (1, 128, 128, 256), (300, 256, 256, 64)])
def test_forward_with_partial_logits_over_later_sections(T, H, I, E):
    """moe_forward on a workspace of exactly the stated size against its steps, which have scratch of their own."""
    wl = syn.Workload("overlaid", T=T, H=H, I=I, E=E, top_k=4, fp8=True)
    gpu = syn.make_inputs(wl, seed=5).to("cuda:0")
    cfg = moe.MoEConfig.from_workload(wl)
    ids, w = moe.moe_route(cfg, gpu.x, gpu.x_scale, gpu.router_w, gpu.bias)
    _, pair, inv, tiles, sched = moe.moe_permute(cfg, ids)
    act, act_scale = moe.moe_grouped_gemm_swiglu(cfg, gpu.x, gpu.x_scale, gpu.w1, gpu.w1_scale, pair, tiles, sched)
    ref = moe.moe_combine(cfg, moe.moe_grouped_gemm_down(cfg, act, act_scale, gpu.w2, gpu.w2_scale, tiles, sched), w, inv)
    size = moe.moe_workspace_size(cfg)
    for fill in (0, 0xff):
        ws = torch.full((size + 4096,), fill, dtype=torch.uint8, device="cuda:0")
        ws[size:] = 0xa5
        out = moe.moe_forward(cfg, gpu.x, gpu.x_scale, gpu.router_w, gpu.bias, gpu.w1, gpu.w1_scale, gpu.w2, gpu.w2_scale,
                              workspace=ws[:size])
        torch.cuda.synchronize()
        assert torch.equal(out.view(torch.int16), ref.view(torch.int16))
        assert bool((ws[size:] == 0xa5).all())
