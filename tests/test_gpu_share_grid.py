"""Grouped GEMMs of a share of the experts whose grid is made for a balanced router: lists of few tiles, of as many as the grid
expects, and of several times that (every token routed to an expert held here)."""
import pytest
import torch

from paper_2602_19128_amd import binding as moe
from paper_2602_19128_amd import synthetic as syn

pytestmark = pytest.mark.gpu


def _dequantise(q, scale, rows):
    N, K = q.shape
    return (q.double().view(N // rows, rows, K // 128, 128) * scale.double()[:, None, :, None]).view(N, K)


@pytest.mark.parametrize("dtype, H, I", [("bf16", 448, 320), ("fp8", 512, 384)])
@pytest.mark.parametrize("T, E, EL, lo, local", [
    (40, 256, 3, 250, 1), (40, 64, 8, 16, 40), (700, 128, 16, 0, 90), (900, 64, 8, 16, 900), (4096, 16, 2, 6, 512),
    (6000, 64, 8, 56, 6000), (6000, 512, 70, 3, 6000),
])
def test_share_of_the_experts(T, E, EL, lo, local, dtype, H, I):
    fp8 = dtype == "fp8"
    cfg = moe.MoEConfig(T, H, I, E, 1, 0, 1, 1, 1, 1, 1 if fp8 else 0, 1.0, lo, EL, 0)
    gen = torch.Generator("cuda").manual_seed(T + E)
    draw = lambda r, c: torch.randn((r, c), generator=gen, device="cuda")
    ids = torch.randint(lo, lo + EL, (T,), generator=gen, device="cuda")
    ids[:local // 3] = lo                                    # one expert above the others
    away = [e for e in (lo - 1, lo + EL) if 0 <= e < E][0]
    ids[local:] = away
    ids = ids[torch.randperm(T, generator=gen, device="cuda")].to(torch.int32).view(T, 1)
    x, w1, w2 = draw(T, H), draw(EL * 2 * I, H) * H ** -0.5, draw(EL * H, I) * I ** -0.5
    xs = s1 = s2 = None
    if fp8:
        (x, xs), (w1, s1), (w2, s2) = syn.quantize_rows_1x128(x), syn.quantize_blocks_128x128(w1), syn.quantize_blocks_128x128(w2)
        xd, w1d, w2d = _dequantise(x, xs, 1), _dequantise(w1, s1, 128), _dequantise(w2, s2, 128)
        s1, s2 = s1.view(EL, 2 * I // 128, H // 128), s2.view(EL, H // 128, I // 128)
    else:
        x, w1, w2 = x.bfloat16(), w1.bfloat16(), w2.bfloat16()
        xd, w1d, w2d = x.double(), w1.double(), w2.double()
    w1, w2, w1d, w2d = w1.view(EL, 2 * I, H), w2.view(EL, H, I), w1d.view(EL, 2 * I, H), w2d.view(EL, H, I)
    offsets, pair, inv, tiles, sched = moe.moe_permute(cfg, ids)
    act, act_s = moe.moe_grouped_gemm_swiglu(cfg, x, xs, w1, s1, pair, tiles, sched)
    y = moe.moe_grouped_gemm_down(cfg, act, act_s, w2, s2, tiles, sched)
    off = offsets.tolist()
    assert off[-1] == local
    for e in range(EL):
        a, b = off[e], off[e + 1]
        if a == b:
            continue
        xe = xd[pair[a:b].long()]
        gu = xe @ w1d[e].t()
        ref = torch.nn.functional.silu(gu[:, :I]) * gu[:, I:]
        if fp8:      # half a step of e4m3 (2^-4 of the value, 2^-10 of the scale among the subnormals), the fp32 sums
            got, sc = _dequantise(act[a:b], act_s[a:b], 1), act_s[a:b].double().repeat_interleave(128, dim=1)
            bound = ref.abs() * 2.0 ** -4 + sc * 2.0 ** -10 + 1e-5 * gu.abs().max() ** 2
        else:        # one bf16 rounding (2^-9 of the value) of fp32 sums
            got = act[a:b].double()
            bound = ref.abs() * 2.0 ** -8 + (xe.abs() @ w1d[e].abs().t()).max() ** 2 * 2.0 ** -20
        assert ((got - ref).abs() <= bound).all(), f"gate/up, expert {e} of {b - a} rows"
        ref, mag = got @ w2d[e].t(), got.abs() @ w2d[e].abs().t()
        # one bf16 rounding; the fp8 matrix instruction adds its products on a grid fixed by the largest of them (2^-14 of
        # the sum of magnitudes), fp32 sums add 2^-24 a term
        bound = ref.abs() * 2.0 ** -8 + mag * 2.0 ** (-13 if fp8 else -20)
        assert ((y[a:b].double() - ref).abs() <= bound).all(), f"down, expert {e} of {b - a} rows"
