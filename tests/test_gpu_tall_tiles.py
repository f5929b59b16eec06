"""Tall tiles of the grouped GEMMs.  fp8: every height of eight row blocks and more, ragged and whole, experts of
several tiles, the shortest K loop they take and one past the first register of weight scales, a ragged last slab.
bf16: experts of three tiles and more, odd and even numbers of 32-row blocks, one K step and up, K in halves."""
import pytest
import torch

from paper_2602_19128_amd import binding as moe
from paper_2602_19128_amd import synthetic as syn

pytestmark = pytest.mark.gpu


def _dequantise(q, scale, rows):
    N, K = q.shape
    return (q.double().view(N // rows, rows, K // 128, 128) * scale.double()[:, None, :, None]).view(N, K)


HEIGHTS = [113, 128, 129, 144, 145, 160, 161, 176, 177, 192, 193, 208, 209, 224, 225, 240, 241, 256]


@pytest.mark.parametrize("rows, H, I, down_wide", [
    (HEIGHTS, 512, 256, False),                                  # gate/up: four K steps, every height
    ([700, 600, 300, 16, 0, 250], 8704, 128, False),             # gate/up: 68 K steps, experts of two and three tiles
    ((HEIGHTS + [300, 520])[:16] * 2, 4224, 512, True),          # down: four K steps, a last slab of 128 columns
    (([20, 300, 520, 800] + HEIGHTS)[:16] * 2, 4096, 1536, True),   # down: 12 K steps, rotated starts, shared weights
])
def test_tall_fp8_tiles(rows, H, I, down_wide):
    E, T = len(rows), sum(rows)
    cfg = moe.MoEConfig(T, H, I, E, 1, 0, 1, 1, 1, 1, 1, 1.0, 0, 0, 0)
    assert moe.moe_gemm_plan(cfg, "gateup")["tile_rows"] == 256
    assert (moe.moe_gemm_plan(cfg, "down")["wavefronts"] == 8) == down_wide
    gen = torch.Generator("cuda").manual_seed(H + I)
    ids = torch.repeat_interleave(torch.arange(E), torch.tensor(rows)).cuda()[torch.randperm(T, generator=gen, device="cuda")]
    ids = ids.to(torch.int32).view(T, 1)
    draw = lambda r, c: torch.randn((r, c), generator=gen, device="cuda")
    x, xs = syn.quantize_rows_1x128(draw(T, H))
    w1, s1 = syn.quantize_blocks_128x128(draw(E * 2 * I, H) * H ** -0.5)
    w2, s2 = syn.quantize_blocks_128x128(draw(E * H, I) * I ** -0.5)
    w1, s1, w2, s2 = w1.view(E, 2 * I, H), s1.view(E, -1, H // 128), w2.view(E, H, I), s2.view(E, -1, I // 128)
    offsets, pair, inv, tiles, sched = moe.moe_permute(cfg, ids)
    act, act_s = moe.moe_grouped_gemm_swiglu(cfg, x, xs, w1, s1, pair, tiles, sched)
    y = moe.moe_grouped_gemm_down(cfg, act, act_s, w2, s2, tiles, sched)
    # again with scales off the 16-byte grid, which the other K loop serves: the same sums, unless K loops start at
    # rotated columns (rows of a multiple of 4 KiB), which here are whole blocks of four steps
    xs_off = torch.empty(xs.numel() + 1, device="cuda")[1:].view_as(xs).copy_(xs)
    act2, _ = moe.moe_grouped_gemm_swiglu(cfg, x, xs_off, w1, s1, pair, tiles, sched)
    act3, _ = moe.moe_grouped_gemm_swiglu(cfg, x, xs, w1, s1, pair, tiles, sched)
    torch.cuda.synchronize()
    assert torch.equal(act.view(torch.uint8), act3.view(torch.uint8)), "not run-to-run identical"
    if H % 4096:
        assert torch.equal(act.view(torch.uint8), act2.view(torch.uint8)), "the K loops differ"
    off, xd = offsets.tolist(), _dequantise(x, xs, 1)
    for e in range(E):
        lo, hi = off[e], off[e + 1]
        if lo == hi:
            continue
        gu = xd[pair[lo:hi].long()] @ _dequantise(w1[e], s1[e], 128).t()
        ref = torch.nn.functional.silu(gu[:, :I]) * gu[:, I:]
        got, sc = _dequantise(act[lo:hi], act_s[lo:hi], 1), act_s[lo:hi].double().repeat_interleave(128, dim=1)
        # half a step of e4m3 (2^-4 of the value, 2^-10 of the scale among the subnormals), and the fp32 sums behind it
        bound = ref.abs() * 2.0 ** -4 + sc * 2.0 ** -10 + 1e-5 * gu.abs().max() ** 2
        assert ((got - ref).abs() <= bound).all(), f"gate/up, expert {e} of {hi - lo} rows"
        w = _dequantise(w2[e], s2[e], 128).t()
        ref = got @ w
        # one bf16 rounding (2^-9 of the value) of the sum; the fp8 matrix instruction adds its 128 products on a
        # grid fixed by the largest of them (2^-14 of the sum of magnitudes measured, in gemm_tile as well)
        bound = ref.abs() * 2.0 ** -8 + (got.abs() @ w.abs()) * 2.0 ** -13
        assert ((y[lo:hi].double() - ref).abs() <= bound).all(), f"down, expert {e} of {hi - lo} rows"


@pytest.mark.parametrize("H, I", [
    (64, 8192), (128, 8192), (192, 8256), (1024, 8192),          # gate/up: 1, 2, 3 and 16 K steps, a ragged last slab
    (16384, 64), (16448, 192),                                   # down: 1 and 3 K steps, a ragged last slab
])
def test_tall_bf16_tiles(H, I):
    rows = [1825, 1024, 700, 600, 513, 257, 40, 0]               # eight, four and three tiles, of 5 to 8 blocks of 32 rows
    E, T = len(rows), sum(rows)
    cfg = moe.MoEConfig(T, H, I, E, 1, 0, 1, 1, 1, 1, 0, 1.0, 0, 0, 0)
    which = "gateup" if I > H else "down"
    plan = moe.moe_gemm_plan(cfg, which)
    assert plan["tile_rows"] == 256 and plan["wavefronts"] == 8 and plan["k_split"] == 1
    gen = torch.Generator("cuda").manual_seed(H + I)
    ids = torch.repeat_interleave(torch.arange(E), torch.tensor(rows)).cuda()[torch.randperm(T, generator=gen, device="cuda")]
    offsets, pair, inv, tiles, sched = moe.moe_permute(cfg, ids.to(torch.int32).view(T, 1))
    draw = lambda *shape: torch.randn(shape, generator=gen, device="cuda")
    off = offsets.tolist()
    # one bf16 rounding (2^-9 of the value) of fp32 sums (2^-24 a term, of the sum of magnitudes)
    if which == "gateup":
        x, w1 = draw(T, H).bfloat16(), (draw(E, 2 * I, H) * H ** -0.5).bfloat16()
        act, _ = moe.moe_grouped_gemm_swiglu(cfg, x, None, w1, None, pair, tiles, sched)
        for e in range(E):
            lo, hi = off[e], off[e + 1]
            xe, w = x[pair[lo:hi].long()].double(), w1[e].double().t()
            gu = xe @ w
            ref = torch.nn.functional.silu(gu[:, :I]) * gu[:, I:]
            slack = (xe.abs() @ w.abs()).max() ** 2 * 2.0 ** -20 if hi > lo else 0.0
            assert ((act[lo:hi].double() - ref).abs() <= ref.abs() * 2.0 ** -8 + slack).all(), f"expert {e}"
    else:
        act, w2 = draw(T, I).bfloat16(), (draw(E, H, I) * I ** -0.5).bfloat16()
        y = moe.moe_grouped_gemm_down(cfg, act, None, w2, None, tiles, sched)
        for e in range(E):
            lo, hi = off[e], off[e + 1]
            a, w = act[lo:hi].double(), w2[e].double().t()
            ref = a @ w
            assert ((y[lo:hi].double() - ref).abs() <= ref.abs() * 2.0 ** -8 + (a.abs() @ w.abs()) * 2.0 ** -20).all(), f"expert {e}"


@pytest.mark.parametrize("T", [700, 1825])
def test_tall_bf16_tiles_with_k_in_halves(T):
    """Every token goes to both experts: three (eight) tiles each in the forward's K-split down projection."""
    H, I, E = 576, 4096, 2
    cfg = moe.MoEConfig(T, H, I, E, 2, 0, 1, 1, 1, 1, 0, 1.0, 0, 0, 0)
    assert moe.moe_gemm_plan(cfg, "down")["k_split"] == 2
    gen = torch.Generator("cuda").manual_seed(T)
    draw = lambda *shape: torch.randn(shape, generator=gen, device="cuda")
    x, router = draw(T, H).bfloat16(), draw(E, H) * H ** -0.5
    w1, w2 = (draw(E, 2 * I, H) * H ** -0.5).bfloat16(), (draw(E, H, I) * I ** -0.5).bfloat16()
    out = moe.moe_forward(cfg, x, None, router, None, w1, None, w2, None)
    xd = x.double()
    w = torch.softmax(xd @ router.double().t(), dim=1)
    ref, mag = torch.zeros_like(xd), torch.zeros_like(xd)
    for e in range(E):
        gu = xd @ w1[e].double().t()
        act = (torch.nn.functional.silu(gu[:, :I]) * gu[:, I:]).bfloat16().double()
        ref += w[:, e:e + 1] * (act @ w2[e].double().t())
        mag += w[:, e:e + 1] * (act.abs() @ w2[e].double().abs().t())
    # bf16 rows (2^-9 each of what they add) and a bf16 output; activations whose rounding flips (2^-8 of one of 4096 terms)
    bound = ref.abs() * 2.0 ** -8 + mag * 2.0 ** -9
    assert ((out.double() - ref).abs() <= bound).all()
