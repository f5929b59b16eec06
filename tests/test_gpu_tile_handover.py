"""Workgroups that work through a short tile and then a tall one: a hot expert among few, whose work range outgrows its
share of the grid and whose last tile is short.  (That these cases hold such pairs: tests/test_host_item_walk.py.)"""
import pytest
import torch

from paper_2602_19128_amd import binding as moe
from paper_2602_19128_amd import synthetic as syn

pytestmark = pytest.mark.gpu

# which, dtype, rows of the experts, H, I
CASES = [
    ("gateup", "bf16", [2161] + [200] * 7, 192, 8192),           # nine tiles, the last of eight row blocks
    ("gateup", "bf16", [170] * 5 + [2900] + [170] * 2, 2048, 8192),
    ("gateup", "fp8", [2405] + [170] * 7, 512, 8192),            # ten tiles, the last of seven row blocks
    ("gateup", "fp8", [2900] + [170] * 7, 4096, 4096),
    ("down", "bf16", [2900] + [16] * 31, 4096, 192),
    ("down", "fp8", [2900] + [16] * 31, 4096, 512),
]


def config(which, dtype, rows, H, I):
    return moe.MoEConfig(sum(rows), H, I, len(rows), 1, 0, 1, 1, 1, 1, 1 if dtype == "fp8" else 0, 1.0, 0, 0, 0)


def _dequantise(q, scale, rows):
    N, K = q.shape
    return (q.double().view(N // rows, rows, K // 128, 128) * scale.double()[:, None, :, None]).view(N, K)


def check_gemm(which, dtype, rows, H, I):
    """One grouped GEMM on shuffled tokens against float64, three times on the same inputs."""
    E, T, fp8 = len(rows), sum(rows), dtype == "fp8"
    cfg = config(which, dtype, rows, H, I)
    gen = torch.Generator("cuda").manual_seed(H + I)
    ids = torch.repeat_interleave(torch.arange(E), torch.tensor(rows)).cuda()[torch.randperm(T, generator=gen, device="cuda")]
    offsets, pair, inv, tiles, sched = moe.moe_permute(cfg, ids.to(torch.int32).view(T, 1))
    off = offsets.tolist()
    draw = lambda r, c: torch.randn((r, c), generator=gen, device="cuda")
    cols, n = (H, 2 * I) if which == "gateup" else (I, H)
    a, w = draw(T, cols), draw(E * n, cols) * cols ** -0.5
    a, a_s = syn.quantize_rows_1x128(a) if fp8 else (a.bfloat16(), None)
    w, w_s = syn.quantize_blocks_128x128(w) if fp8 else (w.bfloat16(), None)
    w = w.view(E, n, cols)
    w_s = w_s.view(E, n // 128, cols // 128) if fp8 else None
    ad = _dequantise(a, a_s, 1) if fp8 else a.double()
    call = moe.moe_grouped_gemm_swiglu if which == "gateup" else moe.moe_grouped_gemm_down
    args = (cfg, a, a_s, w, w_s) + ((pair, tiles, sched) if which == "gateup" else (tiles, sched))
    for _ in range(3):
        got = call(*args)
        if which == "gateup":
            got, got_s = got
            gotd = _dequantise(got, got_s, 1) if fp8 else got.double()
        for e in range(E):
            lo, hi = off[e], off[e + 1]
            x = ad[pair[lo:hi].long()] if which == "gateup" else ad[lo:hi]
            wd = (_dequantise(w[e], w_s[e], 128) if fp8 else w[e].double()).t()
            ref, mag = x @ wd, x.abs() @ wd.abs()
            if which == "down":
                # one bf16 rounding (2^-9 of the value) of the sum: fp32 sums add 2^-24 a term, the fp8 matrix instruction
                # adds its products on a grid fixed by the largest of them (2^-14 of the sum of magnitudes)
                bound = ref.abs() * 2.0 ** -8 + mag * 2.0 ** (-13 if fp8 else -20)
                assert ((got[lo:hi].double() - ref).abs() <= bound).all(), f"expert {e} of {hi - lo} rows"
                continue
            gu = ref
            ref = torch.nn.functional.silu(gu[:, :I]) * gu[:, I:]
            if fp8:      # half a step of e4m3 (2^-4 of the value, 2^-10 of the scale among the subnormals), the fp32 sums
                sc = got_s[lo:hi].double().repeat_interleave(128, dim=1)
                bound = ref.abs() * 2.0 ** -4 + sc * 2.0 ** -10 + 1e-5 * gu.abs().max() ** 2
            else:        # one bf16 rounding of fp32 sums
                bound = ref.abs() * 2.0 ** -8 + mag.max() ** 2 * 2.0 ** -20
            assert ((gotd[lo:hi] - ref).abs() <= bound).all(), f"expert {e} of {hi - lo} rows"


@pytest.mark.parametrize("which, dtype, rows, H, I", CASES)
def test_short_tile_then_tall_tile(which, dtype, rows, H, I):
    check_gemm(which, dtype, rows, H, I)
