"""Routing with infinite and NaN operands on the matrix cores, which carry a router weight as three bf16 planes: an
infinite weight, one beyond the bf16 range and an infinite hidden state give the logits that fp32 sums give."""
import pytest
import torch

from paper_2602_19128_amd import binding as moe
from paper_2602_19128_amd import synthetic as syn

pytestmark = pytest.mark.gpu

INF = float("inf")


def _layer(T, E, fp8, n_group=1, H=384, k=6):
    cfg = moe.MoEConfig(T, H, 128, E, k, 1, 1, n_group, max(1, n_group // 2), 2, 1 if fp8 else 0, 1.0, 0, 0, 0)
    gen = torch.Generator("cuda").manual_seed(T + E)
    x = torch.randn((T, H), generator=gen, device="cuda")
    x, xs = syn.quantize_rows_1x128(x) if fp8 else (x.bfloat16(), None)
    router = torch.randn((E, H), generator=gen, device="cuda") * H ** -0.5
    bias = torch.rand((E,), generator=gen, device="cuda") * 0.2
    return cfg, x, xs, router, bias


def _reference(cfg, x, xs, router, bias):
    xd = x.double() if xs is None else (x.double().view(cfg.T, -1, 128) * xs.double()[:, :, None]).view(cfg.T, cfg.H)
    s = torch.sigmoid((xd[:, None, :] * router.double()[None]).sum(dim=2))      # (no matrix product: inf * 0 is NaN here)
    key = s + bias.double()
    if cfg.n_group > 1:
        grouped = key.view(cfg.T, cfg.n_group, -1)
        best = grouped.topk(2, dim=2).values.sum(dim=2).topk(cfg.topk_group, dim=1).indices
        kept = torch.zeros(grouped.shape[:2], dtype=torch.bool, device="cuda").scatter_(1, best, True)
        key = key.masked_fill(~kept[:, :, None].expand_as(grouped).reshape(key.shape), -INF)
    order = torch.sort(key, dim=1, descending=True, stable=True)
    ids = order.indices[:, :cfg.top_k]
    margin = (order.values[:, :cfg.top_k] - order.values[:, 1:cfg.top_k + 1]).amin(dim=1)
    w = s.gather(1, ids)
    return ids, w / w.sum(dim=1, keepdim=True), margin


@pytest.mark.parametrize("fp8", [False, True])
@pytest.mark.parametrize("T, E, n_group", [(3, 512, 1), (200, 256, 8), (511, 40, 1), (512, 512, 1), (700, 130, 1)])
def test_infinite_operands(T, E, n_group, fp8):
    cfg, x, xs, router, bias = _layer(T, E, fp8, n_group)
    H = cfg.H
    router[7, 5] = INF                                     # sigmoid 1 or 0 by the sign of the hidden value
    router[E - 1, H - 1] = -INF
    router[2, 130] = 3.4e38                                # finite weights that round to an infinite bf16: times 0 ...
    router[3, 131] = 3.4e38                                # ... and times 2^-126
    x = x.clone()
    if not fp8:
        x[:, 130] = 0.0
        x[:, 131] = 2.0 ** -126
        x[T - 1, 17] = INF                                 # ties of infinite logits: the lower index first
    else:
        x.view(torch.uint8)[:, 130:132] = 0
        xs[T - 1, 1] = 2.0 ** 126                          # logits of any size, and infinite ones
    ids, w = moe.moe_route(cfg, x, xs, router, bias)
    ids_r, w_r, margin = _reference(cfg, x, xs, router, bias)
    clear = (margin > 1e-6) & ~torch.isnan(w_r).any(dim=1)
    clear[T - 1] = False
    assert int(clear.sum()) >= T // 2
    assert torch.equal(ids[clear].long(), ids_r[clear])
    assert torch.allclose(w[clear].double(), w_r[clear], rtol=2e-5, atol=2e-6)
    assert bool(((ids >= 0) & (ids < E)).all())
    assert all(len(set(row)) == cfg.top_k for row in ids.tolist())
    if not fp8:
        # infinite logits of either sign, NaN only where a weight is infinite as well
        s = torch.sigmoid((x[T - 1].double() * router.double()).sum(dim=1))
        keyed = torch.where(torch.isnan(s), torch.full_like(s, -INF), s + bias.double())
        finite_top = [e for e in ids[T - 1].tolist() if not bool(torch.isnan(s[e]))]
        assert all(float(s[e]) == 1.0 for e in finite_top)
        assert torch.isfinite(keyed[finite_top]).all()


@pytest.mark.parametrize("T, E", [(5, 64), (511, 256), (600, 512)])
def test_nan_keys_give_distinct_experts(T, E):
    cfg, x, xs, router, bias = _layer(T, E, True)
    bits = bias.view(torch.int32)
    bits.fill_(-1)                                         # NaN with every bit set: the smallest key there is
    ids, _ = moe.moe_route(cfg, x, xs, router, bias)
    assert all(sorted(row) == list(range(cfg.top_k)) for row in ids.tolist())
    x.view(torch.uint8)[0] = 0x7f                          # a hidden state of NaNs
    ids, _ = moe.moe_route(cfg, x, xs, router, torch.zeros_like(bias))
    assert bool(((ids >= 0) & (ids < E)).all()) and all(len(set(row)) == cfg.top_k for row in ids.tolist())
