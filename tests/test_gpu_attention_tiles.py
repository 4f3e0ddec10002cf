"""Selected-row attention at the edges of its key tiles (64 keys, fragments of 16 and 32): contexts that end just before,
at and just behind them, from a single key on, against a plain 64-bit softmax; every head size and group size."""
import pytest
import torch

from paper_2605_24022_amd import binding as B
from tests.gpu_util import say

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("hq,hkv,d", [(2, 2, 64), (8, 2, 128), (16, 1, 64), (32, 2, 128), (4, 2, 128)])
def test_contexts_around_the_key_tiles(hq, hkv, d):
    assert torch.cuda.is_available()
    B.load()
    g = torch.Generator(device="cuda").manual_seed(hq + d)
    cfg = B.make_cfg(64, hq, hkv, d, 1.0e4)
    for n_ctx in (1, 2, 15, 17, 31, 33, 63, 64, 65, 127, 128, 129, 191, 192, 193, 257, 321):
        say(f"attention tiles heads={hq}/{hkv} d={d} n_ctx={n_ctx}")
        n_sel = min(n_ctx, 70)
        sel = torch.randperm(n_ctx, generator=g, device="cuda")[:n_sel]
        sel[-1] = n_ctx - 1
        sel = torch.unique(sel).to(torch.int32)
        n_sel = sel.numel()
        q, k, v = (torch.randn(n, h, d, generator=g, device="cuda").to(torch.bfloat16) for n, h in ((n_sel, hq), (n_ctx, hkv), (n_ctx, hkv)))
        out = torch.full((n_sel, hq, d), float("nan"), device="cuda", dtype=torch.bfloat16)
        lse = torch.full((n_sel, hq), float("nan"), device="cuda")
        B.ct_selected_attention(cfg, q, k, v, n_ctx, sel, n_sel, out, lse, None, 0)
        hidden = torch.arange(n_ctx, device="cuda")[None, :] > sel[:, None]
        for h in range(hq):
            kv = h // (hq // hkv)
            s = (q[:, h].double() @ k[:, kv].double().T.contiguous() * d ** -0.5).masked_fill(hidden, float("-inf"))
            p, val = torch.softmax(s, 1), v[:, kv].double()
            want, size = p @ val, p @ val.abs()
            # probabilities are rounded to bf16 (by up to 2^-8 of each; their sum is not) and so is the result
            assert ((out[:, h].double() - want).abs() <= 2.0 ** -8 * (size + want.abs()) + 1e-4 * size).all(), (n_ctx, h)
            assert ((lse[:, h].double() - torch.logsumexp(s, 1)).abs() <= 1e-4).all(), (n_ctx, h)


@pytest.mark.parametrize("n_sel,split", [(3072, False), (40, True)])
def test_row_sum_over_a_long_flat_row(n_sel, split):
    """Every key but the first has the same score, so what a sum loses per addition adds up along the row."""
    assert torch.cuda.is_available()
    B.load()
    n_ctx, hq, hkv, d = 65536, 32, 8, 128
    say(f"attention flat row n_ctx={n_ctx} n_sel={n_sel}")
    cfg = B.make_cfg(64, hq, hkv, d, 1.0e4)
    sel = torch.arange(n_ctx - n_sel, n_ctx, device="cuda", dtype=torch.int32)
    # one dimension carries the scores: a bf16 product, exact in fp32; the first key is twice the others
    q = torch.zeros(n_sel, hq, d, device="cuda", dtype=torch.bfloat16)
    a = torch.rand(n_sel, hq, generator=torch.Generator(device="cuda").manual_seed(3), device="cuda") * 40 + 1
    q[:, :, 0] = a.to(torch.bfloat16)
    k = torch.zeros(n_ctx, hkv, d, device="cuda", dtype=torch.bfloat16)
    k[:, :, 0] = 1.0
    k[0, :, 0] = 2.0
    v = torch.ones(n_ctx, hkv, d, device="cuda", dtype=torch.bfloat16)
    out = torch.empty(n_sel, hq, d, device="cuda", dtype=torch.bfloat16)
    lse = torch.empty(n_sel, hq, device="cuda")
    ws = torch.empty(B.ct_workspace_bytes(cfg, n_ctx, n_sel), dtype=torch.uint8, device="cuda")
    B.ct_selected_attention(cfg, q, k, v, n_ctx, sel, n_sel, out, lse, ws if split else None, ws.numel() if split else 0)
    s = q[:, :, 0].double() * d ** -0.5
    want = 2 * s + torch.log1p(sel.double()[:, None] * torch.exp(-s))
    # a lane adds n_ctx / 64 tiles to a growing sum, each addition off by half a unit of the sum so far (2^-24 of half the
    # final one on average), after 16 within a tile; then roundings of exponents and logarithms up to 32
    bound = (n_ctx / 128 + 16 + 4 * 32) * 2.0 ** -24
    err = float((lse.double() - want).abs().max())
    assert err <= bound, (err, bound)
    assert (out.double() - 1).abs().max() <= 2.0 ** -8
