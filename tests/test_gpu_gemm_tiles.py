"""The GEMM of the selected rows at the edges of its tiles and of its load pipeline: reductions of one, two
and three K steps (shorter than the look-ahead), rows and features that end inside a tile, in both tile
widths, against a plain fp32 product of the same bf16 operands."""
import pytest
import torch

from paper_2605_24022_amd import binding as B
from tests.gpu_util import say

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module", autouse=True)
def _need_gpu():
    assert torch.cuda.is_available()
    B.load()
    torch.cuda.set_device(0)


def _rand(g, *shape):
    return torch.randn(*shape, generator=g, device="cuda").to(torch.bfloat16)


def _check(got, want, scale):
    """One rounding to bf16 (up to 2^-8 of the value) and fp32 sums in another order (K <= 4096 products of
    size `scale`: 4096 * 2^-24, with a factor of four)."""
    err = (got.float() - want).abs()
    assert torch.isfinite(got).all()
    assert (err <= 2.0 ** -8 * want.abs() + 1e-3 * scale).all(), float(err.max())


# few tiles take 128 tokens each; 2500 rows of 4096 features fill one round of 256-token tiles, of SwiGLU, whose tiles
# hold 128 features of each half, 2500 rows of 2048
@pytest.mark.parametrize("k_len", [64, 128, 192, 704])
@pytest.mark.parametrize("n,n_out", [(1, 64), (127, 320), (129, 256), (300, 1088), (2500, 4096), (2305, 4032), (2500, 2048), (2305, 1984)])
def test_linear_and_swiglu(n, k_len, n_out):
    say(f"gemm tiles n={n} k={k_len} out={n_out}")
    g = torch.Generator(device="cuda").manual_seed(n + k_len)
    x, w, u, r = _rand(g, n, k_len), _rand(g, n_out, k_len), _rand(g, n_out, k_len), _rand(g, n, n_out)
    prod = x.float() @ w.float().T
    out = torch.full((n, n_out), float("nan"), device="cuda", dtype=torch.bfloat16)
    scale = k_len ** 0.5
    B.ct_linear(x, n, k_len, w, n_out, None, out)
    _check(out, prod, scale)
    out.copy_(r)                                    # the residual is the output buffer itself
    B.ct_linear(x, n, k_len, w, n_out, out, out)
    _check(out, prod + r.float(), scale)
    out.fill_(float("nan"))
    B.ct_swiglu(x, n, k_len, w, u, n_out, out)
    _check(out, torch.nn.functional.silu(prod) * (x.float() @ u.float().T), scale * scale)


@pytest.mark.parametrize("n,hq,hkv,d,style", [(1, 4, 2, 64, 0), (129, 8, 2, 64, 1), (300, 5, 5, 128, 0), (255, 8, 1, 128, 1),
                                              (2500, 32, 8, 128, 0), (2500, 64, 16, 64, 0), (2305, 32, 8, 128, 1)])
@pytest.mark.parametrize("hidden", [64, 192])
def test_qkv(n, hq, hkv, d, style, hidden):
    say(f"qkv tiles n={n} heads={hq}/{hkv} d={d} style={style} hidden={hidden}")
    g = torch.Generator(device="cuda").manual_seed(n + d)
    cfg = B.make_cfg(hidden, hq, hkv, d, 1.0e4, style)
    x, w = _rand(g, n, hidden), _rand(g, (hq + 2 * hkv) * d, hidden)
    pos = torch.arange(n, device="cuda", dtype=torch.int32) * 3 + 5
    q, k, v = (torch.full((n, h, d), float("nan"), device="cuda", dtype=torch.bfloat16) for h in (hq, hkv, hkv))
    B.ct_qkv_selected(cfg, x, None, pos, n, w, None, q, k, v)
    y = (x.double() @ w.double().T).view(n, hq + 2 * hkv, d)
    ang = pos.double()[:, None] * 1.0e4 ** (-2.0 * torch.arange(d // 2, device="cuda", dtype=torch.float64) / d)
    c, s = ang.cos()[:, None], ang.sin()[:, None]
    a, b = (y[..., :d // 2], y[..., d // 2:]) if style == 0 else (y[..., 0::2], y[..., 1::2])
    rot = torch.cat([a * c - b * s, a * s + b * c], -1) if style == 0 else torch.stack([a * c - b * s, a * s + b * c], -1).flatten(-2)
    scale = hidden ** 0.5
    _check(q, rot[:, :hq].float(), scale)
    _check(k, rot[:, hq:hq + hkv].float(), scale)
    _check(v, y[:, hq + hkv:].float(), scale)
