"""Frequency scores at lengths that take the run-time plan: every radix in every place, strips of one to 64
column pairs, both factors of the lengths beyond 4096 tokens, against a 64-bit FFT of the same values."""
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


@pytest.mark.parametrize("n,row,n_batch,alpha", [
    (1, 2, 2, 0.5), (5, 6, 1, 1.0), (27, 64, 2, 0.5), (96, 1024, 1, 0.5), (100, 128, 3, 0.3), (486, 256, 1, 0.5),
    (625, 64, 2, 0.5), (640, 1000, 1, 0.7), (1500, 1024, 1, 0.5), (1500, 6, 1, 0.5), (1536, 128, 2, 0.0), (1944, 64, 1, 0.5),
    (2025, 48, 1, 0.4), (2048, 10, 1, 0.5), (2187, 32, 1, 0.5), (2500, 128, 1, 0.5), (3645, 16, 1, 0.5), (4050, 1000, 1, 0.5),
    (4096, 6, 1, 0.5), (4860, 128, 2, 0.5), (9375, 20, 1, 0.5), (15625, 16, 1, 0.5), (100000, 8, 1, 0.2)])
def test_scores_against_fp64(n, row, n_batch, alpha):
    say(f"frequency lengths n={n} row={row} batch={n_batch} alpha={alpha}")
    g = torch.Generator(device="cuda").manual_seed(n)
    k, v = (torch.randn(n_batch, n, row, generator=g, device="cuda").to(torch.bfloat16) for _ in range(2))
    ws_bytes = B.ct_frequency_workspace_bytes(n_batch, n, row)
    assert ws_bytes > 0
    ws = torch.empty(ws_bytes, dtype=torch.uint8, device="cuda")
    scores = torch.full((n_batch, n), -1.0, device="cuda")
    B.ct_frequency_scores(k, v, n_batch, n * row, n, row, alpha, scores, ws, ws_bytes)
    kept = (torch.arange(n // 2 + 1, device="cuda") < int(alpha * (n // 2 + 1) + 1e-9)).double()[None, :, None]
    want = 0
    for x in (k, v):
        want = want + 0.5 * torch.fft.irfft(torch.fft.rfft(x.double(), dim=1) * kept, n=n, dim=1).norm(dim=2)
    # roundings of 2^-24, about 4 log2(n) <= 68 of them deep, relative to the largest score
    err = float((scores.double() - want).abs().max())
    assert torch.isfinite(scores).all() and err <= 4.1e-6 * max(float(want.max()), 1e-30), err


@pytest.mark.parametrize("n", [256, 512, 1024, 2048, 4096])
@pytest.mark.parametrize("row,n_batch", [(128, 1), (1024, 4), (384, 3)])
def test_power_of_two_lengths_around_half_the_spectrum(n, row, n_batch):
    """Cutoffs at and on both sides of N / 4 (where half of the last pass is left out), strips of one and several
    rounds, sequences that fill whole XCDs and not."""
    for cutoff in (1, n // 8 + 1, n // 4 - 1, n // 4, n // 4 + 1, n // 2):
        test_scores_against_fp64(n, row, n_batch, (cutoff + 0.5) / (n // 2 + 1))


@pytest.mark.parametrize("n", [1023, 1025, 2047, 2048, 2049, 3000, 4096, 4097, 8191, 8193, 9001, 16384, 16385, 20481, 32767, 32768, 32769])
@pytest.mark.parametrize("levels", [3, 1 << 20])
def test_topk_where_scores_per_thread_change(n, levels):
    """Both sides of every number of scores that a thread holds, with many ties and with few, of either sign."""
    say(f"topk n={n} levels={levels}")
    g = torch.Generator(device="cuda").manual_seed(n)
    scores = (torch.randint(0, levels, (3, n), generator=g, device="cuda") - levels // 2).float() / levels
    order = torch.sort(scores.cpu(), dim=1, descending=True, stable=True).indices
    for k in (1, n // 7, n):
        idx = torch.full((3, k), -1, dtype=torch.int32, device="cuda")
        B.ct_topk_indices(scores, 3, n, k, idx)
        assert torch.equal(idx.cpu().long(), order[:, :k].sort(dim=1).values)


@pytest.mark.parametrize("n", [256, 512, 1024, 2048, 4096])
@pytest.mark.parametrize("alpha", [0.5, 0.75])
def test_power_of_two_lengths_at_every_magnitude(n, alpha):
    """Data scaled by a power of two give the same scores scaled by it, to the bit, from where squares are far from underflow
    to where they are just finite; beyond that, up to the largest spectrum that bf16 data of one size have, scores are
    infinite and never NaN."""
    say(f"frequency magnitudes n={n} alpha={alpha}")
    row = 128
    g = torch.Generator(device="cuda").manual_seed(n)
    k, v = (torch.randn((1, n, row), generator=g, device="cuda").to(torch.bfloat16) for _ in range(2))
    ws = torch.empty(B.ct_frequency_workspace_bytes(1, n, row), dtype=torch.uint8, device="cuda")

    def scores(by):
        out = torch.empty(1, n, device="cuda")
        B.ct_frequency_scores((k.float() * by).to(torch.bfloat16), (v.float() * by).to(torch.bfloat16), 1, n * row, n, row, alpha, out,
                              ws, ws.numel())
        return out

    want = scores(1.0)
    for e in (-45, -20, 20, 40):
        assert torch.equal(scores(2.0 ** e), want * 2.0 ** e), e
    for e in (70, 95, 105, 112):          # (bins reach 2^(e + 8))
        assert torch.isposinf(scores(2.0 ** e)).all(), e
