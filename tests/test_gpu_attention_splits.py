"""Attention of few selected rows: the layer call splits the key range as far as its workspace goes.  Every amount of
scratch, from what a call needs at least to what ct_workspace_bytes asks for, gives the same rows, against a plain
64-bit softmax; lengths around the limits of the rule, rows that see one key, and rows whose splits are empty.  The
attention entry points split only where they always needed scratch, and leave it alone where they did not."""
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


SHAPES = [(8, 2, 64, 512, 9), (8, 2, 64, 513, 1), (8, 2, 64, 1024, 153), (32, 8, 128, 1025, 65), (16, 16, 64, 4097, 3),
          (16, 1, 128, 3000, 200), (32, 8, 128, 8192, 81), (4, 4, 128, 2049, 2000), (32, 2, 128, 700, 700)]


@pytest.mark.parametrize("hq,hkv,d,n_ctx,n_sel", SHAPES)
def test_any_scratch_gives_the_same_rows(hq, hkv, d, n_ctx, n_sel):
    say(f"attention splits heads={hq}/{hkv} d={d} n_ctx={n_ctx} n_sel={n_sel}")
    g = torch.Generator(device="cuda").manual_seed(n_ctx + n_sel)
    cfg = B.make_cfg(64, hq, hkv, d, 1.0e4)
    q, k, v = (torch.randn(n, h, d, generator=g, device="cuda").to(torch.bfloat16) for n, h in ((n_sel, hq), (n_ctx, hkv), (n_ctx, hkv)))
    sel = torch.randperm(n_ctx, generator=g, device="cuda")[:n_sel]
    sel[0] = 0                                   # one key
    sel = torch.unique(sel).to(torch.int32)      # ascending
    n_sel = sel.numel()
    q = q[:n_sel].contiguous()
    want, size = (torch.empty(n_sel, hq, d, device="cuda", dtype=torch.float64) for _ in range(2))
    want_lse = torch.empty(n_sel, hq, device="cuda", dtype=torch.float64)
    hidden = torch.arange(n_ctx, device="cuda")[None, :] > sel[:, None]
    for h in range(hq):
        kv = h // (hq // hkv)
        s = (q[:, h].double() @ k[:, kv].double().T.contiguous() * d ** -0.5).masked_fill(hidden, float("-inf"))
        want[:, h] = torch.softmax(s, 1) @ v[:, kv].double()
        size[:, h] = torch.softmax(s, 1) @ v[:, kv].double().abs()
        want_lse[:, h] = torch.logsumexp(s, 1)
    most = B.ct_workspace_bytes(cfg, n_ctx, n_sel)
    ws = torch.empty(most, dtype=torch.uint8, device="cuda")
    ran = 0
    for share in (0.0, 0.1, 0.4, 0.7, 1.0):
        out = torch.full((n_sel, hq, d), float("nan"), device="cuda", dtype=torch.bfloat16)
        lse = torch.full((n_sel, hq), float("nan"), device="cuda")
        try:
            B.ct_selected_attention(cfg, q, k, v, n_ctx, sel, n_sel, out, lse, ws, int(most * share))
        except B.CacheTuneError:                 # less than the call needs at least
            assert share < 1.0 and n_ctx > 2048
            continue
        ran += 1
        # probabilities are rounded to bf16 (8 significant bits: by up to 2^-8 of each; their sum is not) and so is the
        # result; fp32 sums and exponents take the rest
        err = (out.double() - want).abs()
        assert (err <= 2.0 ** -8 * (size + want.abs()) + 1e-4 * size).all(), (share, float(err.max()))
        assert ((lse.double() - want_lse).abs() <= 1e-4).all()
    assert ran >= 1


@pytest.mark.parametrize("hq,hkv,d,n_ctx,n_sel", SHAPES)
def test_any_workspace_of_the_layer_gives_the_same_rows(hq, hkv, d, n_ctx, n_sel):
    say(f"layer splits heads={hq}/{hkv} d={d} n_ctx={n_ctx} n_sel={n_sel}")
    g = torch.Generator(device="cuda").manual_seed(n_ctx + n_sel)
    hidden = 64
    cfg = B.make_cfg(hidden, hq, hkv, d, 1.0e4)
    sel = torch.randperm(n_ctx, generator=g, device="cuda")[:n_sel]
    sel[0] = 0                                   # one key
    sel = torch.unique(sel).to(torch.int32)      # ascending
    n_sel = sel.numel()
    x, w, k, v = (torch.randn(*s, generator=g, device="cuda").to(torch.bfloat16)
                  for s in ((n_sel, hidden), ((hq + 2 * hkv) * d, hidden), (n_ctx, hkv, d), (n_ctx, hkv, d)))
    w *= hidden ** -0.5
    q, ks, vs = (torch.empty(n_sel, h, d, device="cuda", dtype=torch.bfloat16) for h in (hq, hkv, hkv))
    B.ct_qkv_selected(cfg, x, None, sel, n_sel, w, None, q, ks, vs)
    chunks = B.make_chunks([dict(k=k, v=v, n_tokens=n_ctx, old_pos_start=0, new_pos_start=0, location=0)])
    keys, values = k.clone(), v.clone()          # (a chunk that does not move is rotated by nothing)
    keys[sel.long()], values[sel.long()] = ks, vs
    want, size = (torch.empty(n_sel, hq, d, device="cuda", dtype=torch.float64) for _ in range(2))
    later = torch.arange(n_ctx, device="cuda")[None, :] > sel[:, None]
    for h in range(hq):
        kv = h // (hq // hkv)
        s = (q[:, h].double() @ keys[:, kv].double().T.contiguous() * d ** -0.5).masked_fill(later, float("-inf"))
        want[:, h] = torch.softmax(s, 1) @ values[:, kv].double()
        size[:, h] = torch.softmax(s, 1) @ values[:, kv].double().abs()
    most = B.ct_workspace_bytes(cfg, n_ctx, n_sel)
    ws = torch.empty(most, dtype=torch.uint8, device="cuda")
    ran = 0
    for share in (0.1, 0.4, 0.7, 1.0):
        kb, vb = (torch.zeros(n_ctx, hkv, d, device="cuda", dtype=torch.bfloat16) for _ in range(2))
        out = torch.full((n_sel, hq, d), float("nan"), device="cuda", dtype=torch.bfloat16)
        try:
            B.ct_partial_prefill_layer(cfg, chunks, 1, x, None, sel, n_sel, -1.0, w, None, kb, vb, out, ws, int(most * share),
                                       None, torch.cuda.Stream())
        except B.CacheTuneError as e:            # less than the call needs at least
            assert share < 1.0 and e.status == B.CT_ERR_WORKSPACE
            continue
        ran += 1
        err = (out.double() - want).abs()        # as above
        assert (err <= 2.0 ** -8 * (size + want.abs()) + 1e-4 * size).all(), (share, float(err.max()))
    assert ran >= 1


@pytest.mark.parametrize("hq,hkv,d,n_ctx,n_sel", [(8, 2, 64, 1024, 153), (32, 8, 128, 2048, 307), (16, 16, 64, 2048, 3)])
def test_attention_that_needs_no_scratch_leaves_it_alone(hq, hkv, d, n_ctx, n_sel):
    """Calls on several streams may share a workspace (and do share the library's array) as long as none needs it."""
    say(f"attention without scratch heads={hq}/{hkv} d={d} n_ctx={n_ctx} n_sel={n_sel}")
    g = torch.Generator(device="cuda").manual_seed(n_sel)
    cfg = B.make_cfg(64, hq, hkv, d, 1.0e4)
    q, k, v = (torch.randn(n, h, d, generator=g, device="cuda").to(torch.bfloat16) for n, h in ((n_sel, hq), (n_ctx, hkv), (n_ctx, hkv)))
    sel = (torch.arange(n_sel, device="cuda") * (n_ctx // n_sel) + n_ctx // n_sel - 1).to(torch.int32)
    plain, given, static = (torch.full((n_sel, hq, d), float("nan"), device="cuda", dtype=torch.bfloat16) for _ in range(3))
    B.ct_selected_attention(cfg, q, k, v, n_ctx, sel, n_sel, plain, None, None, 0)
    ws = torch.full((B.ct_workspace_bytes(cfg, n_ctx, n_sel),), 0xa5, dtype=torch.uint8, device="cuda")
    B.ct_selected_attention(cfg, q, k, v, n_ctx, sel, n_sel, given, None, ws, ws.numel())
    B.ct_set_profiling(True)
    B.ct_profile_reset()
    B.ct_selected_attention_static(cfg, q, k, v, n_ctx, sel, n_sel, static, None)
    B.ct_set_profiling(False)
    assert B.ct_profile_read("merge")[0] == 0    # nothing was put into the array to be merged
    B.ct_profile_reset()
    assert bool((ws == 0xa5).all())
    assert torch.isfinite(plain).all() and torch.equal(plain, given) and torch.equal(plain, static)


def test_host_pool_takes_the_state_from_room_asked_for():
    """The room for splits in ct_workspace_bytes is none of the attention state's: with that amount a short context in
    pinned memory comes in one launch and is followed by one attention launch, with the state's bytes on top by several."""
    hq, hkv, d, n_chunks, length, n_sel, hidden = 32, 8, 128, 4, 512, 307, 128
    n_ctx = n_chunks * length
    g = torch.Generator(device="cuda").manual_seed(5)
    cfg = B.make_cfg(hidden, hq, hkv, d, 1.0e4)
    x, w, k, v = (torch.randn(*s, generator=g, device="cuda").to(torch.bfloat16)
                  for s in ((n_sel, hidden), ((hq + 2 * hkv) * d, hidden), (n_ctx, hkv, d), (n_ctx, hkv, d)))
    w *= hidden ** -0.5
    kp, vp = (torch.empty(n_ctx, hkv, d, dtype=torch.bfloat16, pin_memory=True) for _ in range(2))
    kp.copy_(k)
    vp.copy_(v)
    chunks = B.make_chunks([dict(k=kp[c * length:], v=vp[c * length:], n_tokens=length, old_pos_start=0, new_pos_start=c * length,
                                 location=1) for c in range(n_chunks)])
    sel = (torch.arange(n_sel, device="cuda") * n_ctx // n_sel).to(torch.int32)
    need, state = B.ct_workspace_bytes(cfg, n_ctx, n_sel), B.ct_attention_state_bytes(cfg, n_ctx, n_sel)
    ws = torch.empty(need + state, dtype=torch.uint8, device="cuda")
    copy, got = torch.cuda.Stream(), []
    for amount in (need, need + state):
        say(f"host pool, workspace of {amount} bytes")
        kb, vb = (torch.zeros(n_ctx, hkv, d, device="cuda", dtype=torch.bfloat16) for _ in range(2))
        out = torch.full((n_sel, hq, d), float("nan"), device="cuda", dtype=torch.bfloat16)
        B.ct_profile_reset()
        B.ct_set_profiling(True)
        B.ct_partial_prefill_layer(cfg, chunks, n_chunks, x, None, sel, n_sel, -1.0, w, None, kb, vb, out, ws, amount, None, copy)
        B.ct_set_profiling(False)
        torch.cuda.synchronize()
        got.append((B.ct_profile_read("attention")[0], kb, vb, out))
        B.ct_profile_reset()
    assert got[0][0] == 1 and got[1][0] == 2
    assert torch.equal(got[0][1], got[1][1]) and torch.equal(got[0][2], got[1][2])
    # the same sums in another order, probabilities and results rounded to bf16 (2^-8)
    size = float(got[0][2].float().abs().max())
    assert float((got[0][3].float() - got[1][3].float()).abs().max()) <= 2.0 ** -7 * size
