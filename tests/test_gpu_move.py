"""Reused chunks brought in beside the projection: what the layer call leaves in its buffers is, bit for bit, what the
single steps give (rotation of the chunks, projection, scatter), and what it returns is, bit for bit, what a layer call on
those buffers returns and, up to the order of the sums, what the attention of the steps gives; for
projections that leave compute units free and for one that does not, chunks in place and elsewhere, more of
them than one table holds, and a chunk whose source lies in the buffer it is moved into."""
import numpy as np
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


@pytest.mark.parametrize("hq,hkv,d,style,lengths,n_sel,where", [
    (8, 2, 64, 0, [130, 1, 67], 20, "pool"), (16, 8, 128, 0, [200, 56, 300], 129, "pool"),
    (4, 4, 128, 1, [64] * 40, 100, "pool"),           # more chunks than one table holds; runtime head count
    (8, 8, 64, 1, [333], 300, "own"),                 # chunks stand in their own place
    (16, 8, 128, 0, [256, 256], 64, "shifted"),       # a source in the layer buffer
    (32, 8, 128, 0, [1300], 1228, "pool"),            # 240 tiles: a launch of its own
    (16, 8, 128, 0, [1300, 1, 1299], 2100, "pool"), (16, 8, 128, 1, [1300, 1, 1299], 2100, "pool"),    # 256-token tiles,
    (32, 16, 64, 0, [1300, 1, 1299], 2100, "pool"), (32, 16, 64, 1, [1300, 1, 1299], 2100, "own"),     # any head count
    (8, 2, 64, 0, [100, 28], 128, "pool")])           # nothing reused
def test_layer_equals_its_steps(hq, hkv, d, style, lengths, n_sel, where):
    say(f"move heads={hq}/{hkv} d={d} chunks={len(lengths)} n_sel={n_sel} {where}")
    g = torch.Generator(device="cuda").manual_seed(n_sel)
    n_ctx, hidden = sum(lengths), 128
    starts = np.concatenate([[0], np.cumsum(lengths)])
    cfg = B.make_cfg(hidden, hq, hkv, d, 1.0e4, style)
    sel = torch.from_numpy(np.sort(np.random.default_rng(n_sel).permutation(n_ctx)[:n_sel]).astype(np.int32)).cuda()
    x, w = _rand(g, n_sel, hidden), _rand(g, (hq + 2 * hkv) * d, hidden)
    kp, vp = _rand(g, n_ctx, hkv, d), _rand(g, n_ctx, hkv, d)
    kb, vb = (torch.zeros(n_ctx, hkv, d, device="cuda", dtype=torch.bfloat16) for _ in range(2))
    src_k, src_v = kp, vp
    if where != "pool":
        kb.copy_(kp)
        vb.copy_(vp)
        src_k, src_v = kb, vb
    rows = [(int(starts[c]), int(starts[c + 1])) for c in range(len(lengths))]
    # shifted: the first chunk comes from the place of the second, which stays as it is but for the selected rows
    taken = rows[1:] + rows[1:] if where == "shifted" else rows
    old = [rows[1][0] if where == "shifted" and c == 1 else 3 * c for c in range(len(rows))]
    chunks = [dict(k=src_k[lo:hi], v=src_v[lo:hi], n_tokens=hi - lo, old_pos_start=old[c], new_pos_start=rows[c][0], location=0)
              for c, (lo, hi) in enumerate(taken)]
    # the steps, on copies
    want_k, want_v = kb.clone(), vb.clone()
    for c, (lo, hi) in enumerate(taken):
        to = slice(*rows[c])
        B.ct_rerope_chunk(cfg, kp[lo:hi], want_k[to], vp[lo:hi], want_v[to], hi - lo, old[c], rows[c][0], 0)
    q, ks, vs = (torch.empty(n_sel, h, d, device="cuda", dtype=torch.bfloat16) for h in (hq, hkv, hkv))
    B.ct_qkv_selected(cfg, x, None, sel, n_sel, w, None, q, ks, vs)
    want_k[sel.long()], want_v[sel.long()] = ks, vs
    ws_bytes = max(B.ct_workspace_bytes(cfg, n_ctx, n_sel), 256)
    ws = torch.empty(ws_bytes, dtype=torch.uint8, device="cuda")
    want, out = (torch.empty(n_sel, hq, d, device="cuda", dtype=torch.bfloat16) for _ in range(2))
    B.ct_selected_attention(cfg, q, want_k, want_v, n_ctx, sel, n_sel, want, None, ws, ws_bytes)
    B.ct_partial_prefill_layer(cfg, B.make_chunks(chunks), len(chunks), x, None, sel, n_sel, -1.0, w, None, kb, vb, out, ws,
                               ws_bytes, None, torch.cuda.Stream())
    torch.cuda.synchronize()
    assert torch.equal(kb, want_k) and torch.equal(vb, want_v)
    # every chunk in its own place and at its own position: nothing is moved or turned, the attention is the layer's
    place = [dict(k=want_k[lo:hi], v=want_v[lo:hi], n_tokens=hi - lo, old_pos_start=lo, new_pos_start=lo, location=0) for lo, hi in rows]
    again = torch.empty_like(out)
    B.ct_partial_prefill_layer(cfg, B.make_chunks(place), len(place), x, None, sel, n_sel, -1.0, w, None, want_k, want_v, again, ws,
                               ws_bytes, None, torch.cuda.Stream())
    torch.cuda.synchronize()
    assert torch.equal(kb, want_k) and torch.equal(vb, want_v) and torch.equal(out, again)
    # the key range may be split in another way: probabilities and results are rounded to bf16 (2^-8) from other sums
    size = float(vb.float().abs().max())
    assert float((out.float() - want.float()).abs().max()) <= 2.0 ** -7 * size


@pytest.mark.parametrize("hq,hkv,d,n_ctx,n_sel,apart", [
    (16, 16, 64, 32768, 9830, 1),      # 44 units left, 6.1 MB to move for each, any number of heads
    (32, 2, 128, 131072, 1310, 1),     # 58 units, 4.6 MB
    (16, 16, 64, 32768, 1638, 0),      # 100 units, 2.7 MB
    (32, 8, 128, 32768, 4915, 0)])     # 32 units, 8.4 MB, but eight heads
def test_much_to_move_has_a_launch_of_its_own(hq, hkv, d, n_ctx, n_sel, apart):
    say(f"move rule heads={hq}/{hkv} d={d} n_ctx={n_ctx} n_sel={n_sel}")
    g = torch.Generator(device="cuda").manual_seed(n_sel)
    hidden = 64
    cfg = B.make_cfg(hidden, hq, hkv, d, 1.0e4)
    sel = (torch.arange(n_sel, device="cuda") * n_ctx // n_sel).to(torch.int32)
    x, w, k, v = _rand(g, n_sel, hidden), _rand(g, (hq + 2 * hkv) * d, hidden), _rand(g, n_ctx, hkv, d), _rand(g, n_ctx, hkv, d)
    kb, vb = (torch.zeros_like(k) for _ in range(2))
    want_k, want_v = (torch.zeros_like(k) for _ in range(2))
    B.ct_rerope_chunk(cfg, k, want_k, v, want_v, n_ctx, 7, 0, 0)
    q, ks, vs = (torch.empty(n_sel, h, d, device="cuda", dtype=torch.bfloat16) for h in (hq, hkv, hkv))
    B.ct_qkv_selected(cfg, x, None, sel, n_sel, w, None, q, ks, vs)
    want_k[sel.long()], want_v[sel.long()] = ks, vs
    chunks = B.make_chunks([dict(k=k, v=v, n_tokens=n_ctx, old_pos_start=7, new_pos_start=0, location=0)])
    ws_bytes = B.ct_workspace_bytes(cfg, n_ctx, n_sel)
    ws = torch.empty(ws_bytes, dtype=torch.uint8, device="cuda")
    B.ct_profile_reset()
    B.ct_set_profiling(True)
    B.ct_partial_prefill_layer(cfg, chunks, 1, x, None, sel, n_sel, -1.0, w, None, kb, vb, q, ws, ws_bytes, None, torch.cuda.Stream())
    B.ct_set_profiling(False)
    torch.cuda.synchronize()
    launches = B.ct_profile_read("rerope")[0]
    B.ct_profile_reset()
    assert launches == apart
    assert torch.equal(kb, want_k) and torch.equal(vb, want_v)
