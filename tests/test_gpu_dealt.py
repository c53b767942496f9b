"""GPU parity of the dealt launch (da_decode_attn_dealt) against the fp64
oracle: a batch's 32-key tiles shared evenly among the workgroups, sequences
cut wherever a share ends and merged inside the launch.  Same bar as the other
paths: max-abs <= 2e-2 and mean-abs <= 2e-3 on O, lse within 1e-3, bit-identical
repeats."""

import numpy as np
import pytest
import torch

import paper_2604_00028_amd as da
from oracle import decode_attention
from workloads import custom_shape, make_inputs, paged_layout
from tests.dealt_cases import CASES, MOST_PIECES, PAGE_WINDOWS, PAGE_WINDOWS_CUS, deal
from tests.gpu_helpers import assert_parity, dev_inputs, say, to_dev, to_f64

pytestmark = pytest.mark.gpu

LSE_TOL = 1e-3

def check(out, lse_t, O, lse, what):
    assert_parity(out, O, what)
    lg = lse_t.cpu().numpy().astype(np.float64)
    fin = np.isfinite(lse)
    assert np.array_equal(np.isfinite(lg), fin), what
    assert np.max(np.abs(lg[fin] - lse[fin]), initial=0.0) <= LSE_TOL, what


@pytest.mark.parametrize("page", [None, 32, 96])
@pytest.mark.parametrize("H_Q,H_KV,lengths", CASES, ids=lambda x: str(x)[:24])
def test_dealt_parity(H_Q, H_KV, lengths, page):
    B = len(lengths)
    inp = make_inputs(custom_shape(B, H_Q, H_KV, max(lengths), varlen=True), seed=B + H_Q, lengths=lengths)
    O, lse = decode_attention(inp.q, inp.k, inp.v, inp.lengths, inp.cu_seqlens_k)
    q, k, v, cu = dev_inputs(inp)
    kw = dict(cu_seqlens_k=cu)
    if page is not None:
        pg = paged_layout(inp, page, seed=page + 3)
        k, v = to_dev(pg.k_cache), to_dev(pg.v_cache)
        kw = dict(block_table=torch.from_numpy(pg.block_table).cuda(), seq_lens=torch.from_numpy(pg.seq_lens).cuda())
    ws = torch.zeros(da.da_dealt_workspace_bytes(B, H_Q, H_KV), dtype=torch.uint8, device="cuda")
    first = None
    for r in range(3):
        say(f"dealt B{B} {H_Q}/{H_KV} {str(lengths)[:40]} page={page} run {r}")
        ws[:-(1 << 20)].fill_(255)      # chunk states need no initialisation (NaN bits here)
        lse_t = torch.empty(B, H_Q, dtype=torch.float32, device="cuda")
        out = da.da_decode_attn_dealt(q, k, v, max(lengths), lse_out=lse_t, workspace=ws, **kw)
        torch.cuda.synchronize()
        check(out, lse_t, O, lse, f"dealt {H_Q}/{H_KV} page={page}")
        assert int(ws[-(1 << 20):].max()) == 0      # the arrival counters are back at zero
        first = first or (out, lse_t)
        assert torch.equal(out.view(torch.int16), first[0].view(torch.int16)) and torch.equal(lse_t, first[1])


@pytest.mark.parametrize("page", [None, 64])
def test_planning_entries_deal_a_mixed_batch(page):
    """da_decode_attn and da_decode_attn_paged give the dealt launch's bits
    where it is preferred, and their own plan's with a forced split count or
    while a graph is captured; a captured da_decode_attn_dealt follows the
    lengths from replay to replay."""
    H_Q, H_KV = 64, 8
    lengths = [int(x) for x in np.random.default_rng(3).integers(500, 5000, 31)] + [8000]
    B, top = len(lengths), 8000
    assert da.da_prefers_dealt(B, H_Q, H_KV, top, sum(lengths))
    inp = make_inputs(custom_shape(B, H_Q, H_KV, max(lengths), varlen=True), seed=11, lengths=lengths)
    q, k, v, cu = dev_inputs(inp)
    if page is None:
        call = lambda s, ws=None: da.da_decode_attn(q, k, v, cu, L_K_max=top, num_splits=s, workspace=ws)  # noqa: E731
        dealt = lambda: da.da_decode_attn_dealt(q, k, v, top, cu)  # noqa: E731
    else:
        pg = paged_layout(inp, page, seed=5, max_pages=-(-top // page))
        k, v = to_dev(pg.k_cache), to_dev(pg.v_cache)
        bt, sl = torch.from_numpy(pg.block_table).cuda(), torch.from_numpy(pg.seq_lens).cuda()
        call = lambda s, ws=None: da.da_decode_attn_paged(q, k, v, bt, sl, top, num_splits=s, workspace=ws)  # noqa: E731
        dealt = lambda: da.da_decode_attn_dealt(q, k, v, top, block_table=bt, seq_lens=sl)  # noqa: E731
    say(f"dealt route page={page}")
    a, b, forced = call(0), dealt(), call(2)
    torch.cuda.synchronize()
    assert torch.equal(a.view(torch.int16), b.view(torch.int16))
    picks = [0, int(np.argmax(lengths)), 9]
    cuh = inp.cu_seqlens_k
    for s in picks:
        O, _ = decode_attention(inp.q[s:s + 1], inp.k[cuh[s]:cuh[s + 1]][None], inp.v[cuh[s]:cuh[s + 1]][None])
        assert_parity(a[s:s + 1], O, f"dealt route sequence {s}")
        assert_parity(forced[s:s + 1], O, f"forced splits sequence {s}")
    # the plan the entry point makes for itself, which a workspace of the caller's keeps
    plan_ws = torch.zeros(da.da_workspace_bytes(B, H_Q, 128, 64), dtype=torch.uint8, device="cuda")
    own = lambda: call(0, plan_ws)  # noqa: E731
    assert not torch.equal(a.view(torch.int16), own().view(torch.int16))
    torch.cuda.synchronize()
    stream = torch.cuda.Stream()
    with torch.cuda.stream(stream):
        call(0), call(2), dealt()       # workspace of this stream
    stream.synchronize()
    g = torch.cuda.CUDAGraph()
    with torch.cuda.graph(g, stream=stream):
        got, got_dealt = call(0), dealt()
    for r in range(4):
        if page is not None:
            sl.copy_(torch.from_numpy(pg.seq_lens) - 37 * r)
        g.replay()
        torch.cuda.synchronize()
        assert torch.equal(got.view(torch.int16), own().view(torch.int16)), f"replay {r}"
        assert torch.equal(got_dealt.view(torch.int16), dealt().view(torch.int16)), f"dealt replay {r}"


@pytest.mark.parametrize("page", [None, 64])
@pytest.mark.parametrize("H_Q,H_KV,lengths,scale", [
    (64, 8, [8192, 3000, 6001], 2.0), (8, 1, [20000, 700], 2.0), (16, 2, [5000] * 6, 1.0), (32, 1, [4100, 9000], 1.0)])
def test_dealt_is_no_further_from_64_bits(H_Q, H_KV, lengths, scale, page):
    """The deal cuts a batch into fewer and longer pieces than a launch with
    many splits.  A piece's largest probability is exactly 1, so fewer pieces
    leave more probabilities to rounding; the dealt launch carries their
    remainders, and its error is no larger than that of 16 splits (whose own
    probabilities are rounded to bf16 once)."""
    B, L = len(lengths), max(lengths)
    inp = make_inputs(custom_shape(B, H_Q, H_KV, L, varlen=True), seed=23, lengths=lengths)
    q, k, v, cu = dev_inputs(inp)
    q = q * scale                        # exact: a power of two
    qh = (inp.q if scale == 1.0 else q.cpu().view(torch.int16).numpy().view(np.uint16))
    O, _ = decode_attention(qh, inp.k, inp.v, inp.lengths, inp.cu_seqlens_k)
    kw, ukw = dict(cu_seqlens_k=cu), dict(cu_seqlens_k=cu, L_K_max=L)
    if page is not None:
        pg = paged_layout(inp, page, seed=2)
        k, v = to_dev(pg.k_cache), to_dev(pg.v_cache)
        kw = dict(block_table=torch.from_numpy(pg.block_table).cuda(), seq_lens=torch.from_numpy(pg.seq_lens).cuda())
    say(f"dealt error {H_Q}/{H_KV} {lengths} page={page}")
    dealt = da.da_decode_attn_dealt(q, k, v, L, **kw)
    if page is None:
        split = da.da_decode_attn(q, k, v, num_splits=16, **ukw)
    else:
        split = da.da_decode_attn_paged(q, k, v, kw["block_table"], kw["seq_lens"], L, num_splits=16)
    torch.cuda.synchronize()
    rel = [float(np.linalg.norm(to_f64(x) - O) / np.linalg.norm(O)) for x in (dealt, split)]
    say(f"  dealt {rel[0]:.3e} 16 splits {rel[1]:.3e}")
    assert rel[0] <= rel[1]


def test_dealt_on_a_masked_stream():
    """On a CU-masked stream the batch is dealt over the CUs the stream has:
    a workspace for that many suffices there and not on a stream with all."""
    from paper_2604_00028_amd.streams import cu_mask_stream, destroy_stream, split_masks
    H_Q, H_KV, lengths = 64, 8, [3000, 17, 0, 900, 2100]
    B, L = len(lengths), max(lengths)
    inp = make_inputs(custom_shape(B, H_Q, H_KV, L, varlen=True), seed=29, lengths=lengths)
    O, lse = decode_attention(inp.q, inp.k, inp.v, inp.lengths, inp.cu_seqlens_k)
    q, k, v, cu = dev_inputs(inp)
    cus = da.da_device_info()[0]
    stream, enabled = cu_mask_stream(split_masks(cus, 8)[1])
    try:
        assert enabled < cus
        ws = torch.zeros(da.da_dealt_workspace_bytes(B, H_Q, H_KV, enabled), dtype=torch.uint8, device="cuda")
        lse_t = torch.empty(B, H_Q, dtype=torch.float32, device="cuda")
        out = torch.empty(B, H_Q, 128, dtype=torch.bfloat16, device="cuda")
        torch.cuda.synchronize()
        say(f"dealt on {enabled} of {cus} CUs")
        da.da_decode_attn_dealt(q, k, v, L, cu, out=out, lse_out=lse_t, workspace=ws, stream=stream)
        torch.cuda.synchronize()
        check(out, lse_t, O, lse, "dealt on a masked stream")
        with pytest.raises(da.DecodeAttnError):
            da.da_decode_attn_dealt(q, k, v, L, cu, out=out, workspace=ws)
    finally:
        destroy_stream(stream)


def close(out, lse_t, O, lse, what):
    """check(), and a relative error that a missed or doubled page would exceed (bf16 output: 1.7e-3)."""
    check(out, lse_t, O, lse, what)
    rel = float(np.linalg.norm(to_f64(out) - O) / np.linalg.norm(O))
    assert rel <= 4e-3, f"{what}: {rel:.2e}"


def test_dealt_most_pieces():
    """A sequence in 64 pieces, the most the merge holds."""
    H_Q, H_KV, lengths = MOST_PIECES
    assert da.da_device_info()[0] != 256 or max(deal(lengths, H_Q, H_KV)["pieces"]) == 64
    inp = make_inputs(custom_shape(2, H_Q, H_KV, max(lengths), varlen=True), seed=31, lengths=lengths)
    O, lse = decode_attention(inp.q, inp.k, inp.v, inp.lengths, inp.cu_seqlens_k)
    q, k, v, cu = dev_inputs(inp)
    say("dealt 64 pieces")
    lse_t = torch.empty(2, H_Q, dtype=torch.float32, device="cuda")
    out = da.da_decode_attn_dealt(q, k, v, max(lengths), cu, lse_out=lse_t)
    torch.cuda.synchronize()
    close(out, lse_t, O, lse, "64 pieces")


@pytest.mark.parametrize("H_Q,H_KV,lengths", PAGE_WINDOWS, ids=lambda x: str(x)[:24])
def test_dealt_page_windows(H_Q, H_KV, lengths):
    """Waves that pass more than the 64 page ids they hold at a time."""
    from paper_2604_00028_amd.streams import cu_mask_stream, destroy_stream, split_masks
    B, L = len(lengths), max(lengths)
    inp = make_inputs(custom_shape(B, H_Q, H_KV, L, varlen=True), seed=37, lengths=lengths)
    O, lse = decode_attention(inp.q, inp.k, inp.v, inp.lengths, inp.cu_seqlens_k)
    pg = paged_layout(inp, 32, seed=6)
    q, k, v = to_dev(inp.q), to_dev(pg.k_cache), to_dev(pg.v_cache)
    bt, sl = torch.from_numpy(pg.block_table).cuda(), torch.from_numpy(pg.seq_lens).cuda()
    stream, enabled = cu_mask_stream(split_masks(da.da_device_info()[0], 24)[1])
    try:
        assert enabled != PAGE_WINDOWS_CUS or deal(lengths, H_Q, H_KV, enabled)["pages"] > 64
        lse_t = torch.empty(B, H_Q, dtype=torch.float32, device="cuda")
        torch.cuda.synchronize()
        say(f"dealt page windows {H_Q}/{H_KV} on {enabled} CUs")
        out = da.da_decode_attn_dealt(q, k, v, L, block_table=bt, seq_lens=sl, lse_out=lse_t, stream=stream)
        torch.cuda.synchronize()
        close(out, lse_t, O, lse, f"page windows {H_Q}/{H_KV}")
    finally:
        destroy_stream(stream)


@pytest.mark.parametrize("page", [None, 32])
def test_dealt_lengths_and_pages_out_of_range(page):
    """Lengths above L_K_max count as L_K_max and, paged, below 0 as 0; a
    page id outside the cache reads as zero keys and values."""
    H_Q, H_KV, lengths, L = 16, 2, [1000, 700, 350, 600], 640
    inp = make_inputs(custom_shape(4, H_Q, H_KV, 1000, varlen=True), seed=41, lengths=lengths)
    cuh = inp.cu_seqlens_k
    q, k, v, cu = dev_inputs(inp)
    kw = dict(cu_seqlens_k=cu)
    keep = [L, L, 350, 600]
    kn, vn = inp.k.copy(), inp.v.copy()
    if page is not None:
        pg = paged_layout(inp, page, seed=9)
        for b, j, bad in ((0, 3, -1), (2, 0, pg.k_cache.shape[0]), (3, 18, 2**31 - 1)):
            pg.block_table[b, j] = bad
            rows = slice(cuh[b] + page * j, min(cuh[b] + page * (j + 1), cuh[b + 1]))
            kn[rows], vn[rows] = 0, 0
        pg.seq_lens[1] = -5
        keep[1] = 0
        k, v = to_dev(pg.k_cache), to_dev(pg.v_cache)
        kw = dict(block_table=torch.from_numpy(pg.block_table).cuda(), seq_lens=torch.from_numpy(pg.seq_lens).cuda())
    cut = np.concatenate([np.arange(cuh[b], cuh[b] + n) for b, n in enumerate(keep)])
    O, lse = decode_attention(inp.q, kn[cut], vn[cut], np.array(keep, dtype=np.int64),
                              np.concatenate([[0], np.cumsum(keep)]).astype(np.int32))
    say(f"dealt out of range page={page}")
    lse_t = torch.empty(4, H_Q, dtype=torch.float32, device="cuda")
    out = da.da_decode_attn_dealt(q, k, v, L, lse_out=lse_t, **kw)
    torch.cuda.synchronize()
    close(out, lse_t, O, lse, f"out of range page={page}")
