"""Host side of the dealt launch: where it is preferred, its workspace, and
the argument checks that run before any device access."""

import pytest

import paper_2604_00028_amd as da
from paper_2604_00028_amd import _binding as bnd

FAKE = 0x100000


def test_preferred_where_the_longest_chunk_exceeds_the_share():
    p = lambda *a: da.da_prefers_dealt(*a, num_cus=256)  # noqa: E731
    assert p(32, 64, 8, 16384, 32 * 8000) and p(64, 8, 1, 32768, 64 * 5000)
    # one long sequence among short ones
    assert p(32, 64, 8, 20000, 50000) and not p(4, 64, 8, 8000, 9000)
    assert not p(16, 32, 4, 512, 16 * 300) and not p(1, 64, 8, 8192, 8192)     # short shares
    assert not p(32, 64, 8, 0, 0)                                              # nothing to read
    assert not p(512, 64, 8, 8192, 512 * 1000)                                 # many workgroups balance themselves
    assert not p(8, 10, 5, 0, 0)
    # equal lengths, and batches of which only B * L_K_max is known: one split count is even already
    for B, H_Q, H_KV, L in ((58, 64, 4, 5180), (110, 16, 2, 6661), (34, 32, 2, 9741), (82, 64, 8, 1670), (16, 128, 2, 26847)):
        assert not p(B, H_Q, H_KV, L, B * L) and not p(B, H_Q, H_KV, L, 0), (B, H_Q, H_KV, L)
    # the lines: 80 tiles over a share of 6.25, and 1.7 shares of 200 tiles
    assert next(t for t in range(1, 4000) if p(100, 64, 8, 32 * t, 3200)) == 87
    assert next(t for t in range(1, 4000) if p(32, 64, 8, 32 * t, 32 * 6368)) == 340
    # wide head tiles need four times the difference and 3 shares
    assert next(t for t in range(1, 4000) if p(64, 128, 2, 32 * t, 32 * 6336)) == 420
    assert next(t for t in range(1, 4000) if p(64, 128, 2, 32 * t, 32 * 12736)) == 600
    # what the Python entry points assume without asking
    assert p(129, 8, 1, bnd.DEALT_MIN_KEYS, 1) and not p(129, 8, 1, bnd.DEALT_MIN_KEYS - 1, 1)
    # head tiles that leave more than a tenth of the CUs idle, or more than the arrival counters
    assert not p(32, 160, 160, 16384, 0) and da.da_dealt_workspace_bytes(32, 160, 160, 256) == 0
    assert da.da_dealt_workspace_bytes(1024, 64, 8, 256) == 0
    assert not p(-1, 64, 8, 512, 0) and not p(4, 64, 7, 512, 0)


def test_workspace_bytes():
    # two chunk states for each of 256 / 8 workgroups of every head tile: Otilde | m | l, then the counters
    assert da.da_dealt_workspace_bytes(32, 64, 8, 256) == 2 * 32 * 64 * (128 * 4 + 4 + 4) + (1 << 20)
    assert da.da_dealt_workspace_bytes(3, 8, 1, 256) == 2 * 256 * 8 * (128 * 4 + 4 + 4) + (1 << 20)
    # chunk states stay below 2 GiB (their offsets have 32 bits): no shape of more CUs than that
    most = (1 << 31) // (2 * 8 * 512)
    assert da.da_dealt_workspace_bytes(3, 8, 1, most - 1) > 0 and da.da_dealt_workspace_bytes(3, 8, 1, most) == 0
    for cus in (1 << 28, (1 << 30) + 1, (1 << 31) - 1):
        assert da.da_dealt_workspace_bytes(3, 8, 1, cus) == 0 and not da.da_prefers_dealt(32, 64, 8, 16384, 1000, cus)


def call(q=FAKE, k=FAKE, v=FAKE, cu=FAKE, bt=None, sl=None, page=64, mp=8, npg=8, out=FAKE, lse=None, B=2, H_Q=8,
         H_KV=1, L=512, d=128, ws=FAKE, ws_bytes=1 << 30):
    return da.load().da_decode_attn_dealt(q, k, v, cu, bt, sl, page, mp, npg, out, lse, B, H_Q, H_KV, L, d, 0.0, 0,
                                          ws, ws_bytes, None)


@pytest.mark.parametrize("kw,code", [
    (dict(q=None), bnd.DA_ERR_NULL), (dict(k=None), bnd.DA_ERR_NULL), (dict(out=None), bnd.DA_ERR_NULL),
    (dict(cu=None), bnd.DA_ERR_NULL), (dict(bt=FAKE), bnd.DA_ERR_NULL),
    (dict(q=FAKE + 8), bnd.DA_ERR_ALIGN), (dict(out=FAKE + 8), bnd.DA_ERR_ALIGN), (dict(cu=FAKE + 2), bnd.DA_ERR_ALIGN),
    (dict(lse=FAKE + 2), bnd.DA_ERR_ALIGN), (dict(ws=FAKE + 8), bnd.DA_ERR_ALIGN),
    (dict(d=64), bnd.DA_ERR_UNSUPPORTED), (dict(H_Q=9, H_KV=2), bnd.DA_ERR_SHAPE), (dict(L=-1), bnd.DA_ERR_SHAPE),
    (dict(bt=FAKE, sl=FAKE, page=48), bnd.DA_ERR_UNSUPPORTED), (dict(bt=FAKE, sl=FAKE, mp=7), bnd.DA_ERR_SHAPE),
    (dict(ws=None), bnd.DA_ERR_WORKSPACE),
])
def test_argument_errors(kw, code):
    assert call(**kw) == code


def test_mixed_schedules_stream_beyond_the_mall():
    """A schedule marks its K/V loads nontemporal above 288 MiB where one
    workgroup reads each key, of mixed lengths as of equal ones: below, the
    hint slows a call that finds its K/V in the MALL."""
    at = (288 << 20) // (512 * 8)               # keys of 8 KV heads in 288 MiB
    for keys, want in ((at - 4096, 0), (at + 4096, 1)):
        lens = [keys - 10 * 2000 - 7] + [2000] * 10
        sched, _ = da.da_make_schedule(lens, 64, 8, num_cus=256)
        assert sched.kv_nontemporal == want
    equal, _ = da.da_make_schedule([at // 8 - 32] * 8, 64, 8, num_cus=256)
    shared, _ = da.da_make_schedule([at * 5, 3000], 128, 2, num_cus=256)      # two head tiles read each key
    assert equal.kv_nontemporal == 0 and shared.kv_nontemporal == 0


def test_schedules_keep_their_chunks():
    """A long schedule of mixed lengths launches the chunks it lists: its
    kv_fetch is a plan's, and its workspace holds its chunk states and the
    arrival counters, no more."""
    for lens, H_Q, H_KV in (([1024 + 480 * i for i in range(32)], 64, 8), ([9117] * 11 + [800] * 79, 16, 16)):
        sched, _ = da.da_make_schedule(lens, H_Q, H_KV, num_cus=256)
        assert sched.kv_fetch in (0, 1, 2) and sched.state_rows > 0
        states = -(-sched.state_rows * H_Q * 128 * 4 // 256) * 256 + 2 * (-(-sched.state_rows * H_Q * 4 // 256) * 256)
        assert da.da_schedule_workspace_bytes(sched) == states + (1 << 20)


def test_the_gpu_cases_reach_what_they_name():
    from tests.dealt_cases import CASES, MOST_PIECES, PAGE_WINDOWS, PAGE_WINDOWS_CUS, deal
    got = [deal(lens, H_Q, H_KV) for H_Q, H_KV, lens in CASES]
    assert got[4]["per"] == 11 and got[4]["pieces"] == [26]
    assert got[6]["passed"] >= 3 and got[7]["passed"] >= 3
    assert {d["hpt"] for d in got} >= {1, 3, 8, 32}
    H_Q, H_KV, lens = MOST_PIECES
    assert deal(lens, H_Q, H_KV)["pieces"][1] == 64
    for H_Q, H_KV, lens in PAGE_WINDOWS:
        d = deal(lens, H_Q, H_KV, PAGE_WINDOWS_CUS)
        assert d["pages"] > 64 and d["passed"] >= 2
