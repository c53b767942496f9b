"""The zero fill of a workspace the binding allocates comes before the call
that needs it, whichever of the call's stream and torch's current one is busy
or captured.  The allocator's block holds 0xff bytes beforehand, so that a
call whose arrival counters are not cleared leaves its output unwritten."""

import pytest
import torch

import paper_2604_00028_amd as da
from paper_2604_00028_amd import _binding as bnd
from tests.gpu_helpers import say

pytestmark = pytest.mark.gpu

B, H_Q, H_KV, L, S = 1, 64, 8, 2048, 4


@pytest.fixture
def call():
    """call(stream, out): a split call merged in the launch, into NaNs; and its expected output."""
    g = torch.Generator(device="cuda").manual_seed(3)
    q, k, v = (torch.randn(s, device="cuda", generator=g).to(torch.bfloat16)
               for s in ((B, H_Q, 128), (B, L, H_KV, 128), (B, L, H_KV, 128)))
    plan = da.da_make_plan(B, H_Q, H_KV, L, 128, S, 1)
    plan.group_waves, plan.wg_per_cu, plan.combine = 4, 0, 1
    run = lambda stream, out, ws=None: da.da_decode_attn_planned(q, k, v, plan, out=out, stream=stream,  # noqa: E731
                                                                 workspace=ws)
    nbytes = da.da_workspace_bytes(B, H_Q, 128, S)
    ref = run(None, torch.empty_like(q), torch.zeros(nbytes, dtype=torch.uint8, device="cuda"))
    # Load what the tests launch (a first launch may load code, which a capture forbids)
    nan = torch.full_like(q, float("nan"))
    torch.cuda.synchronize()
    return run, nan, ref, nbytes


def dirty_block(nbytes):
    """Leave a freed block of 0xff bytes for the current stream's next allocation of that size."""
    t = torch.full((nbytes,), 255, dtype=torch.uint8, device="cuda")
    torch.cuda.synchronize()
    del t


def same(a, b):
    return torch.equal(a.view(torch.int16), b.view(torch.int16))


def test_the_call_waits_for_a_fill_on_a_busy_stream(call):
    run, nan, ref, nbytes = call
    busy, own = torch.cuda.Stream(), torch.cuda.Stream()
    m = torch.randn(4096, 4096, device="cuda")
    out = nan.clone()
    with torch.cuda.stream(busy):
        dirty_block(nbytes)
    torch.cuda.synchronize()
    say("call on its own stream, current stream busy")
    with torch.cuda.stream(busy):
        for _ in range(20):
            m = torch.mm(m, m).mul_(1e-4)
        run(own, out)
    torch.cuda.synchronize()
    assert same(out, ref)
    bnd._workspaces.pop((torch.cuda.current_device(), own.cuda_stream))


def test_eager_call_beside_a_capture(call):
    """The current stream is captured, the call's is not: the fill runs now."""
    run, nan, ref, nbytes = call
    cap, own = torch.cuda.Stream(), torch.cuda.Stream()
    out, x = nan.clone(), torch.zeros(8, device="cuda")
    with torch.cuda.stream(own):
        dirty_block(nbytes)
        x.add_(0)
    torch.cuda.synchronize()
    say("eager call beside a capture")
    g = torch.cuda.CUDAGraph()
    with torch.cuda.graph(g, stream=cap, capture_error_mode="relaxed"):
        x.add_(1)
        run(own, out)
    torch.cuda.synchronize()
    assert same(out, ref)
    g.replay()
    torch.cuda.synchronize()
    assert float(x[0]) == 1.0
    ws = bnd._workspaces.pop((torch.cuda.current_device(), own.cuda_stream))
    assert int(ws[-(1 << 20):].max()) == 0


def test_captured_call_from_an_eager_stream(call):
    """The call's stream is captured, the current one is not: the capture goes
    on, and every replay is right."""
    run, nan, ref, nbytes = call
    cur, own = torch.cuda.Stream(), torch.cuda.Stream()
    out = nan.clone()
    with torch.cuda.stream(cur):
        dirty_block(nbytes)
    torch.cuda.synchronize()
    say("captured call from an eager stream")
    g = torch.cuda.CUDAGraph()
    with torch.cuda.stream(own):
        g.capture_begin(capture_error_mode="relaxed")
        with torch.cuda.stream(cur):
            run(own, out)
        g.capture_end()
    torch.cuda.synchronize()
    for r in range(3):
        out.copy_(nan)
        g.replay()
        torch.cuda.synchronize()
        assert same(out, ref), f"replay {r}"
    del g
    bnd._workspaces.pop((torch.cuda.current_device(), own.cuda_stream))
