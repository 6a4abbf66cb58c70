"""Workspaces kept between calls on the null stream: results do not depend on which block a
call gets -- a fresh one, one left by a call of another size or kind, one allocated after
ring_attn_release_workspace() -- nor does a call on another stream between them matter."""
import threading

import pytest
import torch

import paper_2310_01889_amd as ra
from paper_2310_01889_amd import synth
from tests.gpu_util import dev, log

pytestmark = pytest.mark.gpu


def _calls(ins):
    out = []
    for q, k, v, do, kc, vc in ins:
        o, lse = ra.attention_fwd(q, k, v, 2, True)
        out += [o, lse, *ra.attention_bwd(q, k, v, o, lse, do, 2, True)]
        out += list(ra.attention_decode(q[:, :3].contiguous(), kc, vc, 2, True))
    torch.cuda.synchronize()
    return out


def test_kept_workspaces():
    ins = []
    for S in (256, 2048, 512, 1024):
        q, k, v, do = dev(*synth.attention_inputs(S, 1, S, 3, 64, with_grad=True))
        ins.append((q, k, v, do, k, v))
    ra.release_workspace()
    ref = _calls(ins)
    for turn in ("again", "reversed", "released"):
        log("workspace %s" % turn)
        if turn == "released":
            ra.release_workspace()
        got = _calls(ins[::-1] if turn == "reversed" else ins)
        if turn == "reversed":
            n = len(got) // len(ins)
            got = [t for i in range(len(ins)) for t in got[(len(ins) - 1 - i) * n:(len(ins) - i) * n]]
        assert all(torch.equal(a, b) for a, b in zip(ref, got))


def test_other_stream_between():
    """A stream of its own takes nothing of the null stream's kept blocks."""
    q, k, v, do = dev(*synth.attention_inputs(3, 1, 256, 2, 128, with_grad=True))
    ref = _calls([(q, k, v, do, k, v)])
    s = torch.cuda.Stream()
    with torch.cuda.stream(s):
        got = _calls([(q, k, v, do, k, v)])
    again = _calls([(q, k, v, do, k, v)])
    assert all(torch.equal(a, b) and torch.equal(a, c) for a, b, c in zip(ref, got, again))


def test_release_returns_kept_blocks():
    """Blocks kept for the null stream go back to the driver with the rest of the pool."""
    bf = torch.bfloat16
    T, dm, dff = 512, 256, 8192
    x, dy = torch.randn(T, dm, device="cuda").to(bf), torch.randn(T, dm, device="cuda").to(bf)
    w1, w2 = torch.randn(dm, dff, device="cuda").to(bf), torch.randn(dff, dm, device="cuda").to(bf)
    dx, dw1, dw2 = torch.empty_like(x), torch.empty(dm, dff, device="cuda"), torch.empty(dff, dm, device="cuda")
    call = lambda: ra.blockwise_ffn_bwd(x, w1, None, w2, dy, dx, dw1, None, dw2, None, T)
    call()  # what the runtime allocates for the kernels' first launches
    torch.cuda.synchronize()
    ra.release_workspace()
    free0 = torch.cuda.mem_get_info()[0]
    call()
    torch.cuda.synchronize()
    free1 = torch.cuda.mem_get_info()[0]
    ra.release_workspace()
    free2 = torch.cuda.mem_get_info()[0]
    log("  MiB free: %.1f, after a call %.1f, after the release %.1f" % tuple(f / 2 ** 20 for f in (free0, free1, free2)))
    assert free1 <= free0 - T * dff * 8  # the call's intermediates are kept
    assert abs(free2 - free0) <= 4 << 20  # the driver's own


def test_two_host_threads_on_the_null_stream():
    """Calls of two host threads, all on the null stream, take each other's kept blocks in turn; every
    result is that of the call made alone."""
    ins = [[dev(*synth.attention_inputs(S + i, 1, S, 3, 64, with_grad=True)) for S in (256, 1024)] for i in range(2)]
    ins = [[(q, k, v, do, k, v) for q, k, v, do in one] for one in ins]
    ref = [_calls(one) for one in ins]
    got, errors = [[], []], []

    def work(i):
        try:
            for _ in range(8):
                got[i].append(_calls(ins[i]))
        except Exception as e:  # reported below, in the main thread
            errors.append(repr(e))

    threads = [threading.Thread(target=work, args=(i,)) for i in range(2)]
    for t in threads:
        t.start()
    for t in threads:
        t.join(timeout=100)
    assert not errors and not any(t.is_alive() for t in threads), errors
    for i in range(2):
        for out in got[i]:
            assert all(torch.equal(a, b) for a, b in zip(ref[i], out))
