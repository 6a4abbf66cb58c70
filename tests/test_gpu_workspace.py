"""Workspaces kept between calls on the null stream: results do not depend on which block a
call gets -- a fresh one, one left by a call of another size or kind, one allocated after
ring_attn_release_workspace() -- nor does a call on another stream between them matter."""
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
