"""The whole ring in one launch against the same call made of one launch a ring step.

With RINGATTN_SERIAL_COPY a whole-ring bf16 call, forward or backward, runs step by step, its
blocks copied from host to host; both forms fold the same tiles in the same order, so their
results are equal bit for bit.  The shapes sit where
the one-launch form can go wrong: (batch, head) groups that do not divide over the 8 XCDs,
one tile per workgroup, blocks of one tile row, more hosts than full blocks, ragged ends one
row past and one row short of a tile, the eight-wave kernel.
"""
import pytest
import torch

import paper_2310_01889_amd as ra
from oracle import attention as OA
from paper_2310_01889_amd import synth
from tests.gpu_util import dev, log, max_err, np64

pytestmark = pytest.mark.gpu

TOL_O = 2e-2  # bf16 outputs against float64, as in test_gpu_attention
TOL_G = 5e-2

# B, S, H, D, N, causal
SHAPES = [
    (1, 128, 1, 128, 1, 1),
    (1, 128, 3, 64, 1, 0),
    (1, 1, 1, 128, 4, 1),
    (1, 127, 5, 64, 2, 1),
    (2, 129, 3, 128, 3, 1),
    (1, 257, 6, 128, 2, 1),
    (3, 640, 2, 64, 5, 1),
    (1, 1023, 7, 128, 8, 1),
    (1, 1025, 12, 64, 4, 1),
    (2, 1024, 4, 128, 8, 0),
    (1, 8192, 2, 128, 64, 1),
    (1, 8192, 1, 64, 64, 0),
    (1, 32768, 1, 128, 2, 1),
    (1, 32700, 1, 128, 2, 1),
]


@pytest.mark.parametrize("B,S,H,D,N,causal", SHAPES)
def test_one_launch_equals_steps(B, S, H, D, N, causal, monkeypatch):
    log("one launch B=%d S=%d H=%d D=%d N=%d causal=%d" % (B, S, H, D, N, causal))
    q, k, v, do = synth.attention_inputs(S + H, B, S, H, D, with_grad=True)
    qd, kd, vd, dod = dev(q, k, v, do)
    o, lse = ra.attention_fwd(qd, kd, vd, N, causal)
    grads = ra.attention_bwd(qd, kd, vd, o, lse, dod, N, causal)
    torch.cuda.synchronize()
    monkeypatch.setenv("RINGATTN_SERIAL_COPY", "1")
    o1, lse1 = ra.attention_fwd(qd, kd, vd, N, causal)
    grads1 = ra.attention_bwd(qd, kd, vd, o, lse, dod, N, causal)
    torch.cuda.synchronize()
    assert torch.equal(o, o1) and torch.equal(lse, lse1)
    for g, g1 in zip(grads, grads1):
        assert torch.equal(g, g1)
    if S <= 8192:
        o_ref, lse_ref = OA.attention_fwd(np64(q), np64(k), np64(v), bool(causal))
        assert max_err(o, o_ref) <= TOL_O and max_err(lse, lse_ref) <= TOL_O
        ref = OA.attention_bwd(np64(q), np64(k), np64(v), np64(do), bool(causal))
        assert max(max_err(g, r) for g, r in zip(grads, ref)) <= TOL_G
