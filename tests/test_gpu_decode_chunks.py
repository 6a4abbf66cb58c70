"""Ring decode around the chunking rule and the merge's split of the chunks, against the fp64
oracle: fewer chunks than the merge has waves, chunk counts that do not divide over them, one
chunk a block, blocks of an odd number of tiles, and caches on both sides of the rule."""
import numpy as np
import pytest
import torch

import paper_2310_01889_amd as ra
from oracle import decode as OD
from paper_2310_01889_amd import synth
from tests.gpu_util import dev, log, max_err, np64

pytestmark = pytest.mark.gpu


def _rel(got, ref):
    return float(np.linalg.norm(np64(got) - ref) / np.linalg.norm(ref))


# split: probabilities in two bf16 parts (chunks longer than 4096 workgroups would have)
@pytest.mark.parametrize("B,S,H,D,Tq,N,split", [
    (1, 32, 1, 64, 1, 1, False), (1, 96, 2, 128, 3, 3, False), (1, 288, 1, 64, 32, 1, False),
    (2, 352, 3, 128, 2, 11, False), (1, 8192, 1, 128, 1, 1, False), (1, 8192, 2, 64, 5, 64, False),
    (4, 2048, 300, 64, 1, 2, False), (1, 65536, 4, 128, 1, 4, True)])
def test_decode_chunks(B, S, H, D, Tq, N, split):
    # o: probabilities (not split) and output rounded to bf16, each 1.7e-3 of the 2-norm; lse: a
    # probability rounded to bf16 is off by up to 2^-8 of itself, independently of the others: over
    # the dozen keys that make up the shortest case's sum 5e-4 rms, of which four are allowed.  A
    # chunk of a head's at most 256 left out or doubled moves lse by 4e-3 and o by 6e-2 of its norm.
    log("decode chunks B=%d S=%d H=%d D=%d Tq=%d N=%d" % (B, S, H, D, Tq, N))
    q, k, v = synth.attention_inputs(S + H, B, Tq, H, D, kv_len=S)
    o, lse = ra.attention_decode(*dev(q, k, v), N, True)
    torch.cuda.synchronize()
    for h in sorted({0, H // 2, H - 1}):
        hs = slice(h, h + 1)
        o_ref, l_ref = OD.ring_decode_fwd(np64(q[:, :, hs]), np64(k[:, :, hs]), np64(v[:, :, hs]), N, True)
        eo, el = _rel(o[:, :, hs], o_ref), max_err(lse[:, hs], l_ref)
        log("  head %d: o %.2e lse %.2e" % (h, eo, el))
        assert eo <= 5e-3 and el <= (2e-5 if split else 2.0 ** -9)


@pytest.mark.parametrize("B,S,H,D,Tq,N", [(2, 4096, 16, 64, 4, 4), (4, 2048, 16, 128, 8, 1)])
def test_decode_probabilities_carry_two_bf16_parts(B, S, H, D, Tq, N):
    # the denominator sums probabilities in float32: its sums and lse's own rounding (values near 9)
    # are a few 1e-6; rounded to bf16 once, probabilities put errors of 1e-4 on lse
    log("decode lse precision B=%d S=%d H=%d D=%d Tq=%d N=%d" % (B, S, H, D, Tq, N))
    q, k, v = synth.attention_inputs(S + D, B, Tq, H, D, kv_len=S)
    # o then carries the rounding of its bf16 storage alone: uniform in half an ulp either way, for
    # mantissas spread over [1, 2) about 2^-8 / sqrt(3) * 0.74 of the 2-norm, 1.7e-3;
    # probabilities rounded once measure 2.0e-3 and more
    o, lse = ra.attention_decode(*dev(q, k, v), N, True)
    o_ref, l_ref = OD.ring_decode_fwd(np64(q), np64(k), np64(v), N, True)
    log("  o %.2e lse %.2e" % (_rel(o, o_ref), max_err(lse, l_ref)))
    assert max_err(lse, l_ref) <= 2e-5 and _rel(o, o_ref) <= 1.8e-3
