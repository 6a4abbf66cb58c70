"""float32 ring attention at the edges of its tiling, against the fp64 oracle.

32-row tiles taken in turn by 2 (D = 128) or 4 (D = 64) waves of a workgroup: sequences of one
block of 64, tile counts that leave some waves without a last tile or without any, blocks of
an odd number of tiles, heads that do not divide over the XCDs, up to 64 hosts, both masks.
Tolerance: the float32 path's 1e-5 (absolute; sums of float32 products in float32).
"""
import pytest
import torch

import paper_2310_01889_amd as ra
from oracle import attention as OA
from paper_2310_01889_amd import synth
from tests.gpu_util import dev, log, max_err, np64

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("D", [64, 128])
@pytest.mark.parametrize("B,S,H,N,causal", [(1, 64, 1, 1, 1), (1, 64, 3, 1, 0), (2, 128, 2, 2, 1), (1, 192, 1, 3, 0),
                                            (1, 320, 5, 1, 1), (1, 576, 2, 3, 1), (1, 576, 2, 9, 0),
                                            (3, 448, 7, 7, 1), (1, 4096, 1, 64, 1), (1, 1024, 8, 2, 0)])
def test_f32_tiles(B, S, H, N, causal, D):
    log("f32 B=%d S=%d H=%d D=%d N=%d causal=%d" % (B, S, H, D, N, causal))
    q, k, v, do = synth.attention_inputs(S + H + D, B, S, H, D, torch.float32, with_grad=True)
    qd, kd, vd, dod = dev(q, k, v, do)
    o, lse = ra.attention_fwd(qd, kd, vd, N, causal)
    grads = ra.attention_bwd(qd, kd, vd, o, lse, dod, N, causal)
    torch.cuda.synchronize()
    o_ref, lse_ref = OA.attention_fwd(np64(q), np64(k), np64(v), bool(causal))
    ref = OA.attention_bwd(np64(q), np64(k), np64(v), np64(do), bool(causal))
    errs = [max_err(o, o_ref), max_err(lse, lse_ref)] + [max_err(g, r) for g, r in zip(grads, ref)]
    log("  errs %s" % ["%.1e" % e for e in errs])
    assert max(errs) <= 1e-5
