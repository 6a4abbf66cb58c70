"""float32 ring attention where finite inputs give scores of -inf, against the fp64 oracle.

A mask carried in the last dimension (k = -max float, q = 4) overflows to a score of -inf in
float32, which weighs 0 (float64: a finite score whose weight underflows to 0).  The masked keys
come first in the walk of the rows that see them, so that a wave's first tiles, or all tiles
of some waves, hold nothing but them.  Tolerance as in test_gpu_f32_tiles.
"""
import numpy as np
import pytest
import torch

import paper_2310_01889_amd as ra
from oracle import attention as OA
from paper_2310_01889_amd import synth
from tests.gpu_util import dev, log, max_err, np64

pytestmark = pytest.mark.gpu

FMAX = float(np.finfo(np.float32).max)


def _inputs(S, H, D, lo, n):
    q, k, v, do = synth.attention_inputs(S + n + D, 1, S, H, D, torch.float32, with_grad=True)
    q[..., -1] = 4.0
    k[..., -1] = 0.0
    k[:, lo:lo + n, :, -1] = -FMAX
    return q, k, v, do


# masked keys [lo, lo + n): one tile, one for every wave of a row group, all of some waves
@pytest.mark.parametrize("D", [64, 128])
@pytest.mark.parametrize("causal,N,lo", [(0, 1, 0), (0, 2, 256), (1, 2, 256)])
@pytest.mark.parametrize("n", [32, 64, 160, 256])
def test_f32_masked_first_tiles(n, causal, N, lo, D):
    log("f32 masked n=%d lo=%d D=%d N=%d causal=%d" % (n, lo, D, N, causal))
    S, H = 512, 2
    q, k, v, do = _inputs(S, H, D, lo, n)
    qd, kd, vd, dod = dev(q, k, v, do)
    o, lse = ra.attention_fwd(qd, kd, vd, N, causal)
    grads = ra.attention_bwd(qd, kd, vd, o, lse, dod, N, causal)
    torch.cuda.synchronize()
    o_ref, lse_ref = OA.attention_fwd(np64(q), np64(k), np64(v), bool(causal))
    ref = OA.attention_bwd(np64(q), np64(k), np64(v), np64(do), bool(causal))
    errs = [max_err(o, o_ref), max_err(lse, lse_ref)] + [max_err(g, r) for g, r in zip(grads, ref)]
    log("  errs %s" % ["%.1e" % e for e in errs])
    assert max(errs) <= 1e-5  # false for NaN


@pytest.mark.parametrize("D", [64, 128])
@pytest.mark.parametrize("n", [32, 96])
def test_f32_left_padding(n, D):
    """One host, causal: rows past the padding are right, rows inside it see no key (lse -inf)."""
    log("f32 left padding n=%d D=%d" % (n, D))
    S, H = 256, 3
    q, k, v, _ = _inputs(S, H, D, 0, n)
    o, lse = ra.attention_fwd(*dev(q, k, v), 1, True)
    torch.cuda.synchronize()
    o_ref, lse_ref = OA.attention_fwd(np64(q), np64(k), np64(v), True)
    assert max_err(o[:, n:], o_ref[:, n:]) <= 1e-5 and max_err(lse[:, :, n:], lse_ref[:, :, n:]) <= 1e-5
    assert bool((lse[:, :, :n] == -float("inf")).all())
