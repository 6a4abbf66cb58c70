"""RMSNorm backward at the edges of its slabs and column chunks, against the fp64 oracle.

Slabs of 32 rows shared by four waves: one row, one row short of and past a slab, several
slabs; widths at and around the 512-column chunks where a kernel instance ends (1024, 2048,
4096 columns) and the largest.  dx is bf16: half an ulp, 2^-8 of the value, and a thousandth of
it for the float32 sum that is rounded.  dg is a float32 sum of T
terms, some ten roundings of 2^-24 each on the way from x to a term and T partial sums
rounded, which add up as a random walk: (10 + sqrt(T)) 2^-24 of sqrt(T) terms' rms, times 5 for
the largest of the columns."""
import numpy as np
import pytest
import torch

import paper_2310_01889_amd as ra
from oracle import llama as OL
from tests.gpu_util import dev, log, np64

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("T,d", [(1, 8), (31, 512), (33, 520), (64, 1024), (100, 1032), (300, 2048), (5, 2056),
                                 (97, 4096), (40, 4104), (65, 8192), (1200, 768)])
def test_rmsnorm_bwd_slabs(T, d):
    log("rmsnorm bwd T=%d d=%d" % (T, d))
    gen = torch.Generator().manual_seed(T + d)
    x = (torch.randn(T, d, generator=gen) * 3).to(torch.bfloat16)
    g = (1 + 0.1 * torch.randn(d, generator=gen)).to(torch.bfloat16)
    dy = torch.randn(T, d, generator=gen)
    dres = torch.randn(T, d, generator=gen).to(torch.bfloat16)
    dx, dg = torch.empty(T, d, dtype=torch.bfloat16, device="cuda"), torch.empty(d, device="cuda")
    ra.rms_norm_bwd(*dev(x, g, dy, dres), dx, dg)
    torch.cuda.synchronize()
    dx_ref, dg_ref = OL.rmsnorm_bwd(np64(x), np64(g), dy.numpy())
    dx_ref = dx_ref + np64(dres)
    # an element of dx is a sum of three terms of up to a few units: their roundings in float32
    scale = np.maximum(np.abs(dx_ref), 1.0)
    x64 = np64(x)
    terms = dy.numpy() * x64 / np.sqrt(np.mean(x64 ** 2, axis=1, keepdims=True))
    bound = 5 * (10 + T ** 0.5) * 2.0 ** -24 * T ** 0.5 * float(np.sqrt(np.mean(terms ** 2)))
    ex, eg = (np.abs(np64(dx) - dx_ref) / scale).max(), np.abs(np64(dg) - dg_ref).max()
    log("  dx %.2e dg %.2e (bound %.2e)" % (ex, eg, bound))
    assert ex <= 1.001 * 2.0 ** -8 and eg <= bound
