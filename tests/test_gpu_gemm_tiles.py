"""Products on both sides of the tile-size rule, and row groups of unequal size.

The GEMM takes 128 x 128 tiles where 256 x 256 ones would leave the chip part empty; the
smallest shapes, and shapes with just under and just over one round of big tiles, are
compared with float32 products of the same bf16 values (errors: bf16 output 2^-9 relative,
float32 sums of K terms).  The feed-forward networks work on as many whole blocks at a time as
their workspace limit holds: a length of five blocks, cut 3 + 2, against the two calls it is
cut into.
"""
import pytest
import torch

import paper_2310_01889_amd as ra
from tests.gpu_util import log

pytestmark = pytest.mark.gpu

BF = torch.bfloat16


def _rand(seed, *shape, std=1.0):
    g = torch.Generator(device="cuda").manual_seed(seed)
    return (torch.randn(*shape, generator=g, device="cuda") * std).to(BF)


def _close(got, ref, tol):
    # relative to the row of sums' own scale: entries of a random product are near its rms
    err = (got.float() - ref).abs().max().item() / ref.pow(2).mean().sqrt().item()
    assert err <= tol, err


# T, d_in, d_out: smallest; ragged counts of small tiles; 128, 240, 256, 272 big tiles
@pytest.mark.parametrize("T,di,do", [(256, 256, 256), (768, 256, 1280), (512, 1280, 512), (2048, 1024, 4096),
                                     (3840, 512, 4096), (4096, 512, 4096), (4352, 512, 4096)])
def test_linear_tiles(T, di, do):
    log("linear T=%d d_in=%d d_out=%d" % (T, di, do))
    x, w, res, dy = _rand(1, T, di), _rand(2, di, do, std=0.02), _rand(3, T, do), _rand(4, T, do)
    y, dx = torch.empty(T, do, dtype=BF, device="cuda"), torch.empty_like(x)
    dw = torch.empty(di, do, device="cuda")
    ra.blockwise_linear(x, w, res, y, 256)
    ra.blockwise_linear_bwd(x, w, dy, dx, dw, 256)
    # one bf16 rounding of values up to ~5 rms: half an ulp 2^-9 * 8 = 1.6e-2 rms
    _close(y, x.float() @ w.float() + res.float(), 2e-2)
    _close(dx, dy.float() @ w.float().t(), 2e-2)
    # float32 output, sums of T terms in another order: T * 2^-24 times a few rms
    _close(dw, x.float().t() @ dy.float(), 1e-3)


@pytest.mark.parametrize("glu", [False, True])
def test_row_groups_of_unequal_size(glu):
    blk, dm = 8192, 256
    dff = 8192 if glu else 16384  # five blocks are cut 3 + 2 in the backward of both
    T, cut = 5 * blk, 3 * blk
    x, dy = _rand(5, T, dm), _rand(6, T, dm)
    w1, w3, w2 = _rand(7, dm, dff, std=0.02), _rand(8, dm, dff, std=0.02), _rand(9, dff, dm, std=0.02)

    def call(lo, hi):
        n = hi - lo
        y, dx = torch.empty(n, dm, dtype=BF, device="cuda"), torch.empty(n, dm, dtype=BF, device="cuda")
        dws = [torch.empty(*s, device="cuda") for s in ((dm, dff), (dm, dff), (dff, dm))]
        xs, gs = x[lo:hi].contiguous(), dy[lo:hi].contiguous()
        if glu:
            ra.swiglu_ffn(xs, w1, w3, w2, xs, y, blk)
            ra.swiglu_ffn_bwd(xs, w1, w3, w2, gs, dx, dws[0], dws[1], dws[2], blk)
        else:
            ra.blockwise_ffn(xs, w1, None, w2, None, y, blk)
            ra.blockwise_ffn_bwd(xs, w1, None, w2, gs, dx, dws[0], None, dws[2], None, blk)
            dws[1].zero_()
        return y, dx, dws

    y, dx, dws = call(0, T)
    ya, dxa, dwa = call(0, cut)
    yb, dxb, dwb = call(cut, T)
    assert torch.equal(y, torch.cat([ya, yb])) and torch.equal(dx, torch.cat([dxa, dxb]))
    for d, a, b in zip(dws, dwa, dwb):
        assert torch.equal(d, a + b)  # the second group's sums are added to the first's
