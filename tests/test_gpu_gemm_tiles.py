"""Products on both sides of the tile-size rule, weight gradients block by block, and row groups.

The GEMM takes 128 x 128 tiles where 256 x 256 ones would leave the chip part empty; the
smallest shapes, and shapes with just under and just over one round of big tiles, are
compared with float32 products of the same bf16 values (errors: bf16 output 2^-9 relative,
float32 sums of K terms).  A weight gradient is the sum of its blocks' own, added up in order:
the same, bit for bit, as calls on one block each.  The feed-forward networks work on several
whole blocks at a time: a length of seven, cut into groups, against the same calls.
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
    err = (got.to(ref.dtype) - ref).abs().max().item() / ref.pow(2).mean().sqrt().item()
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
    # float32 sums: T / 16 products and T / 256 blocks each round a partial sum of up to ~5 rms by
    # at most 2^-24 of it, which adds up as a random walk: sqrt(289) * 5 * 6e-8 = 5e-6 rms
    _close(dw.double(), x.double().t().contiguous() @ dy.double(), 1e-5)


# big and small tiles, one to 18 blocks of 8 to 64 steps, several products of one input
@pytest.mark.parametrize("T,di,do,blk", [(512, 256, 256, 512), (1024, 256, 512, 512), (4608, 256, 256, 256),
                                         (3840, 1280, 512, 768), (6144, 4096, 4096, 2048), (1280, 4096, 4096, 256)])
def test_weight_gradient_adds_up_blocks(T, di, do, blk):
    log("wgrad T=%d d_in=%d d_out=%d block=%d" % (T, di, do, blk))
    x, w, dy = _rand(1, T, di), _rand(2, di, do, std=0.02), _rand(4, T, do)
    dw, one, ref = (torch.empty(di, do, device="cuda") for _ in range(3))
    ra.blockwise_linear_bwd(x, w, dy, None, dw, blk)
    for r in range(0, T, blk):
        ra.blockwise_linear_bwd(x[r:r + blk], w, dy[r:r + blk], None, one, blk)
        ref = one.clone() if r == 0 else ref + one
    assert torch.equal(dw, ref)


# a slab of fewer rows than waves, odd counts of rows a wave, long slabs
@pytest.mark.parametrize("T,blk", [(256, 256), (1280, 256), (16384, 2048), (65536, 1024)])
def test_bias_gradient_precision(T, blk):
    log("bias gradient T=%d block=%d" % (T, blk))
    dm, dff = 512, 256
    x, dy, w1, w2 = _rand(1, T, dm), _rand(2, T, dm), _rand(3, dm, dff, std=0.02), _rand(4, dff, dm, std=0.02)
    b1, dx = _rand(5, dff), torch.empty_like(x)
    dws = [torch.empty(*s, device="cuda") for s in ((dm, dff), (dff,), (dff, dm), (dm,))]
    ra.blockwise_ffn_bwd(x, w1, b1, w2, dy, dx, *dws, blk)
    ref = dy.double().sum(0)
    err = ((dws[3].double() - ref).norm() / ref.norm()).item()
    log("  relative error %.2e" % err)
    # in units of a float32's half ulp, 2^-24: four sums of T / 1024 rows a thread measure 0.9 at
    # 16384 rows and 1.1 at 65536 (bf16 terms add up exactly while sums are small), one sum of
    # T / 256 rows a thread 1.8 and 2.5, a call a block 1.1 and 2.6
    assert err <= 1.25 * 2.0 ** -24


@pytest.mark.parametrize("dm", [256, 512])  # weight gradients in 128 x 128 and in 256 x 128 tiles
@pytest.mark.parametrize("glu", [False, True])
def test_row_groups_of_unequal_size(glu, dm):
    blk = 2048
    dff = 8192 if glu else 16384  # five blocks fit in the backward of both: groups of 4 + 3
    T = 7 * blk
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
    ys, dxs, sums = zip(*(call(r, r + blk) for r in range(0, T, blk)))
    assert torch.equal(y, torch.cat(ys)) and torch.equal(dx, torch.cat(dxs))
    for i, d in enumerate(dws):
        ref = sums[0][i]
        for s in sums[1:]:
            ref = ref + s[i]
        assert torch.equal(d, ref)


def test_row_groups_hold_little_memory():
    """The intermediates of a long, narrow network stay within the header's 1.25 GiB."""
    T, dm, dff, blk = 32768, 256, 16384, 1024
    x, dy, w1, w2 = _rand(1, T, dm), _rand(2, T, dm), _rand(3, dm, dff, std=0.02), _rand(4, dff, dm, std=0.02)
    dx, dw1, dw2 = torch.empty_like(x), torch.empty(dm, dff, device="cuda"), torch.empty(dff, dm, device="cuda")
    torch.cuda.synchronize()
    ra.release_workspace()
    free = torch.cuda.mem_get_info()[0]
    ra.blockwise_ffn_bwd(x, w1, None, w2, dy, dx, dw1, None, dw2, None, blk)
    torch.cuda.synchronize()
    used = free - torch.cuda.mem_get_info()[0]
    ra.release_workspace()
    log("  workspace %.3f GiB" % (used / 2 ** 30))
    assert 0 < used <= 1.25 * 2 ** 30 + 64 * 2 ** 20  # column sums and the pool's granularity
