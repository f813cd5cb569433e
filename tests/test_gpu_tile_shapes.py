"""GPU parity of the tile kernel's shapes (64 x 128, 64 x 256, 128 x 256 work-group tiles) against fp64 matrix products of the dequantized
weights: every format, buckets at the edges of 64- and 128-row tiles, weight rows that do not fill a tile, one, two, odd and even
numbers of k-steps.

Bound per element: the codes enter the matrix cores exactly, so every error is an fp32 rounding of a partial sum.  A partial sum is at
most sum_k |x| s (|q - z| + offset) with an offset of at most 128 code units; there are at most k/32 matrix-core additions, each
rounding within a handful of ulps (the 32 products of one are added in a few steps), and four roundings per group of 64: fewer
than k/4 + 16 roundings of 2^-24."""
import numpy as np
import pytest
import torch

pytestmark = pytest.mark.gpu
DEV = "cuda:0"

FORMATS = [(8, 0, True, 1.0, 0), (6, 0, True, 1.0, 0), (4, 0, True, 1.0, 0), (4, 128, False, 0.9, 0), (4, 64, False, 1.0, 0),
           (3, 128, False, 1.0, 0), (3, 64, False, 0.9, 0), (8, 0, True, 1.0, 1)]
# rows of the eight buckets: below, at and above the heights of a tile, and what a last tile of 1 .. 128 rows leaves
EDGES = [[33, 64, 65, 127, 128, 129, 192, 193], [256, 257, 319, 320, 321, 384, 40, 100], [191, 63, 48, 0, 255, 448, 130, 66]]


def _codes(can):
    """Canonical codes -> (code - zero) * scale and scale, fp64 [n, k]."""
    q = can.qdata.double()
    if can.symmetric:
        s = can.scale.double()[:, None].expand_as(q)
        return q * s, s
    g = can.group
    s = can.scale.double().repeat_interleave(g, dim=1)
    return (q - can.zero.double().repeat_interleave(g, dim=1)) * s, s


@pytest.mark.parametrize("n,k", [(80, 128), (80, 384), (400, 512), (2064, 256), (4112, 640), (17568, 128), (17568, 256), (17568, 384)])
@pytest.mark.parametrize("rows", EDGES)
def test_tile_shapes_against_fp64(rows, n, k):
    from paper_2508_09204_amd import binding as mq
    from paper_2508_09204_amd import experts as ex
    g = torch.Generator(device=DEV)
    g.manual_seed(n + k + rows[0])
    K, M = len(FORMATS), sum(rows)
    w = torch.randn((n, k), generator=g, device=DEV) * 0.02
    pairs = [ex.quantize_and_pack(w, *f, keep_canonical=True) for f in FORMATS]
    x = (torch.randn((M, k), generator=g, device=DEV) + 0.25).to(torch.bfloat16)
    idx = torch.from_numpy(np.repeat(np.arange(K, dtype=np.int32), rows)).to(DEV)[torch.randperm(M, generator=g, device=DEV)].contiguous()
    off, perm = torch.zeros(K + 1, dtype=torch.int32, device=DEV), torch.zeros(M, dtype=torch.int32, device=DEV)
    mq.moqe_bucket(idx, M, K, None, off, perm, None)
    y = torch.full((M, n), float("nan"), device=DEV)
    mq.moqe_grouped_qgemm(x, off, perm, M, 1, [p for p, _ in pairs], y, mq.SCATTER_OUTPUT)
    for e, (_, can) in enumerate(pairs):
        at = (idx == e).nonzero().squeeze(1)
        if at.numel() == 0:
            continue
        xe = x[at].double()
        if can.act_mode:                                   # rows rounded to int8 steps in fp32, as defined for W8A8
            sx = (xe.abs().amax(dim=1, keepdim=True) / 127.0).float()
            xe = torch.round((x[at].float() / sx)).clamp(-127, 127).double() * sx.double()
        wd, s = _codes(can)
        ref = xe @ wd.t()
        bound = (k / 4 + 16) * 2.0 ** -24 * (xe.abs() @ (wd.abs() + 128 * s).t())
        got = y[at].double()
        assert torch.isfinite(got).all(), (e, at.numel())
        worst = float(((got - ref).abs() / bound).max())
        assert worst <= 1.0, (FORMATS[e], at.numel(), worst)
