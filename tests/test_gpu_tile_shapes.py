"""GPU parity of the tile kernel's shapes against fp64 matrix products of the dequantized weights: every format, weight rows that do not
fill a tile, one, two, odd and even numbers of k-steps.  The 64-row tiles (64 x 128 and 64 x 256) at the edges of a bucket; the 128 x 256 tile, for
the formats that have it, with 65, 100 and 127 rows left and with a rest that takes a 64-row tile, plain and SiLU-gated, in launches of
4096 such tiles and more, where it is the shape taken whatever the times of the others.

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


LARGE = [(8, 0, True, 1.0, 0), (4, 0, True, 1.0, 0), (4, 128, False, 0.9, 0), (3, 128, False, 1.0, 0), (8, 0, True, 1.0, 1)]
REST = [833, 868, 895, 767, 802]                    # rows of the five buckets: 65, 100, 127, 127 and 34 in the last tile
LARGE_TILES = sum(REST) // 128


def _rows(xe, act_mode):
    """Activation rows in fp64, as the expert sees them."""
    if not act_mode:
        return xe.double()
    sx = (xe.double().abs().amax(dim=1, keepdim=True) / 127.0).float()
    return torch.round(xe.float() / sx).clamp(-127, 127).double() * sx.double()


def _product(xe, can):
    """x W^T in fp64 and the bound of its fp32 error (see above)."""
    wd, s = _codes(can)
    return xe @ wd.t(), (xe.shape[1] / 4 + 16) * 2.0 ** -24 * (xe.abs() @ (wd.abs() + 128 * s).t())


def _large_case(k, seed):
    g = torch.Generator(device=DEV)
    g.manual_seed(seed)
    M = sum(REST)
    x = (torch.randn((M, k), generator=g, device=DEV) + 0.25).to(torch.bfloat16)
    idx = torch.from_numpy(np.repeat(np.arange(5, dtype=np.int32), REST)).to(DEV)[torch.randperm(M, generator=g, device=DEV)].contiguous()
    return g, M, x, idx


@pytest.mark.parametrize("k", [128, 384, 512, 640])
@pytest.mark.parametrize("turn", range(5))
def test_large_tile_with_rows_missing(turn, k):
    from paper_2508_09204_amd import binding as mq
    from paper_2508_09204_amd import experts as ex
    n = 32768
    assert LARGE_TILES * (n // 256) >= 4096
    fm = LARGE[turn:] + LARGE[:turn]
    g, M, x, idx = _large_case(k, 10 * k + turn)
    pairs = [ex.quantize_and_pack(torch.randn((n, k), generator=g, device=DEV) * 0.02, *f, keep_canonical=True) for f in fm]
    off, perm = torch.zeros(6, dtype=torch.int32, device=DEV), torch.zeros(M, dtype=torch.int32, device=DEV)
    mq.moqe_bucket(idx, M, 5, None, off, perm, None)
    y = torch.full((M, n), float("nan"), device=DEV)
    mq.moqe_grouped_qgemm(x, off, perm, M, 1, [p for p, _ in pairs], y, mq.SCATTER_OUTPUT)
    for e, (_, can) in enumerate(pairs):
        at = (idx == e).nonzero().squeeze(1)
        ref, bound = _product(_rows(x[at], can.act_mode), can)
        worst = float(((y[at].double() - ref).abs() / bound).nan_to_num(nan=float("inf")).max())
        assert worst <= 1.0, (fm[e], at.numel(), worst)


@pytest.mark.parametrize("k", [128, 640])
@pytest.mark.parametrize("turn", range(5))
def test_large_gated_tile_with_rows_missing(turn, k):
    """The bf16 intermediate of a SiLU-gated block, in bucket order.  silu' is at most 1.1, so errors a of the gate and b of the up product move
    silu(g) u by at most 1.1 (|u| + b) a + |silu(g)| b; its own fp32 arithmetic and the bf16 rounding stay within 2^-8 of it."""
    from paper_2508_09204_amd import binding as mq
    from paper_2508_09204_amd import experts as ex
    F = 16384
    assert LARGE_TILES * (F // 128) >= 4096
    fm = LARGE[turn:] + LARGE[:turn]
    g, M, x, idx = _large_case(k, 20 * k + turn)
    make = lambda n, kk, f: ex.quantize_and_pack(torch.randn((n, kk), generator=g, device=DEV) * 0.02, *f, keep_canonical=True)
    gate, up, down = ([make(*shape, f) for f in fm] for shape in ((F, k), (F, k), (k, F)))
    blk = mq.Block(mq.KIND_SILU_MLP, mq.Router(None, None, None, None, k, 0, 5), [p for p, _ in gate], [p for p, _ in up], [p for p, _ in down])
    y = torch.full((M, k), float("nan"), device=DEV)
    h = torch.zeros((M, F), dtype=torch.bfloat16, device=DEV)
    perm = torch.zeros(M, dtype=torch.int32, device=DEV)
    mq.moqe_forward_routed(blk, idx, x, M, 1, y, mq.Aux(perm=perm, h=h))
    at = 0
    for e, n_rows in enumerate(REST):
        xe = _rows(x[perm[at:at + n_rows].long()], fm[e][4])
        assert bool((idx[perm[at:at + n_rows].long()] == e).all())
        (gr, ga), (ur, ua) = _product(xe, gate[e][1]), _product(xe, up[e][1])
        sg = gr * torch.sigmoid(gr)
        bound = 1.1 * (ur.abs() + ua) * ga + sg.abs() * ua + 2.0 ** -8 * (sg * ur).abs()
        worst = float(((h[at:at + n_rows].double() - sg * ur).abs() / bound).nan_to_num(nan=float("inf")).max())
        assert worst <= 1.0, (fm[e], n_rows, worst)
        at += n_rows
    assert bool(torch.isfinite(y).all())


@pytest.mark.parametrize("F,k", [(128, 128), (384, 384), (2176, 256), (6144, 640)])
@pytest.mark.parametrize("rows", EDGES[:2])
def test_gated_tile_shapes(rows, F, k):
    """The bf16 intermediate of every format on the 64-row tiles (narrow ones hold gate and up rows in one block of 32); bound as above."""
    from paper_2508_09204_amd import binding as mq
    from paper_2508_09204_amd import experts as ex
    g = torch.Generator(device=DEV)
    g.manual_seed(F + k + rows[0])
    K, M = len(FORMATS), sum(rows)
    make = lambda n, kk, f: ex.quantize_and_pack(torch.randn((n, kk), generator=g, device=DEV) * 0.02, *f, keep_canonical=True)
    gate, up = ([make(F, k, f) for f in FORMATS] for _ in range(2))
    down = [make(k, F, f) for f in FORMATS]
    x = (torch.randn((M, k), generator=g, device=DEV) + 0.25).to(torch.bfloat16)
    idx = torch.from_numpy(np.repeat(np.arange(K, dtype=np.int32), rows)).to(DEV)[torch.randperm(M, generator=g, device=DEV)].contiguous()
    perm = torch.zeros(M, dtype=torch.int32, device=DEV)
    y = torch.zeros((M, k), device=DEV)
    h = torch.zeros((M, F), dtype=torch.bfloat16, device=DEV)
    blk = mq.Block(mq.KIND_SILU_MLP, mq.Router(None, None, None, None, k, 0, K), [p for p, _ in gate], [p for p, _ in up], [p for p, _ in down])
    mq.moqe_forward_routed(blk, idx, x, M, 1, y, mq.Aux(perm=perm, h=h))
    at = 0
    for e, n_rows in enumerate(rows):
        xe = _rows(x[perm[at:at + n_rows].long()], FORMATS[e][4])
        (gr, ga), (ur, ua) = _product(xe, gate[e][1]), _product(xe, up[e][1])
        sg = gr * torch.sigmoid(gr)
        bound = 1.1 * (ur.abs() + ua) * ga + sg.abs() * ua + 2.0 ** -8 * (sg * ur).abs()
        worst = float(((h[at:at + n_rows].double() - sg * ur).abs() / bound).nan_to_num(nan=float("inf")).max())
        assert worst <= 1.0, (FORMATS[e], n_rows, worst)
        at += n_rows


def _spoil(x, at):
    """A copy of x whose rows `at` (positions of x) hold an infinity of either sign or a NaN each, in turn, at different columns."""
    bad = x.clone()
    for i, r in enumerate(at.tolist()):
        bad[r, (37 * i) % x.shape[1]] = (float("inf"), float("nan"), float("-inf"))[i % 3]
    return bad


def _spoiled_places(rows):
    """Places in bucket order, some in every bucket: the first and the last row, and of every 32 rows one, in their first and second half in turn."""
    places, at = [], 0
    for n in rows:
        places += [at + r for r in sorted({0, n - 1} | {32 * i + 16 * (i & 1) + i % 16 for i in range(n // 32)}) if r < n]
        at += n
    return places


@pytest.mark.parametrize("n,k,large", [(32768, 384, True), (4112, 256, False), (400, 640, False)])
def test_rows_that_are_not_finite_stay_by_themselves(n, k, large):
    """Rows of one bucket share tiles and matrix operands: an infinite or NaN activation in some leaves the bits of all others as they are."""
    from paper_2508_09204_amd import binding as mq
    from paper_2508_09204_amd import experts as ex
    rows, fm = (REST, LARGE) if large else (EDGES[0], FORMATS)
    g = torch.Generator(device=DEV)
    g.manual_seed(n + k)
    K, M = len(fm), sum(rows)
    x = (torch.randn((M, k), generator=g, device=DEV) + 0.25).to(torch.bfloat16)
    idx = torch.from_numpy(np.repeat(np.arange(K, dtype=np.int32), rows)).to(DEV)[torch.randperm(M, generator=g, device=DEV)].contiguous()
    packs = [ex.quantize_and_pack(torch.randn((n, k), generator=g, device=DEV) * 0.02, *f) for f in fm]
    off, perm = torch.zeros(K + 1, dtype=torch.int32, device=DEV), torch.zeros(M, dtype=torch.int32, device=DEV)
    mq.moqe_bucket(idx, M, K, None, off, perm, None)
    at = perm[torch.tensor(_spoiled_places(rows), device=DEV)].long()
    out = []
    for a in (x, _spoil(x, at)):
        out.append(torch.zeros((M, n), device=DEV))
        mq.moqe_grouped_qgemm(a, off, perm, M, 1, packs, out[-1], mq.SCATTER_OUTPUT)
    same = (out[0].view(torch.int32) == out[1].view(torch.int32)).all(dim=1)
    same[at] = True
    assert bool(torch.isfinite(out[0]).all())
    assert bool(same.all()), [(fm[int(idx[r])], int(r)) for r in (~same).nonzero().squeeze(1)[:8]]


@pytest.mark.parametrize("F,k,large", [(16384, 256, True), (2176, 384, False), (6144, 256, False)])
def test_rows_that_are_not_finite_stay_by_themselves_gated(F, k, large):
    """The same for the bf16 intermediate of a SiLU-gated block and its output."""
    from paper_2508_09204_amd import binding as mq
    from paper_2508_09204_amd import experts as ex
    rows, fm = (REST, LARGE) if large else (EDGES[0], FORMATS)
    g = torch.Generator(device=DEV)
    g.manual_seed(F + k)
    K, M = len(fm), sum(rows)
    x = (torch.randn((M, k), generator=g, device=DEV) + 0.25).to(torch.bfloat16)
    idx = torch.from_numpy(np.repeat(np.arange(K, dtype=np.int32), rows)).to(DEV)[torch.randperm(M, generator=g, device=DEV)].contiguous()
    make = lambda n, kk: [ex.quantize_and_pack(torch.randn((n, kk), generator=g, device=DEV) * 0.02, *f) for f in fm]
    blk = mq.Block(mq.KIND_SILU_MLP, mq.Router(None, None, None, None, k, 0, K), make(F, k), make(F, k), make(k, F))
    perm = torch.zeros(M, dtype=torch.int32, device=DEV)
    places = torch.tensor(_spoiled_places(rows), device=DEV)
    hs, ys, at = [], [], None
    for spoiled in (False, True):
        hs.append(torch.zeros((M, F), dtype=torch.bfloat16, device=DEV))
        ys.append(torch.zeros((M, k), device=DEV))
        mq.moqe_forward_routed(blk, idx, _spoil(x, at) if spoiled else x, M, 1, ys[-1], mq.Aux(perm=perm, h=hs[-1]))
        at = perm[places].long()
    for (a, b), own, expert in (((hs[0].view(torch.int16), hs[1].view(torch.int16)), places, idx[perm.long()]), ((ys[0].view(torch.int32), ys[1].view(torch.int32)), at, idx)):
        same = (a == b).all(dim=1)
        same[own] = True
        assert bool(same.all()), [(fm[int(expert[r])], int(r)) for r in (~same).nonzero().squeeze(1)[:8]]
    assert bool(torch.isfinite(ys[0]).all())


@pytest.mark.parametrize("k", [128, 384])
@pytest.mark.parametrize("fm", [LARGE[2], LARGE[3]])
@pytest.mark.parametrize("n", [65536, 52224, 49152])
def test_large_tile_whose_last_round_is_half_empty(n, fm, k):
    """One sample of 600 rows, so that the rows of its bucket are known: five 128-row tiles, 2.5, 2 and 1.9 rounds of work-groups (without and with priorities)."""
    from paper_2508_09204_amd import binding as mq
    from paper_2508_09204_amd import experts as ex
    g = torch.Generator(device=DEV)
    g.manual_seed(n + k)
    T = 600
    x = (torch.randn((T, k), generator=g, device=DEV) + 0.25).to(torch.bfloat16)
    packed, can = ex.quantize_and_pack(torch.randn((n, k), generator=g, device=DEV) * 0.02, *fm, keep_canonical=True)
    off = torch.tensor([0, 1], dtype=torch.int32, device=DEV)
    y = torch.full((T, n), float("nan"), device=DEV)
    mq.moqe_grouped_qgemm(x, off, None, 1, T, [packed], y, 0)
    ref, bound = _product(x.double(), can)
    worst = float(((y.double() - ref).abs() / bound).nan_to_num(nan=float("inf")).max())
    assert worst <= 1.0, worst
