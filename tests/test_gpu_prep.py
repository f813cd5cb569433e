"""GPU parity: round-to-nearest quantizer, packed layout round trip, int8 activation quantization.

Integer results (codes, zero-points, code - zero) must match the oracle bit for bit.
"""
import numpy as np
import pytest
import torch

from oracle import moqe_oracle as oc

pytestmark = pytest.mark.gpu

FORMATS = [(8, 0, True, 1.0, 0), (8, 0, True, 1.0, 1), (6, 0, True, 1.0, 0), (4, 0, True, 1.0, 0),
           (4, 64, False, 1.0, 0), (4, 128, False, 1.0, 0), (3, 64, False, 1.0, 0), (3, 128, False, 1.0, 0),
           (4, 128, False, 0.9, 0), (3, 128, False, 0.85, 0)]


def _w(n, k, seed):
    w = (np.random.default_rng(seed).standard_normal((n, k)) * 0.02).astype(np.float32)
    w[0, :128] = 0.0            # an all-zero group / (almost) zero row start
    w[1, :] = 0.0               # an all-zero row
    w[2, :128] = 0.01           # a constant group
    return w


@pytest.mark.parametrize("bits,group,sym,clip,act", FORMATS)
@pytest.mark.parametrize("n,k", [(48, 384), (16, 128)])
def test_quantize_rtn_matches_oracle_bit_exact(bits, group, sym, clip, act, n, k):
    from paper_2508_09204_amd import binding as mq, experts as ex
    from tests import gpu_blocks as gb
    w = _w(n, k, seed=bits * 7 + group)
    ref = oc.quantize(w, bits, group, sym, clip)
    can = ex.alloc_canonical(n, k, bits, group, sym, 0, gb.DEV)
    mq.moqe_quantize_rtn(gb.to_dev(w), clip, can)
    torch.cuda.synchronize()
    assert np.array_equal(can.qdata.cpu().numpy(), ref.q)
    assert np.array_equal(can.scale.cpu().numpy().view(np.uint32), ref.scale.view(np.uint32))
    if not sym:
        assert np.array_equal(can.zero.cpu().numpy(), ref.zero)


@pytest.mark.parametrize("bits,group,sym,clip,act", FORMATS)
@pytest.mark.parametrize("n,k", [(48, 384), (16, 128), (256, 256)])
def test_pack_unpack_round_trip_bit_exact(bits, group, sym, clip, act, n, k):
    from paper_2508_09204_amd import binding as mq
    from tests import gpu_blocks as gb
    w = _w(n, k, seed=bits * 11 + group + n)
    ref = oc.quantize(w, bits, group, sym, clip, act)
    packed = gb.packed_dev(ref)
    assert packed.qdata.numel() == mq.moqe_packed_bytes(n, k, bits, group, sym, act)
    out = torch.full((n, k), -999, dtype=torch.int16, device=gb.DEV)
    sc = torch.zeros(ref.scale.shape, dtype=torch.float32, device=gb.DEV)
    mq.moqe_unpack_qmat(packed, out, sc)
    torch.cuda.synchronize()
    assert np.array_equal(out.cpu().numpy(), oc.dequant_int(ref))
    assert np.array_equal(sc.cpu().numpy().view(np.uint32), ref.scale.view(np.uint32))


def test_quantize_full_llama_matrix_matches_oracle():
    """One full-size matrix (11008 x 4096, int4 g128): codes, scales and zero-points bit-exact."""
    from paper_2508_09204_amd import binding as mq, experts as ex
    from tests import gpu_blocks as gb
    w = (np.random.default_rng(5).standard_normal((11008, 4096)) * 0.02).astype(np.float32)
    ref = oc.quantize_asym_group(w, 4, 128, 0.9)
    can = ex.alloc_canonical(11008, 4096, 4, 128, False, 0, gb.DEV)
    mq.moqe_quantize_rtn(gb.to_dev(w), 0.9, can)
    torch.cuda.synchronize()
    assert np.array_equal(can.qdata.cpu().numpy(), ref.q)
    assert np.array_equal(can.scale.cpu().numpy(), ref.scale)
    assert np.array_equal(can.zero.cpu().numpy(), ref.zero)


@pytest.mark.parametrize("bits,group,sym,clip,act", FORMATS)
@pytest.mark.parametrize("n,k", [(16, 128), (80, 640), (16, 13312)])
def test_quantize_and_pack_take_any_alignment_and_write_every_byte(bits, group, sym, clip, act, n, k):
    """fp32 weights 4 bytes and codes 1 byte off a 16-byte boundary give the codes of the oracle; the packed blob does not depend on the
    alignment of the codes nor on what was in the blob before; rows longer than the quantizer's registers hold (12288)."""
    from paper_2508_09204_amd import binding as mq
    from tests import gpu_blocks as gb
    w = _w(n, k, seed=bits + group + n)
    ref = oc.quantize(w, bits, group, sym, clip)
    room = torch.zeros(n * k + 4, dtype=torch.float32, device=gb.DEV)
    room[1:1 + n * k] = gb.to_dev(w).reshape(-1)
    q = torch.zeros(n * k + 16, dtype=torch.uint8, device=gb.DEV)
    can = gb.canonical_dev(ref)
    off = mq.QMat(q.data_ptr() + 1, torch.zeros_like(can.scale), None if sym else torch.zeros_like(can.zero), n, k, bits, group, sym, 0,
                  mq.LAYOUT_CANONICAL)
    mq.moqe_quantize_rtn(room[1:], clip, off)
    torch.cuda.synchronize()
    codes = q[1:1 + n * k].cpu().numpy().reshape(n, k)
    assert np.array_equal(codes.view(ref.q.dtype), ref.q)
    assert np.array_equal(off.scale.cpu().numpy().view(np.uint32), ref.scale.view(np.uint32))
    off.act_mode = can.act_mode = act
    nbytes = mq.moqe_packed_bytes(n, k, bits, group, sym, act)
    blobs = [torch.full((nbytes,), fill, dtype=torch.uint8, device=gb.DEV) for fill in (0, 255)]
    mq.moqe_pack_qmat(can, blobs[0])
    mq.moqe_pack_qmat(off, blobs[1])
    torch.cuda.synchronize()
    assert torch.equal(blobs[0], blobs[1])


@pytest.mark.parametrize("k", [128, 4096, 4224, 12288, 12416, 20480, 20608])       # rows in registers of 2, 6 and 10 vectors a thread, and longer ones
@pytest.mark.parametrize("S,T", [(3, 1), (130, 20)])
def test_activation_rows_are_rounded_to_the_nearest_step(S, T, k):
    """The int8 rows and scales that a grouped launch leaves at the start of its workspace, bit-exact with the IEEE quotient; zeros, rows of extreme scale, and
    more rows than work-groups."""
    from paper_2508_09204_amd import binding as mq
    from paper_2508_09204_amd import experts as ex
    from tests import gpu_blocks as gb
    g = torch.Generator(device=gb.DEV)
    g.manual_seed(k + S)
    x = torch.randn((S * T, k), generator=g, device=gb.DEV) * 10.0 ** torch.randint(-3, 4, (S * T, 1), generator=g, device=gb.DEV)
    x[0], x[1], x[2] = 0.0, x[1] * 1e-37, x[2].sign() * 3e38
    x[-1, 5:] = 0.0
    x = x.to(torch.bfloat16)
    e = [ex.quantize_and_pack(torch.randn((16, k), generator=g, device=gb.DEV), 8, 0, True, 1.0, 1)]
    perm = torch.randperm(S, generator=g, device=gb.DEV).to(torch.int32)
    offsets = torch.tensor([0, S], dtype=torch.int32, device=gb.DEV)
    ws = torch.zeros(mq.moqe_grouped_qgemm_workspace_bytes(e, S, T), dtype=torch.uint8, device=gb.DEV)
    y = torch.zeros((S * T, 16), device=gb.DEV)
    mq.moqe_grouped_qgemm(x, offsets, perm, S, T, e, y, mq.SCATTER_OUTPUT, ws)
    torch.cuda.synchronize()
    M = S * T
    got = ws[:M * k].view(torch.int8).view(M, k).cpu().numpy()
    at = (M * k + 255) // 256 * 256
    scale = ws[at:at + 4 * M].view(torch.float32).cpu().numpy()
    xf = x.float().view(S, T, k)[perm.long()].reshape(M, k).cpu().numpy()
    a = np.abs(xf).max(axis=1)
    sx = np.where(a == 0, np.float32(1), (a / np.float32(127)).astype(np.float32))
    assert np.array_equal(scale.view(np.uint32), sx.view(np.uint32))
    want = np.clip(np.rint(xf / sx[:, None]), -127, 127).astype(np.int8)
    assert np.array_equal(got, want)
