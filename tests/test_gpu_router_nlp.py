"""GPU parity of the NLP router model (moqe_route_nlp, Section 3.2: Transformer encoder -> self-attention module
-> MLP) against the oracle with the same bf16 operand rounding.

Logits: |gpu - ref| <= 2e-3 * max(1, max|ref|) (fp32 accumulation, fp32 exp and the rare bf16 rounding decision
that differs between an fp32 and an fp64 intermediate).  The selected expert is an integer decided by fp32 logits: it
must be the first arg-max of the logits the library wrote (bit-exact) and the oracle's expert wherever the oracle's
margin between the two largest logits exceeds twice that tolerance."""
import numpy as np
import pytest
import torch

import workloads as wl
from oracle import moqe_oracle as oc
from oracle import router_nlp_oracle as rn
from tests import oracle_router_nlp as orn

pytestmark = pytest.mark.gpu

#         S   T    d    dm  heads d_ff head_h K
CASES = {
    "small_dh32": (5, 7, 192, 128, 4, 256, 32, 4),
    "one_token": (6, 1, 128, 128, 4, 128, 16, 3),
    "ragged_tiles_dh64": (2, 70, 128, 256, 4, 256, 64, 5),
    "dh16_many_heads": (3, 19, 64, 128, 8, 128, 32, 2),
    "dh128": (2, 33, 64, 256, 2, 128, 32, 4),
    "many_rows": (3, 200, 256, 128, 2, 256, 32, 4),
    "paper_size": (4, 37, 4096, 384, 6, 1536, 384, 4),
}


def _gpu_router(p, d, dm, heads, dff, hh, K):
    from paper_2508_09204_amd import binding as mq
    from tests import gpu_blocks as gb
    dev = {k: gb.to_dev(np.ascontiguousarray(v)) for k, v in p.items()}
    head = mq.Router(dev["head_w1"], dev["head_b1"], dev["head_w2"], dev["head_b2"], dm, hh, K)
    return mq.NlpRouter(dev, head, d, dm, heads, dff)


def _run(case, seed=21):
    from paper_2508_09204_amd import binding as mq
    from tests import gpu_blocks as gb
    S, T, d, dm, heads, dff, hh, K = CASES[case]
    p = wl.make_nlp_router(d, dm, heads, dff, hh, K, seed)
    bits = wl.make_token_activations(S, T, d, seed + 1)
    r = _gpu_router(p, d, dm, heads, dff, hh, K)
    x = gb.bf16_dev(bits.reshape(S * T, d))
    idx = torch.full((S,), -1, dtype=torch.int32, device=gb.DEV)
    logits = torch.full((S, K), float("nan"), dtype=torch.float32, device=gb.DEV)
    mq.moqe_route_nlp(x, S, T, r, idx, logits)
    torch.cuda.synchronize()
    ref_idx, ref_logits, _ = rn.route_nlp(oc.bf16_bits_to_f64(bits), orn.make(p, heads), round_operands=True)
    return idx.cpu().numpy(), logits.cpu().numpy(), ref_idx, ref_logits


@pytest.mark.parametrize("case", list(CASES))
def test_route_nlp_matches_oracle(case):
    idx, logits, ref_idx, ref_logits = _run(case)
    tol = 2e-3 * max(1.0, float(np.abs(ref_logits).max()))
    err = float(np.abs(logits.astype(np.float64) - ref_logits).max())
    assert err <= tol, (err, tol)
    first_max = np.array([int(np.flatnonzero(row == row.max())[0]) for row in logits])
    assert np.array_equal(idx, first_max)
    srt = np.sort(ref_logits, axis=1)
    clear = (srt[:, -1] - srt[:, -2]) > 2 * tol
    assert np.array_equal(idx[clear], ref_idx[clear])
    assert clear.mean() >= 0.5          # the seeded cases are not all near-ties


def test_route_nlp_is_deterministic_and_feeds_the_bucket():
    from paper_2508_09204_amd import binding as mq
    from tests import gpu_blocks as gb
    a = _run("small_dh32")
    b = _run("small_dh32")
    assert np.array_equal(a[0], b[0]) and np.array_equal(a[1], b[1])
    S, K = CASES["small_dh32"][0], CASES["small_dh32"][7]
    idx = gb.to_dev(a[0].astype(np.int32))
    counts = torch.zeros(K, dtype=torch.int32, device=gb.DEV)
    offsets = torch.zeros(K + 1, dtype=torch.int32, device=gb.DEV)
    perm = torch.zeros(S, dtype=torch.int32, device=gb.DEV)
    inv = torch.zeros(S, dtype=torch.int32, device=gb.DEV)
    mq.moqe_bucket(idx, S, K, counts, offsets, perm, inv)
    torch.cuda.synchronize()
    c, o, pm, iv = oc.bucket(a[0], K)
    assert np.array_equal(counts.cpu().numpy(), c) and np.array_equal(perm.cpu().numpy(), pm)


@pytest.mark.parametrize("S,T", [(11, 6), (5, 70)])         # a batch that buckets itself in the first launch / one that does not
def test_router_model_drives_the_routed_mlp_block(S, T):
    """The paper's router in front of the routed experts: moqe_route_nlp -> moqe_forward_routed (bucketing, grouped
    gate/up GEMM with the SiLU gate, grouped down GEMM, scatter).  The experts the GPU router chose are checked against the
    oracle's router, the block's output against the oracle's block run on those experts."""
    from paper_2508_09204_amd import binding as mq
    from tests import gpu_blocks as gb
    from tests import oracle_blocks as ob
    cfg = wl.scaled(wl.get_config("llama7b_mlp_decode"), S=S, T=T, D=256, F=384, router_hidden=32)
    blk = ob.make_block(cfg)
    dm, heads, dff, hh = 128, 4, 256, 32
    p = wl.make_nlp_router(cfg.D, dm, heads, dff, hh, cfg.K, 31)
    bits = wl.make_token_activations(cfg.S, cfg.T, cfg.D, 32)
    x64 = oc.bf16_bits_to_f64(bits)
    r = _gpu_router(p, cfg.D, dm, heads, dff, hh, cfg.K)
    x = gb.bf16_dev(bits.reshape(cfg.M, cfg.D))
    idx = torch.full((cfg.S,), -1, dtype=torch.int32, device=gb.DEV)
    mq.moqe_route_nlp(x, cfg.S, cfg.T, r, idx)
    dblk = gb.block_dev(blk)
    y = torch.full((cfg.M, cfg.D), float("nan"), dtype=torch.float32, device=gb.DEV)
    aux = gb.new_aux(cfg.S, cfg.K, cfg.M, cfg.F)
    aux.expert_idx = None
    aux.logits = None
    mq.moqe_forward_routed(dblk, idx, x, cfg.S, cfg.T, y, aux)
    torch.cuda.synchronize()
    e = idx.cpu().numpy()
    assert len(set(e.tolist())) > 1
    ref_idx, _, _ = rn.route_nlp(x64, orn.make(p, heads), round_operands=True)
    assert np.mean(e == ref_idx) >= 0.8
    c, o, pm, iv = oc.bucket(e, cfg.K)
    assert np.array_equal(aux.counts.cpu().numpy(), c) and np.array_equal(aux.offsets.cpu().numpy(), o)
    assert np.array_equal(aux.perm.cpu().numpy(), pm) and np.array_equal(aux.inv_perm.cpu().numpy(), iv)
    # stage-wise, as for moqe_forward: H against the oracle's H, the down projection against the oracle's on the GPU's H
    from tests.test_gpu_forward import _check_mlp_stages
    _check_mlp_stages(cfg, blk, x64, aux, y.cpu().numpy().reshape(cfg.S, cfg.T, cfg.D), e)


@pytest.mark.timeout(900)
@pytest.mark.parametrize("S,T", [(64, 1), (16, 512)])
def test_route_nlp_full_size_workload_shapes(S, T):
    """The 16 MB router at the decode and prefill batch shapes the bench times (d = 4096): all logits against the oracle."""
    from paper_2508_09204_amd import binding as mq
    from tests import gpu_blocks as gb
    d, dm, heads, dff, hh, K = 4096, 384, 6, 1536, 384, 4
    p = wl.make_nlp_router(d, dm, heads, dff, hh, K, 51)
    bits = wl.make_token_activations(S, T, d, 52)
    r = _gpu_router(p, d, dm, heads, dff, hh, K)
    x = gb.bf16_dev(bits.reshape(S * T, d))
    idx = torch.full((S,), -1, dtype=torch.int32, device=gb.DEV)
    logits = torch.full((S, K), float("nan"), dtype=torch.float32, device=gb.DEV)
    mq.moqe_route_nlp(x, S, T, r, idx, logits)
    torch.cuda.synchronize()
    ref_idx, ref_logits, _ = rn.route_nlp(oc.bf16_bits_to_f64(bits), orn.make(p, heads), round_operands=True)
    tol = 2e-3 * max(1.0, float(np.abs(ref_logits).max()))
    lg = logits.cpu().numpy()
    assert float(np.abs(lg - ref_logits).max()) <= tol
    srt = np.sort(ref_logits, axis=1)
    clear = (srt[:, -1] - srt[:, -2]) > 2 * tol
    assert np.array_equal(idx.cpu().numpy()[clear], ref_idx[clear]) and clear.mean() >= 0.5


@pytest.mark.parametrize("T", [31, 32, 33, 64, 65, 96, 128, 129])
@pytest.mark.parametrize("dm,heads", [(128, 8), (128, 4), (128, 2), (256, 2), (640, 10)])
def test_route_nlp_attention_and_linear_tile_edges(T, dm, heads):
    """Token counts around the attention's tiles (32 keys, 64 or 128 queries per work-group) for every head width, with 2 to 3 samples:
    rows that do not fill the linear kernel's 128 and batches below and above its 512-row split; one and several chunks of the pooled
    LayerNorm, widths on both sides of its 512-column variant.  Same tolerance and input
    distribution as the cases above."""
    name = "edge"
    CASES[name] = (3 if T % 2 else 5, T, 192, dm, heads, 256, 32, 4)
    try:
        idx, logits, ref_idx, ref_logits = _run(name, seed=T + dm + heads)
    finally:
        del CASES[name]
    tol = 2e-3 * max(1.0, float(np.abs(ref_logits).max()))
    assert float(np.abs(logits.astype(np.float64) - ref_logits).max()) <= tol
    assert np.array_equal(idx, np.array([int(np.flatnonzero(row == row.max())[0]) for row in logits]))


@pytest.mark.parametrize("S,T,d", [(513, 1, 64), (20, 32, 192), (300, 3, 320), (1030, 1, 128), (40, 1, 1088), (70, 2, 1216)])
def test_route_nlp_linear_ring_and_row_tiles(S, T, d):
    """Up to 512 rows the linear kernel's four-buffer ring with k-tiles in shares of 8, 9 and 10.  The batches above take the kernels of whole rows
    at this width; the linear kernel has them in the test below.  Same tolerance and input distribution as the cases above."""
    name = "ring"
    CASES[name] = (S, T, d, 128, 2, 256, 32, 4)
    try:
        idx, logits, ref_idx, ref_logits = _run(name, seed=S + T + d)
    finally:
        del CASES[name]
    tol = 2e-3 * max(1.0, float(np.abs(ref_logits).max()))
    assert float(np.abs(logits.astype(np.float64) - ref_logits).max()) <= tol
    assert np.array_equal(idx, np.array([int(np.flatnonzero(row == row.max())[0]) for row in logits]))


@pytest.mark.parametrize("S,T,d,dm,heads,dff", [
    (513, 1, 64, 256, 4, 384),           # 2 k-tiles; five row tiles, one row in the last
    (20, 32, 192, 256, 2, 384),          # 6
    (300, 3, 320, 256, 8, 384),          # 10; eight row tiles, dealt to the XCDs as one group
    (1030, 1, 128, 256, 4, 640),         # 4; a ninth row tile, beside the group
    (461, 5, 64, 640, 10, 640),          # 19 row tiles, 285 work-groups in the widest product: the two-buffer form
    (33, 157, 128, 512, 4, 512),         # 41 row tiles, and 492 work-groups
    (44, 12, 64, 384, 6, 8064),          # a width that whole rows take, with a feed-forward that they do not
])
def test_route_nlp_launch_per_stage_of_many_rows(S, T, d, dm, heads, dff):
    """More than 512 rows of widths and feed-forwards that stay on a launch per stage: the linear kernel's rings of four and two buffers with whole and
    broken rounds of k-tiles, row tiles below, at and above the eight from which they are dealt to the XCDs.

    Bound: a bf16 rounding that fp32 and fp64 decide differently moves its sample's logits by up to what all the roundings together move them, the
    distance of the oracle to itself without them; all but such samples are held to the tolerance above.  (1030 samples of one token, which average
    nothing: noise of 2^-23 ahead of the oracle's roundings moves 3 % of the samples by more than 1e-4 and one of them by 4.3e-3 to
    6.3e-3 over four seeds; the roundings together move one by 1.4e-2.)"""
    name = "stages"
    CASES[name] = (S, T, d, dm, heads, dff, 32, 4)
    seed = S + T + d + dm
    try:
        idx, logits, _, ref_logits = _run(name, seed=seed)
    finally:
        del CASES[name]
    x64 = oc.bf16_bits_to_f64(wl.make_token_activations(S, T, d, seed + 1))
    plain = rn.route_nlp(x64, orn.make(wl.make_nlp_router(d, dm, heads, dff, 32, 4, seed), heads), round_operands=False)[1]
    err = np.abs(logits.astype(np.float64) - ref_logits).max(axis=1)
    assert float(err.max()) <= float(np.abs(plain - ref_logits).max())
    assert np.mean(err <= 2e-3 * max(1.0, float(np.abs(ref_logits).max()))) >= 0.97
    assert np.array_equal(idx, np.array([int(np.flatnonzero(row == row.max())[0]) for row in logits]))


@pytest.mark.parametrize("weight", [-3e38, -1e25, 1e25])
@pytest.mark.parametrize("T", [9, 20, 48, 100])
@pytest.mark.parametrize("dm,heads", [(128, 8), (128, 4), (128, 2), (256, 2)])
def test_route_nlp_keys_of_very_low_score_have_weight_zero(dm, heads, T, weight):
    """Keys whose score with every query of one head is minus infinity (their product overflows fp32) or hugely negative get weight 0 and
    leave the other keys' weights alone, as in exact arithmetic; the router's logits stay finite.  A column of the token vectors marks
    these keys: it reaches dimension 0 of the head's keys with `weight` times 2, and the head's queries have 1 there.
    weight 1e25: hugely positive, all the weight is on the marked keys (of equal score up to fp32, so only one token is marked)."""
    from paper_2508_09204_amd import binding as mq
    from tests import gpu_blocks as gb
    S, d, dff, hh, K, head, dh = 3, 64, 128, 32, 4, 1, dm // heads
    p = wl.make_nlp_router(d, dm, heads, dff, hh, K, 77 + T)
    p["w_in"][0], p["b_in"][0] = 0.0, 0.0
    p["w_in"][0, 0] = 1.0
    q0, k0 = head * dh, dm + head * dh
    p["wqkv1"][q0], p["bqkv1"][q0] = 0.0, 1.0
    p["wqkv1"][k0], p["bqkv1"][k0] = 0.0, 0.0
    p["wqkv1"][k0, 0] = weight
    bits = wl.make_token_activations(S, T, d, 78).reshape(S, T, d).copy()
    bits[:, :, 0] = 0
    marked = [T // 2] if weight > 0 else [1, T // 2, T - 1]
    bits[:, marked, 0] = wl.f32_to_bf16_bits(np.array([2.0], dtype=np.float32))[0]
    r = _gpu_router(p, d, dm, heads, dff, hh, K)
    idx = torch.full((S,), -1, dtype=torch.int32, device=gb.DEV)
    logits = torch.full((S, K), float("nan"), dtype=torch.float32, device=gb.DEV)
    mq.moqe_route_nlp(gb.bf16_dev(bits.reshape(S * T, d)), S, T, r, idx, logits)
    torch.cuda.synchronize()
    _, ref = rn.route_nlp(oc.bf16_bits_to_f64(bits), orn.make(p, heads), round_operands=True)[:2]
    lg = logits.cpu().numpy().astype(np.float64)
    assert np.isfinite(lg).all()
    assert float(np.abs(lg - ref).max()) <= 2e-3 * max(1.0, float(np.abs(ref).max()))


@pytest.mark.parametrize("T", [1, 2, 15, 16, 17, 48, 49, 191, 192, 193])
@pytest.mark.parametrize("dm,heads", [(128, 8), (128, 4), (128, 2), (256, 2)])
def test_route_nlp_attention_dispatch_edges(T, dm, heads):
    """Token counts on both sides of the lines between the attention's forms (16 and 48 tokens, 64, 128 to 192), for every head width.  Same
    tolerance and input distribution as the cases above."""
    name = "dispatch"
    CASES[name] = (9 if T < 64 else 2, T, 64, dm, heads, 128, 32, 4)
    try:
        idx, logits, ref_idx, ref_logits = _run(name, seed=T + dm + 3 * heads)
    finally:
        del CASES[name]
    tol = 2e-3 * max(1.0, float(np.abs(ref_logits).max()))
    assert float(np.abs(logits.astype(np.float64) - ref_logits).max()) <= tol
    assert np.array_equal(idx, np.array([int(np.flatnonzero(row == row.max())[0]) for row in logits]))


@pytest.mark.parametrize("S,T,d,dm,heads,dff", [
    (9, 57, 64, 128, 2, 128),            # 513 rows: 16-row tiles, one row in the last, samples that share tiles, half a buffer of x
    (521, 1, 192, 384, 6, 384),          # a sample per row
    (2, 300, 576, 384, 12, 1152),        # samples of many tiles; five buffers of x, the last half full
    (3, 201, 320, 256, 2, 512),
    (241, 17, 64, 128, 4, 256),          # 4097 rows: 32-row tiles
    (2731, 3, 128, 128, 2, 128),         # 8193 rows: 64-row tiles
    (33, 251, 64, 256, 4, 256),
    (7, 1171, 64, 384, 3, 768),
])
def test_route_nlp_rows_kept_through_the_stages(S, T, d, dm, heads, dff):
    """The kernels that take 16, 32 or 64 whole rows through several stages: row counts on both sides of the lines between them, last tiles of one
    row, samples shorter and longer than a tile, every width, inputs of whole and half buffers.  Same tolerance and input
    distribution as the cases above."""
    name = "rows"
    CASES[name] = (S, T, d, dm, heads, dff, 32, 4)
    try:
        idx, logits, ref_idx, ref_logits = _run(name, seed=S + T + d + dm)
    finally:
        del CASES[name]
    tol = 2e-3 * max(1.0, float(np.abs(ref_logits).max()))
    assert float(np.abs(logits.astype(np.float64) - ref_logits).max()) <= tol
    assert np.array_equal(idx, np.array([int(np.flatnonzero(row == row.max())[0]) for row in logits]))


@pytest.mark.parametrize("S,T,d", [(2341, 7, 64), (131, 127, 192), (37, 444, 448), (23, 713, 832), (257, 127, 320), (192, 128, 64),
                                   (16385, 1, 128), (257, 64, 192), (5483, 3, 64), (2064, 8, 128)])
def test_route_nlp_128_rows_a_work_group(S, T, d):
    """More rows than a round of 64-row work-groups: input widths of half, whole and several buffers of x, a last work-group of 1, 3, 15, 44, 64, 65, 125, 127 and 128 rows.
    Every token row goes through the same sums as in a batch of 513 to 16384 rows (fewer take other kernels), in the same order; only the rows' grouping into tiles for the mean over a
    sample differs: a few roundings of 2^-24 of logits of size 1, so 1e-5 of the largest."""
    from paper_2508_09204_amd import binding as mq
    from tests import gpu_blocks as gb
    p = wl.make_nlp_router(d, 384, 6, 384, 32, 4, S + d)
    r = _gpu_router(p, d, 384, 6, 384, 32, 4)
    g = torch.Generator(device=gb.DEV)
    g.manual_seed(S + T + d)
    x = (torch.randn((S, 1, d), generator=g, device=gb.DEV) + torch.randn((S, T, d), generator=g, device=gb.DEV)).to(torch.bfloat16)

    def run(xs):
        n = xs.shape[0]
        idx = torch.full((n,), -1, dtype=torch.int32, device=gb.DEV)
        logits = torch.full((n, 4), float("nan"), device=gb.DEV)
        mq.moqe_route_nlp(xs.reshape(n * T, d).contiguous(), n, T, r, idx, logits)
        assert torch.equal(idx.long(), (logits == logits.amax(dim=1, keepdim=True)).int().argmax(dim=1))
        return logits

    half = (S + 1) // 2
    assert 16384 < S * T <= 32768 and 512 < (S - half) * T and half * T <= 16384
    whole, parts = run(x), torch.cat([run(x[:half]), run(x[half:])])
    assert float((whole - parts).abs().max()) <= 1e-5 * float(parts.abs().max().clamp(min=1.0))


@pytest.mark.parametrize("S,T,d,dm,heads,dff", [(9, 57, 64, 128, 2, 128), (20, 30, 128, 384, 6, 768), (7, 11, 128, 128, 2, 256), (3, 201, 64, 256, 4, 384)])
def test_route_nlp_layer_norm_vectors_on_any_float(S, T, d, dm, heads, dff):
    """LayerNorm gains and offsets that do not start on 16 bytes (slices of one flat parameter buffer) give the logits of aligned ones, through the
    kernels of whole rows (513 and 600 rows) and a launch per stage (77 rows; 603 of a feed-forward those do not take)."""
    from paper_2508_09204_amd import binding as mq
    from tests import gpu_blocks as gb
    K, hh = 4, 32
    p = wl.make_nlp_router(d, dm, heads, dff, hh, K, 61)
    x = gb.bf16_dev(wl.make_token_activations(S, T, d, 62).reshape(S * T, d))
    dev = {k: gb.to_dev(np.ascontiguousarray(v)) for k, v in p.items()}
    names = [k for k in dev if k.startswith("ln")]
    assert len(names) == 6
    out = []
    for shift in (0, 1, 2, 3):
        flat = torch.zeros(shift + len(names) * (dm + 4 * (shift > 0)), device=gb.DEV)
        q, at = dict(dev), shift
        for k in names:
            q[k] = flat[at:at + dm]
            q[k].copy_(dev[k])
            assert q[k].data_ptr() % 16 == 4 * shift
            at += dm + 4 * (shift > 0)
        head = mq.Router(q["head_w1"], q["head_b1"], q["head_w2"], q["head_b2"], dm, hh, K)
        idx = torch.full((S,), -1, dtype=torch.int32, device=gb.DEV)
        logits = torch.full((S, K), float("nan"), dtype=torch.float32, device=gb.DEV)
        mq.moqe_route_nlp(x, S, T, mq.NlpRouter(q, head, d, dm, heads, dff), idx, logits)
        torch.cuda.synchronize()
        out.append(logits.cpu().numpy())
    assert np.isfinite(out[0]).all()
    for o in out[1:]:
        assert np.array_equal(o, out[0])


@pytest.mark.parametrize("S,T,dm,heads,dff", [(47, 11, 128, 2, 256), (600, 1, 384, 6, 384), (500, 9, 256, 4, 512), (1100, 8, 128, 4, 128),     # whole rows: 16, 16, 32 and 64
                                              (47, 11, 256, 4, 384), (19, 21, 128, 2, 256)])                                                    # a launch per stage
def test_route_nlp_rows_that_are_not_finite_stay_with_their_sample(S, T, dm, heads, dff):
    """A NaN and two infinite token rows change nothing for the samples they do not belong to, though these share tiles of rows with them."""
    from paper_2508_09204_amd import binding as mq
    from tests import gpu_blocks as gb
    d, K, hh = 64, 4, 32
    r = _gpu_router(wl.make_nlp_router(d, dm, heads, dff, hh, K, 71), d, dm, heads, dff, hh, K)
    bits = wl.make_token_activations(S, T, d, 72).reshape(S, T, d).copy()
    bad = {2: 0x7fc0, S // 2: 0x7f80, S - 1: 0xff80}

    def logits_of(b):
        idx = torch.full((S,), -1, dtype=torch.int32, device=gb.DEV)
        lg = torch.full((S, K), 7.0, dtype=torch.float32, device=gb.DEV)
        mq.moqe_route_nlp(gb.bf16_dev(b.reshape(S * T, d)), S, T, r, idx, lg)
        torch.cuda.synchronize()
        return lg.cpu().numpy(), idx.cpu().numpy()

    clean, clean_idx = logits_of(bits)
    for s, v in bad.items():
        bits[s, T // 2, 5] = v
    lg, idx = logits_of(bits)
    rest = np.array([s not in bad for s in range(S)])
    assert np.isfinite(clean).all()
    assert np.array_equal(lg[rest], clean[rest]) and np.array_equal(idx[rest], clean_idx[rest])
    assert ((idx >= 0) & (idx < K)).all()
