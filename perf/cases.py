"""Performance cases of the routed quantization-expert library: the calls a serving or training program makes.

`listed()` names the cases, `draw(rng)` gives further ones of the same ranges, `prepare` builds what a program
holds before the call (weights quantized and packed once, inputs, workspace), `run` makes one call through the public
binding, `work` states the bytes and operations the call cannot do without, `exact` is the same call in 64-bit
arithmetic by plain torch.

Kinds of calls:
  block   moqe_forward on a routed block (`shape`: linear, mlp, conv), arguments marshalled once (ForwardCall)
  ragged  moqe_forward_ragged on sequences of different lengths
  layer   moqe_grouped_qgemm inside a stack of layers: bf16 rows in bucket order in and out
  nlp     moqe_route_nlp, the Transformer router model
  cv      moqe_route_cv, the convolutional router model
  label   moqe_label_pass, the training labels of the router
  build   quantize_and_pack, how an expert's matrix is made from fp32 weights
"""
import math
import random

import torch

import workloads as wl
from paper_2508_09204_amd import binding as mq
from paper_2508_09204_amd import experts as ex

DEV = "cuda"
W_STD = 0.02

# expert sets by name; an expert is bits, group, symmetric, clip, act_mode
_FORMATS = {
    "toy": ((8, 0, True, 1.0, 0), (4, 64, False, 1.0, 0), (3, 64, False, 1.0, 0)),
    "llama": ((4, 128, False, 1.0, 0), (4, 128, False, 0.9, 0), (3, 128, False, 1.0, 0), (8, 0, True, 1.0, 0)),
    "qwen": tuple((4, 128, False, c, 0) for c in (1.0, 0.95, 0.9, 0.85)) + (
        (3, 128, False, 1.0, 0), (3, 128, False, 0.9, 0), (8, 0, True, 1.0, 1), (8, 0, True, 1.0, 0)),
    "conv": ((8, 0, True, 1.0, 0), (6, 0, True, 1.0, 0), (4, 0, True, 1.0, 0), (4, 64, False, 1.0, 0)),
}
# router models: widths of the 16 MB Transformer router, and of the convolutional one (16/32/64 channels, strides 1/2/2)
NLP = dict(dm=384, heads=6, d_ff=1536, head=384)
CV = dict(mlp=(64, 32, 16), stages=(16, 32, 64), strides=(1, 2, 2), heads=8)


def listed():
    return [
        # the smallest routed layer (256 x 256, 32 sequences of 16 tokens): what a call costs when there is little to do
        dict(name="linear_small", kind="block", shape="linear", S=32, T=16, D=256, F=256, formats="toy", hidden=0, bias=0.0),
        # one request being decoded: one token through a LLaMA-7B-shaped MLP block, one expert's weights read
        dict(name="decode_one", kind="block", shape="mlp", S=1, T=1, D=4096, F=11008, formats="llama", hidden=256, bias=0.0),
        # decode of a batch of 64 requests: the experts' weights are read once for a few rows each
        dict(name="decode_batch", kind="block", shape="mlp", S=64, T=1, D=4096, F=11008, formats="llama", hidden=256, bias=0.0),
        # prefill of 16 prompts of 512 tokens on the same block
        dict(name="prefill", kind="block", shape="mlp", S=16, T=512, D=4096, F=11008, formats="llama", hidden=256, bias=0.0),
        # the largest: 128 sequences on a Qwen-shaped block with eight experts, most sequences on one of them
        dict(name="prefill_skewed", kind="block", shape="mlp", S=128, T=256, D=3584, F=18944, formats="qwen", hidden=256,
             bias=wl.configs.QWEN_SKEW_BIAS0),
        # image classification: a ResNet-50-shaped 3x3 stage on a batch of 256 images
        dict(name="conv_stage", kind="block", shape="conv", S=256, T=196, D=256, F=256, formats="conv", hidden=64, bias=0.0),
        # a served batch of prompts of mixed lengths, short follow-ups beside long documents
        dict(name="ragged_prompts", kind="ragged", S=40, rows_lo=1, rows_hi=900, lengths=7, D=4096, F=11008, formats="llama",
             hidden=256),
        # an inner layer of a stack bucketed once: short continuations (9 tokens each) of 96 requests, eight experts
        dict(name="stack_layer", kind="layer", S=96, T=9, k=4096, n=4096, formats="qwen"),
        # the Transformer router model scoring 128 sequences
        dict(name="router_nlp", kind="nlp", S=128, T=256, D=3584, K=8),
        # the convolutional router model scoring a batch of feature maps
        dict(name="router_cv", kind="cv", S=256, h=14, w=14, c=256, K=4),
        # router training: 128 short sequences through all experts
        dict(name="label_pass", kind="label", S=128, T=4, D=4096, F=11008, formats="llama"),
        # loading a model: one fp32 matrix quantized and packed
        dict(name="build_expert", kind="build", n=11008, k=4096, bits=4, group=128, symmetric=False, clip=0.9, act_mode=0),
    ]


def _log(rng, lo, hi, step=1):
    """Spread over the logarithm of lo .. hi, in multiples of step."""
    v = math.exp(rng.uniform(math.log(lo), math.log(hi)))
    return max(lo, min(hi, int(round(v / step)) * step))


def _most_rows(D, F):
    """Rows of an MLP block that cost no more than the largest listed case."""
    return int(32768 * 3584 * 18944 / (D * F))


def draw(rng):
    kind = rng.choice(("linear", "decode", "mlp", "mlp", "conv", "ragged", "layer", "nlp", "cv", "label", "build"))
    D = 128 * rng.randint(4, 32)
    F = 128 * rng.randint(8, 148)
    fmt = rng.choice(("toy", "llama", "qwen"))
    if kind == "linear":
        return dict(kind="block", shape="linear", S=_log(rng, 1, 256), T=_log(rng, 1, 64), D=128 * rng.randint(1, 16),
                    F=16 * rng.randint(4, 128), formats=fmt, hidden=rng.choice((0, 64)), bias=0.0)
    if kind == "decode":
        return dict(kind="block", shape="mlp", S=_log(rng, 1, 128), T=1, D=D, F=F, formats=fmt, hidden=256, bias=0.0)
    if kind == "mlp":
        T = _log(rng, 2, 700)
        S = _log(rng, 1, max(1, min(256, 16384 // T, _most_rows(D, F) // T)))
        return dict(kind="block", shape="mlp", S=S, T=T, D=D, F=F, formats=fmt, hidden=256,
                    bias=rng.choice((0.0, wl.configs.QWEN_SKEW_BIAS0)))
    if kind == "conv":
        h, w = rng.randint(5, 28), rng.randint(5, 28)
        return dict(kind="block", shape="conv", S=_log(rng, 1, 256), T=h * w, h=h, D=128 * rng.randint(1, 4),
                    F=16 * rng.randint(4, 32), formats="conv", hidden=64, bias=0.0)
    if kind == "ragged":
        return dict(kind="ragged", S=_log(rng, 2, 64), rows_lo=1, rows_hi=_log(rng, 8, 1200), lengths=rng.randint(1, 1 << 20), D=D,
                    F=min(F, 11008), formats=fmt, hidden=256)
    if kind == "layer":
        T = _log(rng, 1, 256)
        return dict(kind="layer", S=_log(rng, 8, max(8, 8192 // T)), T=T, k=D, n=16 * rng.randint(32, 512), formats=fmt)
    if kind == "nlp":
        return dict(kind="nlp", S=_log(rng, 101, 384), T=_log(rng, 1, 160), D=64 * rng.randint(8, 64), K=rng.randint(2, 8))
    if kind == "cv":
        return dict(kind="cv", S=_log(rng, 1, 256), h=rng.randint(5, 24), w=rng.randint(5, 24), c=4 * rng.randint(4, 64),
                    K=rng.randint(2, 8))
    if kind == "label":
        return dict(kind="label", S=_log(rng, 101, 256), T=rng.randint(1, 6), D=D, F=min(F, 8192), formats=rng.choice(("toy", "llama")))
    bits, group, symmetric, clip, act = rng.choice(_FORMATS["toy"] + _FORMATS["llama"] + _FORMATS["conv"] + _FORMATS["qwen"])
    return dict(kind="build", n=16 * _log(rng, 8, 1184), k=D, bits=bits, group=group, symmetric=symmetric, clip=clip, act_mode=act)


# ---- inputs -----------------------------------------------------------------------------------------------------------
class _Source:
    """Tensors drawn on the GPU, in a fixed order, from one seed."""

    def __init__(self, seed):
        self.g = torch.Generator(device=DEV)
        self.g.manual_seed(int(seed) + 250809200)

    def normal(self, *shape, std=1.0, mean=0.0):
        return torch.randn(shape, generator=self.g, device=DEV, dtype=torch.float32).mul_(std).add_(mean)

    def uniform(self, *shape):
        return torch.rand(shape, generator=self.g, device=DEV, dtype=torch.float32)

    def below(self, n, *shape):
        return torch.randint(0, n, shape, generator=self.g, device=DEV, dtype=torch.int32)


def _lengths(case):
    r = random.Random(case["lengths"])
    return [_log(r, case["rows_lo"], case["rows_hi"]) for _ in range(case["S"])]


def _router(src, D, hidden, K, bias):
    """Router weights as workloads.make_router draws them: zero-sum last layer behind a hidden layer, bias on expert 0."""
    w1 = b1 = None
    if hidden:
        w1 = src.normal(hidden, D, std=0.02)
        b1 = torch.zeros(hidden, device=DEV)
        w2 = src.normal(K, hidden, std=0.02)
        w2 -= w2.mean(dim=1, keepdim=True)
    else:
        w2 = src.normal(K, D, std=0.1)
    b2 = torch.zeros(K, device=DEV)
    b2[0] = bias
    return mq.Router(w1, b1, w2.contiguous(), b2, D, hidden, K)


def _matrices(case):
    """(out, in) of the block's matrices."""
    if case.get("shape") == "linear":
        return [(case["F"], case["D"])]
    if case.get("shape") == "conv":
        return [(case["F"], 9 * case["D"])]
    if case["kind"] == "layer":
        return [(case["n"], case["k"])]
    return [(case["F"], case["D"])] * 2 + [(case["D"], case["F"])]


def _draw_all(case, seed):
    """Everything random of a case, as a dict of fp32 / bf16 / int32 tensors: weights first, then the router, then inputs."""
    src, kind = _Source(seed), case["kind"]
    if kind == "build":
        return dict(w=src.normal(case["n"], case["k"], std=W_STD))
    if kind == "nlp":
        return _draw_nlp(case, src)
    if kind == "cv":
        return _draw_cv(case, src)
    K = len(_FORMATS[case["formats"]])
    d = dict(w=[src.normal(n, k, std=W_STD) for n, k in _matrices(case)])
    if kind == "layer":
        d["expert_idx"] = src.below(K, case["S"])
        d["x"] = src.normal(case["S"] * case["T"], case["k"]).to(torch.bfloat16)
        return d
    if kind != "label":
        d["router"] = _router(src, case["D"], case["hidden"], K, case.get("bias", 0.0))
    rows = sum(_lengths(case)) if kind == "ragged" else case["S"] * case["T"]
    d["x"] = src.normal(rows, case["D"]).to(torch.bfloat16)
    if kind == "label":
        d["targets"] = src.below(case["D"], case["S"], case["T"])
    return d


def _draw_nlp(case, src):
    """The Transformer router's parameters (N(0, 1/fan-in) matrices) and token vectors with a topic per sequence."""
    dm, ff, hd, D, K = NLP["dm"], NLP["d_ff"], NLP["head"], case["D"], case["K"]
    mat = lambda n, k: src.normal(n, k, std=k ** -0.5)
    vec = lambda n, mean=0.0, std=0.02: src.normal(n, std=std, mean=mean)
    p = dict(w_in=mat(dm, D), b_in=vec(dm))
    for t in "12":
        p.update({"wqkv" + t: mat(3 * dm, dm), "bqkv" + t: vec(3 * dm), "wo" + t: mat(dm, dm), "bo" + t: vec(dm)})
    p.update(w_ff1=mat(ff, dm), b_ff1=vec(ff), w_ff2=mat(dm, ff), b_ff2=vec(dm))
    for t in "123":
        p.update({"ln%s_g" % t: vec(dm, 1.0, 0.05), "ln%s_b" % t: vec(dm)})
    h1, hb1, h2, hb2 = mat(hd, dm), vec(hd), mat(K, hd), vec(K)
    h2 = (h2 - h2.mean(dim=1, keepdim=True)).contiguous()
    x = src.normal(case["S"], 1, D) + src.normal(case["S"], case["T"], D)
    return dict(p=p, head=mq.Router(h1, hb1, h2, hb2, dm, hd, K), x=x.to(torch.bfloat16).reshape(-1, D))


def _draw_cv(case, src):
    """The convolutional router's parameters and images with a channel offset, a spatial slope and noise per pixel."""
    mat = lambda *s: src.normal(*s, std=math.prod(s[1:]) ** -0.5)
    vec = lambda n, mean=0.0, std=0.05: src.normal(n, std=std, mean=mean)
    p = {}

    def bn(pre, n):
        p[pre + "_g"], p[pre + "_o"], p[pre + "_m"] = vec(n, 1.0, 0.1), vec(n, 0.0, 0.1), vec(n, 0.0, 0.1)
        p[pre + "_v"] = src.uniform(n) + 0.5

    prev = case["c"]
    for i, n in enumerate(CV["mlp"]):
        p["mlp%d_w" % i], p["mlp%d_b" % i] = mat(n, prev), vec(n)
        bn("mlp%d_bn" % i, n)
        prev = n
    for i, (n, st) in enumerate(zip(CV["stages"], CV["strides"])):
        p["st%d_a" % i], p["st%d_b" % i] = mat(n, 3, 3, prev), mat(n, 3, 3, n)
        bn("st%d_abn" % i, n)
        bn("st%d_bbn" % i, n)
        p["st%d_se1" % i], p["st%d_se1b" % i] = mat(n // 4, n), vec(n // 4)
        p["st%d_se2" % i], p["st%d_se2b" % i] = mat(n, n // 4), vec(n)
        if st != 1 or n != prev:
            p["st%d_s" % i] = mat(n, prev)
            bn("st%d_sbn" % i, n)
        prev = n
    p["wqkv"], p["bqkv"], p["wo"], p["bo"] = mat(3 * prev, prev), vec(3 * prev), mat(prev, prev), vec(prev)
    w = mat(case["K"], prev)
    p["w_out"], p["b_out"] = (w - w.mean(dim=1, keepdim=True)).contiguous(), vec(case["K"])
    S, h, w_, c = case["S"], case["h"], case["w"], case["c"]
    x = src.normal(S, 1, 1, c) + src.normal(S, h, w_, c)
    yy = torch.linspace(-1, 1, h, device=DEV).view(1, h, 1, 1)
    xx = torch.linspace(-1, 1, w_, device=DEV).view(1, 1, w_, 1)
    x += src.normal(S, 1, 1, c) * yy + src.normal(S, 1, 1, c) * xx
    return dict(p=p, x=x.to(torch.bfloat16).reshape(-1, c))


# ---- the call -----------------------------------------------------------------------------------------------------------
def _pack(w, f):
    return ex.quantize_and_pack(w, f[0], f[1], f[2], f[3], f[4])


def _workspace(nbytes):
    return torch.empty(max(int(nbytes), 256), dtype=torch.uint8, device=DEV)


def _i32(*shape):
    return torch.zeros(shape, dtype=torch.int32, device=DEV)


def prepare(case, seed):
    kind, d = case["kind"], _draw_all(case, seed)
    st = dict(case=case)
    if kind == "build":
        st["w"] = d["w"]
        return st
    S = case["S"]
    if kind == "nlp":
        r = mq.NlpRouter(d["p"], d["head"], case["D"], NLP["dm"], NLP["heads"], NLP["d_ff"])
        st.update(x=d["x"], r=r, idx=_i32(S), logits=torch.zeros(S, case["K"], device=DEV),
                  ws=_workspace(mq.moqe_route_nlp_workspace_bytes(S, case["T"], r)))
        return st
    if kind == "cv":
        r = mq.CvRouter(d["p"], case["c"], CV["strides"], CV["heads"], case["K"])
        st.update(x=d["x"], r=r, idx=_i32(S), logits=torch.zeros(S, case["K"], device=DEV),
                  ws=_workspace(mq.moqe_route_cv_workspace_bytes(S, case["h"], case["w"], r)))
        return st
    fm = _FORMATS[case["formats"]]
    K = len(fm)
    packed = [[_pack(w, f) for f in fm] for w in d["w"]]
    if kind == "layer":
        T, n = case["T"], case["n"]
        offsets, perm = _i32(K + 1), _i32(S)
        mq.moqe_bucket(d["expert_idx"], S, K, None, offsets, perm, None)
        st.update(x=d["x"], offsets=offsets, experts=packed[0], y=torch.zeros(S * T, n, dtype=torch.bfloat16, device=DEV),
                  ws=_workspace(mq.moqe_grouped_qgemm_workspace_bytes(packed[0], S, T)))
        return st
    mlp = len(packed) == 3
    blk = mq.Block(kind=mq.KIND_SILU_MLP if mlp else mq.KIND_LINEAR, router=d.get("router") or mq.Router(None, None, None, None, case["D"], 0, K),
                   w0=packed[0], w1=packed[1] if mlp else None, w2=packed[2] if mlp else None)
    if case.get("shape") == "conv":
        h = case.get("h") or math.isqrt(case["T"])
        blk.kind, blk.img_h, blk.img_w, blk.cin = mq.KIND_CONV3X3, h, case["T"] // h, case["D"]
    x = d["x"]
    if kind == "label":
        st.update(blk=blk, x=x, targets=d["targets"], losses=torch.zeros(S, K, device=DEV), labels=_i32(S),
                  ws=_workspace(mq.moqe_label_pass_workspace_bytes(blk, S, case["T"])))
        return st
    y = torch.zeros(x.shape[0], case["D"] if mlp else case["F"], device=DEV)
    aux = mq.Aux(expert_idx=_i32(S))
    if kind == "ragged":
        cu = torch.tensor([0] + _lengths(case), device=DEV).cumsum(0).to(torch.int32)
        st.update(blk=blk, x=x, cu=cu, y=y, aux=aux, ws=_workspace(mq.moqe_workspace_bytes_ragged(blk, S, x.shape[0])))
        return st
    st.update(call=mq.ForwardCall(blk, x, S, case["T"], y, aux), y=y, aux=aux)
    return st


def run(st):
    case = st["case"]
    kind = case["kind"]
    if kind == "block":
        st["call"]()
        return dict(y=st["y"], expert_idx=st["aux"].expert_idx)
    if kind == "ragged":
        mq.moqe_forward_ragged(st["blk"], st["x"], st["cu"], case["S"], st["x"].shape[0], st["y"], st["aux"], st["ws"])
        return dict(y=st["y"], expert_idx=st["aux"].expert_idx)
    if kind == "layer":
        mq.moqe_grouped_qgemm(st["x"], st["offsets"], None, case["S"], case["T"], st["experts"], st["y"], mq.OUTPUT_BF16, st["ws"])
        return dict(y=st["y"])
    if kind == "nlp":
        mq.moqe_route_nlp(st["x"], case["S"], case["T"], st["r"], st["idx"], st["logits"], st["ws"])
        return dict(logits=st["logits"], expert_idx=st["idx"])
    if kind == "cv":
        mq.moqe_route_cv(st["x"], case["S"], case["h"], case["w"], st["r"], st["idx"], st["logits"], st["ws"])
        return dict(logits=st["logits"], expert_idx=st["idx"])
    if kind == "label":
        mq.moqe_label_pass(st["blk"], st["x"], st["targets"], case["S"], case["T"], st["losses"], st["labels"], st["ws"])
        return dict(losses=st["losses"], labels=st["labels"])
    packed, can = ex.quantize_and_pack(st["w"], case["bits"], case["group"], case["symmetric"], case["clip"], case["act_mode"],
                                       keep_canonical=True)
    return dict(blob=packed.qdata, codes=can.qdata, scale=can.scale, **({} if can.zero is None else dict(zero=can.zero)))


# ---- what a call cannot do without ----------------------------------------------------------------------------------------
def _weight_bytes(n, k, f):
    meta = n * (k // f[1]) * (4 if f[2] else 5) if f[1] else 4 * n
    return n * k * f[0] / 8 + meta


def work(case):
    kind = case["kind"]
    if kind == "build":
        n, k = case["n"], case["k"]
        f = (case["bits"], case["group"], case["symmetric"])
        canonical = n * k + _weight_bytes(n, k, (0,) + f[1:])
        return dict(bytes=4 * n * k + canonical + _weight_bytes(n, k, f), flops=4 * n * k)
    S = case["S"]
    if kind == "nlp":
        M, D, dm, ff = S * case["T"], case["D"], NLP["dm"], NLP["d_ff"]
        mats = dm * D + 8 * dm * dm + 2 * dm * ff
        return dict(bytes=2 * M * D + 4 * (mats + NLP["head"] * dm) + 4 * S * (case["K"] + 1),
                    flops=2 * M * mats + 2 * 4 * M * case["T"] * dm + 2 * S * NLP["head"] * dm)
    if kind == "cv":
        h, w, prev, mac, params = case["h"], case["w"], case["c"], 0, 0
        for n in CV["mlp"]:
            mac += S * h * w * prev * n
            params += prev * n
            prev = n
        for n, stride in zip(CV["stages"], CV["strides"]):
            h, w = (h - 1) // stride + 1, (w - 1) // stride + 1
            short = n * prev if stride != 1 or n != prev else 0
            mac += S * h * w * (9 * prev * n + 9 * n * n + short)
            params += 9 * prev * n + 9 * n * n + short
            prev = n
        mac += S * h * w * (3 * prev * prev + 2 * h * w * prev)
        return dict(bytes=2 * S * case["h"] * case["w"] * case["c"] + 4 * (params + 4 * prev * prev) + 4 * S * (case["K"] + 1), flops=2 * mac)
    fm, mats = _FORMATS[case["formats"]], _matrices(case)
    K = len(fm)
    rows = sum(_lengths(case)) if kind == "ragged" else S * case["T"]
    used = min(S, K) / K if kind != "label" else 1.0
    weights = used * sum(_weight_bytes(n, k, f) for n, k in mats for f in fm)
    macs = rows * sum(n * k for n, k in mats)
    if kind == "layer":
        return dict(bytes=weights + 2 * rows * (case["k"] + case["n"]), flops=2 * macs)
    if kind == "label":
        return dict(bytes=weights + 2 * rows * case["D"] + 4 * rows + 4 * S * (K + 1), flops=2 * K * macs)
    n_out = case["D"] if len(mats) == 3 else case["F"]
    hid = case["hidden"]
    router = 4 * (hid * (case["D"] + K) if hid else K * case["D"])
    return dict(bytes=weights + router + 2 * rows * case["D"] + 4 * rows * n_out + 4 * S, flops=2 * macs + S * router / 2)


def tolerance(case):
    """About four times what the outputs were seen to be off their 64-bit values: 2e-3 where an intermediate or the result is held in
    bf16 (3e-3 with an expert on int8 activations, 4e-3 through the whole Transformer router), 1e-6 where all is 32-bit (1e-5 stated).
    Whole numbers are decided by sums; one sample in a hundred may sit on a tie where those are not 32-bit throughout."""
    kind = case["kind"]
    if kind == "build":
        return "exact"
    if kind == "nlp":
        return dict(rel=1.4e-2, max=0.2, differ=0.01)
    if kind == "cv":
        return dict(rel=1e-5, max=1e-4)
    if kind == "layer":
        return dict(rel=7e-3, max=4e-2)
    if kind == "label":
        return dict(rel=6e-4, max=6e-3, differ=0.01)
    a8 = any(f[4] for f in _FORMATS[case["formats"]])
    if case.get("shape") in ("linear", "conv"):
        return dict(rel=1e-3, max=1e-1) if a8 else dict(rel=1e-5, max=1e-3)
    return dict(rel=1.2e-2 if a8 else 6e-3, max=0.2)


# ---- the same call in 64 bits ------------------------------------------------------------------------------------------------
def _codes(w, f):
    """Round-to-nearest quantization, fp32 steps (a quotient of two fp32 numbers taken in 64 bits and rounded is the fp32
    quotient): (codes minus zero, scale) as fp64 with the group axis last, codes, zero."""
    bits, group, symmetric, clip = f[:4]
    n, k = w.shape
    div = lambda a, b: (a.double() / b.double()).float()
    if symmetric:
        qmax = float(2 ** (bits - 1) - 1)
        a = w.abs().amax(dim=1, keepdim=True)
        s = torch.where(a == 0, torch.ones_like(a), div(a, torch.full_like(a, qmax)))
        q = torch.round(div(w, s)).clamp_(-qmax, qmax)
        return q.double(), s.double(), q, None
    v = w.view(n, k // group, group)
    c = torch.full((1,), clip, dtype=torch.float32, device=w.device)
    lo, hi = c * v.amin(dim=2, keepdim=True).clamp(max=0), c * v.amax(dim=2, keepdim=True).clamp(min=0)
    top = float(2 ** bits - 1)
    s = torch.where(hi == lo, torch.ones_like(hi), div(hi - lo, torch.full_like(hi, top)))
    z = torch.round(div(-lo, s)).clamp_(0, top)
    q = (torch.round(div(v, s)) + z).clamp_(0, top)
    return (q - z).double(), s.double(), q, z


def _dequantized(w, f):
    q, s = _codes(w, f)[:2]
    return (q * s).reshape(w.shape)


def _times(x, wd, act_mode):
    """x W^T in 64 bits; act_mode 1: the rows are first rounded to 127 steps of their largest value."""
    if act_mode:
        a = x.abs().amax(dim=1, keepdim=True)
        s = torch.where(a == 0, torch.ones_like(a), a / 127.0)
        x = torch.round(x / s).clamp_(-127, 127) * s
    return x @ wd.t()


def _expert(case, weights, f, x):
    """One expert of the block on fp64 rows (conv: on NHWC images [s, h, w, c])."""
    wd = [_dequantized(w, f) for w in weights]
    if case.get("shape") == "conv":
        s, h, w, c = x.shape
        out = torch.zeros(s * h * w, wd[0].shape[0], dtype=torch.float64, device=x.device)
        xp = torch.nn.functional.pad(x, (0, 0, 1, 1, 1, 1))
        for t in range(9):
            part = xp[:, t // 3:t // 3 + h, t % 3:t % 3 + w].reshape(-1, c)
            out += part @ wd[0][:, t * c:(t + 1) * c].t()
        return out
    if len(wd) == 1:
        return _times(x, wd[0], f[4])
    g = _times(x, wd[0], f[4])
    h = g * torch.sigmoid(g)
    del g
    h *= _times(x, wd[1], f[4])
    return _times(h, wd[2], f[4])


def _scores(r, feat):
    h = feat
    if r.w1 is not None:
        h = torch.relu(feat @ r.w1.double().t() + r.b1.double())
    return h @ r.w2.double().t() + (r.b2.double() if r.b2 is not None else 0.0)


def exact(case, seed):
    kind, d = case["kind"], _draw_all(case, seed)
    if kind == "build":
        _, s, q, z = _codes(d["w"], (case["bits"], case["group"], case["symmetric"], case["clip"]))
        out = dict(blob=None, codes=None, scale=s.reshape(-1) if case["symmetric"] else s.squeeze(2))
        return out if z is None else dict(out, zero=None)
    if kind == "nlp":
        return dict(logits=_exact_nlp(case, d), expert_idx=None)
    if kind == "cv":
        return dict(logits=_exact_cv(case, d), expert_idx=None)
    fm = _FORMATS[case["formats"]]
    K, S, mats = len(fm), case["S"], _matrices(case)
    x = d["x"]
    if kind == "layer":
        # rows are in bucket order: expert e owns as many samples as chose it
        counts = torch.bincount(d["expert_idx"].long(), minlength=K).tolist()
        y, at = [], 0
        for f, c in zip(fm, counts):
            y.append(_expert(case, d["w"], f, x[at:at + c * case["T"]].double()))
            at += c * case["T"]
        return dict(y=torch.cat(y))
    if kind == "label":
        losses = torch.zeros(S, K, dtype=torch.float64, device=DEV)
        tg = d["targets"].reshape(-1).long()
        for e, f in enumerate(fm):
            y = _expert(case, d["w"], f, x.double())
            row = torch.logsumexp(y, dim=1) - y.gather(1, tg[:, None]).squeeze(1)
            losses[:, e] = row.view(S, case["T"]).mean(dim=1)
        return dict(losses=losses, labels=None)
    lens = _lengths(case) if kind == "ragged" else [case["T"]] * S
    first = [0]
    for n in lens:
        first.append(first[-1] + n)
    feat = torch.stack([x[a:b].double().mean(dim=0) for a, b in zip(first, first[1:])])
    idx = _scores(d["router"], feat).argmax(dim=1).tolist()
    y = torch.zeros(x.shape[0], mats[-1][0], dtype=torch.float64, device=DEV)
    for e, f in enumerate(fm):
        mine = [s for s in range(S) if idx[s] == e]
        if not mine:
            continue
        rows = torch.cat([torch.arange(first[s], first[s + 1], device=DEV) for s in mine])
        xe = x[rows].double()
        if case.get("shape") == "conv":
            h = case.get("h") or math.isqrt(case["T"])
            xe = xe.view(len(mine), h, case["T"] // h, case["D"])
        y[rows] = _expert(case, d["w"], f, xe)
    return dict(y=y, expert_idx=None)


def _exact_nlp(case, d):
    p = {k: v.double() for k, v in d["p"].items()}
    S, T, dm, H = case["S"], case["T"], NLP["dm"], NLP["heads"]
    dh = dm // H
    lin = lambda v, w, b: v @ p[w].t() + p[b]

    def norm(v, t):
        return torch.nn.functional.layer_norm(v, (dm,), p["ln%s_g" % t], p["ln%s_b" % t], 1e-5)

    def attention(v, t):
        out = torch.empty_like(v)
        for a in range(0, S, 32):                       # 32 sequences at a time: the scores stay small
            b = min(S, a + 32)
            q, k, u = (z.reshape(b - a, T, H, dh).transpose(1, 2).contiguous()
                       for z in lin(v[a * T:b * T], "wqkv" + t, "bqkv" + t).split(dm, dim=1))
            s = torch.matmul(q, k.transpose(2, 3).contiguous()) / math.sqrt(dh)
            o = torch.matmul(torch.softmax(s, dim=3), u)
            out[a * T:b * T] = o.transpose(1, 2).reshape(-1, dm)
        return lin(out, "wo" + t, "bo" + t)

    u = lin(d["x"].double(), "w_in", "b_in")
    v = norm(u + attention(u, "1"), "1")
    w = norm(v + torch.relu(lin(v, "w_ff1", "b_ff1")) @ p["w_ff2"].t() + p["b_ff2"], "2")
    z = norm(w + attention(w, "2"), "3")
    return _scores(d["head"], z.view(S, T, dm).mean(dim=1))


def _exact_cv(case, d):
    p = {k: v.double() for k, v in d["p"].items()}
    S, h, w = case["S"], case["h"], case["w"]

    def bn(v, pre):
        return (v - p[pre + "_m"]) / torch.sqrt(p[pre + "_v"] + 1e-5) * p[pre + "_g"] + p[pre + "_o"]

    def conv3(v, wt, stride):
        ho, wo = (v.shape[1] - 1) // stride + 1, (v.shape[2] - 1) // stride + 1
        vp = torch.nn.functional.pad(v, (0, 0, 1, 1, 1, 1))
        out = 0.0
        for t in range(9):
            i, j = t // 3, t % 3
            out = out + vp[:, i:i + stride * (ho - 1) + 1:stride, j:j + stride * (wo - 1) + 1:stride] @ wt[:, i, j].t()
        return out

    v = d["x"].double().view(S, h, w, case["c"])
    for i in range(3):
        v = torch.relu(bn(v @ p["mlp%d_w" % i].t() + p["mlp%d_b" % i], "mlp%d_bn" % i))
    for i, stride in enumerate(CV["strides"]):
        a = torch.relu(bn(conv3(v, p["st%d_a" % i], stride), "st%d_abn" % i))
        u = bn(conv3(a, p["st%d_b" % i], 1), "st%d_bbn" % i)
        z = torch.relu(u.mean(dim=(1, 2)) @ p["st%d_se1" % i].t() + p["st%d_se1b" % i])
        g = torch.sigmoid(z @ p["st%d_se2" % i].t() + p["st%d_se2b" % i])
        s = v
        if "st%d_s" % i in p:
            s = bn(v[:, ::stride, ::stride] @ p["st%d_s" % i].t(), "st%d_sbn" % i)
        v = torch.relu(u * g[:, None, None] + s)
    dm, H = CV["stages"][2], CV["heads"]
    t = v.reshape(S, -1, dm)
    q, k, u = ((t @ p["wqkv"].t() + p["bqkv"]).view(S, -1, 3, H, dm // H).permute(2, 0, 3, 1, 4).contiguous()).unbind(0)
    a = torch.softmax(torch.matmul(q, k.transpose(2, 3).contiguous()) / math.sqrt(dm // H), dim=3)
    o = torch.matmul(a, u).transpose(1, 2).reshape(S, -1, dm) @ p["wo"].t() + p["bo"]
    return o.mean(dim=1) @ p["w_out"].t() + p["b_out"]
