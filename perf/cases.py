"""What is timed: the calls that a program using this library makes, over the range of shapes it makes them with.

A shape is known only when the call is made, so every pass over a plain operator looks its plan up
(ft_plan_cached) and launches it, as a serving loop does.  The operators, their uKernel sets, the
weights and the output buffers are what such a program keeps; the plan of a ragged batch is made
once per batch and launched by every layer, so it belongs to what is in hand too.

Kinds of cases
  dense    one Matmul: M tokens against a weight [K, N]
  encoder  the dense layers of a BERT-base encoder, chained: four Matmuls per layer with fused bias
           and 16-bit outputs, each layer with weights of its own
  attn     scores Q K^T and context P V of one batch of equally long sequences (batched Matmuls)
  ragged   the same two products for sequences of different lengths, one grouped launch each
  conv     3x3 NHWC Conv2d of one batch of images
"""
import math
import random

import torch

import paper_2407_21418_amd as ft

HEADS, DHEAD, MAX_LEN = 12, 64, 512
HIDDEN, FFN = 768, 3072
ENCODER_GEMMS = (("qkv", 3 * HIDDEN, HIDDEN), ("o", HIDDEN, HIDDEN), ("ffn1", FFN, HIDDEN), ("ffn2", HIDDEN, FFN))  # name, N, K
BERT_LAYERS = ((768, 768), (768, 3072), (3072, 768))  # (K, N)
LLM_K, LLM_N = 4096, (4096, 11008)
CONV_C_IN, CONV_C_OUT, CONV_TAPS = 64, 128, 3
MAX_TOKENS = 8192
MAX_SEQS = 64


def listed():
    return [
        # one short sentence through one 768-wide layer: the smallest call, an odd row count
        dict(name="dense 77x768x768", kind="dense", m=77, k=768, n=768, dtype="f16", out="f32"),
        # 16 sentences of 17 tokens down the feed-forward layer: few tiles, a long reduce axis
        dict(name="dense 272x768x3072", kind="dense", m=272, k=3072, n=768, dtype="f16", out="f32"),
        # 16 sentences of 128 tokens up the feed-forward layer: the largest of the BERT sweep
        dict(name="dense 2048x3072x768", kind="dense", m=2048, k=768, n=3072, dtype="f16", out="f32"),
        # 16 sentences of 43 tokens through all dense layers of an encoder
        dict(name="encoder 12x688", kind="encoder", m=688, layers=12, dtype="f16"),
        # a decode step of a few requests: bound by reading the weight once
        dict(name="decode 7x11008x4096", kind="dense", m=7, k=4096, n=11008, dtype="bf16", out="same"),
        # a decode step of many requests together with a short prompt
        dict(name="mixed 403x4096x4096", kind="dense", m=403, k=4096, n=4096, dtype="bf16", out="f32"),
        # prefill of a long prompt: the largest matrix product
        dict(name="prefill 8192x11008x4096", kind="dense", m=8192, k=4096, n=11008, dtype="bf16", out="same"),
        # attention of a small batch at an odd length
        dict(name="attention 8x131", kind="attn", batch=8, length=131, dtype="f16", out="f32", k_layout="kn"),
        # attention of a full batch at full length, keys stored as the projection leaves them
        dict(name="attention 64x512", kind="attn", batch=64, length=512, dtype="f16", out="f32", k_layout="nk"),
        # attention of a full batch of sentences of their own lengths
        dict(name="ragged attention 64", kind="ragged", seqs=64, lengths=1, dtype="f16", out="f32", k_layout="nk"),
        # an inner layer of a convolutional network
        dict(name="conv 8x56x56", kind="conv", images=8, size=56, dtype="f16", out="f32"),
        # the same layer on a full-size image
        dict(name="conv 8x224x224", kind="conv", images=8, size=224, dtype="f16", out="f32"),
    ]


def _log_int(rng, lo, hi):
    return min(hi, max(lo, int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))))


def draw(rng):
    kind = rng.choice(("dense", "dense", "llm", "llm", "encoder", "attn", "ragged", "conv"))
    if kind == "dense":  # the BERT layers at any row count
        k, n = rng.choice(BERT_LAYERS)
        return dict(kind="dense", m=_log_int(rng, 1, 2048), k=k, n=n, dtype=rng.choice(("f16", "bf16")), out=rng.choice(("f32", "same")))
    if kind == "llm":  # decode to prefill
        m = _log_int(rng, 1, MAX_TOKENS)
        return dict(kind="dense", m=m, k=LLM_K, n=rng.choice(LLM_N), dtype=rng.choice(("bf16", "bf16", "f16")),
                    out=rng.choice(("f32", "same")) if m <= MAX_TOKENS // 2 else "same")
    if kind == "encoder":
        return dict(kind="encoder", m=16 * rng.randint(1, 128), layers=12, dtype=rng.choice(("f16", "bf16")))
    if kind == "attn":
        return dict(kind="attn", batch=rng.choice((1, 8, 32, 64)), length=_log_int(rng, 8, MAX_LEN), dtype="f16", out=rng.choice(("f32", "f32", "same")),
                    k_layout=rng.choice(("kn", "nk")))
    if kind == "ragged":
        return dict(kind="ragged", seqs=_log_int(rng, 4, MAX_SEQS), lengths=rng.randint(2, 1 << 20), dtype="f16", out="f32", k_layout=rng.choice(("kn", "nk")))
    return dict(kind="conv", images=8, size=_log_int(rng, 28, 224), dtype=rng.choice(("f16", "f16", "bf16")), out=rng.choice(("f32", "f32", "same")))


def _lengths(case):
    r = random.Random(case["lengths"])
    return [r.randint(1, MAX_LEN) for _ in range(case["seqs"])]


# ---- what a program keeps: registered operators and their uKernel sets ---------------------------


def _operator(case, **desc):
    op = ft.ft_op_register(ft.ft_op_desc(dtype=ft.FT_F16 if case["dtype"] == "f16" else ft.FT_BF16,
                                         out_dtype=ft.FT_OUT_SAME if case.get("out", "same") == "same" else ft.FT_OUT_F32, **desc))
    return op, ft.ft_ukernels_derive(op, ft.ft_hw_query(torch.cuda.current_device()))


def _scores_operator(case):
    return _operator(case, kind=ft.FT_OP_BMM, k=DHEAD, m_lo=0, m_hi=MAX_LEN, n_lo=0, n_hi=MAX_LEN, batch_hi=MAX_SEQS * HEADS,
                     b_layout=ft.FT_B_NK if case["k_layout"] == "nk" else ft.FT_B_KN)


def _context_operator(case):
    return _operator(case, kind=ft.FT_OP_BMM, n=DHEAD, m_lo=0, m_hi=MAX_LEN, k_lo=0, k_hi=MAX_LEN, batch_hi=MAX_SEQS * HEADS)


class _Inputs:
    """Seeded values of a case's type on the GPU."""

    def __init__(self, case, seed):
        self.gen = torch.Generator(device="cuda").manual_seed(seed)
        self.dtype = torch.float16 if case["dtype"] == "f16" else torch.bfloat16
        self.out = torch.float32 if case.get("out", "same") == "f32" else self.dtype

    def normal(self, *shape, std=1.0):
        return torch.randn(shape, generator=self.gen, device="cuda", dtype=torch.float32).mul_(std).to(self.dtype)

    def probabilities(self, *shape):  # rows as a softmax leaves them
        return torch.softmax(torch.randn(shape, generator=self.gen, device="cuda", dtype=torch.float32), dim=-1).to(self.dtype)

    def output(self, *shape):
        return torch.empty(shape, dtype=self.out, device="cuda")


def prepare(case, seed):
    x = _Inputs(case, seed)
    kind = case["kind"]
    s = dict(kind=kind, stream=torch.cuda.current_stream().cuda_stream)
    if kind == "dense":
        m, n, k = case["m"], case["n"], case["k"]
        s["op"], s["set"] = _operator(case, kind=ft.FT_OP_MATMUL, n=n, k=k, m_lo=1, m_hi=MAX_TOKENS)
        s["m"], s["a"], s["b"], s["c"] = m, x.normal(m, k), x.normal(k, n, std=0.02), x.output(m, n)
        ft.ft_plan_cached(s["op"], s["set"], ft.ft_shape(m=m))
    elif kind == "encoder":
        m = case["m"]
        s["m"] = m
        s["ops"] = {name: _operator(case, kind=ft.FT_OP_MATMUL, n=n, k=k, m_lo=1, m_hi=MAX_TOKENS, epilogue=ft.FT_EPI_BIAS) for name, n, k in ENCODER_GEMMS}
        s["weights"] = [{name: x.normal(k, n, std=0.02) for name, n, k in ENCODER_GEMMS} for _ in range(case["layers"])]
        s["bias"] = [{name: torch.randn(n, generator=x.gen, device="cuda").mul_(0.02) for name, n, _ in ENCODER_GEMMS} for _ in range(case["layers"])]
        s["x"], s["context"] = x.normal(m, HIDDEN), x.normal(m, HIDDEN)
        s["qkv"], s["o"], s["h"] = x.output(m, 3 * HIDDEN), x.output(m, HIDDEN), x.output(m, FFN)
        s["y"] = [x.output(m, HIDDEN), x.output(m, HIDDEN)]
        for op, uks in s["ops"].values():
            ft.ft_plan_cached(op, uks, ft.ft_shape(m=m))
    elif kind == "attn":
        b, length = case["batch"] * HEADS, case["length"]
        s["scores_op"], s["context_op"] = _scores_operator(case), _context_operator(case)
        s["b"], s["length"] = b, length
        s["q"], s["v"] = x.normal(b, length, DHEAD), x.normal(b, length, DHEAD)
        s["k"] = x.normal(b, length, DHEAD) if case["k_layout"] == "nk" else x.normal(b, DHEAD, length)
        s["p"] = x.probabilities(b, length, length)
        s["scores"], s["context"] = x.output(b, length, length), x.output(b, length, DHEAD)
        ft.ft_plan_cached(*s["scores_op"], ft.ft_shape(batch=b, m=length, n=length))
        ft.ft_plan_cached(*s["context_op"], ft.ft_shape(batch=b, m=length, k=length))
    elif kind == "ragged":
        lengths = _lengths(case)
        s["scores_op"], s["context_op"] = _scores_operator(case), _context_operator(case)
        s["scores_plan"] = ft.ft_plan_create_grouped(*s["scores_op"], [ft.ft_shape(batch=HEADS, m=n, n=n) for n in lengths])
        s["context_plan"] = ft.ft_plan_create_grouped(*s["context_op"], [ft.ft_shape(batch=HEADS, m=n, k=n) for n in lengths])
        tokens, pairs = HEADS * sum(lengths), HEADS * sum(n * n for n in lengths)
        s["q"], s["k"], s["v"] = x.normal(tokens * DHEAD), x.normal(tokens * DHEAD), x.normal(tokens * DHEAD)
        s["p"] = torch.cat([x.probabilities(HEADS, n, n).reshape(-1) for n in lengths])
        s["scores"], s["context"] = x.output(pairs), x.output(tokens * DHEAD)
    else:
        n, size = case["images"], case["size"]
        s["op"], s["set"] = _operator(case, kind=ft.FT_OP_CONV2D, c_in=CONV_C_IN, c_out=CONV_C_OUT, r=CONV_TAPS, s=CONV_TAPS, stride=1, pad=1, m_lo=1, m_hi=1 << 22)
        s["images"], s["size"] = n, size
        s["x"] = x.normal(n, size, size, CONV_C_IN)
        s["w"] = x.normal(CONV_TAPS, CONV_TAPS, CONV_C_IN, CONV_C_OUT, std=(CONV_TAPS * CONV_TAPS * CONV_C_IN) ** -0.5)
        s["y"] = x.output(n, size, size, CONV_C_OUT)
        ft.ft_plan_cached(s["op"], s["set"], ft.ft_shape(img_n=n, img_h=size, img_w=size))
    return s


def run(s):
    kind, stream = s["kind"], s["stream"]
    if kind == "dense":
        plan = ft.ft_plan_cached(s["op"], s["set"], ft.ft_shape(m=s["m"]))
        ft.ft_launch(plan, s["a"].data_ptr(), s["b"].data_ptr(), s["c"].data_ptr(), stream)
        return s["c"]
    if kind == "encoder":
        src, m, ops = s["x"], s["m"], s["ops"]
        for layer, (w, bias) in enumerate(zip(s["weights"], s["bias"])):
            dst = s["y"][layer % 2]
            for name, a, c in (("qkv", src, s["qkv"]), ("o", s["context"], s["o"]), ("ffn1", s["o"], s["h"]), ("ffn2", s["h"], dst)):
                op, uks = ops[name]
                plan = ft.ft_plan_cached(op, uks, ft.ft_shape(m=m))
                ft.ft_launch_epilogue(plan, a.data_ptr(), w[name].data_ptr(), c.data_ptr(), bias[name].data_ptr(), stream)
            src = dst
        return s["qkv"], s["o"], s["h"], *s["y"]
    if kind == "attn":
        b, length = s["b"], s["length"]
        plan = ft.ft_plan_cached(*s["scores_op"], ft.ft_shape(batch=b, m=length, n=length))
        ft.ft_launch(plan, s["q"].data_ptr(), s["k"].data_ptr(), s["scores"].data_ptr(), stream)
        plan = ft.ft_plan_cached(*s["context_op"], ft.ft_shape(batch=b, m=length, k=length))
        ft.ft_launch(plan, s["p"].data_ptr(), s["v"].data_ptr(), s["context"].data_ptr(), stream)
        return s["scores"], s["context"]
    if kind == "ragged":
        ft.ft_launch(s["scores_plan"], s["q"].data_ptr(), s["k"].data_ptr(), s["scores"].data_ptr(), stream)
        ft.ft_launch(s["context_plan"], s["p"].data_ptr(), s["v"].data_ptr(), s["context"].data_ptr(), stream)
        return s["scores"], s["context"]
    plan = ft.ft_plan_cached(s["op"], s["set"], ft.ft_shape(img_n=s["images"], img_h=s["size"], img_w=s["size"]))
    ft.ft_launch(plan, s["x"].data_ptr(), s["w"].data_ptr(), s["y"].data_ptr(), stream)
    return s["y"]


def _product(batch, m, n, k, out_bytes):
    return batch * (2 * (m * k + k * n) + out_bytes * m * n), 2 * batch * m * n * k


def work(case):
    """Every operand of every launch read once and every result written once."""
    kind = case["kind"]
    ob = 4 if case.get("out", "same") == "f32" else 2
    if kind == "dense":
        parts = [_product(1, case["m"], case["n"], case["k"], ob)]
    elif kind == "encoder":
        parts = [_product(1, case["m"], n, k, ob) for _, n, k in ENCODER_GEMMS] + [(4 * n, 0) for _, n, _ in ENCODER_GEMMS]
        parts *= case["layers"]
    elif kind in ("attn", "ragged"):
        lengths = [case["length"]] * case["batch"] if kind == "attn" else _lengths(case)
        parts = [p for n in lengths for p in (_product(HEADS, n, n, DHEAD, ob), _product(HEADS, n, DHEAD, n, ob))]
    else:
        pixels = case["images"] * case["size"] ** 2
        taps = CONV_TAPS * CONV_TAPS * CONV_C_IN
        parts = [(2 * (pixels * CONV_C_IN + taps * CONV_C_OUT) + ob * pixels * CONV_C_OUT, 2 * pixels * taps * CONV_C_OUT)]
    return {"bytes": sum(p[0] for p in parts), "flops": sum(p[1] for p in parts)}


def tolerance(case):
    """Sums are kept in fp32 (any order); 16-bit outputs are rounded once, and those of an encoder are the next
    Matmul's inputs (three roundings in a row reach a layer's output)."""
    if case.get("out", "same") == "f32":
        return {"rel": 1e-5}
    return {"rel": 2e-3 if case["dtype"] == "f16" else 1e-2}
