"""Cases that stand for the work a user of libgdy has it do: submissions of
independent GEMMs (and element-wise adds) run under the dynamic selector.

A case is a dict of plain values.  "set" lists the submission's members,
"MxNxK:layout" separated by commas; layout nn, nt, tn or tt names the
transposes of A and B, "add" an element-wise add over M x N.  "batch" > 1
makes every member a strided batch of that many items, "pad" widens every
row pitch by that many elements, "dtype" is the input type.
"""
import functools
import math
import os

import torch

from paper_2409_02227_amd import gdy

TORCH = {"bf16": torch.bfloat16, "f16": torch.float16, "fp8": torch.float8_e4m3fn, "f32": torch.float32}
OUT = {"bf16": torch.bfloat16, "f16": torch.float16, "fp8": torch.bfloat16, "f32": torch.float32}
SIZE = {"bf16": 2, "f16": 2, "fp8": 1, "f32": 4}
OUT_SIZE = {"bf16": 2, "f16": 2, "fp8": 2, "f32": 4}

# One GPU's share of an 8-way tensor-sliced transformer layer, hidden size
# 12288, 512 tokens: QKV, out-projection, FFN up and down.
LAYER = "512x4608x12288:nn,512x12288x1536:nn,512x6144x12288:nn,512x12288x6144:nn"

# Two tenants' inference requests of different batch sizes, interleaved.
TENANTS = ",".join("%dx%dx%d:nn" % (m, nk, nk) for m, nk in (
    (256, 4096), (1, 8192), (2048, 8192), (32, 4096), (1, 4096), (256, 8192), (32, 8192), (2048, 4096),
    (2048, 4096), (32, 8192), (1, 8192), (256, 8192), (32, 4096), (2048, 8192), (1, 4096), (256, 4096)) * 2)


def case(name, dtype, members, batch=0, pad=0):
    return {"name": name, "dtype": dtype, "set": members, "batch": batch, "pad": pad}


def listed():
    return [
        # two tiny GEMMs: what a call costs when there is next to nothing to compute
        case("pair_256_f16", "f16", "256x256x256:nn,256x256x256:nn"),
        # the four gate projections of one LSTM step at batch 64 (decode, weights read once)
        case("lstm_gates_bf16", "bf16", ",".join(["64x4096x1024:nn"] * 4)),
        # a transformer layer's share for two independent microbatches (prefill, training forward)
        case("layer_share_bf16", "bf16", LAYER + "," + LAYER),
        # the same in full precision
        case("layer_share_f32", "f32", LAYER + "," + LAYER),
        # backward of two linear layers with K x N weights, 2048 tokens:
        # input gradients dY W^T (nt) and weight gradients X^T dY (tn)
        case("linear_backward_bf16", "bf16", ",".join(["2048x4096x4096:nt", "4096x4096x2048:tn"] * 2)),
        # two fp8 tenants, decode to prefill batch sizes in one submission
        case("two_tenant_fp8", "fp8", TENANTS),
        # a submission of unrelated bf16 GEMMs with token counts as they come
        case("heterogeneous_bf16", "bf16",
             "1913x2048x1024:nn,37x8192x4096:nn,402x1024x8192:nn,96x4096x2048:nn,731x4096x4096:nn,"
             "18x1024x1024:nn,2660x1024x2048:nn,155x8192x1024:nn,59x2048x8192:nn"),
        # attention scores Q K^T of four sequence-length buckets, 16 heads x 4 sequences, head size 64
        case("attention_scores_bf16", "bf16", "128x128x64:nt,256x256x64:nt,384x384x64:nt,512x512x64:nt", batch=64),
        # a memory-bound GEMM and the element-wise add of another branch
        case("gemm_and_add_bf16", "bf16", "8192x1024x512:nn,8192x1024x0:add"),
        # sizes that no tile divides, rows still 16-byte aligned
        case("ragged_bf16", "bf16", "377x1000x2040:nn,1290x3000x1000:nt,83x2504x5000:nn,645x1112x3080:nt"),
        # odd sizes, rows packed without any alignment
        case("odd_f16", "f16", "509x2047x1021:nn,1023x1025x777:nt,65x3001x2999:nn"),
        # one square GEMM alone, weight stored N x K as linear layers keep it
        case("single_4096_bf16", "bf16", "4096x4096x4096:nt"),
    ]


def spread(rng, lo, hi, step):
    """A size between lo and hi, even over its logarithm, on multiples of step."""
    x = math.exp(rng.uniform(math.log(lo), math.log(hi)))
    return max(int(round(x / step)) * step, step, lo if step == 1 else 0)


def draw(rng):
    kind = rng.choice(["concurrent", "concurrent", "skinny", "fp8", "backward", "attention", "add", "odd", "single",
                       "full"])
    pad = rng.choice([0, 0, 0, 16])
    if kind == "attention":
        sls = [spread(rng, 64, 512, rng.choice([64, 8])) for _ in range(rng.randint(1, 6))]
        head = rng.choice([64, 128])
        return case(None, rng.choice(["bf16", "f16"]), ",".join("%dx%dx%d:nt" % (s, s, head) for s in sls),
                    rng.choice([8, 16, 32, 64]), pad)
    if kind == "add":
        m, n, k = spread(rng, 1024, 16384, 1), spread(rng, 512, 4096, 64), spread(rng, 512, 4096, 64)
        return case(None, rng.choice(["bf16", "f16"]), "%dx%dx%d:nn,%dx%dx0:add" % (m, n, k, m, n), 0, pad)
    dtype = {"fp8": "fp8", "full": "f32"}.get(kind) or rng.choice(["bf16", "bf16", "f16"])
    layouts = {"backward": ["nt", "tn"], "odd": ["nn", "nt", "tn"]}.get(kind, ["nn", "nt"])
    count = 1 if kind == "single" else rng.randint(2, 16)
    top = {"skinny": 64, "odd": 1500, "single": 8192}.get(kind, 4096)
    large = 4096 if kind == "odd" else 8192
    step = {"odd": 1, "concurrent": rng.choice([128, 64, 8])}.get(kind, rng.choice([64, 256]))
    budget = {"fp8": 1.4e12, "f32": 3e11}.get(dtype, 4e11) / (4 if kind == "odd" else 1)
    members = []
    for _ in range(count):
        m = spread(rng, 1 if kind == "skinny" else 16, top, 1)
        n, k = spread(rng, 512, large, step), spread(rng, 512, large, step)
        lay = rng.choice(layouts)
        if lay == "tn":  # A is stored K x M: its row pitch is M
            m = max(m // 16, 1) * 16 if step > 1 else m
        flops = 2.0 * m * n * k
        if flops > budget:
            continue
        budget -= flops
        members.append("%dx%dx%d:%s" % (m, n, k, lay))
    return case(None, dtype, ",".join(members or ["512x1024x1024:nn"]), 0, 0 if kind == "odd" else pad)


def members(c):
    """(m, n, k, layout) of each member."""
    out = []
    for text in c["set"].split(","):
        size, lay = text.split(":")
        out.append(tuple(int(x) for x in size.split("x")) + (lay,))
    return out


@functools.lru_cache(maxsize=1)
def context():
    """The handle a program creates once and keeps."""
    table = os.path.join(os.path.dirname(os.path.abspath(gdy.__file__)), "tables", "gfx950.table")
    return gdy.Context(0, table=table)


def operand(gen, c, rows, cols, weight):
    """(matrix, scale): rows x cols (of every batch item) with padded rows.
    Activations are uniform in [-1, 1], weights normal with deviation 0.02;
    fp8 tensors are uniform with a scale of their own."""
    shape = (c["batch"], rows, cols + c["pad"]) if c["batch"] else (rows, cols + c["pad"])
    scale = 1.0
    if c["dtype"] == "fp8":
        amax = 2.0 ** float(torch.rand((), generator=gen, device="cuda") * 8 - 4)
        scale = float(torch.tensor(amax / 448.0, dtype=torch.float32))
        x = (torch.rand(shape, generator=gen, device="cuda") * 2 - 1) * 448.0
    elif weight:
        x = torch.randn(shape, generator=gen, device="cuda") * 0.02
    else:
        x = torch.rand(shape, generator=gen, device="cuda") * 2 - 1
    return x.to(TORCH[c["dtype"]])[..., :cols], scale


def inputs(c, seed):
    """Operands of every member, from the seed alone."""
    gen = torch.Generator(device="cuda").manual_seed(seed)
    out = []
    for m, n, k, lay in members(c):
        if lay == "add":
            (a, sa), (b, sb) = operand(gen, c, m, n, False), operand(gen, c, m, n, False)
        else:
            activations = c["batch"] > 1  # attention multiplies two activations
            a, sa = operand(gen, c, *((k, m) if lay[0] == "t" else (m, k)), False)
            b, sb = operand(gen, c, *((n, k) if lay[1] == "t" else (k, n)), not activations and lay != "tn")
        out.append((a, b, sa, sb))
    return out


def prepare(c, seed):
    subs = []
    for (m, n, k, lay), (a, b, sa, sb) in zip(members(c), inputs(c, seed)):
        shape = (c["batch"], m, n + c["pad"]) if c["batch"] else (m, n + c["pad"])
        out = torch.empty(shape, dtype=OUT[c["dtype"]], device="cuda")[..., :n]
        if lay == "add":
            subs.append(gdy.Add(a, b, out))
        else:
            subs.append(gdy.Gemm(a, b, out, int(lay[0] == "t"), int(lay[1] == "t"), sa, sb))
    stream = gdy.ctypes.c_void_p(torch.cuda.current_stream().cuda_stream)
    return {"ctx": context(), "subs": subs, "descs": gdy.descs(subs), "stream": stream, "out": [s.c for s in subs]}


def run(state):
    state["ctx"].execute_descs(state["descs"], len(state["subs"]), gdy.SELECTOR, 0, state["stream"])
    return state["out"]


def work(c):
    es, os_ = SIZE[c["dtype"]], OUT_SIZE[c["dtype"]]
    items = max(c["batch"], 1)
    total, flops = 0, 0
    for m, n, k, lay in members(c):
        if lay == "add":
            total += 3 * m * n * es * items
            flops += m * n * items
        else:
            total += ((m * k + k * n) * es + m * n * os_) * items
            flops += 2 * m * n * k * items
    return {"bytes": total, "flops": flops}


def tolerance(c):
    """Rounding of the output type: bf16 keeps 8 bits, fp16 11; fp32 results
    carry the error of an fp32 sum of up to 12288 products."""
    return {"bf16": {"rel": 7e-3, "max": 2e-2}, "fp8": {"rel": 7e-3, "max": 2e-2}, "f16": {"rel": 1e-3, "max": 3e-3},
            "f32": {"rel": 1e-5, "max": 1e-4}}[c["dtype"]]


def exact(c, seed):
    out = []
    for (m, n, k, lay), (a, b, sa, sb) in zip(members(c), inputs(c, seed)):
        a, b = a.double(), b.double()
        if lay == "add":
            out.append(a + b)
            continue
        a = a.transpose(-1, -2).contiguous() if lay[0] == "t" else a.contiguous()
        b = b.transpose(-1, -2).contiguous() if lay[1] == "t" else b.contiguous()
        if c["batch"]:
            out.append(torch.stack([torch.mm(x, y) for x, y in zip(a, b)]))
        else:
            out.append(torch.mm(a, b) * (sa * sb))
    return out
