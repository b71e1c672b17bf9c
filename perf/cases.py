"""The cases this framework's speed is measured on: operator mixes of several inference streams, each run as one
plan through the C ABI's Python binding.

A case is a mix of operators ("mix", with its sizes), how many streams run it ("tenants") or how many operators it
has ("count"), the element type, a number that fixes the shapes ("shapes") and the call that runs it ("via"):

  launch   sk_launch of a device-resident plan, the ordinary case
  static   sk_launch_static of a host-only plan, for programs that cannot allocate
  queue    sk_queue_submit / sk_queue_poll: a burst of requests is planned, launched and waited for

All outputs of a plan lie in one buffer per element type, as a serving program's output arena would; `run` returns
these buffers.
"""
from __future__ import annotations

import ctypes
import math
import random
from dataclasses import dataclass

import torch

import paper_1901_10008_amd as sk

ES = {"f32": 4, "bf16": 2, "f16": 2}
TORCH = {"f32": torch.float32, "bf16": torch.bfloat16, "f16": torch.float16}


@dataclass
class Operator:
    op: str  # gemm: C[M,N] = A[M,K] . B[N,K]^T; conv, conv_nchw: image layout of a convolution
    dtype: str
    M: int = 0
    N: int = 0
    K: int = 0
    Nb: int = 0
    H: int = 0
    W: int = 0
    Cin: int = 0
    Cout: int = 0
    R: int = 0
    S: int = 0
    pad_h: int = 0
    pad_w: int = 0
    stride: int = 1
    deadline_ms: float = math.inf
    lda: int = 0  # row strides of a GEMM in elements, 0: packed
    ldb: int = 0
    ldc: int = 0

    def out_hw(self):
        return (self.H + 2 * self.pad_h - self.R) // self.stride + 1, (self.W + 2 * self.pad_w - self.S) // self.stride + 1

    def a_elems(self):
        return self.M * (self.lda or self.K) if self.op == "gemm" else self.Nb * self.H * self.W * self.Cin

    def b_elems(self):
        return self.N * (self.ldb or self.K) if self.op == "gemm" else self.Cout * self.R * self.S * self.Cin

    def c_elems(self):
        if self.op == "gemm":
            return self.M * (self.ldc or self.N)
        ho, wo = self.out_hw()
        return self.Nb * ho * wo * self.Cout


def _gemm(dtype, m, n, k, **more):
    return Operator("gemm", dtype, M=m, N=n, K=k, **more)


def _conv(dtype, hw, cin, cout, r, stride=1, pad=None, op="conv", nb=1, **more):
    p = (r - 1) // 2 if pad is None else pad
    return Operator(op, dtype, Nb=nb, H=hw, W=hw, Cin=cin, Cout=cout, R=r, S=r, pad_h=p, pad_w=p, stride=stride, **more)


# ---- the mixes --------------------------------------------------------------------------------------------

RESNET = [(56, 64, 256, 1), (56, 64, 64, 3), (28, 128, 512, 1), (28, 128, 128, 3),
          (14, 256, 1024, 1), (14, 256, 256, 3), (7, 512, 2048, 1), (7, 512, 512, 3)]
STRIDE2 = [(224, 3, 64, 7, 3), (56, 128, 128, 3, 1), (56, 256, 512, 1, 0), (28, 256, 256, 3, 1),
           (28, 512, 1024, 1, 0), (14, 512, 512, 3, 1), (14, 1024, 2048, 1, 0)]
BERT = [(768, 768), (768, 768), (768, 768), (768, 3072), (3072, 768)]  # (K, N)


def _log_uniform(r, lo, hi):
    return max(lo, min(hi, int(math.exp(r.uniform(math.log(lo), math.log(hi + 1))))))


def _mixed_operator(r, dtype):
    """One request of the main workload: a low-batch GEMM or a convolution, with a latency budget."""
    deadline = r.uniform(0.5, 5.0)
    if r.random() < 0.6:
        m = _log_uniform(r, 1, 64)
        return _gemm(dtype, m, 256 * r.randint(1, 32), 256 * r.randint(1, 32), deadline_ms=deadline)
    return _conv(dtype, r.choice([7, 14, 28, 56]), r.choice([64, 128, 256, 512]), r.choice([64, 128, 256, 512]),
                 r.choice([1, 3]), deadline_ms=deadline)


def _ragged_operator(r, dtype):
    """Sizes as they come: class heads, odd feature counts, images with few channels, padded rows."""
    kind = r.random()
    if kind < 0.35:  # a linear layer with odd sizes
        return _gemm(dtype, _log_uniform(r, 1, 300), _log_uniform(r, 33, 1500), _log_uniform(r, 31, 2000))
    if kind < 0.6:  # even sizes in padded rows
        k, n = 8 * _log_uniform(r, 8, 250), 8 * _log_uniform(r, 8, 190)
        return _gemm(dtype, _log_uniform(r, 1, 300), n, k, lda=k + 8 * r.randint(0, 4), ldb=k + 8 * r.randint(0, 4),
                     ldc=n + r.randint(0, 9))
    if kind < 0.8:  # a stem: an RGB image
        return _conv(dtype, r.randint(24, 112), 3, r.choice([32, 48, 64]), r.choice([3, 5, 7]), stride=r.choice([1, 2]))
    # a convolution with channel counts outside the powers of two
    return _conv(dtype, r.randint(7, 40), r.randint(9, 200), r.randint(9, 200), r.choice([1, 3]), stride=r.choice([1, 2]))


def operators(case):
    r = random.Random(case["shapes"])
    mix, dtype, n = case["mix"], case["dtype"], case.get("tenants", 1)
    if mix == "fp32_gemm":
        shapes = [(1, 256, 256), (4, 256, 512), (8, 512, 256), (2, 128, 384)]
        return [_gemm(dtype, *s) for _ in range(n) for s in shapes]
    if mix == "lowbatch":
        step, hi = case["step"], 4096 // case["step"]
        return [_gemm(dtype, r.choice([1, 2, 4, 8, 16, 32]), step * _log_uniform(r, max(1, 512 // step), hi),
                      step * _log_uniform(r, max(1, 512 // step), hi)) for _ in range(case["count"])]
    if mix == "resnet":
        op = "conv_nchw" if case["channel_major"] else "conv"
        return [_conv(dtype, hw, ci, co, f, op=op, nb=case["batch"]) for _ in range(n) for hw, ci, co, f in RESNET]
    if mix == "stride2":
        return [_conv(dtype, hw, ci, co, f, stride=2, pad=p) for _ in range(n) for hw, ci, co, f, p in STRIDE2]
    if mix == "conv3x3":
        return [_conv(dtype, case["hw"], case["channels"], case["channels"], 3) for _ in range(n)]
    if mix == "bert":
        out = []
        for _ in range(32 * n):
            k, nn = r.choice(BERT)
            out.append(_gemm(dtype, r.randint(1, 128), nn, k))
        return out
    if mix == "lstm":
        hidden = [r.choice([256, 512, 1024, 2048]) for _ in range(case["count"])]
        return [_gemm(dtype, 1, 4 * h, 2 * h) for h in hidden]
    if mix == "square":
        return [_gemm(dtype, case["size"], case["size"], case["size"]) for _ in range(n)]
    if mix == "mixed":
        return [_mixed_operator(r, dtype) for _ in range(case["count"])]
    if mix == "ragged":
        types = [dtype] if dtype != "mixed" else ["bf16", "f16", "f32"]
        return [_ragged_operator(r, types[i % len(types)]) for i in range(case["count"])]
    raise ValueError(mix)


def listed():
    return [
        # Four small fp32 layers in one launch, the smallest call there is: what counts is the launch itself.
        {"name": "fp32_gemm4", "mix": "fp32_gemm", "tenants": 1, "dtype": "f32", "shapes": 1, "via": "launch"},
        # Sixteen low-batch linear layers of different models, one decode step of each: a short weight-streaming launch.
        {"name": "lowbatch16", "mix": "lowbatch", "count": 16, "step": 512, "dtype": "bf16", "shapes": 2, "via": "launch"},
        # The eight distinct convolutions of a 50-layer residual network at batch 1, for sixteen tenants.
        {"name": "resnet_x16", "mix": "resnet", "tenants": 16, "batch": 1, "channel_major": False, "dtype": "bf16", "shapes": 3,
         "via": "launch"},
        # The same layers handed over in the other storage order that frameworks use.
        {"name": "resnet_nchw_x8", "mix": "resnet", "tenants": 8, "batch": 1, "channel_major": True, "dtype": "f16", "shapes": 3,
         "via": "launch"},
        # The down-sampling layers with the 7x7 stem on an RGB image, for sixteen tenants.
        {"name": "stride2_x16", "mix": "stride2", "tenants": 16, "dtype": "bf16", "shapes": 4, "via": "launch"},
        # One 3x3 layer (64 channels on 56x56) of 32 tenants, the experiment of the paper's Section 5.3, sixteen requests each.
        {"name": "conv2_2_x512", "mix": "conv3x3", "hw": 56, "channels": 64, "tenants": 512, "dtype": "bf16", "shapes": 5,
         "via": "launch"},
        # Linear layers of a BERT-base encoder at sequence lengths 1 to 128, for eight tenants: tile and streaming classes mixed.
        {"name": "bert_x8", "mix": "bert", "tenants": 8, "dtype": "bf16", "shapes": 6, "via": "launch"},
        # LSTM cells at batch 1 (fp16 matrix-vector products), the paper's second workload: pure weight streaming.
        {"name": "lstm64", "mix": "lstm", "count": 64, "dtype": "f16", "shapes": 7, "via": "launch"},
        # Sixteen square GEMMs: bound by the matrix cores.
        {"name": "square16", "mix": "square", "size": 2048, "tenants": 16, "dtype": "bf16", "shapes": 8, "via": "launch"},
        # The main workload: 256 mixed operators with latency budgets, 60 % low-batch GEMMs, 40 % convolutions, about 5 GB.
        {"name": "mixed256", "mix": "mixed", "count": 256, "dtype": "bf16", "shapes": 9, "via": "launch"},
        # Odd sizes, padded rows, RGB stems and three element types in one plan.
        {"name": "ragged96", "mix": "ragged", "count": 96, "dtype": "mixed", "shapes": 10, "via": "launch"},
        # A burst of requests through the arrival queue: planning, upload, launch and completion are all part of it.
        {"name": "queue24", "mix": "mixed", "count": 24, "dtype": "bf16", "shapes": 11, "via": "queue"},
    ]


def draw(rng):
    mix = rng.choice(["fp32_gemm", "lowbatch", "resnet", "resnet", "stride2", "conv3x3", "bert", "lstm", "square", "mixed", "ragged",
                      "ragged", "queue"])
    half = rng.choice(["bf16", "f16"])
    case = {"mix": mix, "dtype": half, "shapes": rng.randrange(1 << 30), "via": "launch"}
    if mix == "fp32_gemm":
        case.update(dtype="f32", tenants=_log_uniform(rng, 1, 64), via=rng.choice(["launch", "static"]))
    elif mix == "lowbatch":
        case.update(count=_log_uniform(rng, 1, 128), step=rng.choice([8, 64, 512]))
    elif mix == "resnet":
        case.update(tenants=_log_uniform(rng, 1, 16), batch=rng.choice([1, 1, 2, 3]), channel_major=rng.random() < 0.5,
                    dtype=rng.choice([half, half, "f32"]))
        if case["batch"] > 1:
            case["tenants"] = min(case["tenants"], 6)
    elif mix == "stride2":
        case.update(tenants=_log_uniform(rng, 1, 16))
    elif mix == "conv3x3":
        # as much work as the listed case at most
        hw, c = rng.randint(7, 56), rng.choice([64, 128, 192, 256])
        most = 512 * (56 * 56 * 64 * 64) // (hw * hw * c * c)
        case.update(hw=hw, channels=c, tenants=_log_uniform(rng, 1, max(1, min(512, most))))
    elif mix == "bert":
        case.update(tenants=_log_uniform(rng, 1, 16), dtype=rng.choice([half, half, "f32"]))
    elif mix == "lstm":
        case.update(count=_log_uniform(rng, 8, 256))
    elif mix == "square":
        size = _log_uniform(rng, 384, 4096) // 8 * 8
        case.update(size=size, tenants=_log_uniform(rng, 1, max(1, min(64, 16 * 2048 ** 3 // size ** 3))))
    elif mix == "mixed":
        case.update(count=_log_uniform(rng, 8, 200))
    elif mix == "ragged":
        case.update(count=_log_uniform(rng, 4, 96), dtype=rng.choice([half, "f32", "mixed"]))
    else:
        case.update(mix="mixed", count=_log_uniform(rng, 4, 48), via="queue")
    return case


# ---- inputs, plan and one pass ----------------------------------------------------------------------------

def _operands(case, seed):
    """[(operator, A, B, place of C)] and the output buffers.  Activations and weights as the layers meet them: a
    convolution's image is the output of a rectifier (uniform), its weights He-normal; a linear layer's input is
    normal, its weights normal over the square root of the reduction length."""
    gen = torch.Generator(device="cuda")
    gen.manual_seed(int(seed))
    sizes, ops = {}, []
    for o in operators(case):
        at = sizes.get(o.dtype, 0)
        sizes[o.dtype] = at + (o.c_elems() + 127) // 128 * 128
        ops.append((o, at))
    out = {t: torch.zeros(n, dtype=TORCH[t], device="cuda") for t, n in sizes.items()}
    got = []
    for o, at in ops:
        if o.op == "gemm":
            a = torch.randn(o.a_elems(), generator=gen, device="cuda").to(TORCH[o.dtype])
            std = 1.0 / math.sqrt(o.K)
        else:
            a = torch.rand(o.a_elems(), generator=gen, device="cuda").to(TORCH[o.dtype])
            std = math.sqrt(2.0 / (o.R * o.S * o.Cin))
        b = (torch.randn(o.b_elems(), generator=gen, device="cuda") * std).to(TORCH[o.dtype])
        got.append((o, a, b, at))
    return got, out


def prepare(case, seed):
    ops, out = _operands(case, seed)
    problems = (sk.sk_problem * len(ops))()
    for i, (o, a, b, at) in enumerate(ops):
        problems[i] = sk.make_problem(o, a.data_ptr(), b.data_ptr(), out[o.dtype].data_ptr() + at * ES[o.dtype],
                                      lda=o.lda, ldb=o.ldb, ldc=o.ldc)
    state = {"via": case["via"], "out": out, "keep": ops, "problems": problems, "n": len(ops)}
    torch.cuda.synchronize()
    if case["via"] == "queue":
        state["stream"] = torch.cuda.Stream()
        state["queue"] = sk.sk_queue_create(sk.sk_queue_params_default(policy="coalesce"), state["stream"].cuda_stream)
        state["budgets"] = (ctypes.c_double * len(ops))(*[o.deadline_ms for o, _, _, _ in ops])
        state["done"] = (sk.sk_completion * len(ops))()
    else:
        state["plan"] = sk.sk_plan_create(problems, sk.sk_plan_params_default(host_only=int(case["via"] == "static")))
    return state


def run(state):
    if state["via"] == "queue":
        queue, done, got = state["queue"], state["done"], 0
        sk.sk_queue_submit(queue, state["problems"], state["budgets"], 0, state["n"])
        while got < state["n"]:
            got += sk.sk_queue_poll(queue, done, wait=True)
    elif state["via"] == "static":
        sk.sk_launch_static(state["plan"], torch.cuda.current_stream().cuda_stream)
    else:
        sk.sk_launch(state["plan"], torch.cuda.current_stream().cuda_stream)
    return state["out"]


# ---- what a pass cannot do without, and how exact it is ----------------------------------------------------

def _taps(size, out, filt, stride, pad):
    """How many (output, filter tap) pairs of one direction fall into the image."""
    return sum(max(0, min(filt, size + pad - o * stride) - max(0, pad - o * stride)) for o in range(out))


def work(case):
    total = flops = 0
    for o in operators(case):
        if o.op == "gemm":
            total += ES[o.dtype] * (o.M * o.K + o.N * o.K + o.M * o.N)
            flops += 2 * o.M * o.N * o.K
        else:
            total += ES[o.dtype] * (o.a_elems() + o.b_elems() + o.c_elems())
            ho, wo = o.out_hw()
            flops += 2 * o.Nb * o.Cin * o.Cout * _taps(o.H, ho, o.R, o.stride, o.pad_h) * _taps(o.W, wo, o.S, o.stride, o.pad_w)
    return {"bytes": total, "flops": flops}


# Four times the largest distance from 64-bit results that was measured on the listed and some drawn cases.
TOLERANCE = {"f32": {"rel": 4e-6, "max": 4e-5}, "f16": {"rel": 9e-4, "max": 2e-3}, "bf16": {"rel": 7e-3, "max": 1.6e-2}}


def tolerance(case):
    return dict(TOLERANCE["bf16" if case["dtype"] == "mixed" else case["dtype"]])


def exact(case, seed):
    ops, out = _operands(case, seed)
    res = {t: torch.zeros(v.numel(), dtype=torch.float64, device="cuda") for t, v in out.items()}
    for o, a, b, at in ops:
        dst = res[o.dtype][at:at + o.c_elems()]
        if o.op == "gemm":
            x = a.view(o.M, o.lda or o.K)[:, :o.K].double()
            w = b.view(o.N, o.ldb or o.K)[:, :o.K].double()
            dst.view(o.M, o.ldc or o.N)[:, :o.N] = x @ w.t()
            continue
        ho, wo = o.out_hw()
        if o.op == "conv":
            x = a.view(o.Nb, o.H, o.W, o.Cin).permute(0, 3, 1, 2).double()
            w = b.view(o.Cout, o.R, o.S, o.Cin).permute(0, 3, 1, 2).double()
        else:
            x = a.view(o.Nb, o.Cin, o.H, o.W).double()
            w = b.view(o.Cout, o.Cin, o.R, o.S).double()
        cols = torch.nn.functional.unfold(x.contiguous(), (o.R, o.S), padding=(o.pad_h, o.pad_w), stride=o.stride)
        w = w.reshape(o.Cout, -1)
        for i in range(o.Nb):
            y = w @ cols[i]  # [Cout, Ho*Wo]
            one = dst.view(o.Nb, -1)[i]
            one.copy_((y.t() if o.op == "conv" else y).reshape(-1))
    return res
