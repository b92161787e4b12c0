"""The work that users of this library have it do, as cases to time and compare.

A case names a path (a few public calls in the order in which a training program makes them), its sizes and its
quantization block.  The paths:

  forward     one linear forward product: the smallest thing the library is asked for
  linear      a linear layer's forward product and both gradients, INT8 in and out
  master      the same three products for a layer whose FP32 master weights take an FP32 weight gradient
  mlp_step    quantize activation, weight and upstream gradient, LayerNorm, linear, GELU and all their backward passes:
              the step of bench.py, with the buffers and the workspace that such a loop keeps
  residual    the residual connection of a block: Dropout, Add with row partials, the LayerNorm fed by them; backward
              LayerNorm, the gradient Add and Dropout
  attention   the hand-over to FP16 attention and back: Q, K, V to FP16 and the output to INT8, then both gradients
  gelu        GELU forward and backward
  layernorm   LayerNorm forward and backward

Values: activations N(0, 1) with 1 % of the channels scaled by 20, weights N(0, 0.02^2), gradients N(0, 0.001^2), GELU
inputs N(0, 2^2); gamma about 1, beta about 0; the quantized operands come from the library's own quantizer.
"""
import math

import torch

import paper_2403_12422_amd as jf

EPS = 1e-5
DROP_P = 0.1


def listed():
    return [
        # one small product (the single-product configuration): launch latency and the host's share of a call
        dict(name="forward_256", path="forward", tokens=256, inner=256, outer=256, block=32),
        # a micro-batch with sizes that fit no tile: 33, 25 and 65 blocks
        dict(name="mlp_step_ragged", path="mlp_step", tokens=1056, inner=800, outer=2080, block=32),
        # the benchmark's step: GPT-2-small MLP
        dict(name="mlp_step_gpt2s", path="mlp_step", tokens=4096, inner=768, outer=3072, block=32),
        # a square layer with FP32 master weights
        dict(name="master_2048", path="master", tokens=2048, inner=2048, outer=2048, block=32),
        # feed-forward layer of the GPT-2-large block
        dict(name="linear_gpt2l_ffn", path="linear", tokens=8192, inner=1280, outer=5120, block=32),
        # large layers, one for each block size
        dict(name="linear_8192", path="linear", tokens=8192, inner=8192, outer=8192, block=32),
        dict(name="linear_4096_b64", path="linear", tokens=4096, inner=4096, outer=4096, block=64),
        dict(name="linear_llama_b128", path="linear", tokens=16384, inner=4096, outer=11008, block=128),
        # what surrounds the products of the GPT-2-large block
        dict(name="residual_gpt2l", path="residual", tokens=8192, inner=1280, outer=0, block=32),
        dict(name="attention_gpt2l", path="attention", tokens=8192, inner=1280, outer=0, block=32),
        # operands of 0.8 GB, which no cache holds
        dict(name="gelu_hbm", path="gelu", tokens=262144, inner=3072, outer=0, block=32),
        dict(name="layernorm_hbm", path="layernorm", tokens=1048576, inner=768, outer=0, block=32),
    ]


#: smallest and largest tokens, features of a drawn case, and the largest number of elements (products: multiply-adds)
RANGES = {
    "forward": (32, 16384, 64, 11008, 16384 * 4096 * 11008),
    "linear": (128, 16384, 128, 11008, 16384 * 4096 * 11008),
    "master": (128, 16384, 128, 11008, 16384 * 4096 * 11008),
    "mlp_step": (128, 16384, 128, 5120, 16384 * 1280 * 5120),
    "residual": (128, 262144, 128, 8192, 1 << 28),
    "attention": (128, 65536, 128, 8192, 1 << 27),
    "gelu": (128, 262144, 128, 11008, 1 << 29),
    "layernorm": (128, 1 << 20, 128, 8192, 1 << 29),
}


def draw(rng):
    path = rng.choice(sorted(RANGES))
    t0, t1, f0, f1, most = RANGES[path]
    product = path in ("forward", "linear", "master", "mlp_step")
    block = rng.choice((32, 32, 32, 64, 128))

    def size(lo, hi):
        v = math.exp(rng.uniform(math.log(lo), math.log(hi)))
        return block * max(1, round(v / block))

    while True:
        n, c, d = size(t0, t1), size(f0, f1), size(f0, f1)
        if n * c * (d if product else 1) <= most:
            return dict(path=path, tokens=n, inner=c, outer=d if product else 0, block=block)


class State:
    pass


def prepare(case, seed):
    s = State()
    s.path, s.block = case["path"], case["block"]
    n, c, d, b = case["tokens"], case["inner"], case["outer"], case["block"]
    dev = torch.device("cuda:0")
    gen = torch.Generator(device=dev)
    gen.manual_seed(seed)

    def normal(rows, cols, std, outliers=False):
        x = torch.randn((rows, cols), generator=gen, device=dev, dtype=torch.float32)
        x *= std
        if outliers:
            x[:, torch.randperm(cols, generator=gen, device=dev)[:max(1, round(0.01 * cols))]] *= 20.0
        return x

    def q(x):
        return jf.jf_quantize_block(x, b)

    def vector(mean):
        return mean + 0.1 * torch.randn((c,), generator=gen, device=dev, dtype=torch.float32)

    def workspace():
        return torch.empty((max(16, jf.jf_workspace_bytes(7, n, c, 0, b)),), dtype=torch.uint8, device=dev)

    if s.path in ("forward", "linear", "master"):
        s.x, s.sx = q(normal(n, c, 1.0, True))
        s.w, s.sw = q(normal(d, c, 0.02))
        if s.path != "forward":
            s.dy, s.sdy = q(normal(n, d, 1e-3))
    elif s.path == "mlp_step":
        s.x, s.w, s.dh = normal(n, c, 1.0, True), normal(d, c, 0.02), normal(n, d, 1e-3)
        s.gamma, s.beta = vector(1.0), vector(0.0)
        s.ws = workspace()

        def codes(r, k):
            return (torch.empty((r, k), dtype=torch.int8, device=dev),
                    torch.empty((r // b, k // b), dtype=torch.float32, device=dev))

        def row(m):
            return torch.empty((m,), dtype=torch.float32, device=dev)

        s.xq, s.wq, s.gq, s.xn, s.y, s.h = codes(n, c), codes(d, c), codes(n, d), codes(n, c), codes(n, d), codes(n, d)
        s.dy, s.dxn, s.dw, s.dx = codes(n, d), codes(n, c), codes(d, c), codes(n, c)
        s.mean, s.rstd, s.dgamma, s.dbeta = row(n), row(n), row(c), row(c)
    elif s.path == "residual":
        s.x, s.sx = q(normal(n, c, 1.0))
        s.r, s.sr = q(normal(n, c, 1.0, True))
        s.dy, s.sdy = q(normal(n, c, 1e-3))
        s.dr, s.sdr = q(normal(n, c, 1e-3))
        keep = torch.rand((n, c // 8, 8), generator=gen, device=dev, dtype=torch.float16) >= DROP_P
        bit = 2 ** torch.arange(8, device=dev, dtype=torch.int32)
        s.mask = torch.zeros((n, c // 8), dtype=torch.uint8, device=dev)
        for k in range(8):
            s.mask |= keep[:, :, k].to(torch.uint8) * bit[k].to(torch.uint8)
        s.gamma, s.beta = vector(1.0), vector(0.0)
        s.ws = workspace()
    elif s.path == "attention":
        s.qkv, s.sqkv = q(normal(n, 3 * c, 1.0))
        s.o = normal(n, c, 1.0).to(torch.float16)
        s.do, s.sdo = q(normal(n, c, 1e-3))
        s.dqkv = normal(n, 3 * c, 1e-2).to(torch.float16)
    elif s.path == "gelu":
        s.x, s.sx = q(normal(n, c, 2.0))
        s.dy, s.sdy = q(normal(n, c, 1e-3))
    else:
        s.x, s.sx = q(normal(n, c, 1.0, True))
        s.dy, s.sdy = q(normal(n, c, 1e-3))
        s.gamma, s.beta = vector(1.0), vector(0.0)
        s.ws = workspace()
    return s


def run(s):
    b = s.block
    if s.path == "forward":
        return jf.jf_linear_fwd(s.x, s.sx, s.w, s.sw, b)
    if s.path == "linear":
        y = jf.jf_linear_fwd(s.x, s.sx, s.w, s.sw, b)
        return y, jf.jf_linear_bwd(s.dy, s.sdy, s.w, s.sw, s.x, s.sx, b)
    if s.path == "master":
        y = jf.jf_linear_fwd(s.x, s.sx, s.w, s.sw, b)
        dx = jf.jf_linear_dgrad(s.dy, s.sdy, s.w, s.sw, b)
        return y, dx, jf.jf_linear_wgrad(s.dy, s.sdy, s.x, s.sx, b, want_q=False, want_f32=True)
    if s.path == "mlp_step":
        xq, wq, gq = (jf.jf_quantize_block(t, b, out=o) for t, o in ((s.x, s.xq), (s.w, s.wq), (s.dh, s.gq)))
        xn = jf.jf_layernorm_q(*xq, s.gamma, s.beta, EPS, b, out=(*s.xn, s.mean, s.rstd))[:2]
        y = jf.jf_linear_fwd(*xn, *wq, b, out=(*s.y, None))[:2]
        h = jf.jf_gelu_q(*y, b, out=s.h)
        dy = jf.jf_gelu_q_bwd(*gq, *y, b, out=s.dy)
        (dxn, sdxn, _), dw = jf.jf_linear_bwd(*dy, *wq, *xn, b, out=((*s.dxn, None), (*s.dw, None)))
        dx = jf.jf_layernorm_q_bwd(dxn, sdxn, *xq, s.gamma, s.mean, s.rstd, b, workspace=s.ws,
                                   out=(*s.dx, s.dgamma, s.dbeta))
        return xq, wq, gq, xn, s.mean, s.rstd, y, h, dy, dxn, sdxn, dw, dx
    if s.path == "residual":
        z, sz = jf.jf_dropout_q(s.x, s.sx, s.mask, DROP_P, b)
        a, sa, row_mean, row_sumsq = jf.jf_add_q(z, sz, s.r, s.sr, b, want_partials=True)
        y, sy, mean, rstd = jf.jf_layernorm_q_partials(a, sa, row_mean, row_sumsq, s.gamma, s.beta, EPS, b)
        da, sda, dgamma, dbeta = jf.jf_layernorm_q_bwd(s.dy, s.sdy, a, sa, s.gamma, mean, rstd, b, workspace=s.ws)
        dr, sdr = jf.jf_add_q(da, sda, s.dr, s.sdr, b)
        dx = jf.jf_dropout_q(dr, sdr, s.mask, DROP_P, b)
        return z, sz, a, sa, row_mean, row_sumsq, y, sy, mean, rstd, da, sda, dgamma, dbeta, dr, sdr, dx
    if s.path == "attention":
        qkv = jf.jf_dequantize_block(s.qkv, s.sqkv, b, torch.float16)
        o = jf.jf_quantize_block(s.o, b)
        do = jf.jf_dequantize_block(s.do, s.sdo, b, torch.float16)
        return qkv, o, do, jf.jf_quantize_block(s.dqkv, b)
    if s.path == "gelu":
        y = jf.jf_gelu_q(s.x, s.sx, b)
        return y, jf.jf_gelu_q_bwd(s.dy, s.sdy, s.x, s.sx, b)
    y, sy, mean, rstd = jf.jf_layernorm_q(s.x, s.sx, s.gamma, s.beta, EPS, b)
    return y, sy, mean, rstd, jf.jf_layernorm_q_bwd(s.dy, s.sdy, s.x, s.sx, s.gamma, mean, rstd, b, workspace=s.ws)


def work(case):
    """Bytes and operations of one pass: the operands and results of every call, each moved once."""
    n, c, d, b = case["tokens"], case["inner"], case["outer"], case["block"]
    i8 = 1.0 + 4.0 / (b * b)          # an INT8 element with its share of the scale grid
    x, w, y = n * c * i8, d * c * i8, n * d * i8
    p = case["path"]
    if p == "forward":
        return {"bytes": x + w + y, "flops": 2.0 * n * c * d}
    if p == "linear":
        return {"bytes": 3 * (x + w + y), "flops": 6.0 * n * c * d}
    if p == "master":
        return {"bytes": 3 * (x + w + y) - w + 4.0 * d * c, "flops": 6.0 * n * c * d}
    rows = 8.0 * n                    # mean and rstd
    if p == "mlp_step":
        quantize = 4.0 * (n * c + d * c + n * d) + x + w + y
        norm = 2 * x + rows + 8.0 * c + 3 * x + rows + 12.0 * c
        return {"bytes": quantize + norm + 3 * (x + w + y) + 5 * y, "flops": 6.0 * n * c * d + 40.0 * n * (c + d)}
    e = n * c
    if p == "residual":
        dropout = 2 * x + e / 8.0
        partials = 8.0 * e / b
        return {"bytes": 2 * dropout + 6 * x + partials + (2 * x + partials + rows) + (3 * x + rows) + 20.0 * c,
                "flops": 60.0 * e}
    if p == "attention":
        return {"bytes": 8 * e * (i8 + 2.0), "flops": 16.0 * e}
    if p == "gelu":
        return {"bytes": 5 * x, "flops": 40.0 * e}
    return {"bytes": 5 * x + 2 * rows + 20.0 * c, "flops": 40.0 * e}


def tolerance(case):
    p = case["path"]
    if p in ("forward", "linear", "master", "attention"):
        # exact integer products, one fixed FP32 order over the blocks along K, and exactly rounded codes
        return "exact"
    if p == "mlp_step":
        # a LayerNorm or GELU code at a rounding tie goes into the sums of the products that follow
        return {"rel": 1e-3, "differ": 0.01}
    # FP32 evaluation of the functions and of the row and column sums; codes at rounding ties
    return {"rel": 1e-5, "differ": 1e-3}
