"""The work whose time matters for a user of this library, as measurable cases.

A case is one call of ``matmul`` or ``conv2d_nchw`` on device tensors, with the
output allocated by the call, as a program that runs a network layer by layer
makes it.  ``listed`` holds one case per kind of work at sizes that the
benchmark, the tests and the paper's examples use (or generic ones); ``draw``
samples the same kinds over their whole range of sizes, odd ones included.
"""
import math

import torch

import paper_2512_16512_amd as xtc


def _matmul(kind, dtype, M, N, K, relu=False, name=None):
    c = {"op": "matmul", "kind": kind, "dtype": dtype, "M": M, "N": N, "K": K, "relu": relu}
    if name:
        c["name"] = name
    return c


def _conv(kind, dtype, batch, C, H, W, OC, R, S, stride, pad, relu=False, name=None):
    c = {"op": "conv2d", "kind": kind, "dtype": dtype, "batch": batch, "C": C, "H": H, "W": W,
         "OC": OC, "R": R, "S": S, "stride": stride, "pad": pad, "relu": relu}
    if name:
        c["name"] = name
    return c


def listed():
    return [
        # The matmul+relu graph of the paper's Sec. 5.2: a call so small that
        # its latency is the launch, one pass over cold caches and the host path.
        _matmul("small", "f32", 256, 1024, 128, relu=True, name="mm_relu_f32_256x1024x128"),
        # The ragged 1000^3 product of the benchmark: a mid-size dense layer,
        # about one workgroup tile per CU.
        _matmul("mid", "f32", 1000, 1000, 1000, name="mm_f32_1000"),
        # Sizes as a program meets them when nothing was padded: every extent
        # odd, so no row but the first starts on a 16-byte boundary.
        _matmul("odd", "f32", 1531, 1021, 2047, name="mm_f32_odd_1531x1021x2047"),
        # The headline fp32 product.
        _matmul("large", "f32", 4096, 4096, 4096, name="mm_f32_4096"),
        # Tall and skinny (a projection onto a few columns): streams A from HBM.
        _matmul("skinny", "f32", 32768, 16, 4096, name="mm_f32_32768x16x4096"),
        # The headline bf16 product.
        _matmul("large", "bf16", 8192, 8192, 8192, name="mm_bf16_8192"),
        # The bf16 counterpart of the odd sizes: rows at any 2-byte boundary.
        _matmul("odd", "bf16", 2047, 3001, 1999, name="mm_bf16_odd_2047x3001x1999"),
        # The classifier at the end of an image network (the paper's Sec. 6.4
        # networks end in one) on a batch of 32: few rows, a long reduction.
        _matmul("dense", "bf16", 32, 1000, 2048, name="mm_bf16_dense_32x1000x2048"),
        # The benchmark's convolution layer, fp32 and bf16.
        _conv("conv3x3", "f32", 32, 64, 56, 56, 64, 3, 3, 1, 1, name="conv_f32_32x64x56x56"),
        _conv("conv3x3", "bf16", 32, 64, 56, 56, 64, 3, 3, 1, 1, name="conv_bf16_32x64x56x56"),
        # A deeper layer of the same kind of network: half the resolution,
        # twice the channels, relu fused.
        _conv("conv3x3", "bf16", 32, 128, 28, 28, 128, 3, 3, 1, 1, relu=True,
              name="conv_relu_bf16_32x128x28x28"),
        # The paper's first-layer convolution (Sec. 6.2): one image, three
        # channels, 7x7 taps at stride 2.
        _conv("stem", "f32", 1, 3, 224, 224, 16, 7, 7, 2, 3, name="conv_f32_stem_7x7s2"),
    ]


def _log(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def _near(rng, v, step):
    """v rounded to a multiple of ``step`` in two draws of three, else made odd."""
    return max(step, v // step * step) if rng.random() < 0.67 else v | 1


def draw(rng):
    kind = rng.choice(["small", "mid", "odd", "large", "skinny", "dense", "conv3x3", "conv3x3",
                       "conv1x1", "stem"])
    dtype = rng.choice(["f32", "bf16"])
    relu = rng.random() < 0.3
    if kind == "small":
        M, N, K = (_near(rng, _log(rng, 64, 512), 8) for _ in range(3))
        return _matmul(kind, dtype, M, N, K, relu)
    if kind == "mid":
        M, N, K = (max(8, _log(rng, 512, 2048) // 8 * 8) for _ in range(3))
        return _matmul(kind, dtype, M, N, K, relu)
    if kind == "odd":
        M, N, K = (_log(rng, 512, 3000) | 1 for _ in range(3))
        return _matmul(kind, dtype, M, N, K, relu)
    if kind == "large":
        hi = 4096 if dtype == "f32" else 8192
        M, N, K = (_log(rng, 2048, hi) // 8 * 8 for _ in range(3))
        return _matmul(kind, dtype, M, N, K, relu)
    if kind == "skinny":
        # one long operand, streamed once against 8 to 32 columns
        return _matmul(kind, dtype, _log(rng, 4096, 32768), rng.randint(8, 32),
                       _log(rng, 1024, 4096) // 8 * 8, relu)
    if kind == "dense":
        # 1 to 128 rows of activations against a weight matrix
        return _matmul(kind, dtype, _log(rng, 1, 128), _near(rng, _log(rng, 256, 4096), 8),
                       _near(rng, _log(rng, 512, 4096), 8), relu)
    if kind == "conv3x3":
        # the 3x3 layers of an image network: channels double where the image
        # is halved; one in four at stride 2
        level = rng.randint(0, 2)
        size = (56, 28, 14)[level] + rng.choice([0, 0, 0, -1, 1, 8])
        C = (64, 128, 256)[level]
        stride = 2 if rng.random() < 0.25 else 1
        return _conv(kind, dtype, _log(rng, 1, 32), C, size, size, C * rng.choice([1, 1, 2]),
                     3, 3, stride, 1, relu)
    if kind == "conv1x1":
        # pointwise layers, as in squeeze and bottleneck blocks
        size = rng.choice([55, 56, 28, 27, 14, 13])
        C = rng.choice([16, 64, 128, 256, 512])
        return _conv(kind, dtype, _log(rng, 1, 32), C, size, size,
                     rng.choice([16, 64, 128, 256]), 1, 1, 1, 0, relu)
    # first layers: three channels of an image of 160 to 256 pixels
    size = rng.randint(160, 256)
    taps = rng.choice([3, 5, 7])
    return _conv("stem", dtype, _log(rng, 1, 16), 3, size, size, rng.choice([16, 32, 64]),
                 taps, taps, 2, taps // 2, relu)


def _inputs(case, seed):
    """The case's two operands in float32: activations and weights of unit
    scale over the reduction, as a normalised network holds them."""
    g = torch.Generator(device="cuda").manual_seed(seed)

    def normal(*shape):
        return torch.randn(*shape, device="cuda", generator=g)

    if case["op"] == "matmul":
        return (normal(case["M"], case["K"]),
                normal(case["K"], case["N"]).mul_(case["K"] ** -0.5))
    C, R, S = case["C"], case["R"], case["S"]
    return (normal(case["batch"], C, case["H"], case["W"]),
            normal(case["OC"], C, R, S).mul_((C * R * S) ** -0.5))


def prepare(case, seed):
    a, b = _inputs(case, seed)
    if case["dtype"] == "bf16":
        a, b = a.bfloat16(), b.bfloat16()
    return {"case": case, "a": a, "b": b}


def run(state):
    c = state["case"]
    if c["op"] == "matmul":
        return xtc.matmul(state["a"], state["b"], relu=c["relu"])
    return xtc.conv2d_nchw(state["a"], state["b"], stride=c["stride"], pad=c["pad"],
                           relu=c["relu"])


def _gemm_extents(case):
    """(rows, columns, reduction) of the case as a matrix product."""
    if case["op"] == "matmul":
        return case["M"], case["N"], case["K"]
    oh, ow = _out_size(case)
    return case["OC"], case["batch"] * oh * ow, case["C"] * case["R"] * case["S"]


def _out_size(case):
    return ((case["H"] + 2 * case["pad"] - case["R"]) // case["stride"] + 1,
            (case["W"] + 2 * case["pad"] - case["S"]) // case["stride"] + 1)


def work(case):
    M, N, K = _gemm_extents(case)
    elt = 4 if case["dtype"] == "f32" else 2
    if case["op"] == "matmul":
        inputs = M * K + K * N
    else:
        inputs = case["batch"] * case["C"] * case["H"] * case["W"] + M * K
    return {"bytes": inputs * elt + M * N * 4, "flops": 2 * M * N * K}


def tolerance(case):
    # fp32 accumulation in another order.  Against float64 the fp32 sums are
    # off by 1.1e-7 (K = 128) to 1.2e-6 (K = 4096), the bf16-input ones
    # (products exact) by 1.1e-7 to 5.5e-7 (K = 8192): about four times that.
    K = _gemm_extents(case)[2]
    return {"rel": 5e-7 + (1.2e-9 if case["dtype"] == "f32" else 2.5e-10) * K}


def exact(case, seed):
    s = prepare(case, seed)
    a, b = s["a"].double(), s["b"].double()
    if case["op"] == "matmul":
        y = a @ b
    else:
        # one product per tap over the strided, zero-padded input
        oh, ow = _out_size(case)
        st, p = case["stride"], case["pad"]
        x = torch.nn.functional.pad(a, (p, p, p, p)).permute(1, 0, 2, 3).contiguous()
        y = torch.zeros(case["OC"], case["batch"] * oh * ow, dtype=torch.float64, device=a.device)
        for kh in range(case["R"]):
            for kw in range(case["S"]):
                tap = x[:, :, kh:kh + (oh - 1) * st + 1:st, kw:kw + (ow - 1) * st + 1:st]
                y += b[:, :, kh, kw].contiguous() @ tap.reshape(case["C"], -1)
        y = y.view(case["OC"], case["batch"], oh, ow).permute(1, 0, 2, 3).contiguous()
    return y.relu_() if case["relu"] else y
