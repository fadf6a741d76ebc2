"""The work that a user of this package has it do, as cases that can be timed and compared.

A data-parallel training program does two things with the package in every step: it quantizes its own gradient
(`ogq_quantize`), and it decodes and averages the packed streams of all workers (`ogq_dequantize_average`).  A case is
one of the two or both in a row ("round": a worker's share of one step), for a gradient of `n` values in buckets of `d`:

  op       "quantize", "decode" or "round"
  scheme   a key of SCHEMES; `bits` is the width of a level index, `iters` the level updates / re-solve sweeps, `clip`
           the clipping factor (0 = off)
  data     distribution of the gradient's values (the generators of `gradient` below)
  workers  streams that are averaged (for "quantize": 1)
  kept     True: the program hands in its own output buffers, as one does that sends them; False: it lets the package
           allocate them

Gradient sizes are those of the package's benchmark (ResNet-50 25.6 M, AlexNet 61.1 M and VGG-19 143.7 M values, and
single layers of VGG-19); bucket sizes, level counts and clipping are the paper's (bucket 128 to 32768, ORQ with 3, 5
and 9 levels, c = 2.5) and the benchmark's.
"""
import math

import torch

import paper_2002_11082_amd as ogq
from paper_2002_11082_amd import synth

SCHEMES = {
    "bingrad_b": ogq.BINGRAD_B,
    "bingrad_pb": ogq.BINGRAD_PB,
    "orq": ogq.ORQ,
    "orq_paper": ogq.ORQ_PAPER,
    "sign": ogq.SCALED_SIGN,
    "even": ogq.EVEN,
    "linear": ogq.LINEAR,
}


def _case(name, op, scheme, bits, n, d, data, workers=1, iters=0, clip=0.0, kept=True):
    return {"name": name, "op": op, "scheme": scheme, "bits": bits, "n": n, "d": d, "data": data, "workers": workers,
            "iters": iters, "clip": clip, "kept": kept}


def listed():
    return [
        # The smallest call: the first convolution of a network, quantized layer by layer in the paper's ImageNet
        # setting (ORQ-3, bucket 512, c = 2.5).  Launches and the host's share are all there is.
        _case("round_first_conv", "round", "orq_paper", 2, 1728, 512, "student", 1, clip=2.5, kept=False),
        # A gradient of one million values, one bit each, and back.
        _case("round_1m_1bit", "round", "bingrad_b", 1, 1048576, 512, "gaussian", 1),
        # One large layer with its bias: ragged buckets, BinGrad-pb, the streams of four workers.
        _case("round_layer_ragged", "round", "bingrad_pb", 1, 2359808, 1344, "laplace", 4),
        # ResNet-50 at one bit per value: the cheapest quantizer on an ordinary gradient ...
        _case("quantize_resnet_1bit", "quantize", "bingrad_b", 1, 25600000, 2048, "laplace"),
        # ... and what the receiver does with one such stream.
        _case("decode_resnet_1bit", "decode", "bingrad_b", 1, 25600000, 2048, "laplace"),
        # ResNet-50 with four levels, two sweeps.
        _case("quantize_resnet_orq4", "quantize", "orq", 2, 25600000, 2048, "mixture", iters=2),
        # The paper's ImageNet run at its finest: nine levels, bucket 512, clipping, four workers.
        _case("round_resnet_orq9_clip", "round", "orq_paper", 4, 25600000, 512, "mixture", 4, clip=2.5),
        # The two ends of the paper's bucket-size sweep.
        _case("quantize_resnet_orq3_d128", "quantize", "orq_paper", 2, 25600000, 128, "mixture"),
        _case("quantize_resnet_orq3_d32768", "quantize", "orq_paper", 2, 25600000, 32768, "mixture"),
        # The rule that most people come from: TernGrad's three evenly spaced levels.
        _case("quantize_resnet_terngrad", "quantize", "even", 2, 25600000, 2048, "mixture"),
        # The largest gradient: VGG-19 with eight levels, two sweeps.
        _case("quantize_vgg_orq8", "quantize", "orq", 3, 143700000, 4096, "student", iters=2),
        # The server step for eight workers, AlexNet-sized.
        _case("decode_alexnet_8_workers", "decode", "orq", 2, 61100000, 2048, "gaussian", 8, iters=2),
    ]


def draw(rng):
    """One more case: any scheme, any bucket size that the package takes, from a small layer to a whole network."""
    op = rng.choice(("quantize", "quantize", "decode", "round"))
    scheme = rng.choice(("bingrad_b", "bingrad_b", "orq", "orq", "orq_paper", "orq_paper", "bingrad_pb", "sign", "even",
                         "linear"))
    bits = 1 if scheme in ("bingrad_b", "bingrad_pb", "sign") else rng.choice((2, 3)) if scheme == "orq" else rng.choice((2, 3, 4))
    # half of the bucket sizes are those of the paper's sweep, the others any multiple of 64
    if rng.random() < 0.5:
        d = 1 << rng.randint(7, 15)
    else:
        d = 64 * int(round(math.exp(rng.uniform(0.0, math.log(512)))))
    workers = 1 if op == "quantize" else rng.randint(1, 8)
    n = int(math.exp(rng.uniform(math.log(1000), math.log(25600000))))
    iters = 2 if scheme == "orq" else rng.choice((0, 0, 0, 2)) if scheme == "bingrad_b" else 0
    clip = rng.choice((0.0, 0.0, 0.0, 2.5)) if op != "decode" else 0.0
    data = rng.choice(("gaussian", "laplace", "mixture", "student"))
    case = _case("", op, scheme, bits, n, d, data, workers, iters, clip, rng.random() < 0.75)
    del case["name"]
    return case


def gradient(data, n, gen):
    """The distributions of the package's synthetic gradients (synth.py), made on the device."""
    def normal(m):
        return torch.randn(m, generator=gen, device="cuda")

    if data == "gaussian":
        return normal(n).mul_(1e-3)
    if data == "laplace":  # Laplace(0, 5e-4), 1 % of the entries times 20
        g = torch.empty(n, device="cuda").exponential_(1.0 / 5e-4, generator=gen)
        pick = torch.rand(n, generator=gen, device="cuda")
        g *= torch.where(pick < 0.5, -1.0, 1.0)
        g *= torch.where((pick * 64.0).frac_() < 0.01, 20.0, 1.0)
        return g
    if data == "mixture":  # 0.9 N(0, 1e-4^2) + 0.1 N(0, 1e-2^2)
        g = normal(n)
        g *= torch.where(torch.rand(n, generator=gen, device="cuda") < 0.9, 1e-4, 1e-2)
        return g
    # Student-t with three degrees of freedom, each layer of VGG-19 scaled by 1/sqrt(fan_in); a gradient of another
    # size has the layers in proportion
    chi = normal(n).square_()
    for _ in range(2):
        chi += normal(n).square_()
    g = normal(n).div_(chi.div_(3.0).sqrt_())
    layers, pos, scale = synth.vgg19_layer_sizes(), 0, n / 143700000
    for k, (size, fan_in) in enumerate(layers):
        end = n if k == len(layers) - 1 else min(n, pos + int(size * scale))
        g[pos:end] *= 1.0 / math.sqrt(fan_in)
        pos = end
    return g


class _State:
    pass


def prepare(case, seed):
    """The gradient, the other workers' packed streams and the buffers that a training program keeps between steps."""
    gen = torch.Generator(device="cuda")
    gen.manual_seed(seed)
    s = _State()
    s.op, s.n = case["op"], case["n"]

    def params(worker):
        return ogq.make_params(case["d"], case["bits"], SCHEMES[case["scheme"]], case["iters"], 1000 * seed + worker, 0,
                               case["clip"])

    s.params = params(0)
    s.n_levels = ogq.ogq_levels_count(s.n, s.params)
    n_words = ogq.ogq_codes_bytes(s.n, s.params) // 8

    def buffers():
        return (torch.empty(s.n_levels, dtype=torch.float32, device="cuda"),
                torch.empty(n_words, dtype=torch.int64, device="cuda"))

    s.grad = gradient(case["data"], s.n, gen)
    s.levels = s.codes = s.out = None
    if case["kept"]:
        s.levels, s.codes = buffers()
        if s.op != "quantize":
            s.out = torch.empty(s.n, device="cuda")
    # the streams of the workers: of all of them where only decoding is done, of the others in a round
    s.all_codes, s.all_levels = [], []
    if s.op != "quantize":
        for w in range(1 if s.op == "round" else 0, case["workers"]):
            lv, codes = buffers()
            ogq.ogq_quantize(s.grad if w == 0 else gradient(case["data"], s.n, gen), params(w), lv, codes)
            s.all_codes.append(codes)
            s.all_levels.append(lv)
    if s.op == "decode":
        s.grad = None
    return s


def run(s):
    if s.op == "decode":
        return ogq.ogq_dequantize_average(s.all_codes, s.all_levels, s.n, s.params, s.out)
    levels, codes = ogq.ogq_quantize(s.grad, s.params, s.levels, s.codes)
    if s.op == "quantize":
        out = None
    else:
        out = ogq.ogq_dequantize_average([codes] + s.all_codes, [levels] + s.all_levels, s.n, s.params, s.out)
    if levels.numel() > s.n_levels:  # the package's own buffer for very few buckets has spare entries
        levels = levels[:s.n_levels]
    return levels, codes, out


def work(case):
    n, workers = case["n"], case["workers"]
    p = ogq.make_params(case["d"], case["bits"], SCHEMES[case["scheme"]])
    stream = ogq.ogq_codes_bytes(n, p) + 4 * ogq.ogq_levels_count(n, p)
    # quantize: a sum and a compare per value; random rounding also takes the distance, the draw's product and the test
    quantize = {"bytes": 4 * n + stream, "flops": n * (2 if case["scheme"] in ("bingrad_b", "sign") else 5)}
    decode = {"bytes": workers * stream + 4 * n, "flops": n * workers}
    if case["op"] == "quantize":
        return quantize
    if case["op"] == "decode":
        return decode
    # in a round the worker's own stream is written once and need not be read back
    return {"bytes": quantize["bytes"] + decode["bytes"] - stream, "flops": quantize["flops"] + decode["flops"]}


def tolerance(case):
    # Averages, the means of BinGrad-b and of the sign rule and the clipping threshold are double-precision sums rounded
    # once to 32 bits: another order of the additions moves a rare one by its last bit.  Every other level is a value of
    # the bucket (or a quotient specified to the last bit), and the codes follow from the levels bit by bit.
    if case["op"] == "quantize" and case["scheme"] not in ("bingrad_b", "sign") and not case["clip"]:
        return "exact"
    # a threshold moved by its last bit can turn the code of a value that lies on it
    moved = 1e-5 if case["op"] != "decode" and (case["scheme"] == "bingrad_b" or case["clip"]) else 0.0
    return {"rel": 1e-7, "max": 1e-6, "differ": moved}
