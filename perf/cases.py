"""The work that a program using this codec has it do, as cases that can be timed one by one.

A case names an entry point of `paper_2212_01185_amd.binding.Codec` (encode, decode, decode into a caller's buffer
without allocations, or the network's outputs alone), a network and a mixture, the weights' kind and the images'
number and size.  `listed()` gives the cases that are always looked at, `draw()` others of the same ranges,
`prepare()` what the program has in hand before the call, `run()` the call.
"""
from __future__ import annotations

import math

import torch

from paper_2212_01185_amd import binding, synth

# Layer widths of the networks the library takes: the measured workloads', the paper's own (wavefront and diagonal
# order) and the six shapes of its ablation study.
WIDTHS = {"workload": synth.DEFAULT_DIMS, "paper": synth.PAPER_DIMS, "diagonal": synth.PAPER_DIMS}
WIDTHS.update({name: synth.ablation_dims(*shape) for name, shape in synth.ABLATION_SHAPES.items()})
DELAY = {name: synth.PAPER_DELAY for name in WIDTHS}
DELAY.update(workload=synth.DEFAULT_DELAY, diagonal=1)

# A drawn case stays within the largest listed ones: pixels of a call, passes of the decoder, pixels of a `probs`
# call (whose outputs are some 250 bytes a pixel), scratch of the decoder that allocates nothing.
LEAST_PIXELS, MOST_PIXELS, MOST_PASSES, MOST_PROBS_PIXELS = 64 * 64, 4096 * 2160, 8414, 2048 * 1365


def _case(name, call, n, h, w, network="workload", weights="he", dist="gaussian"):
    return {"name": name, "call": call, "network": network, "weights": weights, "dist": dist, "n": n, "h": h, "w": w}


def listed():
    return [
        # a thumbnail or a tile of a larger picture, coded on its own: launches and latency are all there is
        _case("encode 64x64", "encode", 1, 64, 64),
        _case("decode 64x64", "decode", 1, 64, 64),
        # one photograph of ordinary size, each direction
        _case("encode 768x512", "encode", 1, 512, 768),
        _case("decode 768x512", "decode", 1, 512, 768),
        # a batch of photographs handed over together (a folder being archived, a loader filling a batch)
        _case("encode 24 of 768x512", "encode", 24, 512, 768, weights="predictor"),
        _case("decode 24 of 768x512", "decode", 24, 512, 768, weights="predictor"),
        # the distributions themselves, for rate estimates and for a loss: a large picture of odd height
        _case("probs 2048x1365", "probs", 1, 1365, 2048),
        # the largest single pictures, each direction
        _case("encode 4096x2160", "encode", 1, 2160, 4096),
        _case("decode 4096x2160", "decode", 1, 2160, 4096),
        # the paper's own network at the size of its run-time table; a few ragged crops with its other mixture;
        # the order with the fewest passes, from a serving loop that allocates nothing
        _case("decode 512x512 paper", "decode", 1, 512, 512, network="paper"),
        _case("encode 5 of 333x217 seven mixtures", "encode", 5, 217, 333, network="most_mixtures", dist="logistic"),
        _case("decode 513x389 diagonal, static", "decode_static", 1, 389, 513, network="diagonal"),
    ]


def draw(rng):
    call = rng.choice(["encode", "encode", "encode", "decode", "decode", "decode", "decode_static", "probs"])
    network = "workload" if rng.random() < 0.5 else rng.choice(sorted(set(WIDTHS) - {"workload"}))
    weights = "predictor" if network == "workload" and rng.random() < 0.3 else "he"
    dist = "logistic" if weights == "he" and rng.random() < 0.2 else "gaussian"
    n = 1 if rng.random() < 0.6 else round(math.exp(rng.uniform(math.log(2), math.log(24))))
    most = MOST_PROBS_PIXELS if call == "probs" else MOST_PIXELS
    while True:
        pixels = math.exp(rng.uniform(math.log(LEAST_PIXELS), math.log(most))) / n
        aspect = math.exp(rng.uniform(-math.log(2.5), math.log(2.5)))     # width over height
        h, w = max(8, round(math.sqrt(pixels / aspect))), max(8, round(math.sqrt(pixels * aspect)))
        passes = binding.pcc_wavefront_steps(h, w, DELAY[network])
        scratch = 8 * n * -(-h // 16) * w
        if LEAST_PIXELS <= n * h * w <= most and passes <= MOST_PASSES and (call != "decode_static" or scratch <= 4 << 20):
            case = _case("", call, n, h, w, network, weights, dist)
            del case["name"]
            return case


_codecs = {}


def _codec(case):
    """The codec a program keeps: one for a network and its weights, for all images."""
    key = (case["network"], case["weights"], case["dist"])
    if key not in _codecs:
        dist = synth.DIST_LOGISTIC if case["dist"] == "logistic" else synth.DIST_GAUSSIAN
        if case["weights"] == "predictor":
            blob = synth.make_predictor_blob()
        elif case["network"] in synth.ABLATION_SHAPES:
            blob = synth.make_ablation_blob(*synth.ABLATION_SHAPES[case["network"]], dist=dist)
        else:
            make = {"workload": synth.make_blob, "paper": synth.make_paper_blob, "diagonal": synth.make_diagonal_blob}
            blob = make[case["network"]](0, dist=dist)
        _codecs[key] = binding.Codec(blob, 0)
    return _codecs[key]


def _images(n, h, w, seed):
    """Pictures of the kind `synth.make_image` makes, made on the GPU: blobs, a gradient and a little noise."""
    g = torch.Generator(device="cuda").manual_seed(seed)
    rand = lambda *shape: torch.rand(*shape, generator=g, device="cuda")    # noqa: E731
    out = torch.empty((n, h, w, 3), dtype=torch.uint8, device="cuda")
    side, blobs = math.sqrt(h * w), 32
    ys, xs = torch.arange(h, device="cuda", dtype=torch.float32), torch.arange(w, device="cuda", dtype=torch.float32)
    for i in range(n):
        sigma = side * (1 / 64 + (1 / 8 - 1 / 64) * rand(blobs))
        gy = torch.exp(-0.5 * ((ys[:, None] - h * rand(blobs)) / sigma) ** 2)
        gx = torch.exp(-0.5 * ((xs[:, None] - w * rand(blobs)) / sigma) ** 2)
        amplitude, slope = 160 * rand(3, blobs), 128 * rand(3) - 32
        for ch in range(3):
            picture = torch.addmm((slope[ch] * (ys / h)[:, None]).expand(h, w), gy * amplitude[ch], gx.t())
            picture = picture + 3.0 * torch.randn(h, w, generator=g, device="cuda")
            out[i, :, :, ch] = picture.round().clamp(0, 255).to(torch.uint8)
    return out


def prepare(case, seed):
    n, h, w = case["n"], case["h"], case["w"]
    state = {"call": case["call"], "codec": _codec(case), "size": (n, h, w)}
    image = _images(n, h, w, seed)
    if case["call"] in ("encode", "probs"):
        state["image"] = image
    if case["call"] == "encode":
        state["out"] = torch.zeros(binding.pcc_stream_bound(n, h, w), dtype=torch.uint8, device="cuda")
    elif case["call"] != "probs":
        state["stream"] = state["codec"].pcc_encode(image).clone()
        state["out"] = torch.empty_like(image)
    return state


def run(state):
    codec, call = state["codec"], state["call"]
    if call == "encode":
        # the stream is the front of the caller's buffer; the rest of the buffer stays as it was
        return {"bytes": codec.pcc_encode(state["image"], out=state["out"]).numel(), "buffer": state["out"]}
    if call == "decode":
        return codec.pcc_decode(state["stream"], *state["size"], out=state["out"])
    if call == "decode_static":
        return codec.pcc_decode_static(state["stream"], *state["size"], out=state["out"])
    return codec.pcc_encode_probs(state["image"])


def work(case):
    dims, pixels, rows = WIDTHS[case["network"]], case["n"] * case["h"] * case["w"], case["n"] * case["h"]
    macs = sum(a * b for a, b in zip(dims[:-1], dims[1:]))
    weights = 2 * macs                                    # bf16, once
    image = 3 * pixels
    # about 9 bits a sub-pixel with random weights, 4.4 with the plane predictor; an offset and two states a row
    bits = 4.4 if case["weights"] == "predictor" else 9.0
    stream = 3 * pixels * bits / 8 + 24 * rows
    outputs = 4 * (dims[-1] + 1) * pixels                 # head outputs and bits, fp32
    return {"bytes": image + weights + (outputs if case["call"] == "probs" else stream), "flops": 2 * macs * pixels}


def tolerance(case):
    # Streams and images are bytes.  Head outputs are sums of fp32 products of bf16 weights with activations of
    # 16 significant bits (two bf16).
    return {"rel": 2e-5} if case["call"] == "probs" else "exact"
