"""The calls whose speed counts, as a program that serves a quantised model makes them.

A case is one linear layer shape, called through the binding once per weight matrix.  `layers`
matrices of that shape are gone through in turn, each with activations and an output of its own,
as the layers of a decoder are in one step: with many of them the weights come from memory and
not from a cache, with one of them the call's own latency is what counts.

  m             activation rows: sequences in a decode step, or tokens of a prompt (prefill)
  n, k          output and input width
  g             group size of the scales and zero points
  bits          width of the packed fields
  act_order     weights in GPTQ's activation order: sorted once per matrix when the model is loaded,
                the activations gathered on every call

split_k is left to the library everywhere, as it is by a program that does not tune by hand.
"""
import math

import torch

from paper_2402_00025_amd import binding
from paper_2402_00025_amd.inputs import SCALE_HI, SCALE_LO, algorithmic_bytes

#: columns per zero-point word (three words for 3-bit fields): n is a multiple of it
_COLUMNS = {8: 8, 4: 8, 3: 32, 2: 16}
_GEMM = {8: "w8a16_gemm", 4: "w4a16_gemm", 3: "w3a16_gemm", 2: "w2a16_gemm"}


def _case(m, n, k, g=128, bits=4, layers=1, act_order=False):
    return dict(m=m, n=n, k=k, g=g, bits=bits, layers=layers, act_order=act_order)


def listed():
    return [
        # one call on a small matrix: all latency
        dict(_case(1, 1024, 1024), name="call_m1_1024"),
        # decode of one sequence through the square projections of 32 layers
        dict(_case(1, 4096, 4096, layers=32), name="decode_m1_4096"),
        # decode of sixteen sequences through the same: the headline shape
        dict(_case(16, 4096, 4096, layers=32), name="decode_m16_4096"),
        # decode of a few sequences, feed-forward projection, neither side a power of two
        dict(_case(3, 11008, 4096, layers=8), name="decode_m3_11008x4096"),
        # decode with fine groups, the feed-forward's projection back down
        dict(_case(1, 5120, 13824, g=32, layers=4), name="decode_m1_5120x13824_g32"),
        # decode on the largest square matrix: a stream
        dict(_case(8, 16384, 16384, layers=2), name="decode_m8_16384"),
        # decode of a large batch
        dict(_case(64, 8192, 8192, layers=4), name="batch_m64_8192"),
        # a short prompt, or one chunk of a long one, of no round length
        dict(_case(333, 11008, 4096, layers=2), name="chunk_m333_11008x4096"),
        # a long prompt: as much arithmetic as memory traffic is the least of it
        dict(_case(2048, 8192, 8192), name="prefill_m2048_8192"),
        # 8-bit fields, decode
        dict(_case(16, 8192, 8192, bits=8, layers=4), name="decode_w8_m16_8192"),
        # 3-bit fields (2-bit ones take the same route), decode
        dict(_case(2, 4096, 4096, bits=3, layers=16), name="decode_w3_m2_4096"),
        # weights in activation order, decode
        dict(_case(16, 4096, 4096, layers=16, act_order=True), name="decode_m16_4096_act_order"),
    ]


def _between(rng, low, high):
    """A whole number from low to high, evenly over its logarithm."""
    return min(high, max(low, round(math.exp(rng.uniform(math.log(low), math.log(high))))))


def draw(rng):
    bits = rng.choice((4, 4, 4, 4, 4, 4, 8, 8, 3, 2))
    g = rng.choice((128, 128, 128, 128, 64, 32, 256))
    low, high = rng.choice(((1, 16), (1, 16), (17, 64), (65, 2048)))
    m = _between(rng, low, high)
    unit_n, unit_k = _COLUMNS[bits], g
    if rng.random() < 0.5:  # half of all widths are multiples of 128, as most models' are
        unit_n, unit_k = 128, max(128, g)
    while True:
        n = _between(rng, 1024, 28672) // unit_n * unit_n
        k = _between(rng, 1024, 28672) // unit_k * unit_k
        # a matrix of at most 2^28 fields, and half of the arithmetic of the largest listed case
        # (a sixteenth where the groups are fine: a long prompt may then cost more time per operation)
        most = 1 << (36 if g >= 128 else 33)
        if n >= 1024 and k >= 1024 and n * k <= 1 << 28 and m * n * k <= most:
            break
    most = max(1, min(32, (256 << 20) * 8 // (n * k * bits), most // (m * n * k)))
    layers = _between(rng, 1, most)
    act_order = bits == 4 and rng.random() < 0.15
    return _case(m, n, k, g, bits, layers, act_order)


def _words(gen, *shape):
    return torch.randint(-(1 << 31), 1 << 31, shape, dtype=torch.int32, device="cuda", generator=gen)


def prepare(case, seed):
    m, n, k, g, bits = (case[x] for x in ("m", "n", "k", "g", "bits"))
    gen = torch.Generator(device="cuda").manual_seed(seed)
    layers = []
    for _ in range(case["layers"]):
        a = torch.randn((m, k), dtype=torch.float32, device="cuda", generator=gen).half()
        qweight = _words(gen, k * bits // 32, n)
        scales = torch.rand((k // g, n), dtype=torch.float32, device="cuda", generator=gen)
        scales = (SCALE_LO + (SCALE_HI - SCALE_LO) * scales).half()
        qzeros = _words(gen, k // g, n * bits // 32)
        c = torch.zeros((m, n), dtype=torch.float16, device="cuda")
        if case["act_order"]:
            g_idx = (torch.randperm(k, device="cuda", generator=gen) // g).int()
            packed, perm = torch.empty_like(qweight), torch.empty_like(g_idx)
            status = torch.empty(1, dtype=torch.int32, device="cuda")
            binding.w4a16_actorder_prepare(qweight, g_idx, packed, perm, status, n, k, g)
            layers.append((a, packed, scales, qzeros, perm, torch.empty_like(a), c))
        else:
            layers.append((a, qweight, scales, qzeros, c))
    gemm = binding.w4a16_gemm_actorder if case["act_order"] else getattr(binding, _GEMM[bits])
    return gemm, layers, (m, n, k, g)


def run(state):
    gemm, layers, (m, n, k, g) = state
    for tensors in layers:
        gemm(*tensors, m, n, k, g, 0)
    return [tensors[-1] for tensors in layers]


def work(case):
    m, n, k, g, bits, layers = (case[x] for x in ("m", "n", "k", "g", "bits", "layers"))
    order = 4 * k if case["act_order"] else 0  # the permutation
    return {"bytes": layers * (algorithmic_bytes(m, n, k, g, bits) + order), "flops": layers * 2 * m * n * k}


def tolerance(case):
    # fp16 results (2e-4 of rounding in the 2-norm) whose partial sums along k may meet in fp16 as well,
    # up to 32 of them in either implementation
    return {"rel": 2e-3, "max": 1e-2}
