"""The transforms a program runs through this library, as timing cases.

Every case goes through the torch entry points (torch_api.fft, torch_api.ifft,
torch_api.fft_batched) with the plan, the output and the workspace made once,
as a program that transforms many signals of one shape keeps them.  Shapes,
bases and slab counts are those of inputs.CONFIGS, of the tests and of
bench.py; sizes are powers of two by the library's contract, so the ragged
ones are odd exponents, unequal sides and bases of which a side is no power
(mixed radix).
"""
from __future__ import annotations

import math

import torch

from paper_2609_06449_amd import inputs, paco, torch_api

DTYPES = {"fp32": paco.PACO_C64, "fp16x3": paco.PACO_C64_MFMA_FP16X3, "bf16x3": paco.PACO_C64_MFMA_BF16X3,
          "bf16x6": paco.PACO_C64_MFMA_BF16X6}


def _single(op, l1, l2, p, b, mixed=False, dt="fp32", gen="normal"):
    return dict(op=op, l1=l1, l2=l2, p=p, b=b, mixed=mixed, dt=dt, gen=gen)


def _batch(count, kmin, kmax, size_seed):
    return dict(op="batch", count=count, kmin=kmin, kmax=kmax, size_seed=size_seed, gen="normal")


def listed():
    cases = {
        # the smallest configured problem: one short signal, a call is latency
        "fft_2p12_64x64": _single("fft", 6, 6, 4, 4, gen="uniform"),
        # one audio- or radar-sized block, called in a loop
        "fft_2p16_256x256": _single("fft", 8, 8, 4, 4),
        # odd exponent, unequal sides, the way back
        "ifft_2p17_512x256": _single("ifft", 9, 8, 4, 2),
        # the ordinary call: a megapoint transform
        "fft_2p20_1024x1024": _single("fft", 10, 10, 8, 4),
        # the same a size up, the way back
        "ifft_2p22_2048x2048": _single("ifft", 11, 11, 16, 2),
        # the headline problem
        "fft_2p24_4096x4096": _single("fft", 12, 12, 64, 16),
        # the headline size in the most used matrix-core form, wide dynamic range
        "fft_2p24_4096x4096_fp16x3": _single("fft", 12, 12, 64, 16, dt="fp16x3", gen="loguniform"),
        # the configured 2^26 problem: unequal sides, wide dynamic range
        "fft_2p26_4096x16384": _single("fft", 12, 14, 64, 4, gen="loguniform"),
        # the largest size, square, literal base (mixed radix)
        "fft_2p28_16384x16384": _single("fft", 14, 14, 256, 16, mixed=True),
        # the largest size, non-square, literal base, the way back
        "ifft_2p28_8192x32768": _single("ifft", 13, 15, 128, 8, mixed=True),
        # the configured batch: thousands of transforms of uneven sizes, one launch
        "batch_4096_2p8_2p20": _batch(4096, 8, 20, 6),
        # many short transforms (spectrogram frames), one launch
        "batch_8192_2p6_2p12": _batch(8192, 6, 12, 6),
    }
    return [dict(case, name=name) for name, case in cases.items()]


def draw(rng):
    if rng.random() < 0.25:
        kmin = rng.randint(2, 14)
        kmax = rng.randint(kmin, min(20, kmin + 12))
        count = int(round(math.exp(rng.uniform(0.0, math.log(8192)))))
        count = max(1, min(count, (1 << 27) >> kmax))
        return _batch(count, kmin, kmax, rng.randint(1, 10**6))
    l = rng.randint(8, 27)
    l1 = min(max(l // 2 + rng.randint(-2, 2), max(2, l - 15)), 14, l - 2)
    l2 = l - l1
    t = rng.choice([1, 2, 3, 4])
    mixed = bool(l1 % t or l2 % t)
    p = 1 << rng.randint(1, max(1, min(l1, l2) - 4))
    dt = "fp32" if l < 18 or rng.random() < 0.75 else rng.choice(["fp16x3", "bf16x3", "bf16x6"])
    return _single(rng.choice(["fft", "ifft"]), l1, l2, p, 1 << t, mixed, dt,
                   rng.choice(["normal", "uniform", "loguniform"]))


def _sizes(case):
    return [int(n) for n in inputs.batch_sizes(case["count"], case["size_seed"], case["kmin"], case["kmax"])]


def _items(case):
    return sum(_sizes(case)) if case["op"] == "batch" else 1 << (case["l1"] + case["l2"])


def _signal(case, seed):
    """The case's input: the value distributions of inputs.py, drawn on the GPU."""
    n = _items(case)
    g = torch.Generator(device="cuda").manual_seed(seed)
    if case["gen"] == "normal":
        return torch.view_as_complex(torch.randn(n, 2, generator=g, device="cuda"))
    u = torch.rand(n, 2, generator=g, device="cuda")
    if case["gen"] == "uniform":
        return torch.view_as_complex(2.0 * u - 1.0)
    return torch.polar(10.0 ** (8.0 * u[:, 0] - 4.0), 2.0 * math.pi * u[:, 1])


def prepare(case, seed):
    x = _signal(case, seed)
    state = dict(case=case, x=x, out=torch.empty_like(x), ws=torch.empty_like(x))
    if case["op"] == "batch":
        # the default per-size plans: no timing runs at plan creation
        state["plan"] = paco.BatchPlan(_sizes(case), flags=paco.PACO_BATCH_NO_TUNE)
    else:
        state["args"] = (1 << case["l1"], 1 << case["l2"], case["p"], case["b"])
        state["kw"] = dict(dt=DTYPES[case["dt"]], mixed=case["mixed"])
        torch_api.get_plan(*state["args"], **state["kw"])
    return state


def run(state):
    op = state["case"]["op"]
    if op == "batch":
        return torch_api.fft_batched(state["x"], state["plan"], out=state["out"], workspace=state["ws"])
    f = torch_api.fft if op == "fft" else torch_api.ifft
    return f(state["x"], *state["args"], out=state["out"], workspace=state["ws"], **state["kw"])


def work(case):
    if case["op"] == "batch":
        return {"bytes": 16 * _items(case), "flops": sum(5 * n * (n.bit_length() - 1) for n in _sizes(case))}
    n = _items(case)
    return {"bytes": 16 * n, "flops": 5 * n * (n.bit_length() - 1)}


def exact(case, seed):
    x = _signal(case, seed).to(torch.complex128)
    if case["op"] == "fft":
        return torch.fft.fft(x)
    if case["op"] == "ifft":
        return torch.fft.ifft(x)
    # transforms of one size together, each back to its own place
    sizes = _sizes(case)
    offsets = [0]
    for n in sizes:
        offsets.append(offsets[-1] + n)
    y = torch.empty_like(x)
    for n in sorted(set(sizes)):
        at = [o for o, m in zip(offsets, sizes) if m == n]
        for s in range(0, len(at), max(1, (1 << 26) // n)):
            part = at[s:s + max(1, (1 << 26) // n)]
            f = torch.fft.fft(torch.stack([x[o:o + n] for o in part]))
            for i, o in enumerate(part):
                y[o:o + n] = f[i]
    return y
