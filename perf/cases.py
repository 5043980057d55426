"""The work that users of the library have it do, as measurable cases.

A case is one of
  plan    one execute of a plan: `batch` transforms of `n` points, out of place
  uneven  one replay of an uneven batch: `count` transforms, N = 2^U with U
          uniform in log_lo .. log_hi
  slot    one step of a serving slot: `count` requests of the serving trace
          (N = 2^U as above, 1 .. batch_hi transforms each) put into the
          slot's buffer and transformed there in place
Inputs are drawn on the GPU from the seed: uniform [-1, 1), N(0, 1), or eight
unit tones with N(0, 0.01) noise (binary16: scaled down by a power of two, so
that the unnormalised transform of a long signal stays in range).
"""
import math
import random

import torch

from paper_2604_00567_amd import binding

_STORE = {"f16": torch.float16, "f32": torch.float32, "f16f32": torch.float16}
_BYTES = {"f16": 4, "f32": 8, "f16f32": 4}
_MAX_ELEMS = 1 << 26


def _plan(dtype, n, batch, data, direction="forward", radix=2):
    return {"kind": "plan", "dtype": dtype, "n": n, "batch": batch, "data": data, "direction": direction,
            "radix": radix}


def _uneven(dtype, count, log_lo, log_hi, sizes_seed):
    return {"kind": "uneven", "dtype": dtype, "count": count, "log_lo": log_lo, "log_hi": log_hi,
            "sizes_seed": sizes_seed, "data": "uniform"}


def _slot(dtype, count, log_lo, log_hi, batch_hi, sizes_seed):
    return {"kind": "slot", "dtype": dtype, "count": count, "log_lo": log_lo, "log_hi": log_hi,
            "batch_hi": batch_hi, "sizes_seed": sizes_seed, "data": "normal"}


def listed():
    return [
        # a few binary32 transforms: the call's latency
        dict(_plan("f32", 1024, 16, "normal"), name="f32 1024 x 16"),
        # one serving request of long binary16 transforms, alone on the GPU
        dict(_plan("f16", 1 << 16, 3, "normal"), name="f16 2^16 x 3"),
        # one serving request of the longest size, binary32, on the way back
        dict(_plan("f32", 1 << 18, 7, "normal", direction="inverse"), name="f32 2^18 x 7 inverse"),
        # an odd number of mid-size binary32 transforms, inverse (filter and return)
        dict(_plan("f32", 1 << 13, 1001, "normal", direction="inverse"), name="f32 2^13 x 1001 inverse"),
        # the benchmark's batched fixed-size workload
        dict(_plan("f16", 1024, 65536, "uniform"), name="f16 1024 x 65536"),
        # the same with binary32 butterflies on binary16 data
        dict(_plan("f16f32", 1024, 65536, "uniform"), name="f16f32 1024 x 65536"),
        # the radix-4 form at the benchmark's second fixed size
        dict(_plan("f16", 4096, 16384, "uniform", radix=4), name="f16 4096 x 16384 radix 4"),
        # the long-transform sweep, binary16: the largest whole transform and the smallest split one
        dict(_plan("f16", 1 << 16, 1024, "tones"), name="f16 2^16 x 1024"),
        dict(_plan("f16", 1 << 17, 512, "tones"), name="f16 2^17 x 512"),
        # the end of the same sweep, binary32
        dict(_plan("f32", 1 << 20, 64, "tones"), name="f32 2^20 x 64"),
        # the uneven batch of the benchmark
        dict(_uneven("f16", 4096, 6, 16, 3), name="f16 uneven 4096"),
        # one step of a busy serving slot
        dict(_slot("f16", 12, 8, 18, 64, 6), name="f16 slot 12 requests"),
    ]


def _log_int(rng, lo, hi):
    return max(lo, min(hi, int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))))


def draw(rng):
    what = rng.random()
    if what < 0.12:
        lo = rng.randint(2, 10)
        hi = rng.randint(max(lo, 8), 18 if rng.random() < 0.3 else 16)
        most = max(1, _MAX_ELEMS // 4 // ((1 << hi + 1) // (hi - lo + 1)))
        return _uneven(rng.choice(["f16", "f16", "f32"]), _log_int(rng, 1, min(4096, most)), lo, hi,
                       rng.randrange(1 << 30))
    if what < 0.24:
        lo = rng.randint(6, 10)
        hi = rng.randint(12, 18)
        count = _log_int(rng, 1, 12)
        most = max(1, _MAX_ELEMS // 4 // (count * (1 << hi) // (hi - lo + 1)))
        return _slot(rng.choice(["f16", "f16", "f32"]), count, lo, hi, _log_int(rng, 1, min(64, most)),
                     rng.randrange(1 << 30))
    dtype = rng.choice(["f16", "f16", "f16", "f32", "f32", "f16f32"])
    # sizes from a few points to the largest, the usual ones more often
    log_n = rng.choice([rng.randint(1, 20), rng.randint(8, 18)])
    n = 1 << log_n
    batch = _log_int(rng, 1, max(1, _MAX_ELEMS // n))
    radix = 4 if dtype != "f16f32" and log_n <= 13 and rng.random() < 0.12 else 2
    data = "tones" if log_n >= 10 and rng.random() < 0.3 else ("uniform" if dtype != "f32" else "normal")
    return _plan(dtype, n, batch, data, rng.choice(["forward", "forward", "inverse"]), radix)


def _sizes(case):
    """(points, transforms) of each request of an uneven batch or serving step."""
    rng = random.Random(case["sizes_seed"])
    n = [1 << rng.randint(case["log_lo"], case["log_hi"]) for _ in range(case["count"])]
    return n, [rng.randint(1, case.get("batch_hi", 1)) for _ in n]


def _tones(n, batch, dtype, gen):
    # one tone in each eighth of the band (n >= 1024 here)
    f = (torch.arange(8, device="cuda") * (n // 8) +
         torch.randint(0, n // 8, (batch, 8), device="cuda", generator=gen))
    scale = 2.0 ** -max(0, n.bit_length() - 1 - 12) if dtype != "f32" else 1.0
    x = torch.randn(batch, n, 2, device="cuda", generator=gen).mul_(0.01)
    t = torch.arange(n, device="cuda")
    rows = max(1, (1 << 22) // n)
    for b in range(0, batch, rows):
        for k in range(8):
            phase = (f[b:b + rows, k, None] * t & (n - 1)).double() * (2 * math.pi / n)
            x[b:b + rows, :, 0] += phase.cos()
            x[b:b + rows, :, 1] += phase.sin()
    return x.mul_(scale).to(_STORE[dtype])


def _input(case, seed):
    gen = torch.Generator(device="cuda").manual_seed(seed)
    if case["kind"] == "plan":
        shape = (case["batch"], case["n"], 2)
        if case["data"] == "tones":
            return _tones(case["n"], case["batch"], case["dtype"], gen)
    else:
        shape = (sum(n * b for n, b in zip(*_sizes(case))), 2)
    if case["data"] == "normal":
        x = torch.randn(shape, device="cuda", generator=gen)
    else:
        x = torch.rand(shape, device="cuda", generator=gen).mul_(2).sub_(1)
    return x.to(_STORE[case["dtype"]])


class _Slot:
    """A serving slot, with the capacities that its requests need."""

    def __init__(self, case):
        self.n, self.batch = _sizes(case)
        elems = [n * b for n, b in zip(self.n, self.batch)]
        self.off = [sum(elems[:i]) for i in range(len(elems))]
        transforms = sum(self.batch)
        self.handle = binding.fft_serve_slot_create(case["dtype"], "dual_select", 64 * transforms, transforms,
                                                    transforms, sum(elems) * _BYTES[case["dtype"]])

    def launch(self, data):
        binding.fft_serve_slot_launch(self.handle, self.n, self.batch, self.off, data.data_ptr(),
                                      torch.cuda.current_stream().cuda_stream)

    def __del__(self):
        if getattr(self, "handle", None):
            binding.fft_serve_slot_destroy(self.handle)


def prepare(case, seed):
    x = _input(case, seed)
    state = {"kind": case["kind"], "x": x, "y": torch.empty_like(x)}
    if case["kind"] == "plan":
        state["plan"] = binding.Plan(case["n"], case["batch"], case["dtype"], "dual_select",
                                     direction=case["direction"], radix=case["radix"])
    elif case["kind"] == "uneven":
        state["plan"] = binding.Batch(_sizes(case)[0], case["dtype"], "dual_select")
    else:
        state["plan"] = _Slot(case)
    return state


def run(state):
    x, y, plan = state["x"], state["y"], state["plan"]
    if state["kind"] == "slot":
        y.copy_(x)             # the requests' payload arrives in the slot's buffer
        plan.launch(y)
    else:
        plan.execute(x, y)
    return y


def work(case):
    if case["kind"] == "plan":
        sizes = [(case["n"], case["batch"])]
    else:
        sizes = list(zip(*_sizes(case)))
    elems = sum(n * b for n, b in sizes)
    # six FMAs a butterfly: 6 n log2 n operations of two
    flops = sum(6 * b * n * (n.bit_length() - 1) for n, b in sizes)
    # one read and one write of the data (a slot's step: of the payload's arrival too)
    return {"bytes": elems * _BYTES[case["dtype"]] * (4 if case["kind"] == "slot" else 2), "flops": flops}


def exact(case, seed):
    x = _input(case, seed).cpu()

    def transform(part):
        z = torch.view_as_complex(part.double().contiguous())
        if case.get("direction") == "inverse":
            return torch.view_as_real(torch.fft.ifft(z, norm="forward"))
        return torch.view_as_real(torch.fft.fft(z))

    if case["kind"] == "plan":
        return transform(x)
    out, at = [], 0
    for n, b in zip(*_sizes(case)):
        out.append(transform(x[at:at + n * b].view(b, n, 2)).reshape(-1, 2))
        at += n * b
    return torch.cat(out)
