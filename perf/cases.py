"""The filter bank's work as its users' programs call it: the cases whose
speed is followed, and how to make, run and check one.

A case is a dict of plain values. `kind` says which entry point it goes
through, with C channels, T taps, S filtered spectra per stream, B streams and
the storage type of the samples:

  forward  Plan.execute: frequency spectra of B recorded streams
  fir      the same with FIR_ONLY: filtered spectra, no transform
  stream   Plan.execute_stream: the next S spectra of continuing streams
  step     Plan.execute and Plan.backward with kept buffers: a training step
  autograd pfb.pfb and torch.autograd.grad: the filter bank as a layer
  subbands VegasPlan.execute: NS polarisation-interleaved sub-bands
  beams    BatchedPlan.execute: many beams of uneven shape in one call
"""
from __future__ import annotations

import math

import torch

from paper_1511_03599_amd import pfb, synth

DEVICE = "cuda"
POWERS = (32, 64, 128, 256, 512, 1024, 2048, 4096, 8192)
MIXED = (96, 240, 384, 640, 768, 1000, 1344, 1536, 2560, 3072, 5120, 6144, 7168)
DTYPES = ("c64", "ci16", "ci8", "cf16")


def listed():
    return [
        # the smallest: one short block of a live stream, where latency counts
        dict(name="live_block", kind="stream", C=1024, T=16, S=64, B=1, dtype="ci16"),
        # a short recording through a small filter bank
        dict(name="small_recording", kind="forward", C=256, T=8, S=4096, B=1, dtype="c64"),
        # the filter bank as a layer of a small model: odd sizes, both gradients
        dict(name="small_layer", kind="autograd", C=512, T=12, S=1001, B=3, dtype="c64"),
        # a receiver's stream, chunk after chunk
        dict(name="receiver_chunk", kind="stream", C=1024, T=16, S=16384, B=1, dtype="ci16"),
        # several half-precision streams of a length that fits no tile
        dict(name="ragged_fp16", kind="forward", C=2048, T=12, S=5003, B=3, dtype="cf16"),
        # long filters: the tap sweep's 32-tap point
        dict(name="taps_32", kind="forward", C=1024, T=32, S=65536, B=1, dtype="c64"),
        # 8-bit recordings at high frequency resolution
        dict(name="fine_int8", kind="forward", C=4096, T=16, S=32768, B=1, dtype="ci8"),
        # a channel count that is no power of two
        dict(name="mixed_radix", kind="forward", C=3072, T=16, S=43690, B=1, dtype="c64"),
        # a dual-polarisation spectrometer's sub-bands
        dict(name="subbands_int8", kind="subbands", C=4096, T=16, S=2048, NS=8, dtype="ci8"),
        # a training step at high frequency resolution
        dict(name="fine_step", kind="step", C=4096, T=16, S=8192, B=2, dtype="c64"),
        # the differentiable workload at its full size
        dict(name="full_step", kind="step", C=1024, T=16, S=8192, B=32, dtype="c64"),
        # the largest: a table of 64 uneven beams in one call
        dict(name="beams_64", kind="beams", NB=64, table=1511400),
    ]


def _log(rng, lo, hi):
    """A whole number of [lo, hi], spread evenly over its logarithm."""
    return max(lo, min(hi, int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))))


def draw(rng):
    kind = rng.choice(("forward", "forward", "forward", "stream", "stream", "step", "autograd", "autograd", "fir",
                       "subbands", "beams"))
    if kind == "beams":
        return dict(kind=kind, NB=_log(rng, 4, 48), table=rng.randrange(1, 1 << 24))
    dtype = rng.choice(DTYPES)
    if kind == "subbands":
        C, T = rng.choice((512, 1024, 2048, 4096)), rng.randrange(4, 33)
        total = _log(rng, 1 << 18, 1 << 27)
        NS = rng.randrange(1, 17)
        return dict(kind=kind, C=C, T=T, S=max(1, total // (2 * C * NS)), NS=NS, dtype=dtype)
    total = _log(rng, 1 << 16, 1 << 27)  # new samples of a pass
    if kind in ("step", "autograd"):
        C, T, dtype = rng.choice(POWERS[2:]), rng.randrange(3, 33), "c64"
    elif kind == "stream":
        C, T = rng.choice(POWERS[3:]), rng.randrange(4, 33)
    else:
        C = rng.choice(POWERS if rng.random() < 0.75 else MIXED)
        T = rng.randrange(3, 17) if rng.random() < 0.6 else _log(rng, 17, 192)
    B = min(_log(rng, 1, 32), max(1, total // (8 * C)))
    return dict(kind=kind, C=C, T=T, S=max(1, total // (B * C)), B=B, dtype=dtype)


def _beams(case):
    return [(b.C, b.T, b.S) for b in synth.beam_table(case["NB"], seed=case["table"])]


def _taps(C, T):
    return torch.from_numpy(synth.windowed_sinc_taps(C, T)).to(DEVICE)


def _samples(case, seed, lead, C):
    """Receiver noise and, in the complex64 streams, a tone in one channel."""
    x = synth.device_quantised_noise(lead, case.get("dtype", "c64"), seed, DEVICE)
    if x.is_complex():
        n = torch.arange(C, dtype=torch.float64, device=DEVICE)
        x += torch.polar(torch.ones_like(n), n * (2.0 * math.pi * (1 + seed % (C - 1)) / C)).to(torch.complex64)
    return x


def prepare(case, seed):
    kind = case["kind"]
    if kind == "beams":
        beams = _beams(case)
        return dict(kind=kind, plan=pfb.BatchedPlan(beams),
                    xs=[_samples(case, 64 * seed + i, (S + T - 1, C), C) for i, (C, T, S) in enumerate(beams)],
                    hs=[_taps(C, T) for (C, T, S) in beams])
    C, T, S = case["C"], case["T"], case["S"]
    h = _taps(C, T)
    if kind == "subbands":
        return dict(kind=kind, plan=pfb.VegasPlan(C, case["NS"], T, S, case["dtype"]), h=h,
                    x=_samples(case, seed, (S + T - 1, case["NS"], C, 2), 2))
    B = case["B"]
    s = dict(kind=kind, h=h)
    if kind != "autograd":
        flags = {"stream": pfb.STREAMING, "fir": pfb.FIR_ONLY}.get(kind, 0)
        s["plan"] = pfb.Plan(C, T, S, B, case["dtype"], flags)
    if kind == "stream":
        s["x"] = s["plan"].stream_buffer(DEVICE)
        s["x"][:, T - 1:] = _samples(case, seed, (B, S, C), C)
        return s
    if kind not in ("step", "autograd"):
        s["x"] = _samples(case, seed, (B, S + T - 1, C), C)
        return s
    s["x"] = synth.device_tone_streams(B, C, T, S, seed, DEVICE)
    s["gY"] = synth.device_noise((B, S, C), seed + 1, DEVICE)
    if kind == "autograd":
        s["x"].requires_grad_(True)
        s["h"].requires_grad_(True)
    else:
        s["Y"] = torch.empty_like(s["gY"])
        s["gx"] = torch.empty_like(s["x"])
        s["gh"] = torch.empty_like(h)
    return s


def run(s):
    kind = s["kind"]
    if kind == "beams":
        return s["plan"].execute(s["xs"], s["hs"])
    if kind == "stream":
        return s["plan"].execute_stream(s["x"], s["h"])
    if kind == "step":
        Y = s["plan"].execute(s["x"], s["h"], Y=s["Y"])
        gx, gh = s["plan"].backward(s["x"], s["h"], s["gY"], gx=s["gx"], gh=s["gh"])
        return [Y, gx, gh]
    if kind == "autograd":
        Y = pfb.pfb(s["x"], s["h"])
        gx, gh = torch.autograd.grad(Y, (s["x"], s["h"]), s["gY"])
        return [Y, gx, gh]
    return s["plan"].execute(s["x"], s["h"])


def _one(C, T, S, width, dtype, fft=True):
    """Bytes and operations of one forward stream of `width` columns."""
    bytes_ = (S + T - 1) * width * synth.BYTES_PER_SAMPLE[dtype] + 4 * T * C + 8 * S * width
    return bytes_, S * width * (4 * T + (5 * math.log2(C) if fft else 0))


def work(case):
    if case["kind"] == "beams":
        each = [_one(C, T, S, C, "c64") for (C, T, S) in _beams(case)]
    elif case["kind"] == "subbands":
        each = [_one(case["C"], case["T"], case["S"], 2 * case["C"] * case["NS"], case["dtype"])]
    else:
        C, T, S, B = case["C"], case["T"], case["S"], case["B"]
        each = [_one(C, T, S, C, case["dtype"], case["kind"] != "fir")] * B
        if case["kind"] in ("step", "autograd"):
            # the adjoint reads the spectra's gradient and the samples and
            # writes the samples' gradient; three contractions of T taps in all
            each += [(8 * C * (S + 2 * (S + T - 1)) + 4 * T * C, S * C * (8 * T + 5 * math.log2(C)))] * B
    return {"bytes": float(sum(b for b, _ in each)), "flops": float(sum(f for _, f in each))}


def _wide(x):
    return x.detach().to(torch.complex128) if x.is_complex() else torch.view_as_complex(x.double())


def _fir(x, h, S):
    """y[s][c] = sum over t of h[t][c] x[s+t][c] (rows lead)."""
    y = h[0] * x[:S]
    for t in range(1, h.shape[0]):
        y += h[t] * x[t:t + S]
    return y


def exact(case, seed):
    s = prepare(case, seed)
    kind = s["kind"]
    if kind == "beams":
        return [torch.fft.fft(_fir(_wide(x), h.double(), S))
                for x, h, (C, T, S) in zip(s["xs"], s["hs"], _beams(case))]
    x, h, S, T = s["x"].detach(), s["h"].detach().double(), case["S"], case["T"]
    if kind == "subbands":
        y = _fir(_wide(x), h[:, None, :, None], S)
        return torch.fft.fft(y, dim=2)
    if kind == "fir":
        return torch.stack([_fir(_wide(xb), h, S) for xb in x])
    Y = torch.stack([torch.fft.fft(_fir(_wide(xb), h, S)) for xb in x])
    if kind not in ("step", "autograd"):
        return Y
    gx = torch.zeros(x.shape, dtype=torch.complex128, device=x.device)
    gh = torch.zeros_like(h)
    for b in range(x.shape[0]):
        gy = torch.fft.ifft(s["gY"][b].to(torch.complex128), norm="forward")
        xb = _wide(x[b])
        for t in range(T):
            gx[b, t:t + S] += h[t] * gy
            gh[t] += (gy.real * xb[t:t + S].real + gy.imag * xb[t:t + S].imag).sum(0)
    return [Y, gx, gh]
