"""Performance cases: what users of this library have it do, through its public entry points.

A case is a dict of plain values; `prepare` makes its inputs on the GPU from a seed, `run` is one call, `work` is what
the call cannot do without, `tolerance` how closely two correct implementations agree.  `listed()` names the standing
cases, `draw()` gives further ones of the same ranges.

Every program of this library keeps ONE context for its batches (the example queue of Sec. 2.2 hands it one batch after
another), so all states here share one, on the current stream.  Batches of unequal utterances come in another order, and
so with other offsets, for every seed; batches of equal ones keep theirs.
"""
from __future__ import annotations

import dataclasses
import functools
import math

import numpy as np
import torch

from paper_1912_11040_amd import workloads as W
from paper_1912_11040_amd.binding import Augmenter

FS, C = W.FS, W.SPEED_OF_SOUND
NOISE_KINDS = ("white", "pink", "babble")

# what a case holds, with the values of the plain front end
DEFAULTS = dict(call="pipeline", n_utt=1, min_len=16000, max_len=16000, n_noise=0, rir_len=0, n_mic=0, fixed_room=False,
                snr_lo=0.0, snr_hi=20.0, feature="power", n_mel=40, n_ceps=13, padded=False, warp=True, all_outputs=False)


def _case(name, **kw):
    return dict(DEFAULTS, name=name, **kw)


def listed():
    return [
        # One utterance of 1-4 s into a recogniser whose input holds 4 s: the front end alone, no warp.  The smallest
        # call a user makes; every request has a length of its own.
        _case("features_one", call="mel", n_utt=1, min_len=16000, max_len=64000, warp=False,
              padded=True),
        # A serving loop that may not allocate: 32 requests of 1-16 s, 80 log-mel channels.
        _case("features_static_ragged", call="mel_static", n_utt=32, min_len=16000, max_len=256000, warp=False,
              feature="log", n_mel=80),
        # A training batch of MFCCs in the padded layout of the trainer's queue.
        _case("mfcc_padded", call="mel", n_utt=256, min_len=16000, max_len=256000, feature="mfcc", padded=True),
        # A corpus pass of the front end: 4096 equal utterances of 8 s (the features-only configuration).
        _case("features", call="mel", n_utt=4096, min_len=128000, max_len=128000),
        # The smallest augmented batch: eight utterances of 1 s in one kind of room (the tiny configuration).
        _case("tiny", n_utt=8, n_noise=1, rir_len=4096, fixed_room=True, snr_lo=10.0, snr_hi=10.0),
        # An ordinary training batch: 64 x 4 s, random rooms, 8000-tap responses, one noise (the batch configuration).
        _case("batch", n_utt=64, min_len=64000, max_len=64000, n_noise=1, rir_len=8000),
        # The headline: 256 utterances of 1-16 s packed, three noises, 16000-tap responses.
        _case("varlen", n_utt=256, min_len=16000, max_len=256000, n_noise=3, rir_len=16000, snr_hi=30.0),
        # The largest: 1024 x 10 s, 32768-tap responses, two noises (the throughput configuration).
        _case("throughput", n_utt=1024, min_len=160000, max_len=160000, n_noise=2, rir_len=32768),
        # A bank of responses computed once and used for many epochs.
        _case("rir_bank", call="rir", n_utt=2000, rir_len=8000),
        # A two-microphone device (Sec. 4): the responses of 192 rooms at both microphones.
        _case("rir_two_mics", call="mics", n_utt=192, rir_len=16000, n_mic=2),
        # Reverberation with measured responses of an odd length, the mixture and the gains kept.
        _case("convolve_measured", call="convolve", n_utt=96, min_len=8001, max_len=200003, n_noise=2, rir_len=12001),
        # VTLP on the waveform before the simulator, the paper's own placement.
        _case("vtlp_waveform", call="resynth", n_utt=256, min_len=16000, max_len=256000),
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    """One more case: any of the calls, batch sizes from one utterance up, lengths from a fraction of a second to 16 s,
    responses from 1000 taps to the longest, no more work than the largest listed case."""
    call = rng.choice(["mel", "mel", "mel_static", "pipeline", "pipeline", "pipeline", "rir", "mics", "convolve", "resynth"])
    c = dict(DEFAULTS, call=call)
    c["n_utt"] = _log_int(rng, 1, {"mel": 4096, "mel_static": 1024, "rir": 3000, "mics": 700}.get(call, 1024))
    if call in ("rir", "mics"):
        c["rir_len"] = _log_int(rng, 1000, 32768)
        c["n_mic"] = rng.randint(2, 4) if call == "mics" else 0
    else:
        c["max_len"] = _log_int(rng, 4000, 256000)
        c["min_len"] = rng.choice([c["max_len"], max(1000, c["max_len"] // 16), max(1000, c["max_len"] // 4)])
        c["min_len"] = min(c["min_len"], c["max_len"])
    if call in ("pipeline", "convolve"):
        c["rir_len"] = rng.choice([4096, 8000, 16000, 32768, _log_int(rng, 1000, 32768), _log_int(rng, 1000, 32768)])
        c["n_noise"] = rng.choice([0, 1, 1, 2, 3])
        c["snr_hi"] = rng.choice([20.0, 30.0])
        c["all_outputs"] = call == "pipeline" and rng.random() < 0.25
    if call in ("mel", "mel_static", "pipeline"):
        c["feature"] = rng.choice(["power", "power", "log", "mfcc"])
        c["n_mel"] = rng.choice([40, 40, 23, 64, 80])
        c["n_ceps"] = 13
        c["padded"] = not c["all_outputs"] and c["min_len"] < c["max_len"] and rng.random() < 0.4
        c["warp"] = rng.random() < 0.7
    if call == "mel_static":       # within the entry point's limit on output rows
        c["n_utt"] = min(c["n_utt"], max(1, 4000000 // (c["max_len"] // 160 + 64)))
    cap = work(next(x for x in listed() if x["name"] == "throughput"))
    while c["n_utt"] > 1 and any(work(c)[k] > cap[k] for k in cap):
        c["n_utt"] = c["n_utt"] * 3 // 4
    return c


# ---- inputs ---------------------------------------------------------------------------------------------------------

@functools.lru_cache(maxsize=None)
def _context():
    return Augmenter(0)


def _lengths(c, rng):
    """Lengths of U[min, max]: evenly spread ones in an order of the seed's, so that every seed's packed batch has the same
    size; for padded batches, whose size does not depend on them, drawn one by one."""
    n, lo, hi = c["n_utt"], c["min_len"], c["max_len"]
    if c["padded"]:
        return rng.integers(lo, hi + 1, size=n).astype(np.int64)
    return rng.permutation(lo + ((np.arange(n) + 0.5) * (hi - lo) / n).astype(np.int64))


def _offsets(lengths):
    return np.concatenate([[0], np.cumsum(lengths)]).astype(np.int64)


def _ar2(rows, m, gen, rng):
    """Rows of noise through a two-pole resonance (r = 0.95, angle in [0.05 pi, 0.3 pi]), unit RMS, under a 4 Hz envelope."""
    theta = torch.from_numpy(rng.uniform(0.05 * np.pi, 0.3 * np.pi, (rows, 1))).to("cuda", torch.float32)
    phase = torch.from_numpy(rng.uniform(0.0, 2.0 * np.pi, (rows, 1))).to("cuda", torch.float32)
    w = torch.arange(m // 2 + 1, device="cuda", dtype=torch.float32) * (2.0 * math.pi / m)
    z = torch.polar(torch.ones_like(w), -w)[None, :]
    x = torch.fft.irfft(torch.fft.rfft(torch.randn(rows, m, device="cuda", generator=gen))
                        / (1.0 - 1.9 * torch.cos(theta) * z + 0.9025 * z * z), m)
    x /= x.square().mean(1, keepdim=True).sqrt()
    t = torch.arange(m, device="cuda", dtype=torch.float32) * (2.0 * math.pi * 4.0 / FS)
    return x * (0.55 + 0.45 * torch.sin(t[None, :] + phase))


def _rows(kind, rows, m, gen, rng):
    if kind == "speech":
        return _ar2(rows, m, gen, rng)
    if kind == "white":
        return torch.randn(rows, m, device="cuda", generator=gen)
    if kind == "pink":
        f = torch.arange(m // 2 + 1, device="cuda", dtype=torch.float32) * (FS / m)
        x = torch.fft.irfft(torch.fft.rfft(torch.randn(rows, m, device="cuda", generator=gen)) / f.clamp(min=20.0).sqrt(), m)
    else:
        x = sum(_ar2(rows, m, gen, rng) for _ in range(5))
    return x / x.square().mean(1, keepdim=True).sqrt()


def _packed(kind, lengths, gen, rng):
    """A packed signal array of this kind, in pieces of at most 2^25 samples at a time."""
    m = 1 << max(10, int(lengths.max() - 1).bit_length())
    step, parts = max(1, (1 << 25) // m), []
    for a in range(0, len(lengths), step):
        n = torch.from_numpy(lengths[a:a + step]).cuda()
        x = _rows(kind, len(n), m, gen, rng)
        parts.append(x[torch.arange(m, device="cuda")[None, :] < n[:, None]])
    return torch.cat(parts)


def _rooms(n, n_src, rng, fixed=False):
    """Geometry rows [n][n_src][10]: a room and a microphone per utterance, a position per source (0.5 m from every
    wall and 0.1 m from the microphone at least), as the workloads draw them."""
    dims = np.tile([5.0, 4.0, 3.0], (n, 1)) if fixed else rng.uniform([3.0, 3.0, 2.5], [10.0, 8.0, 4.0], (n, 3))
    beta = np.full(n, 0.7) if fixed else rng.uniform(0.2, 0.9, n)
    mic = 0.5 + rng.random((n, 3)) * (dims - 1.0)
    src = 0.5 + rng.random((n, n_src, 3)) * (dims - 1.0)[:, None]
    near = np.linalg.norm(src - mic[:, None], axis=2) < 0.1
    src[near] += np.array([0.15, 0.0, 0.0]) * np.where(src[near][:, :1] > 2.0, -1.0, 1.0)
    g = np.empty((n, n_src, 10), np.float32)
    g[:, :, 0:3], g[:, :, 3:6], g[:, :, 6:9], g[:, :, 9] = dims[:, None], src, mic[:, None], beta[:, None]
    return g


def _measured(n, n_src, length, gen, rng):
    """Responses as a measurement gives them: a direct path after 1-15 ms, then a noise tail that falls by 60 dB in 0.2-0.8 s."""
    delay = torch.from_numpy(rng.integers(16, min(240, max(17, length // 2)), (n, n_src, 1))).cuda()
    rate = torch.from_numpy(6.9078 / (rng.uniform(0.2, 0.8, (n, n_src, 1)) * FS)).to("cuda", torch.float32)
    t = torch.arange(length, device="cuda")[None, None, :] - delay
    tail = 0.05 * torch.randn(n, n_src, length, device="cuda", generator=gen) * torch.exp(-rate * t.clamp(min=0))
    return torch.where(t > 0, tail, (t == 0).float()).contiguous()


def _frontend(c):
    return dataclasses.replace(W.FrontendConfig(), feature=c["feature"], n_mel=c["n_mel"], n_ceps=c["n_ceps"])


def _frames(lengths, fe):
    return np.where(lengths >= fe.win, 1 + (lengths - fe.win) // fe.hop, 0)


def prepare(case, seed):
    c = dict(DEFAULTS, **case)
    rng = np.random.default_rng([seed & 0x7fffffff, 77])
    gen = torch.Generator("cuda").manual_seed(seed)
    call, n, n_noise = c["call"], c["n_utt"], c["n_noise"]
    s = dict(call=call, context=_context(), rir_len=c["rir_len"])
    dev = lambda a: torch.from_numpy(np.ascontiguousarray(a, np.float32)).cuda()          # noqa: E731
    empty = lambda *shape: torch.empty(shape, device="cuda")                               # noqa: E731
    if call in ("rir", "mics"):
        geom = _rooms(n, 1, rng)[:, 0]
        s["geom"] = dev(geom)
        if call == "mics":
            s["mics"] = dev(W.microphone_arrays(geom, c["n_mic"], seed=seed & 0x7fffffff))
        s["rir_out"] = empty(n, max(1, c["n_mic"]), c["rir_len"])
        return s
    lengths = _lengths(c, rng)
    s["offsets"] = _offsets(lengths)
    total = int(s["offsets"][-1])
    s["speech"] = _packed("speech", lengths, gen, rng)
    s["alpha"] = dev(rng.uniform(0.8, 1.2, n) if c["warp"] else np.ones(n))
    if call == "resynth":
        s["wave_out"] = empty(total)
        return s
    if call in ("pipeline", "convolve"):
        s["noise"] = torch.stack([_packed(NOISE_KINDS[j % 3], lengths, gen, rng) for j in range(n_noise)]) if n_noise else None
        s["snr"] = dev(rng.uniform(c["snr_lo"], c["snr_hi"], (n, n_noise))) if n_noise else None
    whole = call == "convolve" or c["all_outputs"]
    s["mixed_out"] = empty(total) if whole else None
    s["gains_out"] = empty(n, n_noise) if whole and n_noise else None
    s["rir_out"] = empty(n, 1 + n_noise, c["rir_len"]) if whole and call == "pipeline" else None
    if call == "convolve":
        s["rir"] = _measured(n, 1 + n_noise, c["rir_len"], gen, rng)
        return s
    if call == "pipeline":
        s["geom"] = dev(_rooms(n, 1 + n_noise, rng, c["fixed_room"]))
    fe = _frontend(c)
    frames = _frames(lengths, fe)
    s["frontend"] = fe
    most = int(_frames(np.int64(c["max_len"]), fe))                   # rows per utterance of the padded layout
    s["frame_offsets"] = np.arange(n + 1, dtype=np.int64) * most if c["padded"] else _offsets(frames)
    s["feats"] = empty(int(s["frame_offsets"][-1]), fe.feature_dim)
    return s


def run(s):
    aug, call = s["context"], s["call"]
    if call == "rir":
        aug.aug_rir_batch(s["geom"], s["rir_len"], FS, C, s["rir_out"])
        return s["rir_out"]
    if call == "mics":
        aug.aug_rir_mics_batch(s["geom"], s["mics"], s["rir_len"], FS, C, s["rir_out"])
        return s["rir_out"]
    if call == "resynth":
        aug.aug_vtlp_resynth_batch(s["offsets"], s["speech"], s["alpha"], s["wave_out"])
        return s["wave_out"]
    if call == "convolve":
        aug.aug_convolve_mix_batch(s["offsets"], s["speech"], s["noise"], s["rir"], s["rir_len"], s["snr"], s["mixed_out"],
                                   s["gains_out"])
        return [s["mixed_out"], s["gains_out"]]
    if call == "pipeline":
        aug.aug_pipeline_batch(s["offsets"], s["speech"], s["noise"], s["geom"], s["rir_len"], FS, C, s["snr"], s["alpha"],
                               s["frontend"], s["frame_offsets"], s["feats"], s["rir_out"], s["mixed_out"], s["gains_out"])
        return [s["feats"], s["rir_out"], s["mixed_out"], s["gains_out"]]
    features = aug.aug_vtlp_mel_batch_static if call == "mel_static" else aug.aug_vtlp_mel_batch
    features(s["offsets"], s["speech"], s["alpha"], s["frontend"], s["frame_offsets"], s["feats"])
    return s["feats"]


# ---- work and tolerance ---------------------------------------------------------------------------------------------

@functools.lru_cache(maxsize=None)
def _images_per_response(rir_len, fixed):
    """Expected number of image sources that add to a response: those within its reach (one per room volume) whose
    amplitude is at least 2^-57, half a unit of the sums; an image in direction u has about d sum(|u_i| / L_i) reflections."""
    g = _rooms(1 if fixed else 400, 1, np.random.default_rng(1), fixed)[:, 0].astype(np.float64)
    u = np.random.default_rng(2).standard_normal((256, 3))
    u = np.abs(u) / np.linalg.norm(u, axis=1, keepdims=True)
    per_metre = -np.log2(g[:, 9:10]) * ((1.0 / g[:, 0:3]) @ u.T)              # halvings of the amplitude per metre
    reach = rir_len * C / FS
    d = np.full(per_metre.shape, reach)
    for _ in range(30):
        d = np.minimum(reach, (57.0 - np.log2(4.0 * np.pi * np.maximum(d, 0.1))) / per_metre)
    return float(np.mean(4.0 * np.pi / 3.0 * np.mean(d ** 3, axis=1) / np.prod(g[:, 0:3], axis=1)))


def work(case):
    c = dict(DEFAULTS, **case)
    call, n, n_src, taps = c["call"], c["n_utt"], 1 + c["n_noise"], c["rir_len"]
    if call in ("rir", "mics"):
        n_rir = n * max(1, c["n_mic"])
        return {"bytes": 4.0 * n_rir * (10 + taps), "flops": 12.0 * n_rir * _images_per_response(taps, False)}
    mean = 0.5 * (c["min_len"] + c["max_len"])
    total = n * mean
    if call == "resynth":         # two 2048-point real transforms, the window and the interpolation per 400 samples
        return {"bytes": 8.0 * total, "flops": total / 400.0 * (2 * 2.5 * 2048 * 11 + 800 + 6 * 1025)}
    frames = n * max(0.0, 1.0 + (mean - 400) / 160.0)
    rows = n * max(0.0, 1.0 + (c["max_len"] - 400) / 160.0) if c["padded"] else frames
    width = c["n_ceps"] if c["feature"] == "mfcc" else c["n_mel"]
    # a 512-point real transform, window, powers, two weights per bin, the epilogue (a dot product each for cepstra)
    mel = {"bytes": 4.0 * total + 4.0 * rows * width,
           "flops": frames * (2.5 * 512 * 9 + 400 + 3 * 257 + 4 * 257 + 2 * c["n_mel"] + (2 * 13 * c["n_mel"] if width == 13 else 0))}
    if call in ("mel", "mel_static"):
        return mel
    # overlap-save with transforms of the power of two at or above twice the response
    nfft = 2 << max(0, (taps - 1).bit_length())
    conv = total * n_src * (2 * 2.5 * nfft * math.log2(nfft) + 6 * (nfft // 2 + 1)) / (nfft - taps + 1)
    signals = 4.0 * total * n_src
    if call == "convolve":
        return {"bytes": signals + 4.0 * n * n_src * taps + 4.0 * total, "flops": conv + 2.0 * total * (2 * n_src - 1)}
    images = 12.0 * n * n_src * _images_per_response(taps, c["fixed_room"])
    extra = 4.0 * (total + n * n_src * taps) if c["all_outputs"] else 0.0
    return {"bytes": signals + 40.0 * n * n_src + 4.0 * rows * width + extra,
            "flops": images + conv + 2.0 * total * (2 * n_src - 1) + mel["flops"]}


def tolerance(case):
    # 32-bit transforms and sums throughout; a feature of little energy shows more of their rounding than its
    # neighbours (a root or a logarithm of it), a sample next to a large one too
    return {"rel": 1e-5, "max": 1e-3 if case.get("call") in ("mel", "mel_static", "pipeline") else 1e-4}
