"""aug_convolve_mix_batch against the oracle's direct convolution and SNR mix."""
import numpy as np
import pytest

from oracle import aug_oracle as O
from paper_1912_11040_amd import workloads as W
from tests.parity import GAIN_TOL, WAVE_TOL, dev, wave_err

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def aug():
    from paper_1912_11040_amd.binding import Augmenter
    a = Augmenter(0)
    yield a
    a.close()


def _decaying_rirs(rng, n_utt, n_src, L):
    t = np.arange(L)
    h = rng.standard_normal((n_utt, n_src, L)) * np.exp(-t / (0.25 * L + 1.0))
    h[:, :, : min(8, L)] += 1.0
    return h.astype(np.float32)


def _run(aug, offsets, speech, noise, rir, snr):
    import torch
    n_utt = len(offsets) - 1
    n_noise = 0 if noise is None else noise.shape[0]
    mixed = torch.full((int(offsets[-1]),), float("nan"), dtype=torch.float32, device="cuda")
    gains = torch.full((n_utt, max(n_noise, 1)), float("nan"), dtype=torch.float32, device="cuda")
    aug.aug_convolve_mix_batch(offsets, dev(speech), None if noise is None else dev(noise), dev(rir),
                               rir.shape[-1], None if snr is None else dev(snr), mixed,
                               gains if n_noise else None)
    torch.cuda.synchronize()
    return mixed.cpu().numpy(), gains.cpu().numpy()[:, :n_noise]


def _check(aug, offsets, speech, noise, rir, snr, method="direct"):
    mixed, gains = _run(aug, offsets, speech, noise, rir, snr)
    ref, g_ref = O.convolve_mix_batch(offsets, speech, noise, rir.astype(np.float64), snr, method)
    assert not np.isnan(mixed).any()
    err = wave_err(mixed, ref, offsets)
    print(f"waveform max error / RMS = {err:.2e} (tolerance {WAVE_TOL:.0e})", flush=True)
    assert err <= WAVE_TOL
    if g_ref.size:
        np.testing.assert_allclose(gains, g_ref, rtol=GAIN_TOL)
    return mixed, ref


def test_tiny_config_with_oracle_rirs(aug):
    w = W.tiny()
    h, _ = O.rir_batch(w.geom.reshape(-1, 10), w.rir_len, w.fs, w.c)
    rir = h.reshape(w.n_utt, 2, w.rir_len).astype(np.float32)
    print("case: tiny, L=4096, direct oracle", flush=True)
    _check(aug, w.offsets, w.speech, w.noise, rir, w.snr_db)


def test_delta_response_is_a_shift(aug):
    rng = np.random.default_rng(0)
    x = rng.standard_normal(3000).astype(np.float32)
    rir = np.zeros((1, 1, 300), np.float32)
    rir[0, 0, 123] = 1.0
    offsets = np.array([0, 3000], np.int64)
    mixed, _ = _run(aug, offsets, x, None, rir, None)
    ref = np.concatenate([np.zeros(123), x[:-123].astype(np.float64)])
    err = wave_err(mixed, ref, offsets)
    print(f"delta shift: max error / RMS = {err:.2e}", flush=True)
    assert err <= WAVE_TOL


@pytest.mark.parametrize("L", [1, 17, 256, 700, 8000])
def test_ragged_lengths_and_response_sizes(aug, L):
    rng = np.random.default_rng(L)
    lens = [0, 1, 399, 5000, 0, 16384, 16385, 777]
    offsets = np.concatenate([[0], np.cumsum(lens)]).astype(np.int64)
    total = int(offsets[-1])
    speech = rng.standard_normal(total).astype(np.float32)
    noise = rng.standard_normal((2, total)).astype(np.float32)
    rir = _decaying_rirs(rng, len(lens), 3, L)
    snr = rng.uniform(0, 30, (len(lens), 2)).astype(np.float32)
    print(f"case: ragged lens, L={L}", flush=True)
    _check(aug, offsets, speech, noise, rir, snr)


def test_partitioned_response_32768_taps(aug):
    # responses longer than one LDS-resident transform are cut into partitions
    rng = np.random.default_rng(7)
    lens = [40000, 9000, 70001]
    offsets = np.concatenate([[0], np.cumsum(lens)]).astype(np.int64)
    total = int(offsets[-1])
    speech = rng.standard_normal(total).astype(np.float32)
    noise = rng.standard_normal((1, total)).astype(np.float32)
    rir = _decaying_rirs(rng, 3, 2, 32768)
    snr = np.array([[5.0], [0.0], [17.0]], np.float32)
    print("case: L=32768 partitioned, fft oracle + sampled direct sums", flush=True)
    mixed, ref = _check(aug, offsets, speech, noise, rir, snr, method="fft")
    # the fft oracle itself is tied to the direct sum at sampled positions of the speech path
    y_gpu, _ = _run(aug, offsets, speech, None, rir[:, :1], None)
    for u in range(3):
        a, b = offsets[u], offsets[u + 1]
        pos = rng.integers(0, b - a, 48)
        direct = O.convolve_at(speech[a:b], rir[u, 0], pos)
        rms = np.sqrt(np.mean(O.convolve_fft(speech[a:b], rir[u, 0]) ** 2))
        assert np.max(np.abs(y_gpu[a:b][pos] - direct)) <= WAVE_TOL * rms


def test_three_noise_sources_16000_taps(aug):
    rng = np.random.default_rng(11)
    lens = [20000, 33000]
    offsets = np.concatenate([[0], np.cumsum(lens)]).astype(np.int64)
    total = int(offsets[-1])
    speech = rng.standard_normal(total).astype(np.float32)
    noise = rng.standard_normal((3, total)).astype(np.float32)
    rir = _decaying_rirs(rng, 2, 4, 16000)
    snr = rng.uniform(0, 30, (2, 3)).astype(np.float32)
    print("case: L=16000, 3 noises, direct oracle", flush=True)
    _check(aug, offsets, speech, noise, rir, snr)


def test_whole_blocks_and_odd_starts_at_the_largest_transform(aug):
    # 16384-sample blocks: utterances that are exact multiples of the block (every window and output block
    # takes the untested two-sample path), one sample more, one sample in all, and odd start offsets, where
    # those 8-byte accesses are only 4-byte aligned
    rng = np.random.default_rng(13)
    lens = [16385, 32768, 1, 16384, 49155]
    offsets = np.concatenate([[0], np.cumsum(lens)]).astype(np.int64)
    assert offsets[1] % 2 == 1 and offsets[3] % 2 == 0 and offsets[4] % 2 == 0
    total = int(offsets[-1])
    speech = rng.standard_normal(total).astype(np.float32)
    noise = rng.standard_normal((1, total)).astype(np.float32)
    rir = _decaying_rirs(rng, len(lens), 2, 9000)
    snr = rng.uniform(0, 30, (len(lens), 1)).astype(np.float32)
    print("case: L=9000, whole 16384-sample blocks, odd starts", flush=True)
    _check(aug, offsets, speech, noise, rir, snr)


def test_more_blocks_than_work_groups_at_a_small_transform(aug):
    # Many short utterances with short responses: the block list (about 4500 blocks of 1024 samples) is longer
    # than the launch has work groups, so each group takes one or two blocks, a stride apart, of its XCD's
    # eighth of the list; some eighths are not a multiple of the stride long.  Every utterance is checked.
    rng = np.random.default_rng(12)
    n_utt, n_noise, L = 500, 2, 700
    lens = rng.integers(2100, 3100, n_utt)
    lens[:3] = [1, 1024, 3072]
    offsets = np.concatenate([[0], np.cumsum(lens)]).astype(np.int64)
    total = int(offsets[-1])
    speech = rng.standard_normal(total).astype(np.float32)
    noise = rng.standard_normal((n_noise, total)).astype(np.float32)
    rir = _decaying_rirs(rng, n_utt, 1 + n_noise, L)
    snr = rng.uniform(0, 20, (n_utt, n_noise)).astype(np.float32)
    blocks = int(np.sum((lens + 1023) // 1024)) * (1 + n_noise)
    print(f"case: {n_utt} utterances, L={L}, {blocks} blocks of 1024 samples", flush=True)
    assert blocks > 4096
    _check(aug, offsets, speech, noise, rir, snr, method="fft")


def test_most_noise_sources_the_interface_takes(aug):
    rng = np.random.default_rng(12)
    lens = [1500, 0, 2600, 700]
    offsets = np.concatenate([[0], np.cumsum(lens)]).astype(np.int64)
    total = int(offsets[-1])
    speech = rng.standard_normal(total).astype(np.float32)
    noise = rng.standard_normal((8, total)).astype(np.float32)
    rir = _decaying_rirs(rng, 4, 9, 300)
    snr = rng.uniform(-5, 30, (4, 8)).astype(np.float32)
    print("case: 8 noises, L=300, one empty utterance", flush=True)
    _check(aug, offsets, speech, noise, rir, snr)


def test_silent_noise_gets_zero_gain(aug):
    rng = np.random.default_rng(3)
    offsets = np.array([0, 2000], np.int64)
    speech = rng.standard_normal(2000).astype(np.float32)
    noise = np.zeros((1, 2000), np.float32)
    rir = _decaying_rirs(rng, 1, 2, 64)
    mixed, gains = _run(aug, offsets, speech, noise, rir, np.array([[10.0]], np.float32))
    assert gains[0, 0] == 0.0
    ref = O.convolve_direct(speech, rir[0, 0])
    assert wave_err(mixed, ref, offsets) <= WAVE_TOL


def test_noise_that_never_arrives_gets_zero_gain(aug):
    # The noise's response starts after the utterance has ended, so its reverberated signal is exactly zero
    # and the rule "zero energy gives gain 0" applies; a transform-based convolution returns rounding noise
    # there, which must not be mistaken for a signal (its gain would be astronomical).
    rng = np.random.default_rng(17)
    lens = [1500, 900]
    offsets = np.concatenate([[0], np.cumsum(lens)]).astype(np.int64)
    total = int(offsets[-1])
    speech = rng.standard_normal(total).astype(np.float32)
    noise = rng.standard_normal((2, total)).astype(np.float32)
    rir = _decaying_rirs(rng, 2, 3, 4000)
    rir[0, 1, :1500] = 0.0          # utterance 0, noise 0: first tap at 1500 = its length
    rir[1, 0, :900] = 0.0           # utterance 1: the speech itself never arrives
    snr = np.full((2, 2), 5.0, np.float32)
    mixed, gains = _run(aug, offsets, speech, noise, rir, snr)
    ref, g_ref = O.convolve_mix_batch(offsets, speech, noise, rir.astype(np.float64), snr)
    assert g_ref[0, 0] == 0.0 and g_ref[0, 1] > 0.0 and np.all(g_ref[1] == 0.0)
    assert gains[0, 0] == 0.0 and np.all(gains[1] == 0.0)
    np.testing.assert_allclose(gains[0, 1], g_ref[0, 1], rtol=GAIN_TOL)
    assert wave_err(mixed, ref, offsets, silent_scale=speech) <= WAVE_TOL


def test_measured_snr_equals_target(aug):
    rng = np.random.default_rng(5)
    offsets = np.array([0, 30000], np.int64)
    speech = rng.standard_normal(30000).astype(np.float32)
    noise = 4.0 * rng.standard_normal((1, 30000)).astype(np.float32)
    rir = _decaying_rirs(rng, 1, 2, 1000)
    snr = np.array([[7.5]], np.float32)
    mixed, gains = _run(aug, offsets, speech, noise, rir, snr)
    y = O.reverberate(offsets, speech, noise, rir.astype(np.float64))
    got = 10 * np.log10(np.sum(y[0] ** 2) / np.sum((gains[0, 0] * y[1]) ** 2))
    assert got == pytest.approx(7.5, abs=1e-3)


def test_utterances_that_end_as_a_source_arrives(aug):
    # Where the waveform bar stops being attainable, as fixed cases.  The transforms' rounding noise is about
    # 1e-7 of (input RMS x response norm), whatever part of the reverberated signal the utterance still holds.
    # An utterance that ends m samples after a source's direct path arrives holds a sliver of energy
    # E = ratio x E_in x E_h, so the noise is about 1e-7 / sqrt(ratio) of its RMS.  Stated bar, asserted here:
    #   * the utterance ends at or before the speech's first tap: gain 0 and exact zeros on both sides;
    #   * otherwise  max|z - z_ref| <= max(1e-4, 1e-6 / sqrt(ratio)) x RMS(z_ref)  and gains to
    #     max(1e-4, 1e-6 / sqrt(ratio)) relative, ratio = E_0 / (E_in,0 E_h,0) of the reverberated speech.
    # With speech-like onsets (ratio 1e-5 .. 1e-3 in the last few samples) that is the ordinary 1e-4 bar or
    # just above it; an onset of near-zero samples (ratio ~ 1e-11, the case a random sweep once met) is far
    # outside it and only the formula holds.
    L = 600
    row_s = [6, 5, 3, 1, 4, 1, 1, 1, 1, 0.6]          # speech 3 m from the microphone: first tap 140
    row_n = [6, 5, 3, 2, 1, 1, 1, 1, 1, 0.6]          # noise 1 m away: first tap 47
    extra = [1, 2, 3, 5, 10, 50, 400]
    lens = [140 + e for e in extra] + [47 + e for e in extra] + [47, 46, 140, 139, 142]
    offsets = np.concatenate([[0], np.cumsum(lens)]).astype(np.int64)
    total = int(offsets[-1])
    geom = np.array([[row_s, row_n]] * len(lens), np.float32)
    h, _ = O.rir_batch(geom.reshape(-1, 10), L, 16000.0, 343.0)
    rir = h.reshape(len(lens), 2, L).astype(np.float32)
    snr = np.full((len(lens), 1), 10.0, np.float32)
    for seed in (1, 2, 3):
        rng = np.random.default_rng(seed)
        speech = np.concatenate([W.speech_like(rng, int(n)) for n in lens]).astype(np.float32)
        noise = rng.standard_normal((1, total)).astype(np.float32)
        speech[offsets[-2]:offsets[-2] + 2] *= 1e-5          # last utterance: a near-silent onset, two samples arrive
        mixed, gains = _run(aug, offsets, speech, noise, rir, snr)
        ref, g_ref = O.convolve_mix_batch(offsets, speech, noise, rir.astype(np.float64), snr)
        y = O.reverberate(offsets, speech, None, rir[:, :1].astype(np.float64))
        worst_ordinary = 0.0
        for u, n in enumerate(lens):
            a, b = int(offsets[u]), int(offsets[u + 1])
            got, want = mixed[a:b].astype(np.float64), ref[a:b]
            if n <= 140:              # the speech never arrives: no SNR to set, gain 0, and the mixture is silence
                assert g_ref[u, 0] == 0.0 and gains[u, 0] == 0.0
                assert not want.any() and not got.any()
                continue
            e0 = float(np.sum(y[0, a:b] ** 2))
            e_in = float(np.sum(speech[a:b].astype(np.float64) ** 2))
            ratio = e0 / (e_in * float(np.sum(rir[u, 0].astype(np.float64) ** 2)))
            bar = max(WAVE_TOL, 1e-6 / np.sqrt(ratio))
            err = np.max(np.abs(got - want)) / np.sqrt(np.mean(want ** 2))
            assert err <= bar, (seed, n, ratio, err)
            assert abs(gains[u, 0] - g_ref[u, 0]) <= max(GAIN_TOL, 1e-6 / np.sqrt(ratio)) * g_ref[u, 0]
            if u < len(lens) - 1:
                assert ratio > 3e-6                           # speech-like onsets stay near the ordinary bar
                worst_ordinary = max(worst_ordinary, err)
            else:
                assert ratio < 1e-9
        print(f"  seed {seed}: worst error / RMS among speech-like slivers {worst_ordinary:.2e}", flush=True)
        assert worst_ordinary <= 2e-4


@pytest.mark.parametrize("L", [
    1, 2, 129, 130, 258, 386, 514, 642, 770, 898, 1025, 1026, 1282, 1538, 1793, 1794, 2049, 2050, 2561, 2562,
    3074, 3585, 3586, 4097, 4098, 5121, 5122, 6146, 7170, 8193, 8194, 10242, 12001, 12289, 12290, 14337, 14338,
    16384, 16385])
def test_blocks_of_every_number_of_rows(aug, L):
    """Response lengths where a block gains or loses a row of its window, signals that end around a row's and a block's end; the
    responses' last tap is the largest, so that a row kept too many shows.  The last utterance's noise response is all zeros."""
    n = 1024
    while n < min(L, 16384):
        n *= 2
    row = n // 8
    rows = 8 if L > n else 16 - (L - 1 + row - 1) // row
    block = row * rows
    lens = [1, row - 1, row + 1, block - 1, block, block + 1, 2 * n - 1, 2 * n + 1, 2 * block + row, 3 * block - 1, 2 * block + 3]
    offsets = np.concatenate([[0], np.cumsum(lens)]).astype(np.int64)
    rng = np.random.default_rng(L)
    speech, noise = (rng.standard_normal(s).astype(np.float32) for s in (offsets[-1], (1, offsets[-1])))
    rir = 0.3 * _decaying_rirs(rng, len(lens), 2, L)
    rir[..., -1] = 3.0
    rir[-1, 1] = 0.0
    print(f"case: rows of a block, L={L}, block={block}", flush=True)
    mixed, _ = _check(aug, offsets, speech, noise, rir.astype(np.float32), rng.uniform(0, 20, (len(lens), 1)).astype(np.float32), method="fft")


@pytest.mark.parametrize("L,n_utt", [(3000, 256), (4096, 128), (4200, 256), (8000, 64)])
def test_short_responses_in_batches_that_fill_the_chip(aug, L, n_utt):
    """Batches of several rounds of groups, with responses much shorter than the signals."""
    rng = np.random.default_rng(L + n_utt)
    lens = rng.integers(60000, 68001, n_utt)
    offsets = np.concatenate([[0], np.cumsum(lens)]).astype(np.int64)
    speech = rng.standard_normal(offsets[-1]).astype(np.float32)
    rir = _decaying_rirs(rng, n_utt, 1, L)
    print(f"case: full chip, L={L}, {n_utt} signals", flush=True)
    _check(aug, offsets, speech, None, rir, None, method="fft")


@pytest.mark.parametrize("L,n_utt", [(100, 8), (1100, 8), (2049, 256), (4096, 256), (8000, 64), (8193, 8), (12001, 8), (16385, 8)])
def test_pauses_and_neighbours(aug, L, n_utt):
    """Bursts between digital silences.  What the transforms leave in the silences reaches no farther than aug.h says and is as
    small there as rounding makes it, and a signal comes out of a batch with the bits that it has alone."""
    p = 1024
    while p < min(L, 16384):
        p *= 2
    reach = 2 * p if L <= p else 3 * p
    rng = np.random.default_rng(L)
    lens = np.maximum(64000, 7 * p) + rng.integers(0, 2000, n_utt)
    offsets = np.concatenate([[0], np.cumsum(lens)]).astype(np.int64)
    onset, burst = rng.integers(2 * p, 3 * p, n_utt), rng.integers(p // 8, p // 2, n_utt)
    speech = np.zeros(offsets[-1], np.float32)
    for u in range(n_utt):
        a = offsets[u] + onset[u]
        speech[a:a + burst[u]] = rng.standard_normal(burst[u])
    rir = _decaying_rirs(rng, n_utt, 1, L)
    print(f"case: pauses, L={L}, {n_utt} signals", flush=True)
    mixed, _ = _run(aug, offsets, speech, None, rir, None)
    worst = 0.0
    for u in range(n_utt):
        y, end = mixed[offsets[u]:offsets[u + 1]].astype(np.float64), onset[u] + burst[u]
        assert not y[:max(onset[u] - reach + 1, 0)].any() and not y[end - 1 + reach:].any(), u
        # a transform of 2p points in single precision: an error of log2(2p) roundings at most of a spectrum's norm, twice
        # (forward and inverse) and that of the response's, spread evenly over the window (three windows at most hold a burst)
        level = np.sqrt(burst[u]) * np.linalg.norm(rir[u, 0].astype(np.float64)) / np.sqrt(2 * p)
        bound = 3 * 2.0 ** -24 * np.log2(2 * p) * level
        for pause in (y[max(onset[u] - reach + 1, 0):onset[u]], y[end - 1 + L:end - 1 + reach]):
            if pause.size:
                worst = max(worst, np.sqrt(np.mean(pause ** 2)) / bound)
    print(f"  rounding in the pauses, of its bound: {worst:.2f}", flush=True)
    assert worst <= 1.0
    for u in (0, 1, n_utt // 2, n_utt - 1):
        a, b = offsets[u], offsets[u + 1]
        alone, _ = _run(aug, np.array([0, b - a], np.int64), speech[a:b], None, rir[u:u + 1], None)
        np.testing.assert_array_equal(alone, mixed[a:b])
