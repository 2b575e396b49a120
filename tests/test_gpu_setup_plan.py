"""The launch that sets up the front end and plans the image sum: batches whose last group of tables is full, one short and two
short, and one whose responses are planned in launches of their own, against the stages' own entry points bit for bit."""
import numpy as np
import pytest

from paper_1912_11040_amd import workloads as W
from tests.parity import dev

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n_utt,n_noise", [(1, 0), (2, 1), (3, 0), (256, 1), (257, 3), (1025, 3)])
def test_stages_of_one_call(n_utt, n_noise):
    import torch
    from paper_1912_11040_amd.binding import Augmenter
    rng = np.random.default_rng(n_utt)
    fe, fs, c, taps, n_src = W.FrontendConfig(), W.FS, W.SPEED_OF_SOUND, 300, 1 + n_noise
    lens = rng.integers(0, 1200, n_utt)
    lens[-1] = 1199
    offsets = np.concatenate([[0], np.cumsum(lens)]).astype(np.int64)
    frames = np.where(lens >= fe.win, 1 + (lens - fe.win) // fe.hop, 0)
    foff = np.concatenate([[0], np.cumsum(frames)]).astype(np.int64)
    total = int(offsets[-1])
    geom = np.empty((n_utt, n_src, 10), np.float32)
    geom[:, :, 0:3] = rng.uniform([3.0, 3.0, 2.5], [10.0, 8.0, 4.0], (n_utt, 1, 3))
    geom[:, :, 3:6] = geom[:, :, 0:3] * rng.uniform(0.2, 0.8, (n_utt, n_src, 3))
    geom[:, :, 6:9] = geom[:, :, 0:3] * rng.uniform(0.2, 0.8, (n_utt, 1, 3))
    geom[:, :, 9] = rng.uniform(0.2, 0.9, (n_utt, 1))
    speech, alpha, g = dev(rng.standard_normal(total).astype(np.float32)), dev(rng.uniform(0.8, 1.2, n_utt).astype(np.float32)), dev(geom)
    noise = dev(rng.standard_normal((n_noise, total)).astype(np.float32)) if n_noise else None
    snr = dev(rng.uniform(0.0, 20.0, (n_utt, n_noise)).astype(np.float32)) if n_noise else None
    nan = lambda *shape: torch.full(shape, float("nan"), device="cuda")                 # noqa: E731
    feats, rir, mixed, feats2, rir2 = nan(int(foff[-1]), fe.n_mel), nan(n_utt, n_src, taps), nan(total), nan(int(foff[-1]), fe.n_mel), nan(n_utt, n_src, taps)
    print(f"case: {n_utt} utterances, {n_src} sources", flush=True)
    with Augmenter(0) as aug:
        aug.aug_pipeline_batch(offsets, speech, noise, g, taps, fs, c, snr, alpha, fe, foff, feats, rir, mixed)
        aug.aug_rir_batch(g.reshape(-1, 10), taps, fs, c, rir2)
        aug.aug_vtlp_mel_batch(offsets, mixed, alpha, fe, foff, feats2)
        torch.cuda.synchronize()
    assert not torch.isnan(feats).any() and not torch.isnan(rir).any()
    assert torch.equal(rir, rir2)
    assert torch.equal(feats, feats2)


def test_more_items_than_the_plan_keeps_in_lds():
    # six items a response and more, in large rooms whose responses are quickly summed
    import torch
    from paper_1912_11040_amd.binding import Augmenter
    n_utt, taps, fe = 750, 32768, W.FrontendConfig()
    rng = np.random.default_rng(8)
    lens = rng.integers(300, 700, n_utt)
    offsets = np.concatenate([[0], np.cumsum(lens)]).astype(np.int64)
    foff = np.concatenate([[0], np.cumsum(np.where(lens >= fe.win, 1 + (lens - fe.win) // fe.hop, 0))]).astype(np.int64)
    total = int(offsets[-1])
    geom = np.empty((n_utt, 2, 10), np.float32)
    geom[:, :, 0:3] = rng.uniform([48.0, 40.0, 32.0], [80.0, 72.0, 48.0], (n_utt, 1, 3))
    geom[:, :, 3:6] = geom[:, :, 0:3] * rng.uniform(0.2, 0.8, (n_utt, 2, 3))
    geom[:, :, 6:9] = geom[:, :, 0:3] * rng.uniform(0.2, 0.8, (n_utt, 1, 3))
    geom[:, :, 9] = rng.choice([0.0, 0.3, 0.85, 1.0], (n_utt, 1))
    g, nan = dev(geom), lambda *shape: torch.full(shape, float("nan"), device="cuda")                 # noqa: E731
    feats, rir, rir2 = nan(int(foff[-1]), fe.n_mel), nan(n_utt, 2, taps), nan(n_utt, 2, taps)
    print("case: 1500 responses of 32768 taps", flush=True)
    with Augmenter(0) as aug:
        aug.aug_pipeline_batch(offsets, dev(rng.standard_normal(total).astype(np.float32)), dev(rng.standard_normal((1, total)).astype(np.float32)), g, taps,
                               W.FS, W.SPEED_OF_SOUND, dev(np.full((n_utt, 1), 10.0, np.float32)), dev(np.ones(n_utt, np.float32)), fe, foff, feats, rir)
        for at in range(0, n_utt, 250):                       # in parts that need no such room
            aug.aug_rir_batch(g[at:at + 250].reshape(-1, 10).contiguous(), taps, W.FS, W.SPEED_OF_SOUND, rir2[at:at + 250])
        torch.cuda.synchronize()
    assert not torch.isnan(feats).any()
    assert torch.equal(rir, rir2)
