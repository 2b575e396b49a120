"""Amplitudes of images with many reflections, past what the table of powers holds one by one, and of the same response cut
differently: every tap to the arithmetic's own error, and bit for bit whatever the batch."""
import numpy as np
import pytest

from oracle import aug_oracle as O
from tests.parity import dev

pytestmark = pytest.mark.gpu
FS, C = 16000.0, 343.0
L = 5200                                    # 111 m: up to 353 reflections in the small room below


def _run(geom):
    import torch
    from paper_1912_11040_amd.binding import Augmenter
    h = torch.full((len(geom), L), float("nan"), dtype=torch.float32, device="cuda")
    cnt = torch.full((len(geom), L), -7, dtype=torch.int32, device="cuda")
    with Augmenter(0) as aug:
        aug.aug_rir_batch(dev(geom), L, FS, C, h, cnt)
        torch.cuda.synchronize()
    return h.cpu().numpy(), cnt.cpu().numpy()


@pytest.mark.parametrize("beta", [0.97, 0.999])
def test_many_reflections(beta):
    row = np.array([0.5, 0.55, 0.6, 0.2, 0.31, 0.13, 0.41, 0.12, 0.37, beta], np.float32)
    h, cnt = _run(row[None])
    ref, cnt_ref = O.rir_single(row, L, FS, C)
    np.testing.assert_array_equal(cnt[0], cnt_ref)
    # each image: 7.1 * 2^-27 of the hardware's root and half a unit of 2^-56; the tap: half a unit of single precision
    bound = np.abs(ref) * (7.1 * 2.0 ** -27 + 2.0 ** -24) + cnt_ref * 2.0 ** -57 + 1e-12 * np.abs(ref)
    assert np.all(np.abs(h[0] - ref) <= bound)
    # a batch of more responses is cut more coarsely, one of very many by another target
    for n in (24, 600):
        more, _ = _run(np.repeat(row[None], n, axis=0) if n == 24 else np.concatenate([row[None], np.tile(
            np.array([[4.0, 3.0, 2.5, 1.0, 1.0, 1.0, 2.5, 2.0, 1.5, 0.7]], np.float32), (n - 1, 1))]))
        np.testing.assert_array_equal(more[0], h[0])


@pytest.mark.parametrize("beta", [0.9, 0.97, 0.999])
@pytest.mark.parametrize("axis", [0, 1, 2])
def test_many_reflections_of_a_flat_room(axis, beta):
    # up to 1115 reflections along one axis, which has more images than the fast walk takes: inner shells are walked one way and
    # outer ones the other
    dims, src, mic = [2.5, 3.0], [1.1, 1.3], [1.9, 0.7]
    for v, thin in ((dims, 0.1), (src, 0.03), (mic, 0.07)):
        v.insert(axis, thin)
    row = np.array(dims + src + mic + [beta], np.float32)
    print(f"case: flat along {axis}, beta {beta}", flush=True)
    h, cnt = _run(row[None])
    ref, cnt_ref = O.rir_single(row, L, FS, C)
    np.testing.assert_array_equal(cnt[0], cnt_ref)
    bound = np.abs(ref) * (7.1 * 2.0 ** -27 + 2.0 ** -24) + cnt_ref * 2.0 ** -57 + 1e-12 * np.abs(ref)
    assert np.all(np.abs(h[0] - ref) <= bound)
    more, _ = _run(np.repeat(row[None], 40, axis=0))
    np.testing.assert_array_equal(more[0], h[0])
    np.testing.assert_array_equal(more[39], h[0])
