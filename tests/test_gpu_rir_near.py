"""Images on either side of 2.6 m (walked apart from the rest), against the oracle."""
import numpy as np
import pytest

from oracle import aug_oracle as O
from tests.parity import RIR_TOL, dev, rir_err

pytestmark = pytest.mark.gpu
C = 343.0


@pytest.fixture(scope="module")
def aug():
    import torch
    from paper_1912_11040_amd.binding import Augmenter
    assert torch.cuda.is_available()
    a = Augmenter(0)
    yield a
    a.close()


def _rooms(fs):
    """Distances in steps across the boundary, microphone on or near the source, small and large rooms."""
    rows = []
    for d in (0.001, 0.2, 2.3, 2.54, 2.56, 2.6, 2.6 + 0.24 * C / fs, 2.6 + 0.26 * C / fs, 2.7):
        for beta in (0.0, 0.8, 1.0):
            rows.append([6.0, 5.0, 3.0, 1.5, 2.0, 1.25, 1.5 + d, 2.0, 1.25, beta])
        rows.append([1.0, 2.9, 0.4, 0.5, 0.05, 0.21, 0.5, 0.05 + min(d, 2.8), 0.2, 0.9])
    return np.array(rows, np.float32)


@pytest.mark.parametrize("fs", [1000.0, 16000.0, 48000.0])
@pytest.mark.parametrize("length", [1, 62, 121, 122, 128, 700])
def test_near_images(aug, fs, length):
    import torch
    g = _rooms(fs)
    print(f"case: fs={fs} length={length}", flush=True)
    h = torch.full((len(g), length), float("nan"), dtype=torch.float32, device="cuda")
    cnt = torch.full((len(g), length), -7, dtype=torch.int32, device="cuda")
    if fs < 2000 and length > 200:
        length = 200                                    # (more would be millions of images in the small room)
        h, cnt = h[:, :length].contiguous(), cnt[:, :length].contiguous()
    aug.aug_rir_batch(dev(g), length, fs, C, h, cnt)
    torch.cuda.synchronize()
    h_ref, cnt_ref = O.rir_batch(g, length, fs, C)
    np.testing.assert_array_equal(cnt.cpu().numpy(), cnt_ref)
    assert rir_err(h.cpu().numpy(), h_ref) <= RIR_TOL


@pytest.mark.parametrize("beta", [0.3, 0.32, 0.1])
def test_near_columns_past_the_reflection_cut(aug, beta):
    """Rooms so narrow that columns within 2.6 m have more reflections than the cut leaves.  Their amplitudes round to
    nothing, and must not come from the powers of other rooms, which the work groups' tables held in the call before."""
    import torch
    rng = np.random.default_rng(3)
    n, length, fs = 320, 130, 16000.0            # (two shells a response: one begins at a distance above 0, within 2.6 m)
    g = []
    for b in (1.0, beta):
        side = rng.uniform(0.1, 0.11, (n, 3))
        g.append(np.concatenate([side, side * rng.uniform(0.2, 0.8, (n, 3)), side * rng.uniform(0.2, 0.8, (n, 3)),
                                 np.full((n, 1), b)], 1).astype(np.float32))
    h = torch.full((2, n, length), float("nan"), dtype=torch.float32, device="cuda")
    for i in range(2):
        aug.aug_rir_batch(dev(g[i]), length, fs, C, h[i])
    torch.cuda.synchronize()
    got = h[1].cpu().numpy()
    for r in range(0, n, 5):
        h_ref, _ = O.rir_batch(g[1][r:r + 1], length, fs, C)
        assert rir_err(got[r:r + 1], h_ref) <= RIR_TOL, r


@pytest.mark.parametrize("fs,length", [(16000.0, 5569), (16000.0, 5570), (48000.0, 5572), (96000.0, 5570), (48000.0, 5600), (48000.0, 11138)])
def test_rooms_whose_images_all_lie_near(aug, fs, length):
    """Small rooms with walls so dead that every image that counts lies within 2.6 m, in batches where a response is cut into few
    shells: one of them begins a few taps after 0 and has no column beyond 2.6 m, only images within.  Against the
    oracle, and every row as it is alone in a call (where it is cut into other shells)."""
    import torch
    rng = np.random.default_rng(length)
    n, head = 1024, int(2.0 * fs / C)
    print(f"case: images all near, fs={fs} L={length}", flush=True)
    for side in (0.1, 0.3, 0.5, 0.9):
        for beta in (0.1, 1e-2, 1e-3, 1e-6):
            g = np.concatenate([np.full((n, 3), side), rng.uniform(0.05, 0.95, (n, 6)) * side, np.full((n, 1), beta)], 1).astype(np.float32)
            g[0] = [side, side, side, 0.1 * side, 0.5 * side, 0.5 * side, 0.9 * side, 0.5 * side, 0.5 * side, beta]
            d = dev(g)
            h = torch.full((n, length), float("nan"), dtype=torch.float32, device="cuda")
            alone = torch.full((4, length), float("nan"), dtype=torch.float32, device="cuda")
            aug.aug_rir_batch(d, length, fs, C, h)
            for r in range(4):
                aug.aug_rir_batch(d[r:r + 1].contiguous(), length, fs, C, alone[r:r + 1])
            torch.cuda.synchronize()
            assert torch.equal(h[:4], alone), (side, beta)
            got = h[:, :head].cpu().numpy()
            for r in [*range(4), *range(50, n, 200)]:
                h_ref, _ = O.rir_batch(g[r:r + 1], head, fs, C)
                assert rir_err(got[r:r + 1], h_ref) <= RIR_TOL, (side, beta, r)
