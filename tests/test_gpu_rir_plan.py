"""Batches on either side of the limits of the one-launch plan: responses do not depend on how a batch is cut."""
import numpy as np
import pytest

from oracle import aug_oracle as O
from tests.parity import RIR_TOL, dev, rir_err

pytestmark = pytest.mark.gpu
FS, C = 16000.0, 343.0


@pytest.fixture(scope="module")
def aug():
    import torch
    from paper_1912_11040_amd.binding import Augmenter
    assert torch.cuda.is_available()
    a = Augmenter(0)
    yield a
    a.close()


def _rooms(n, side, seed):
    rng = np.random.default_rng(seed)
    room = rng.uniform([0.6 * side, 0.5 * side, 0.4 * side], [side, 0.9 * side, 0.6 * side], (n, 3))
    g = np.concatenate([room, room * rng.uniform(0.1, 0.9, (n, 3)), room * rng.uniform(0.1, 0.9, (n, 3)),
                        rng.choice([0.0, 0.3, 0.85, 1.0], (n, 1))], 1)
    return g.astype(np.float32)


# (the last: more items than the plan keeps in LDS, six or more a response)
@pytest.mark.parametrize("n,length,side", [(1, 200, 6.0), (1024, 200, 6.0), (1025, 65, 6.0), (4096, 64, 6.0), (4097, 64, 6.0), (1500, 32768, 80.0)])
def test_batch_sizes(aug, n, length, side):
    import torch
    g = _rooms(n, side, n)
    print(f"case: {n} responses of {length} taps", flush=True)
    d = dev(g)
    h = torch.full((n, length), float("nan"), dtype=torch.float32, device="cuda")
    cnt = torch.full((n, length), -7, dtype=torch.int32, device="cuda")
    aug.aug_rir_batch(d, length, FS, C, h, cnt)
    part, cnt_part = torch.empty_like(h), torch.empty_like(cnt)
    step = 700
    for at in range(0, n, step):
        end = min(n, at + step)
        aug.aug_rir_batch(d[at:end].contiguous(), length, FS, C, part[at:end], cnt_part[at:end])
    torch.cuda.synchronize()
    assert torch.equal(h, part) and torch.equal(cnt, cnt_part)
    rows = np.unique(np.linspace(0, n - 1, 5).astype(int))
    h_ref, cnt_ref = O.rir_batch(g[rows], length, FS, C)
    np.testing.assert_array_equal(cnt.cpu().numpy()[rows], cnt_ref)
    assert rir_err(h.cpu().numpy()[rows], h_ref) <= RIR_TOL
