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


@pytest.mark.parametrize("dims", [(3.0, 2.0, 0.1), (0.1, 2.5, 3.0), (2.5, 0.1, 3.0), (0.15, 1.5, 0.12)])
@pytest.mark.parametrize("length", [1600, 2300])
def test_rooms_that_fit_the_tables_in_part(aug, dims, length):
    """Rooms so flat or narrow that the outer shells have more images along an axis than the tables hold and the inner ones have
    not.  Alone in a call a response is cut into many shells, in the batch into one or two: the same bits."""
    import torch
    n, rng = 400, np.random.default_rng(length)
    room = np.tile(np.array(dims), (n, 1)) * rng.uniform(1.0, 1.05, (n, 3))
    g = np.concatenate([room, room * rng.uniform(0.05, 0.95, (n, 3)), room * rng.uniform(0.05, 0.95, (n, 3)),
                        rng.choice([0.1, 0.5, 0.9, 1.0], (n, 1))], 1).astype(np.float32)
    g[0] = [*dims, *(0.25 * np.array(dims)), *(0.75 * np.array(dims)), 1.0]
    print(f"case: {dims}, {length} taps", flush=True)
    d = dev(g)
    h = torch.full((n, length), float("nan"), dtype=torch.float32, device="cuda")
    cnt = torch.full((n, length), -7, dtype=torch.int32, device="cuda")
    aug.aug_rir_batch(d, length, FS, C, h, cnt)
    rows = [0, 1, 2, 3, 4, 200, n - 1]
    alone = torch.full((len(rows), length), float("nan"), dtype=torch.float32, device="cuda")
    cnt_alone = torch.full((len(rows), length), -7, dtype=torch.int32, device="cuda")
    for i, r in enumerate(rows):
        aug.aug_rir_batch(d[r:r + 1].contiguous(), length, FS, C, alone[i:i + 1], cnt_alone[i:i + 1])
    torch.cuda.synchronize()
    assert torch.equal(h[rows], alone) and torch.equal(cnt[rows], cnt_alone)
    head = 400                                            # (a response's first taps do not depend on its length)
    h_ref, cnt_ref = O.rir_batch(g[rows], head, FS, C)
    np.testing.assert_array_equal(cnt.cpu().numpy()[rows, :head], cnt_ref)
    assert rir_err(h.cpu().numpy()[rows, :head], h_ref) <= RIR_TOL
