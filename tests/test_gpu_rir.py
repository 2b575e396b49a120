"""aug_rir_batch against the oracle: tap counts bit for bit, amplitudes to 1e-5."""
import numpy as np
import pytest

from oracle import aug_oracle as O
from paper_1912_11040_amd import workloads as W
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


def _run(aug, geom, L, counts=True):
    import torch
    g = dev(np.asarray(geom, np.float32).reshape(-1, 10))
    n = g.shape[0]
    h = torch.full((n, L), float("nan"), dtype=torch.float32, device="cuda")
    cnt = torch.full((n, L), -7, dtype=torch.int32, device="cuda") if counts else None
    aug.aug_rir_batch(g, L, FS, C, h, cnt)
    torch.cuda.synchronize()
    return h.cpu().numpy(), (cnt.cpu().numpy() if counts else None)


def _check(aug, geom, L):
    geom = np.asarray(geom, np.float32).reshape(-1, 10)
    h, cnt = _run(aug, geom, L)
    h_ref, cnt_ref = O.rir_batch(geom, L, FS, C)
    np.testing.assert_array_equal(cnt, cnt_ref)          # integer work: bit exact
    assert rir_err(h, h_ref) <= RIR_TOL
    return h, cnt


def test_tiny_config_rirs(aug):
    w = W.tiny()
    print("case: tiny geom, L=4096", flush=True)
    _check(aug, w.geom, 4096)


@pytest.mark.parametrize("L", [1, 63, 1000, 5000])
def test_ragged_lengths(aug, L):
    w = W.tiny(n_utt=2)
    print(f"case: tiny geom, L={L}", flush=True)
    _check(aug, w.geom, L)


def test_positions_outside_the_room(aug):
    """Not checked, and bounded all the same: the images whose index the room's size allows, and in the rooms beside them
    what they get alone.  (The order of an axis' images that the tables are built in needs |s - m|, |s + m| <= 2 L.)"""
    room = np.array([5.0, 4.0, 3.0])
    inside = np.concatenate([room, 0.4 * room, 0.7 * room, [0.8]])
    rows = []
    for axis in range(3):
        for s, m in ((1.0, 1.0), (1.001, 1.0), (1.3, 1.2), (-0.1, 0.5), (-1.2, -1.3), (2.5, 0.4), (0.3, -2.2), (-1.9, 0.9), (1e4, 0.5), (0.5, -1e15)):
            row = inside.copy()
            row[3 + axis], row[6 + axis] = s * room[axis], m * room[axis]
            rows += [row, inside]
    rows.append(np.concatenate([room, 1.4 * room, 1.3 * room, [1.0]]))
    for axis in range(3):
        row = inside.copy()
        row[3 + axis] = np.nan
        rows.append(row)
    rows = np.array(rows, np.float32)
    known = len(rows) - 3
    for L in (62, 3000):
        print(f"case: positions outside the room, L={L}", flush=True)
        h, cnt = _run(aug, rows, L)
        h_ref, cnt_ref = O.rir_batch(rows[:known], L, FS, C)
        np.testing.assert_array_equal(cnt[:known], cnt_ref)
        for r in range(known):
            assert rir_err(h[r], h_ref[r]) <= RIR_TOL, rows[r]
        assert not h[known:].any() and not cnt[known:].any()
        alone, _ = _run(aug, inside, L)
        np.testing.assert_array_equal(h[1:known - 1:2], np.broadcast_to(alone, (len(h[1:known - 1:2]), L)))


def test_random_rooms_8000_taps(aug):
    w = W.batch(n_utt=6, seconds=0.1)
    print("case: batch geom 12 rirs, L=8000", flush=True)
    _check(aug, w.geom, 8000)


def test_split_over_several_groups_16000_taps(aug):
    # small rooms at 16000 taps hold millions of images and are cut over many work groups
    g = np.array([[3.0, 3.1, 2.5, 1.0, 1.2, 1.1, 2.2, 2.0, 1.4, 0.9],
                  [9.5, 7.5, 3.9, 2.0, 3.0, 1.5, 7.0, 5.0, 2.0, 0.35]], np.float32)
    print("case: two rooms, L=16000", flush=True)
    _, cnt = _check(aug, g, 16000)
    assert cnt[0].sum() > 5_000_000


def test_longest_response_the_interface_takes(aug):
    w = W.throughput(n_utt=1, seconds=0.1)
    print("case: throughput geom, 3 rirs, L=32768", flush=True)
    _check(aug, w.geom, 32768)


def test_unusable_rooms_give_silence_and_leave_the_rest_alone(aug):
    # the library's guard against an unbounded image lattice: a side under 10 cm or not a number
    w = W.tiny(n_utt=2)
    geom = np.asarray(w.geom, np.float32).reshape(-1, 10).copy()
    good = geom.copy()
    geom[1, 0] = 0.05
    geom[2, 1] = np.nan
    h, cnt = _run(aug, geom, 1500)
    for bad_beta in (-0.5, 1.5, np.nan):
        g2 = good.copy()
        g2[1, 9] = bad_beta
        h2, cnt2 = _run(aug, g2, 700)
        assert np.all(h2[1] == 0.0) and np.all(cnt2[1] == 0) and np.any(h2[0] != 0.0)
    assert np.all(h[1] == 0.0) and np.all(cnt[1] == 0) and np.all(h[2] == 0.0) and np.all(cnt[2] == 0)
    h_ref, cnt_ref = O.rir_batch(good[[0, 3]], 1500, FS, C)
    np.testing.assert_array_equal(cnt[[0, 3]], cnt_ref)
    assert rir_err(h[[0, 3]], h_ref) <= RIR_TOL


def test_zero_reflection_closed_form(aug):
    g = np.array([[5, 4, 3, 1.0, 1.5, 1.2, 3.5, 2.0, 1.7, 0.0]], np.float32)
    h, _ = _run(aug, g, 2048)
    gd = g[0].astype(np.float64)
    r = np.sqrt(np.sum((gd[3:6] - gd[6:9]) ** 2))
    n0 = int(np.floor(r * FS / C + 0.5))
    assert np.count_nonzero(h) == 1
    assert h[0, n0] == pytest.approx(1 / (4 * np.pi * r), rel=1e-6)


def test_without_counts_and_empty_batch(aug):
    import torch
    w = W.tiny(n_utt=1)
    h, _ = _run(aug, w.geom, 777, counts=False)
    h_ref, _ = O.rir_batch(w.geom.reshape(-1, 10), 777, FS, C)
    assert rir_err(h, h_ref) <= RIR_TOL
    aug.aug_rir_batch(None, 128, FS, C, None, None)       # n_rir == 0: no-op
    torch.cuda.synchronize()


def test_beta_one_and_repeatable_counts(aug):
    g = np.array([[4.0, 3.0, 2.6, 1.0, 1.1, 1.2, 3.0, 2.0, 1.3, 1.0]], np.float32)
    h, cnt = _check(aug, g, 3000)
    h2, cnt2 = _run(aug, g, 3000)
    np.testing.assert_array_equal(cnt, cnt2)
    assert rir_err(h2, h.astype(np.float64)) <= RIR_TOL


def test_very_flat_room_walks_images_directly(aug):
    # a 12 cm high room has more z images than the kernel's LDS table holds; it then walks them directly
    g = np.array([[3.0, 3.2, 0.12, 1.0, 1.1, 0.04, 2.1, 2.0, 0.08, 0.5],
                  [4.0, 3.0, 2.7, 1.0, 1.1, 1.0, 2.1, 2.0, 1.5, 0.6]], np.float32)
    print("case: flat room, L=2000", flush=True)
    _check(aug, g, 2000)


@pytest.mark.parametrize("axis", [0, 1])
def test_very_narrow_rooms_walk_images_directly(aug, axis):
    # 12 cm wide along x (more than 320 x images per parity inside the response's radius: the rows of the
    # column table do not fit) or along y (the sorted y table does not fit): both take the plain path
    dims = [3.0, 3.2, 2.7]
    src, mic = [1.0, 1.1, 1.0], [2.1, 2.0, 1.5]
    dims[axis], src[axis], mic[axis] = 0.12, 0.04, 0.08
    g = np.array([dims + src + mic + [0.5],
                  [4.0, 3.0, 2.7, 1.0, 1.1, 1.0, 2.1, 2.0, 1.5, 0.6]], np.float32)
    print(f"case: room 12 cm wide along axis {axis}, L=2000", flush=True)
    _, cnt = _check(aug, g, 2000)
    assert cnt[0].sum() > 200_000


def test_symmetric_geometry_with_tied_distances(aug):
    # source and microphone at mid height: images above and below tie exactly in distance
    g = np.array([[4.0, 4.0, 3.0, 1.0, 2.0, 1.5, 3.0, 2.0, 1.5, 0.8],
                  [4.0, 4.0, 3.0, 2.0, 2.0, 1.5, 2.0, 2.0, 1.0, 0.5]], np.float32)
    print("case: symmetric rooms, L=3000", flush=True)
    _check(aug, g, 3000)


@pytest.mark.parametrize("fs,length", [(500.0, 1), (500.0, 200), (16000.0, 1), (16000.0, 700), (16000.0, 1700), (16000.0, 7000)])
def test_edges_of_the_walk_along_z(aug, fs, length):
    """Either side of what the walk in steps of 2 L takes: heights around a quarter of a tap and 16384 taps, walls so close that an
    axis has more images than the tables hold, and positions on floor and ceiling (lists of images that fall together, the
    mirror image at distance zero)."""
    import torch
    z = []
    for h in (0.1, 0.1714, 0.1716, 0.3, 2.9, 351.0, 351.5, 1e4):
        for s, m in ((0.37, 0.62), (0.0, 0.0), (1.0, 1.0), (0.0, 1.0), (0.5, 0.5)):
            z.append((h, s, m))
    floor = 7.0 * max(1.0, length * 16000.0 / fs / 2000.0)
    rows = [[5 * floor, 4 * floor, h, 1.1, 1.3, s * h, 3.2, 2.1, m * h, 0.85] for h, s, m in z if h >= 2.9 or length <= 1700]
    rows += [[w, 3 * floor, 2.4 * floor, 0.4 * w, 1.3, 1.0, 0.7 * w, 2.1, 1.4, 0.9] for w in (0.1, 0.12, 0.15, 0.3)]
    rows += [[3 * floor, w, 2.4 * floor, 1.3, 0.4 * w, 1.0, 2.1, 0.7 * w, 1.4, 0.9] for w in (0.1, 0.12, 0.15, 0.3)]
    geom = np.asarray(rows, np.float32)
    print(f"case: edges of the z walk, fs={fs} L={length}", flush=True)
    h = torch.full((len(rows), length), float("nan"), device="cuda")
    cnt = torch.full((len(rows), length), -7, dtype=torch.int32, device="cuda")
    aug.aug_rir_batch(dev(geom), length, fs, C, h, cnt)
    torch.cuda.synchronize()
    h_ref, cnt_ref = O.rir_batch(geom, length, fs, C)
    np.testing.assert_array_equal(cnt.cpu().numpy(), cnt_ref)
    assert rir_err(h.cpu().numpy(), h_ref) <= RIR_TOL


@pytest.mark.parametrize("fs,length", [(16000.0, 700), (16000.0, 7000), (16000.0, 32768), (48000.0, 20000)])
def test_tall_rooms(aug, fs, length):
    """Heights on either side of 16384 taps, up to 4e5 taps and beyond: images outside a shell lie so far from it that sixteen bits
    of their slots come round.  Against the oracle, and in a batch (where a response is cut into other shells) the same bits."""
    import torch
    rng = np.random.default_rng(length)
    rows = []
    for taps in (16000, 16383, 16385, 24000, 32600, 32768, 33000, 49000, 65500, 65536, 66000, 131072, 390000, 410000):
        h = taps * C / fs
        for s, m in ((0.4, 0.41), (0.0, 0.0), (1.0, 0.999), (0.5, 0.5), (0.01, 0.02), (0.3, 0.7)):
            w, d = rng.uniform(8.0, 30.0, 2)
            rows.append([w, d, h, 0.3 * w, 0.6 * d, s * h, 0.7 * w, 0.2 * d, m * h, rng.choice([0.3, 0.8, 1.0])])
    geom = np.asarray(rows, np.float32)
    n = len(rows)
    print(f"case: tall rooms, fs={fs} L={length}", flush=True)
    h = torch.full((12 * n, length), float("nan"), device="cuda")
    cnt = torch.full((n, length), -7, dtype=torch.int32, device="cuda")
    aug.aug_rir_batch(dev(np.tile(geom, (12, 1))), length, fs, C, h)
    alone = torch.full((n, length), float("nan"), device="cuda")
    aug.aug_rir_batch(dev(geom), length, fs, C, alone, cnt)
    torch.cuda.synchronize()
    for k in range(12):
        assert torch.equal(h[k * n:(k + 1) * n], alone)
    h_ref, cnt_ref = O.rir_batch(geom, length, fs, C)
    np.testing.assert_array_equal(cnt.cpu().numpy(), cnt_ref)
    assert rir_err(alone.cpu().numpy(), h_ref) <= RIR_TOL


@pytest.mark.parametrize("fs,length", [(16000.0, 62), (16000.0, 1500), (16000.0, 6000), (96000.0, 700)])
def test_positions_below_the_floor(aug, fs, length):
    """Positions up to a room's height below it, where the images of one list along z change sides, with short responses (images
    walked apart) and long ones.  Against the oracle, and in a batch the same bits."""
    import torch
    rng = np.random.default_rng(length)
    rows = []
    for h in (0.4, 1.0, 2.5):
        for s, m in ((-0.1, -0.2), (-0.5, 0.2), (0.3, -0.9), (-0.999, -0.99), (-1.0, -1.0), (-1.0, 0.9), (-0.4, 0.4), (-0.001, 0.0), (-0.6, -0.6)):
            for near in (0.05, 0.8):
                w, d = rng.uniform(4.0, 9.0, 2)
                rows.append([w, d, h, 0.4 * w, 0.5 * d, s * h, 0.4 * w + near, 0.5 * d + near, m * h, rng.choice([0.1, 0.6, 0.9, 1.0])])
    geom = np.asarray(rows, np.float32)
    n = len(rows)
    print(f"case: below the floor, fs={fs} L={length}", flush=True)
    h = torch.full((10 * n, length), float("nan"), device="cuda")
    cnt = torch.full((n, length), -7, dtype=torch.int32, device="cuda")
    aug.aug_rir_batch(dev(np.tile(geom, (10, 1))), length, fs, C, h)
    alone = torch.full((n, length), float("nan"), device="cuda")
    aug.aug_rir_batch(dev(geom), length, fs, C, alone, cnt)
    torch.cuda.synchronize()
    for k in range(10):
        assert torch.equal(h[k * n:(k + 1) * n], alone)
    h_ref, cnt_ref = O.rir_batch(geom, length, fs, C)
    np.testing.assert_array_equal(cnt.cpu().numpy(), cnt_ref)
    assert rir_err(alone.cpu().numpy(), h_ref) <= RIR_TOL


def test_images_whose_slots_come_round_in_32_bits(aug):
    """Rooms so high that the image behind the ceiling lies 2^29 taps and a few away: it belongs to no tap."""
    k = np.float64(np.float32(FS)) / np.float64(np.float32(C))
    rows, heights = [], (2.0 ** 29 + np.linspace(50.0, 2900.0, 40)) / (2.0 * k)
    for h in heights.astype(np.float32):
        rows.append([6.0, 5.0, h, 2.0, 3.0, 0.0, 4.0, 1.5, 0.0, 1.0])
    geom = np.asarray(rows, np.float32)
    assert np.any(np.floor(2.0 * geom[:, 2].astype(np.float64) * k + 0.5) % 2 ** 29 < 3000)
    print("case: images 2^29 taps away, L=3000", flush=True)
    _check(aug, geom, 3000)


def test_positions_many_rooms_outside(aug):
    """Source and microphone many sides apart along one axis: the images near the microphone have numbers that only the whole
    response's radius allows.  Against the oracle, and in a batch (where a response is cut into other shells) the same bits."""
    rng = np.random.default_rng(3)
    length = 8000
    rows = []
    for axis in range(3):
        for share in (0.3, 0.6, -0.8, 0.95):
            room = rng.uniform(1.8, 3.0, 3)
            src, mic = 0.4 * room, 0.7 * room
            (src if rng.random() < 0.5 else mic)[axis] += share * length * C / FS
            rows.append(np.concatenate([room, src, mic, [rng.choice([0.6, 0.9, 1.0])]]))
    geom = np.asarray(rows, np.float32)
    print("case: positions many rooms outside, L=8000", flush=True)
    h, _ = _check(aug, geom, length)
    many, _ = _run(aug, np.tile(geom, (15, 1)), length, counts=False)
    np.testing.assert_array_equal(many, np.tile(h, (15, 1)))


def test_heights_so_far_outside_that_rounding_moves_images(aug):
    """Source and microphone 1e16 to 7e16 m above or below the room: the recipe rounds its images' heights to more than the distance between
    two of them."""
    rng = np.random.default_rng(9)
    rows = []
    for i in range(48):
        s = np.float32(rng.uniform(1e16, 7e16) * rng.choice([-1.0, 1.0]))
        rows.append([4.0, 3.0, rng.uniform(0.4, 3.5), 1.0, 1.1, s, 2.5, 1.7, s * rng.choice([-1.0, 1.0]), 0.9])
    print("case: heights far outside the room, L=3000", flush=True)
    _check(aug, np.asarray(rows, np.float32), 3000)
