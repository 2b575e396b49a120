"""How the front end's frames are shared among its work groups: the table on the CPU, and batches whose groups meet several
utterances, several groups one, and some none."""
import os
import shutil
import subprocess

import numpy as np
import pytest

HERE = os.path.dirname(os.path.abspath(__file__))
ROCM_INCLUDE = "/opt/rocm/include"


@pytest.mark.skipif(not shutil.which("g++") or not os.path.isdir(ROCM_INCLUDE), reason="needs g++ and the HIP headers")
def test_table_of_groups(tmp_path):
    exe = str(tmp_path / "frame_shares")
    subprocess.run(["g++", "-std=c++17", "-O1", "-D__HIP_PLATFORM_AMD__", "-I" + ROCM_INCLUDE, "-I" + os.path.join(HERE, "..", "include"),
                    "-I" + os.path.join(HERE, "..", "paper_1912_11040_amd", "csrc"), os.path.join(HERE, "host", "frame_shares.cpp"),
                    "-o", exe], check=True)
    r = subprocess.run([exe], capture_output=True, text=True, timeout=120)
    assert r.returncode == 0, r.stdout


@pytest.mark.gpu
@pytest.mark.parametrize("n_utt,longest,spare", [(1, 1, 0), (5, 300, 0), (2500, 3, 2), (1100, 40, 0), (1100, 17, 40)])
def test_batches(n_utt, longest, spare):
    import torch
    from oracle import aug_oracle as O
    from paper_1912_11040_amd import workloads as W
    from paper_1912_11040_amd.binding import Augmenter
    from tests.parity import FEAT_TOL, dev, feat_err
    fe = W.FrontendConfig()
    rng = np.random.default_rng(n_utt + longest)
    frames = rng.integers(0, longest + 1, n_utt)
    frames[rng.integers(0, n_utt)] = longest
    lens = np.where(frames > 0, 400 + 160 * (frames - 1) + rng.integers(0, 160, n_utt), rng.integers(0, 400, n_utt))
    offsets = np.concatenate([[0], np.cumsum(lens)]).astype(np.int64)
    rows = frames + (rng.integers(0, spare + 1, n_utt) if spare else 0)
    foff = np.concatenate([[0], np.cumsum(rows)]).astype(np.int64)
    x = rng.standard_normal(int(offsets[-1])).astype(np.float32)
    # (a few warps: the oracle forms its bank for every one)
    alpha = rng.choice(np.array([0.85, 1.0, 1.15], np.float32), n_utt)
    feats = torch.full((int(foff[-1]), fe.n_mel), float("nan"), dtype=torch.float32, device="cuda")
    print(f"case: {n_utt} utterances of up to {longest} frames, up to {spare} rows more", flush=True)
    with Augmenter(0) as aug:
        aug.aug_vtlp_mel_batch(offsets, dev(x), dev(alpha), fe, foff, feats)
        torch.cuda.synchronize()
    got, ref = feats.cpu().numpy(), O.vtlp_mel_batch(offsets, x, alpha, fe)
    owner = np.repeat(np.arange(n_utt), rows)
    place = np.arange(int(foff[-1])) - foff[owner]
    is_frame = place < frames[owner]
    assert not got[~is_frame].any()
    assert feat_err(got[is_frame], ref) <= FEAT_TOL


@pytest.mark.gpu
@pytest.mark.parametrize("n_out", [40, 13])
def test_rows_without_frames(n_out):
    """Utterances with nothing but rows to clear, of a few units and of many, beside ordinary ones and ones with more rows than frames."""
    import dataclasses
    import torch
    from oracle import aug_oracle as O
    from paper_1912_11040_amd import workloads as W
    from paper_1912_11040_amd.binding import Augmenter
    from tests.parity import FEAT_TOL, dev, feat_err
    fe = W.FrontendConfig() if n_out == 40 else dataclasses.replace(W.FrontendConfig(), feature="mfcc", n_ceps=13)
    rng = np.random.default_rng(n_out)
    lens = np.array([0, 4000, 399, 0, 400, 0, 16000, 8000, 200, 0, 2800])
    rows = np.array([70001, 23, 255, 256, 257, 513, 5000, 48, 0, 1, 271])
    lens, rows = np.tile(lens, 9), np.tile(rows, 9)
    rows[11:] = np.minimum(rows[11:], 5000)
    frames = np.where(lens >= 400, 1 + (lens - 400) // 160, 0)
    offsets = np.concatenate([[0], np.cumsum(lens)]).astype(np.int64)
    foff = np.concatenate([[0], np.cumsum(rows)]).astype(np.int64)
    x = rng.standard_normal(int(offsets[-1])).astype(np.float32)
    alpha = rng.choice(np.array([0.85, 1.0, 1.15], np.float32), len(lens))
    feats = torch.full((int(foff[-1]), n_out), float("nan"), dtype=torch.float32, device="cuda")
    print(f"case: {n_out} values a row", flush=True)
    with Augmenter(0) as aug:
        aug.aug_vtlp_mel_batch(offsets, dev(x), dev(alpha), fe, foff, feats)
        torch.cuda.synchronize()
    got = feats.cpu().numpy()
    place = np.arange(int(foff[-1])) - np.repeat(foff[:-1], rows)
    is_frame = place < np.repeat(frames, rows)
    assert np.all(got[~is_frame] == 0.0)
    assert feat_err(got[is_frame], O.vtlp_mel_batch(offsets, x, alpha, fe)) <= FEAT_TOL
