"""Front-end calls on one batch that take different numbers of work groups (the mixture on the fly or not, another feature or hop):
a graph that holds one of them still gives its result after the others have run."""
import dataclasses
import os
import shutil
import subprocess

import numpy as np
import pytest

HERE = os.path.dirname(os.path.abspath(__file__))
ROCM_INCLUDE = "/opt/rocm/include"


@pytest.mark.skipif(not shutil.which("g++") or not os.path.isdir(ROCM_INCLUDE), reason="needs g++ and the HIP headers")
def test_tables_of_other_calls(tmp_path):
    exe = str(tmp_path / "frame_tables")
    subprocess.run(["g++", "-std=c++17", "-g", "-O1", "-D__HIP_PLATFORM_AMD__", "-D__align__(n)=__attribute__((aligned(n)))",
                    "-DHIP_SYMBOL(s)=s", "-I" + ROCM_INCLUDE, "-I" + os.path.join(HERE, "..", "include"),
                    "-I" + os.path.join(HERE, "..", "paper_1912_11040_amd", "csrc"), os.path.join(HERE, "host", "frame_tables.cpp"),
                    "-o", exe], check=True)
    r = subprocess.run([exe], capture_output=True, text=True, timeout=120)
    assert r.returncode == 0, (r.returncode, r.stdout)


@pytest.mark.gpu
def test_graphs_of_calls_with_other_groups():
    # 1000 units and more: 1024 groups at most without a mixture, 768 with one, fewer for cepstra of 128 channels
    import torch
    from paper_1912_11040_amd import workloads as W
    from paper_1912_11040_amd.binding import Augmenter
    rng = np.random.default_rng(11)
    fe, n, taps = W.FrontendConfig(), 24, 700
    lens = rng.integers(100000, 120000, n)
    offsets = np.concatenate([[0], np.cumsum(lens)]).astype(np.int64)
    foff = np.concatenate([[0], np.cumsum(1 + (lens - 400) // 160)]).astype(np.int64)
    total = int(offsets[-1])
    dev = lambda a: torch.from_numpy(np.ascontiguousarray(a, np.float32)).cuda()                    # noqa: E731
    geom = np.empty((n, 2, 10), np.float32)
    geom[:, :, 0:3] = [5.0, 4.0, 3.0]
    geom[:, :, 3:6] = rng.uniform(0.5, 2.5, (n, 2, 3))
    geom[:, :, 6:9] = rng.uniform(0.5, 2.5, (n, 1, 3))
    geom[:, :, 9] = 0.6
    speech, noise, g = dev(rng.standard_normal(total)), dev(rng.standard_normal((1, total))), dev(geom)
    snr, alpha = dev(rng.uniform(0.0, 20.0, (n, 1))), dev(rng.uniform(0.8, 1.2, n))
    # (padded rows are the same for another hop)
    calls = [(fe, False), (fe, True), (dataclasses.replace(fe, feature="mfcc", n_mel=128, n_ceps=128), False), (dataclasses.replace(fe, hop=200), False)]
    stream = torch.cuda.Stream()
    print("case: graphs of four front ends of one batch", flush=True)
    with Augmenter(0, stream) as aug, torch.cuda.stream(stream):
        outs = [torch.empty(int(foff[-1]), c.feature_dim, device="cuda") for c, _ in calls]

        def call(i, out):
            c, mix = calls[i]
            if mix:
                aug.aug_pipeline_batch(offsets, speech, noise, g, taps, 16000.0, 343.0, snr, alpha, c, foff, out)
            else:
                aug.aug_vtlp_mel_batch(offsets, speech, alpha, c, foff, out)

        eager = []
        for i in range(len(calls)):
            call(i, outs[i])
            stream.synchronize()
            eager.append(outs[i].clone())
        graphs = []
        for i in range(len(calls)):
            call(i, outs[i])
            stream.synchronize()
            graph = torch.cuda.CUDAGraph()
            with torch.cuda.graph(graph, stream=stream):
                call(i, outs[i])
            graphs.append(graph)
        for turn in range(3):
            for i in np.random.default_rng(turn).permutation(len(calls)):
                outs[i].fill_(float("nan"))
                stream.synchronize()
                graphs[i].replay()
                stream.synchronize()
                assert torch.equal(outs[i], eager[i]), (turn, i)
            other = outs[0].clone()
            call(turn % 2, other)                                  # eager work between the replays
            stream.synchronize()
            assert torch.equal(other, eager[turn % 2])
        del graphs
