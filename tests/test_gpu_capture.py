"""HIP graph capture as the header has it: after one loss call of any sizes outside a capture, the first calls of other sizes,
dtypes and paths may be captured, and every replay gives what the eager call gives."""
import os
import subprocess
import sys

import numpy as np
import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CASES = [(8192, 1024, 4, "bf16", "MATERIALIZED"), (1024, 256, 2, "bf16", "MATERIALIZED"), (5000, 64, 1, "bf16", "FUSED"),
         (5888, 320, 1, "bf16", "SYMMETRIC"), (1024, 128, 2, "bf16", "AUTO"), (4098, 300, 3, "f32", "AUTO"),
         (4098, 100, 3, "bf16", "AUTO"), (2048, 512, 4, "f32", "AUTO"), (256, 64, 2, "f32", "AUTO")]


def _child():
    """In a process of its own: nothing but the one small call has run before the captures."""
    import torch
    from synth import clip_pairs, f32_to_bf16_bits
    import paper_2304_08480_amd as dl
    from tests.gpu_util import Runner, to_device

    def runner(B, d, N, dtype, path):
        I, T = clip_pairs(B, d, 91)
        Id, Td, dt = to_device(I, T, f32_to_bf16_bits(I), f32_to_bf16_bits(T), dtype)
        return Runner(Id, Td, B, d, N, dt, getattr(dl, "DISCO_PATH_" + path))

    warm = runner(16, 8, 2, "f32", "AUTO")
    warm.rank(0, 10.0)
    torch.cuda.synchronize()
    for case in CASES:
        print("case capture", *case, flush=True)
        run, r = runner(*case), case[2] - 1
        outs = (run.loss, run.gs, run.gI, run.gT)
        graph = torch.cuda.CUDAGraph()
        with torch.cuda.graph(graph):
            run.rank(r, 14.285714)
        replays = []
        for _ in range(3):
            for o in outs:
                o.fill_(float("nan"))
            graph.replay()
            torch.cuda.synchronize()
            replays.append([o.cpu().numpy() for o in outs])
            warm.rank(1, 10.0)                              # eager work of the program's between the replays
        run.rank(r, 14.285714)
        torch.cuda.synchronize()
        eager = [o.cpu().numpy() for o in outs]
        assert all(np.isfinite(e).all() for e in eager)
        for got in replays:
            assert all(np.array_equal(g, e) for g, e in zip(got, eager)), case
    print("capture ok", flush=True)


@pytest.mark.gpu
def test_first_calls_may_be_captured_after_one_call_of_any_sizes():
    r = subprocess.run([sys.executable, "-u", "-c", "from tests.test_gpu_capture import _child; _child()"], cwd=ROOT, timeout=100,
                       stdout=subprocess.PIPE, stderr=subprocess.STDOUT, text=True)
    print(r.stdout, flush=True)
    assert r.returncode == 0 and "capture ok" in r.stdout
