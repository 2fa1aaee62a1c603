"""Every call records all the stage events of the path it resolves to, also where other kernels take it over."""
import numpy as np
import pytest
import torch

import paper_2304_08480_amd as dl
from bench import HipEvents
from synth import clip_pairs, f32_to_bf16_bits
from tests.gpu_util import Runner, to_device

pytestmark = pytest.mark.gpu
STAGES = {dl.DISCO_PATH_NAIVE: 5, dl.DISCO_PATH_MATERIALIZED: 6, dl.DISCO_PATH_FUSED: 5, dl.DISCO_PATH_SYMMETRIC: 7}


@pytest.mark.parametrize("B,d,N,dtype,path", [
    (256, 64, 2, "f32", "AUTO"), (2048, 512, 4, "f32", "AUTO"),          # small and split kernels of the fp32 path
    (1024, 128, 2, "bf16", "AUTO"), (512, 128, 1, "bf16", "AUTO"),       # small kernels for a bf16 path
    (1024, 128, 2, "bf16", "MATERIALIZED"), (4096, 128, 2, "bf16", "FUSED"), (5000, 64, 1, "bf16", "FUSED"),
    (1024, 128, 1, "bf16", "SYMMETRIC"), (5888, 320, 1, "bf16", "SYMMETRIC"),   # handed over to the two-block kernels, and not
])
def test_all_stage_events_are_recorded(B, d, N, dtype, path):
    I, T = clip_pairs(B, d, 81)
    Id, Td, dt = to_device(I, T, f32_to_bf16_bits(I), f32_to_bf16_bits(T), dtype)
    path = getattr(dl, "DISCO_PATH_" + path)
    n = STAGES[dl.disco_resolve_path(B, d, N, dt, path)]
    run = Runner(Id, Td, B, d, N, dt, path)
    run.rank(N - 1, 14.0)
    torch.cuda.synchronize()
    ev = HipEvents(n + 1)
    print(f"case stage events B={B} d={d} N={N} {dtype} path={path}: {n}", flush=True)
    dl.disco_set_stage_events(ev.arr, ev.n)
    try:
        run.rank(N - 1, 14.0)
        torch.cuda.synchronize()
    finally:
        dl.disco_set_stage_events(None, 0)
    ms = [ev.elapsed_ms(k, k + 1) for k in range(n)]       # (an event that was not recorded fails here)
    assert all(t >= 0.0 for t in ms) and np.isfinite(run.results()[0])
