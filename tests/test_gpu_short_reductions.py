"""The 16 x 16 similarity tiles of the smallest fp32 calls where a wave's part of the reduction is not whole blocks of four
16-deep pieces: one to three pieces, whole or with a ragged last one, after a whole block or alone.  Values against the float64
oracle at the fp32 bars; and a reduction half as long takes no longer, which it did when those pieces were fetched one element
at a time."""
import pytest
import torch

import paper_2304_08480_amd as dl
from oracle import clip_oracle as oc
from synth import clip_pairs
from tests.gpu_util import Runner, TOL, check_scalar, check_tensor, term_scale, to_device

pytestmark = pytest.mark.gpu
S = 14.285714


def _runner(B, N, d, shift=0):
    I, T = clip_pairs(B, d, 12)
    Id, Td, dt = to_device(I, T, None, None, "f32")
    if shift:
        Id, Td = (torch.empty(x.numel() + shift, device="cuda")[shift:].view(B, d).copy_(x) for x in (Id, Td))
    p = dl.disco_describe_plan(B, d, N, dt, dl.DISCO_PATH_AUTO)
    assert p.kernels == dl.DISCO_KERNELS_SMALL
    return I, T, Runner(Id, Td, B, d, N, dt, dl.DISCO_PATH_AUTO)


# eight waves: d = 160 deals 1 or 2 pieces to each, 300 2 or 3 (the last of them 12 wide), 384 3, 500 3 or 4 (the last 4 wide), 560 4 or 5,
# 700 5 or 6, 1001 7 or 8 (rows off their boundary)
@pytest.mark.parametrize("d", [160, 256, 300, 384, 500, 560, 700, 896, 1001])
@pytest.mark.parametrize("B,N,shift", [(256, 4, 0), (200, 1, 0), (130, 2, 1)])
def test_parts_of_a_block_of_pieces(B, N, shift, d):
    I, T, run = _runner(B, N, d, shift)
    run.rank(N - 1, S)
    ref, scale = oc.disco_rank(I, T, S, N - 1, N), term_scale(oc, I, T, S, N - 1, N)
    loss, gI, gT, gs = run.results()
    check_scalar("loss", loss, ref[0], TOL["f32"]["scalar"])
    check_scalar("gs", gs, ref[3], TOL["f32"]["scalar"] * 10, abs_tol=1e-9)
    check_tensor("gI", gI, ref[1], "f32", scale[0], scale[2])
    check_tensor("gT", gT, ref[2], "f32", scale[1], scale[2])


@pytest.mark.parametrize("B,N", [(256, 1), (512, 4)])
def test_a_shorter_reduction_takes_no_longer(B, N):
    calls = {d: _runner(B, N, d)[2] for d in (256, 512)}
    a, b = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
    best = {d: float("inf") for d in calls}
    for _ in range(12):
        for d, run in calls.items():
            run.rank(0, S)
            a.record()
            for _ in range(50):
                run.rank(0, S)
            b.record()
            b.synchronize()
            best[d] = min(best[d], a.elapsed_time(b) * 20.0)
    print(f"us a call at B={B} N={N}: {best}", flush=True)
    # (measured 15.5 / 17.7 and 17.9 / 20.6; element by element 20.6 / 17.5 and 22.8 / 20.4)
    assert best[256] <= 1.03 * best[512]
