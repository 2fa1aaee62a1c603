"""The small-call kernels of the fp32 path at the sizes where their tiling can go wrong: shares that straddle 32- and 64-row
tiles, widths that leave waves without work or end inside an 8-deep piece, row pitches that are not whole 16-byte
pieces, and features that do not start on a 16-byte boundary.  Against the float64 oracle at the fp32 bars."""
import numpy as np
import pytest
import torch

import paper_2304_08480_amd as dl
from oracle import clip_oracle as oc
from synth import clip_pairs, f32_to_bf16_bits, bf16_bits_to_f32
from tests.gpu_util import Runner, term_scale, check_scalar, check_tensor, to_device, TOL

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("dtype", ["f32", "bf16"])
@pytest.mark.parametrize("B,d,N,shift", [
    (100, 36, 4, 0),        # shares of 25 rows inside 32-row tiles; most waves have no part of the reduction over d
    (99, 44, 3, 0),         # a row pitch of 99 is rounded up to whole pieces
    (130, 100, 2, 1),       # features one element off the boundary: element-wise loads
    (66, 260, 1, 0),        # N = 1, d just past the waves' 256
    (96, 63, 96, 0),        # one row per rank, odd width
    (2178, 68, 2, 0),       # 64 x 64 tiles in the similarities, 32 x 32 in the gradients, shares of 1089 rows
    (4230, 130, 6, 1),      # 64 x 64 tiles in both, shares of 705 rows that straddle them
    (200, 48, 1, 0),        # three 16-deep pieces of d: a wave without one, rows past the last tile
    (513, 128, 1, 0),       # an odd batch: the last row of a pair does not exist
    (150, 77, 2, 2),        # odd width: features one by one; bf16 rows on 4-byte boundaries
    (4098, 68, 1, 0),       # all rows one share, a row pitch that is rounded up
])
def test_small_products(B, d, N, shift, dtype):
    s = 14.285714
    I, T = clip_pairs(B, d, 31)
    Ib = Tb = None
    if dtype == "bf16":
        Ib, Tb = f32_to_bf16_bits(I), f32_to_bf16_bits(T)
        I, T = bf16_bits_to_f32(Ib), bf16_bits_to_f32(Tb)
    Id, Td, dt = to_device(I, T, Ib, Tb, dtype)
    assert dl.disco_describe_plan(B, d, N, dt, dl.DISCO_PATH_NAIVE).kernels == dl.DISCO_KERNELS_SMALL
    if shift:
        moved = []
        for x in (Id, Td):
            y = torch.empty(x.numel() + shift, dtype=x.dtype, device="cuda")[shift:].view(B, d)
            moved.append(y.copy_(x))
        Id, Td = moved
    run = Runner(Id, Td, B, d, N, dt, dl.DISCO_PATH_NAIVE)
    for r in sorted({0, N // 2, N - 1}):
        print(f"case small products B={B} d={d} N={N} rank={r} dtype={dtype} shift={shift}", flush=True)
        run.rank(r, s)
        loss, gI, gT, gs = run.results()
        ref = oc.disco_rank(I, T, s, r, N)
        sI, sT, fl = term_scale(oc, I, T, s, r, N)
        check_scalar("loss", loss, ref[0], TOL["f32"]["scalar"])
        check_scalar("gs", gs, ref[3], TOL["f32"]["scalar"] * 10, abs_tol=1e-9)
        check_tensor("gI", gI, ref[1], "f32", sI, fl)
        check_tensor("gT", gT, ref[2], "f32", sT, fl)
    # the rank's contribution is added to what the buffers hold
    run.gI.fill_(0.5); run.gT.fill_(-0.25); run.loss.fill_(2.0); run.gs.fill_(1.0)
    run.rank(N - 1, s, accumulate=True)
    l2, a2, t2, g2 = run.results()
    assert l2 == pytest.approx(2.0 + loss, rel=1e-6) and g2 == pytest.approx(1.0 + gs, rel=1e-6)
    np.testing.assert_allclose(a2, gI + 0.5, rtol=1e-6)
    np.testing.assert_allclose(t2, gT - 0.25, rtol=1e-6)


@pytest.mark.parametrize("B,d,N", [(256, 128, 1), (512, 256, 2), (1024, 64, 4)])
def test_auto_runs_a_call_of_a_few_tiles_in_fp32_arithmetic(B, d, N):
    # such a call resolves to a bf16 tile path, whose numerators would cost 1e-5 and more of the gradients' 2-norm
    s = 14.285714
    I, T = clip_pairs(B, d, 32)
    Ib, Tb = f32_to_bf16_bits(I), f32_to_bf16_bits(T)
    I, T = bf16_bits_to_f32(Ib), bf16_bits_to_f32(Tb)
    Id, Td, dt = to_device(I, T, Ib, Tb, "bf16")
    assert dl.disco_resolve_path(B, d, N, dt, dl.DISCO_PATH_AUTO) != dl.DISCO_PATH_NAIVE
    assert dl.disco_describe_plan(B, d, N, dt, dl.DISCO_PATH_AUTO).kernels == dl.DISCO_KERNELS_SMALL
    run = Runner(Id, Td, B, d, N, dt, dl.DISCO_PATH_AUTO)
    run.rank(N - 1, s)
    loss, gI, gT, gs = run.results()
    ref = oc.disco_rank(I, T, s, N - 1, N)
    sI, sT, fl = term_scale(oc, I, T, s, N - 1, N)
    check_scalar("loss", loss, ref[0], TOL["f32"]["scalar"])
    check_scalar("gs", gs, ref[3], TOL["f32"]["scalar"] * 10, abs_tol=1e-9)
    check_tensor("gI", gI, ref[1], "f32", sI, fl)
    check_tensor("gT", gT, ref[2], "f32", sT, fl)
