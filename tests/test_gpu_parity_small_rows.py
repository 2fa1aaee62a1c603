"""The row softmax of small calls that keeps a row in one wave's registers, at the edges of what a lane holds (256, 512, 1024 and
2048 columns, and one more, which another kernel takes), and the 16 x 16 similarity tiles of the smallest calls, at remainders of
rows, columns and reduction.  Tolerances of fp32 arithmetic (tests/gpu_util.py), against the float64 oracle."""
import pytest

import paper_2304_08480_amd as dl
from oracle import clip_oracle as oc
from synth import bf16_bits_to_f32, clip_pairs, f32_to_bf16_bits
from tests.gpu_util import Runner, TOL, check_scalar, check_tensor, term_scale, to_device

pytestmark = pytest.mark.gpu


# (B, N, d): shares of 1 to 128 rows; widths with every remainder of a 16-deep piece that a wave's part can end in
@pytest.mark.parametrize("B,N,d", [(1, 1, 1), (2, 2, 3), (16, 1, 16), (17, 1, 15), (33, 3, 17), (255, 5, 40), (256, 4, 64), (257, 1, 129), (260, 4, 512),
                                   (510, 5, 100), (512, 8, 65), (513, 9, 48), (1023, 33, 72), (1024, 32, 31), (1028, 4, 20), (2046, 62, 96), (2048, 64, 512),
                                   (2049, 683, 24), (2052, 54, 36)])
@pytest.mark.parametrize("dtype", ["f32", "bf16"])
def test_rows_and_tiles_at_their_edges(B, N, d, dtype):
    I, T = clip_pairs(B, d, 11)
    Ib = Tb = None
    if dtype == "bf16":
        Ib, Tb = f32_to_bf16_bits(I), f32_to_bf16_bits(T)
        I, T = bf16_bits_to_f32(Ib), bf16_bits_to_f32(Tb)
    Id, Td, dt = to_device(I, T, Ib, Tb, dtype)
    assert dl.disco_describe_plan(B, d, N, dt, dl.DISCO_PATH_NAIVE).kernels == dl.DISCO_KERNELS_SMALL
    run = Runner(Id, Td, B, d, N, dt, dl.DISCO_PATH_NAIVE)
    for r in sorted({0, N - 1}):
        run.rank(r, 14.285714)
        ref, scale = oc.disco_rank(I, T, 14.285714, r, N), term_scale(oc, I, T, 14.285714, r, N)
        loss, gI, gT, gs = run.results()
        check_scalar("loss", loss, ref[0], TOL["f32"]["scalar"])
        check_scalar("gs", gs, ref[3], TOL["f32"]["scalar"] * 10, abs_tol=1e-9)
        check_tensor("gI", gI, ref[1], "f32", scale[0], scale[2])
        check_tensor("gT", gT, ref[2], "f32", scale[1], scale[2])
