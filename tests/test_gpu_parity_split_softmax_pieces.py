"""The row softmax of the fp32 path's large calls where its pieces a thread change (8192 | 16384 columns) and end, with multipliers of both
signs: a negative one makes the smallest logit of a row the one its exponentials are taken against.  Against the float64 oracle at the fp32 bars."""
import pytest

import paper_2304_08480_amd as dl
from oracle import clip_oracle as oc
from synth import clip_pairs
from tests.gpu_util import TOL, Runner, check_scalar, check_tensor, term_scale, to_device

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("s", [14.285714, -9.0])
@pytest.mark.parametrize("B,N", [(2047, 1), (7936, 31), (8192, 32), (8193, 3), (8448, 33), (16384, 64)])
def test_rows_at_the_lengths_where_the_pieces_change(B, N, s):
    d, r = 64, N - 1
    I, T = clip_pairs(B, d, 29)
    Id, Td, dt = to_device(I, T, None, None, "f32")
    assert dl.disco_describe_plan(B, d, N, dt, dl.DISCO_PATH_AUTO).kernels == dl.DISCO_KERNELS_SPLIT
    run = Runner(Id, Td, B, d, N, dt, dl.DISCO_PATH_AUTO)
    print(f"case softmax pieces B={B} N={N} s={s}", flush=True)
    run.rank(r, s)
    loss, gI, gT, gs = run.results()
    ref, scale = oc.disco_rank(I, T, s, r, N), term_scale(oc, I, T, s, r, N)
    check_scalar("loss", loss, ref[0], TOL["f32"]["scalar"])
    check_scalar("gs", gs, ref[3], TOL["f32"]["scalar"] * 10, abs_tol=1e-9)
    check_tensor("gI", gI, ref[1], "f32", scale[0], scale[2])
    check_tensor("gT", gT, ref[2], "f32", scale[1], scale[2])
