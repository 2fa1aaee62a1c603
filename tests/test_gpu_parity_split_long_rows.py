"""The softmax of the fp32 path's large calls at the lengths of a row where it keeps more of it in registers, or none: 16384, 32768
columns, and one tile more.  Tolerances of fp32 arithmetic, against the float64 oracle."""
import pytest

import paper_2304_08480_amd as dl
from tests.gpu_util import Runner
from tests.test_gpu_parity_split import S, _check, _features

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("B,N", [(16384, 64), (16640, 65), (32768, 128), (33024, 129)])
def test_rows_as_long_as_registers_hold(B, N):
    I, T, (Id, Td, dt) = _features(B, 64, "f32")
    run = Runner(Id, Td, B, 64, N, dt, dl.DISCO_PATH_AUTO)
    assert dl.disco_describe_plan(B, 64, N, dt, dl.DISCO_PATH_AUTO).kernels == dl.DISCO_KERNELS_SPLIT
    run.rank(N - 1, S)
    _check(I, T, run, N - 1, N, f"B={B}")
