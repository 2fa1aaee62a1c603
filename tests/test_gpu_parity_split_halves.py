"""The fp32 path's large calls on fp16 planes, and the bf16 planes that replace them on the device where features leave fp16's range:
norms at either end of what the fp16 planes hold and past it, a first row of zeros, whole matrices far from 1, both tile sizes, both
losses, both dtypes.  Against the float64 oracles at the fp32 bars."""
import numpy as np
import pytest
import torch

import paper_2304_08480_amd as dl
from oracle import clip_oracle as oc
from synth import clip_pairs, f32_to_bf16_bits, bf16_bits_to_f32
from tests.gpu_util import Runner, forget_planes, planes_taken, term_scale, check_scalar, check_tensor, to_device, TOL

pytestmark = pytest.mark.gpu


def _features(B, d, dtype, change):
    I, T = clip_pairs(B, d, 43)
    I, T = change(I.copy()), change(T.copy())
    Ib = Tb = None
    if dtype == "bf16":
        Ib, Tb = f32_to_bf16_bits(I), f32_to_bf16_bits(T)
        I, T = bf16_bits_to_f32(Ib), bf16_bits_to_f32(Tb)
    return I, T, to_device(I, T, Ib, Tb, dtype)


def _norms(lo, hi):
    """Rows of norms between 2^lo and 2^hi, the first row's 1."""
    def change(X):
        e = np.linspace(lo, hi, len(X)).astype(np.float32)
        e[0] = 0.0
        return X * (2.0 ** e)[:, None].astype(np.float32)
    return change


def _zero_row(row):
    def change(X):
        X[row] = 0.0
        return X
    return change


def _long_row(X):
    X[-1] *= 100.0
    return X


CHANGES = {
    "unit": lambda X: X,
    "inside": _norms(-4.0, 2.0),           # all on fp16 planes
    "short rows": _norms(-12.0, 0.0),      # past their lower end
    "long row": _long_row,                 # past the upper one, in the last row
    "first row zero": _zero_row(0),        # no power of two to go by
    "other row zero": _zero_row(5),
}
PLANES = {"unit": "fp16", "inside": "fp16", "short rows": "bf16 instead", "long row": "bf16 instead", "first row zero": "bf16 instead", "other row zero": "fp16"}


@pytest.mark.parametrize("change", sorted(CHANGES))
@pytest.mark.parametrize("B,d,N,dtype", [(2048, 512, 4, "f32"), (4098, 300, 3, "f32"), (4099, 130, 1, "f32"), (8192, 64, 16, "f32"), (6145, 333, 5, "bf16")])
def test_norms_inside_and_outside_the_range(B, d, N, dtype, change):
    I, T, (Id, Td, dt) = _features(B, d, dtype, CHANGES[change])
    assert dl.disco_describe_plan(B, d, N, dt, dl.DISCO_PATH_AUTO).kernels == dl.DISCO_KERNELS_SPLIT
    # a multiplier that leaves the longest pair CLIP's largest logit
    s = 14.285714 / max(1.0, float(np.abs((I * T).sum(1)).max()))
    run = Runner(Id, Td, B, d, N, dt, dl.DISCO_PATH_AUTO)
    print(f"case halves {change} B={B} d={d} N={N} dtype={dtype}", flush=True)
    forget_planes(run.ws)
    run.rank(N - 1, s)
    loss, gI, gT, gs = run.results()
    assert planes_taken(run.ws) == (PLANES[change] if d >= 192 else "bf16")      # (narrow fp32 features stay on bf16 planes)
    ref = oc.disco_rank(I, T, s, N - 1, N)
    sI, sT, fl = term_scale(oc, I, T, s, N - 1, N)
    check_scalar("loss", loss, ref[0], TOL["f32"]["scalar"])
    check_scalar("gs", gs, ref[3], TOL["f32"]["scalar"] * 10, abs_tol=1e-9)
    check_tensor("gI", gI, ref[1], "f32", sI, fl)
    check_tensor("gT", gT, ref[2], "f32", sT, fl)


@pytest.mark.parametrize("ki,kt", [(70, -70), (-60, -40), (70, 20), (-85, 85), (3, -9)])
def test_matrices_far_from_one(ki, kt):
    # a power of two on each side and its inverse on s: the same call, on whichever planes hold the features
    B, d, N, s = 2048, 512, 4, 14.285714
    I, T, (Id, Td, dt) = _features(B, d, "f32", CHANGES["unit"])
    out = []
    for a, b in ((0, 0), (ki, kt)):
        run = Runner(Id * 2.0 ** a, Td * 2.0 ** b, B, d, N, dt, dl.DISCO_PATH_AUTO)
        run.rank(1, s * 2.0 ** -(a + b))
        loss, gI, gT, gs = run.results()
        out.append((loss, gI * 2.0 ** a, gT * 2.0 ** b, gs * 2.0 ** -(a + b)))
    assert abs(out[0][0] - out[1][0]) <= 1e-6 * abs(out[0][0]) and abs(out[0][3] - out[1][3]) <= 1e-6 * abs(out[0][3])
    for x, y in zip(out[0][1:3], out[1][1:3]):
        # either form is 6e-7 from 64 bits at this shape
        assert np.linalg.norm(x - y) <= 3e-6 * np.linalg.norm(x)


def test_what_is_not_a_number_stays_so():
    B, d, N = 2048, 512, 4
    _, _, (Id, Td, dt) = _features(B, d, "f32", CHANGES["unit"])
    Id[700, 3] = float("nan")
    run = Runner(Id, Td, B, d, N, dt, dl.DISCO_PATH_AUTO)
    run.rank(1, 14.285714)                                             # rows 512 .. 1023: a row of NaN logits, a column in the other block
    loss, gI, gT, gs = run.results()
    assert np.isnan(loss) and np.isnan(gs) and np.isnan(gI[700]).all() and np.isnan(gT).all()
