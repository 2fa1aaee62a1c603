"""Rows whose softmax total is lost under the exponent reference taken from their own positive: keys of a norm far above the
positives' (the numerators overflow), and rows of large norm with small cosines (they underflow).  The row groups that hold
them are redone against their true maxima inside the merge kernel; the others keep the ordinary route."""
import numpy as np
import pytest
import torch

import paper_2304_08480_amd as dl
from oracle import clip_oracle as oc
from oracle import ntxent_oracle as nx
from synth import clip_pairs, two_views, f32_to_bf16_bits, bf16_bits_to_f32
from tests.gpu_util import Runner, term_scale, check_scalar, check_tensor, to_device, TOL

pytestmark = pytest.mark.gpu
PATHS = {"materialized": dl.DISCO_PATH_MATERIALIZED, "fused": dl.DISCO_PATH_FUSED, "symmetric": dl.DISCO_PATH_SYMMETRIC}


def _spoil(I, T, B):
    """Two keys of each side 40 times longer than the rest, and a few rows 60 times longer whose cosines are small anyway."""
    I, T = I.copy(), T.copy()
    T[[3, B - 2]] *= 40.0
    I[[B // 2, B - 1]] *= 40.0
    I[5] *= 60.0
    return I, T


@pytest.mark.parametrize("path,B,d,N", [("materialized", 1024, 128, 4), ("materialized", 1010, 64, 2), ("fused", 1024, 128, 2),
                                        ("fused", 1500, 64, 3), ("fused", 1581, 64, 3), ("symmetric", 4608, 512, 1)])
def test_rows_are_redone(path, B, d, N):
    s = 14.285714
    I, T = _spoil(*clip_pairs(B, d, 51), B)
    Ib, Tb = f32_to_bf16_bits(I), f32_to_bf16_bits(T)
    I, T = bf16_bits_to_f32(Ib), bf16_bits_to_f32(Tb)
    Id, Td, dt = to_device(I, T, Ib, Tb, "bf16")
    run = Runner(Id, Td, B, d, N, dt, PATHS[path])
    for r in sorted({0, N - 1}):
        print(f"case lost rows {path} B={B} d={d} N={N} rank={r}", flush=True)
        run.rank(r, s)
        loss, gI, gT, gs = run.results()
        ref = oc.disco_rank(I, T, s, r, N)
        sI, sT, fl = term_scale(oc, I, T, s, r, N)
        check_scalar("loss", loss, ref[0], TOL["bf16"]["scalar"])
        check_scalar("gs", gs, ref[3], TOL["bf16"]["scalar"] * 10, abs_tol=1e-6)
        check_tensor("gI", gI, ref[1], "bf16", sI, fl)
        check_tensor("gT", gT, ref[2], "bf16", sT, fl)


@pytest.mark.parametrize("path", ["materialized", "fused"])
@pytest.mark.parametrize("M,d,N", [(512, 128, 2), (505, 64, 1)])
def test_two_view_rows_are_redone(path, M, d, N):
    s, B = 14.285714, 2 * M
    Z = two_views(M, d, 6)
    Z[[3, M + 7, B - 1]] *= 40.0
    bits = f32_to_bf16_bits(Z)
    Z, Zd = bf16_bits_to_f32(bits), torch.from_numpy(bits.view(np.int16)).cuda()
    need = dl.ntxent_workspace_bytes(B, d, N, dl.DISCO_BF16, PATHS[path])
    ws = torch.empty(need, dtype=torch.uint8, device="cuda")
    loss, gs, gZ = torch.zeros(1, device="cuda"), torch.zeros(1, device="cuda"), torch.empty(B, d, device="cuda")
    for r in sorted({0, N - 1}):
        print(f"case lost rows two views {path} M={M} d={d} N={N} rank={r}", flush=True)
        dl.ntxent_loss_fwd_bwd(Zd, B, d, r, N, s, dl.DISCO_BF16, PATHS[path], 0, loss, gZ, gs, ws, need, torch.cuda.current_stream())
        torch.cuda.synchronize()
        ref, scale = nx.ntxent_rank(Z, s, r, N), nx.ntxent_rank_term_scale(Z, s, r, N)
        check_scalar("loss", float(loss.item()), ref[0], TOL["bf16"]["scalar"])
        check_scalar("gs", float(gs.item()), ref[2], TOL["bf16"]["scalar"] * 10, abs_tol=1e-9 + 2.0 ** -8 * scale[1])
        check_tensor("gZ", gZ.cpu().numpy().astype(np.float64), ref[1], "bf16", scale[0], 1e-13 * s / B)


# One key of `length` along the first feature, which some rows of the last rank see `exponent` (base 2) above their positive: less
# than fp32 holds as a numerator, more than it holds once that is multiplied by the key, and those rows are so short that
# bf16 would not hold them divided by such a total.  Every other row sees the key far below its positive.
WINDOW = [(2048.0, 112.0), (16384.0, 118.0), (2.0 ** 26, 104.0)]
SHORT = 2.0 ** -13


def _window(X, rows, key, length, exponent, s):
    """X: the query features, changed in place; returns the long key's features."""
    X[:, 0] = -0.05
    X[key, 0] = 0.0
    X[rows] *= SHORT
    X[rows, 0] = exponent / (s * np.log2(np.e) * length)
    y = np.zeros(X.shape[1], X.dtype)
    y[0] = length
    return y


@pytest.mark.parametrize("length,exponent", WINDOW)
@pytest.mark.parametrize("path,B,d,N", [("materialized", 1024, 64, 4), ("materialized", 8100, 256, 4), ("fused", 1024, 128, 2),
                                        ("fused", 1500, 64, 3), ("fused", 1581, 64, 3), ("materialized", 1100, 192, 2)])
def test_numerators_stay_within_what_the_products_hold(path, B, d, N, length, exponent):
    s, r, key = 14.285714, N - 1, 3
    I, T = clip_pairs(B, d, 53)
    I, T = I.copy(), T.copy()
    T[:, 0] = 0.0
    T[key] = _window(I, [B - B // N + 1, B - 70, B - 1], key, length, exponent, s)
    Ib, Tb = f32_to_bf16_bits(I), f32_to_bf16_bits(T)
    I, T = bf16_bits_to_f32(Ib), bf16_bits_to_f32(Tb)
    Id, Td, dt = to_device(I, T, Ib, Tb, "bf16")
    run = Runner(Id, Td, B, d, N, dt, PATHS[path])
    print(f"case long key {path} B={B} d={d} N={N} length={length} exponent={exponent}", flush=True)
    run.rank(r, s)
    loss, gI, gT, gs = run.results()
    ref = oc.disco_rank(I, T, s, r, N)
    sI, sT, fl = term_scale(oc, I, T, s, r, N)
    check_scalar("loss", loss, ref[0], TOL["bf16"]["scalar"])
    # (the short rows' terms and the others' cancel in d/ds: one bf16 rounding of every P moves it by 2^-8 of their magnitudes)
    check_scalar("gs", gs, ref[3], TOL["bf16"]["scalar"] * 10, abs_tol=1e-9 + 2.0 ** -8 * oc.disco_rank_gs_term_scale(I, T, s, r, N))
    check_tensor("gI", gI, ref[1], "bf16", sI, fl)
    check_tensor("gT", gT, ref[2], "bf16", sT, fl)


@pytest.mark.parametrize("length,exponent", WINDOW)
@pytest.mark.parametrize("path", ["materialized", "fused"])
def test_two_view_numerators_stay_within_what_the_products_hold(path, length, exponent):
    s, M, d, N = 14.285714, 1024, 64, 4
    B, r, key = 2 * M, N - 1, 3                             # (the key and its positive belong to other ranks)
    Z = two_views(M, d, 8).copy()
    Z[key] = _window(Z, [B - B // N + 1, B - 70, B - 1], key, length, exponent, s)
    bits = f32_to_bf16_bits(Z)
    Z, Zd = bf16_bits_to_f32(bits), torch.from_numpy(bits.view(np.int16)).cuda()
    need = dl.ntxent_workspace_bytes(B, d, N, dl.DISCO_BF16, PATHS[path])
    ws = torch.empty(need, dtype=torch.uint8, device="cuda")
    loss, gs, gZ = torch.zeros(1, device="cuda"), torch.zeros(1, device="cuda"), torch.empty(B, d, device="cuda")
    print(f"case long key two views {path} length={length} exponent={exponent}", flush=True)
    dl.ntxent_loss_fwd_bwd(Zd, B, d, r, N, s, dl.DISCO_BF16, PATHS[path], 0, loss, gZ, gs, ws, need, torch.cuda.current_stream())
    torch.cuda.synchronize()
    ref, scale = nx.ntxent_rank(Z, s, r, N), nx.ntxent_rank_term_scale(Z, s, r, N)
    check_scalar("loss", float(loss.item()), ref[0], TOL["bf16"]["scalar"])
    check_scalar("gs", float(gs.item()), ref[2], TOL["bf16"]["scalar"] * 10, abs_tol=1e-9 + 2.0 ** -8 * scale[1])
    check_tensor("gZ", gZ.cpu().numpy().astype(np.float64), ref[1], "bf16", scale[0], 1e-13 * s / B)
