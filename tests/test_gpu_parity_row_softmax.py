"""The row softmaxes at what their first tests leave out: the two-view loss, whose rows leave a column out, at every length that the
softmax of small calls keeps in one wave's registers; rows longer than 16384 and 32768 columns that end inside a 16-byte piece, for both
losses of the split products, accumulated and repeated; and features that are not finite.  Against the float64 oracles at the fp32 bars."""
import numpy as np
import pytest
import torch

import paper_2304_08480_amd as dl
from oracle import clip_oracle as oc
from oracle import ntxent_oracle as nx
from synth import bf16_bits_to_f32, clip_pairs, f32_to_bf16_bits, two_views
from tests.gpu_util import TOL, Runner, check_scalar, check_tensor, term_scale, to_device

pytestmark = pytest.mark.gpu
S = 14.285714


def _two_view_call(Zd, B, d, N, r, dt, path, kernels):
    assert dl.disco_describe_plan(B, d, N, dt, path, two_view=True).kernels == kernels
    need = dl.ntxent_workspace_bytes(B, d, N, dt, path)
    ws = torch.empty(need, dtype=torch.uint8, device="cuda")
    loss, gs, gZ = torch.zeros(1, device="cuda"), torch.zeros(1, device="cuda"), torch.full((B, d), float("nan"), device="cuda")

    def call(accumulate):
        dl.ntxent_loss_fwd_bwd(Zd, B, d, r, N, S, dt, path, accumulate, loss, gZ, gs, ws, need, torch.cuda.current_stream())
        torch.cuda.synchronize()
        return float(loss.item()), gZ.cpu().numpy().astype(np.float64), float(gs.item())

    return call


def _check_two_view(Z, got, r, N, B, tag):
    ref, scale = nx.ntxent_rank(Z, S, r, N), nx.ntxent_rank_term_scale(Z, S, r, N)
    check_scalar(f"{tag} loss", got[0], ref[0], TOL["f32"]["scalar"])
    check_scalar(f"{tag} gs", got[2], ref[2], TOL["f32"]["scalar"] * 10, abs_tol=1e-9 + 1e-5 * scale[1])
    check_tensor(f"{tag} gZ", got[1], ref[1], "f32", scale[0], 1e-13 * S / B)


@pytest.mark.parametrize("dtype", ["f32", "bf16"])
@pytest.mark.parametrize("B,N,d", [(254, 1, 33), (258, 2, 20), (510, 3, 36), (514, 1, 48), (1022, 7, 40), (1024, 1, 36), (1026, 2, 20), (1500, 4, 33),
                                   (2046, 6, 24), (2048, 2, 36), (2050, 5, 20)])
def test_two_view_rows_of_small_calls(B, N, d, dtype):
    Z = two_views(B // 2, d, 21)
    if dtype == "bf16":
        bits = f32_to_bf16_bits(Z)
        Z, Zd, dt = bf16_bits_to_f32(bits), torch.from_numpy(bits.view(np.int16)).cuda(), dl.DISCO_BF16
    else:
        Zd, dt = torch.from_numpy(Z).cuda(), dl.DISCO_F32
    for r in sorted({0, N - 1}):                           # positives behind and before the rank's own rows
        print(f"case two-view rows B={B} N={N} d={d} rank={r} {dtype}", flush=True)
        _check_two_view(Z, _two_view_call(Zd, B, d, N, r, dt, dl.DISCO_PATH_NAIVE, dl.DISCO_KERNELS_SMALL)(0), r, N, B, f"rank {r}")


# lengths just past 16384 (a row kept in registers, 16 pieces a thread) and past 32768 (read again), 2 and 1 columns past whole pieces
@pytest.mark.parametrize("B,N", [(16510, 127), (32890, 253)])
def test_long_two_view_rows(B, N):
    Z = two_views(B // 2, 64, 22)
    r = N - 1
    call = _two_view_call(torch.from_numpy(Z).cuda(), B, 64, N, r, dl.DISCO_F32, dl.DISCO_PATH_AUTO, dl.DISCO_KERNELS_SPLIT)
    print(f"case long two-view rows B={B} N={N}", flush=True)
    first = call(0)
    _check_two_view(Z, first, r, N, B, f"B={B}")
    twice = call(1)                                        # added to its own result
    np.testing.assert_allclose(twice[1], 2.0 * first[1], rtol=1e-6, atol=1e-12)
    again = call(0)
    assert again[0] == first[0] and again[2] == first[2] and np.array_equal(again[1], first[1])


@pytest.mark.parametrize("B,N", [(16641, 129), (32881, 251)])
def test_long_rows_that_end_inside_a_piece(B, N):
    d, r = 64, N - 1
    I, T = clip_pairs(B, d, 23)
    Id, Td, dt = to_device(I, T, None, None, "f32")
    run = Runner(Id, Td, B, d, N, dt, dl.DISCO_PATH_AUTO)
    assert dl.disco_describe_plan(B, d, N, dt, dl.DISCO_PATH_AUTO).kernels == dl.DISCO_KERNELS_SPLIT
    print(f"case long rows B={B} N={N}", flush=True)
    ref, scale = oc.disco_rank(I, T, S, r, N), term_scale(oc, I, T, S, r, N)
    run.rank(r, S)
    loss, gI, gT, gs = run.results()
    check_scalar("loss", loss, ref[0], TOL["f32"]["scalar"])
    check_scalar("gs", gs, ref[3], TOL["f32"]["scalar"] * 10, abs_tol=1e-9)
    check_tensor("gI", gI, ref[1], "f32", scale[0], scale[2])
    check_tensor("gT", gT, ref[2], "f32", scale[1], scale[2])
    run.gI.fill_(0.5); run.gT.fill_(-0.25); run.loss.fill_(2.0); run.gs.fill_(1.0)
    run.rank(r, S, accumulate=True)
    l2, a2, t2, g2 = run.results()
    assert l2 == pytest.approx(2.0 + loss, rel=1e-6) and g2 == pytest.approx(1.0 + gs, rel=1e-6)
    np.testing.assert_allclose(a2, gI + 0.5, rtol=1e-6)
    np.testing.assert_allclose(t2, gT - 0.25, rtol=1e-6)
    run.rank(r, S)
    l3, a3, t3, g3 = run.results()
    assert l3 == loss and g3 == gs and np.array_equal(a3, gI) and np.array_equal(t3, gT)


# every kernel that takes exponentials: small calls (16 x 16 and 32 x 32 similarity tiles, one to eight pieces a lane), split products, tiles
@pytest.mark.parametrize("B,N,d,dtype,path", [
    (200, 2, 40, "f32", "auto"), (500, 2, 40, "f32", "naive"), (1000, 2, 40, "f32", "naive"), (2000, 2, 40, "f32", "naive"), (2100, 2, 40, "f32", "naive"),
    (200, 2, 40, "bf16", "auto"), (1000, 2, 40, "bf16", "naive"), (2000, 2, 40, "bf16", "naive"),
    (2048, 4, 512, "f32", "auto"), (16640, 130, 64, "f32", "auto"), (33024, 258, 64, "f32", "auto"),
    (1024, 2, 128, "bf16", "materialized"), (1000, 2, 64, "bf16", "materialized"), (1024, 2, 128, "bf16", "fused"), (4096, 1, 640, "bf16", "symmetric"),
])
@pytest.mark.parametrize("value", [float("nan"), float("inf")], ids=["nan", "inf"])
def test_what_is_not_finite_reaches_the_outputs(B, N, d, dtype, path, value):
    paths = {"auto": dl.DISCO_PATH_AUTO, "naive": dl.DISCO_PATH_NAIVE, "materialized": dl.DISCO_PATH_MATERIALIZED, "fused": dl.DISCO_PATH_FUSED,
             "symmetric": dl.DISCO_PATH_SYMMETRIC}
    I, T = clip_pairs(B, d, 24)
    q = B // N + 3 if N > 1 else 3                         # a row of the second rank's
    I[q, d // 2] = value
    Ib = Tb = None
    if dtype == "bf16":
        Ib, Tb = f32_to_bf16_bits(np.where(np.isfinite(I), I, 0.0)), f32_to_bf16_bits(T)
        Ib[q, d // 2] = 0x7FC0 if np.isnan(value) else 0x7F80
    Id, Td, dt = to_device(I, T, Ib, Tb, dtype)
    run = Runner(Id, Td, B, d, N, dt, paths[path])
    for r in range(min(N, 2)):
        print(f"case not finite B={B} N={N} d={d} {dtype} {path} {value} rank={r}", flush=True)
        run.rank(r, S)
        torch.cuda.synchronize()
        with np.errstate(invalid="ignore", over="ignore"):
            ref = oc.disco_rank(I, T, S, r, N)
        # what the definition makes not finite is not finite in the outputs (within a tile the kernels may spread it further)
        for name, got, want in (("loss", run.loss, ref[0]), ("gs", run.gs, ref[3]), ("gI", run.gI, ref[1]), ("gT", run.gT, ref[2])):
            lost = ~np.isfinite(want)
            assert lost.any(), name
            finite = np.isfinite(got.cpu().numpy()).reshape(lost.shape)
            assert not (finite & lost).any(), f"{name} rank {r}: {int((finite & lost).sum())} finite values of {int(lost.sum())}"
