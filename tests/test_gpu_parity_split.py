"""The large calls of the fp32 path (operands split into bf16 planes) at the sizes where they can go wrong: shares and
batches that are not whole tiles, widths that are not whole K-steps or 16-byte pieces, one share per 256 rows and all rows in
one, rows past the softmax's smaller set of registers, rows taken in chunks, operands off their 16-byte boundary.  Against the
float64 oracles at the fp32 bars."""
import numpy as np
import pytest
import torch

import paper_2304_08480_amd as dl
from oracle import clip_oracle as oc
from oracle import ntxent_oracle as nx
from synth import clip_pairs, two_views, f32_to_bf16_bits, bf16_bits_to_f32
from tests.gpu_util import Runner, term_scale, check_scalar, check_tensor, to_device, TOL

pytestmark = pytest.mark.gpu
S = 14.285714


def _features(B, d, dtype):
    I, T = clip_pairs(B, d, 41)
    Ib = Tb = None
    if dtype == "bf16":
        Ib, Tb = f32_to_bf16_bits(I), f32_to_bf16_bits(T)
        I, T = bf16_bits_to_f32(Ib), bf16_bits_to_f32(Tb)
    return I, T, to_device(I, T, Ib, Tb, dtype)


def _moved(x, shift):
    return torch.empty(x.numel() + shift, dtype=x.dtype, device="cuda")[shift:].view(x.shape).copy_(x)


def _check(I, T, run, r, N, tag):
    loss, gI, gT, gs = run.results()
    ref = oc.disco_rank(I, T, S, r, N)
    sI, sT, fl = term_scale(oc, I, T, S, r, N)
    check_scalar(f"{tag} loss", loss, ref[0], TOL["f32"]["scalar"])
    check_scalar(f"{tag} gs", gs, ref[3], TOL["f32"]["scalar"] * 10, abs_tol=1e-9)
    check_tensor(f"{tag} gI", gI, ref[1], "f32", sI, fl)
    check_tensor(f"{tag} gT", gT, ref[2], "f32", sT, fl)
    return loss, gI, gT, gs


@pytest.mark.parametrize("B,d,N,dtype,shift", [
    (2048, 512, 4, "f32", 0),          # whole tiles
    (4098, 300, 3, "f32", 0),          # nothing whole but the 16-byte pieces of a row
    (5000, 77, 4, "f32", 1),           # rows that are not whole pieces, features off the boundary: element loads and stores
    (4099, 130, 1, "f32", 0),          # all rows one share, an odd batch
    (16896, 64, 66, "f32", 0),         # rows of twice the registers' first size, one K-step of d
    (2048, 200, 4, "bf16", 0),         # one plane per feature
    (4098, 100, 3, "bf16", 1),
    (6145, 333, 5, "bf16", 0),
])
def test_split_products(B, d, N, dtype, shift):
    I, T, (Id, Td, dt) = _features(B, d, dtype)
    if shift:
        Id, Td = _moved(Id, shift), _moved(Td, shift)
    run = Runner(Id, Td, B, d, N, dt, dl.DISCO_PATH_AUTO)
    # by name the path keeps to its fp32 blocks; a call that is worth it takes more memory through AUTO
    assert run.ws_bytes > dl.disco_workspace_bytes(B, d, N, dt, dl.DISCO_PATH_NAIVE)
    assert dl.disco_describe_plan(B, d, N, dt, dl.DISCO_PATH_AUTO).kernels == dl.DISCO_KERNELS_SPLIT
    for r in sorted({0, N - 1}):
        print(f"case split products B={B} d={d} N={N} rank={r} dtype={dtype} shift={shift}", flush=True)
        run.rank(r, S)
        loss, gI, gT, gs = _check(I, T, run, r, N, f"rank {r}")
    run.gI.fill_(0.5); run.gT.fill_(-0.25); run.loss.fill_(2.0); run.gs.fill_(1.0)
    run.rank(N - 1, S, accumulate=True)
    l2, a2, t2, g2 = run.results()
    assert l2 == pytest.approx(2.0 + loss, rel=1e-6) and g2 == pytest.approx(1.0 + gs, rel=1e-6)
    np.testing.assert_allclose(a2, gI + 0.5, rtol=1e-6)
    np.testing.assert_allclose(t2, gT - 0.25, rtol=1e-6)
    run.rank(N - 1, S)                                     # the same call twice: the same bits
    l3, a3, t3, g3 = run.results()
    assert l3 == loss and g3 == gs and np.array_equal(a3, gI) and np.array_equal(t3, gT)


@pytest.mark.parametrize("B,d,N,dtype,chunks", [
    (4099, 130, 1, "f32", 6),             # a last chunk that is short and ragged, gradients through partial sums (d % 4 != 0)
    (6000, 400, 2, "f32", 6),             # the query side added to rows that a chunk before has written
    (5001, 500, 1, "bf16", 4),
    (4099, 450, 1, "f32", 6),
])
def test_rows_in_chunks_within_the_papers_memory(B, d, N, dtype, chunks):
    I, T, (Id, Td, dt) = _features(B, d, dtype)
    plan = dl.disco_describe_plan(B, d, N, dt, dl.DISCO_PATH_NAIVE)
    assert plan.kernels == dl.DISCO_KERNELS_SPLIT and plan.row_chunks == chunks
    run = Runner(Id, Td, B, d, N, dt, dl.DISCO_PATH_NAIVE)
    assert run.ws_bytes <= 2 * (B // N) * (B + 3) * 4 + 64 * (B // N) + 4096
    print(f"case chunks B={B} d={d} N={N} dtype={dtype}", flush=True)
    run.gI.fill_(0.0); run.gT.fill_(0.0); run.loss.fill_(0.0); run.gs.fill_(0.0)
    run.rank(N - 1, S, accumulate=True)
    _check(I, T, run, N - 1, N, "added to zeros")
    run.rank(N - 1, S)
    _check(I, T, run, N - 1, N, "overwritten")


def test_gradients_off_the_boundary():
    B, d, N = 2048, 512, 4
    I, T, (Id, Td, dt) = _features(B, d, "f32")
    run = Runner(Id, Td, B, d, N, dt, dl.DISCO_PATH_AUTO)
    run.gI, run.gT = _moved(run.gI, 1), _moved(run.gT, 1)
    run.rank(1, S)
    _check(I, T, run, 1, N, "shifted gradients")


def test_powers_of_two_pass_through_exactly():
    # planes, products and sums only shift when one side's features are scaled by 2^k and the other's by 2^-k
    B, d, N = 2048, 512, 4
    I, T, (Id, Td, dt) = _features(B, d, "f32")
    out = []
    for k in (0, 60):
        run = Runner(Id * 2.0 ** k, Td * 2.0 ** -k, B, d, N, dt, dl.DISCO_PATH_AUTO)
        run.rank(2, S)
        out.append(run.results())
    assert out[0][0] == out[1][0] and out[0][3] == out[1][3]
    assert np.array_equal(out[0][1], out[1][1] * 2.0 ** 60) and np.array_equal(out[0][2], out[1][2] * 2.0 ** -60)


@pytest.mark.parametrize("M,d,N,dtype", [(2048, 256, 2, "f32"), (2049, 77, 3, "f32"), (2050, 100, 1, "bf16"), (3075, 200, 6, "bf16")])
def test_two_view_loss_on_split_products(M, d, N, dtype):
    B = 2 * M
    Z = two_views(M, d, 5)
    if dtype == "bf16":
        bits = f32_to_bf16_bits(Z)
        Z, Zd, dt = bf16_bits_to_f32(bits), torch.from_numpy(bits.view(np.int16)).cuda(), dl.DISCO_BF16
    else:
        Zd, dt = torch.from_numpy(Z).cuda(), dl.DISCO_F32
    need = dl.ntxent_workspace_bytes(B, d, N, dt, dl.DISCO_PATH_AUTO)
    assert need > dl.ntxent_workspace_bytes(B, d, N, dt, dl.DISCO_PATH_NAIVE)
    ws = torch.empty(need, dtype=torch.uint8, device="cuda")
    loss, gs, gZ = torch.zeros(1, device="cuda"), torch.zeros(1, device="cuda"), torch.empty(B, d, device="cuda")
    r = N - 1
    print(f"case two views M={M} d={d} N={N} dtype={dtype}", flush=True)
    dl.ntxent_loss_fwd_bwd(Zd, B, d, r, N, S, dt, dl.DISCO_PATH_AUTO, 0, loss, gZ, gs, ws, need, torch.cuda.current_stream())
    torch.cuda.synchronize()
    ref = nx.ntxent_rank(Z, S, r, N)
    scale = nx.ntxent_rank_term_scale(Z, S, r, N)
    check_scalar("loss", float(loss.item()), ref[0], TOL["f32"]["scalar"])
    check_scalar("gs", float(gs.item()), ref[2], TOL["f32"]["scalar"] * 10, abs_tol=1e-9 + 1e-5 * scale[1])
    check_tensor("gZ", gZ.cpu().numpy().astype(np.float64), ref[1], "f32", scale[0], 1e-13 * S / B)
