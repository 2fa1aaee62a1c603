"""Small bf16 calls on tiles of 32 rows and on both sides of the rule that chooses them: shares and batches around whole tiles, reductions
that end inside a 16-deep piece or leave waves without one, widths on both sides of whole 64-column tiles, features one by one.  Against the
float64 oracles at the fp32 bars (features are exact in bf16, the arithmetic is the fp32 path's)."""
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


@pytest.mark.parametrize("B,d,N", [
    (160, 64, 5),           # shares of 32 rows, one piece of d per wave or none
    (165, 66, 5),           # shares of 33, a column tile of two columns
    (31, 33, 1),            # less than a tile of everything, odd width
    (2112, 96, 2),          # own rows on many tiles, the reduction over b in whole pieces
    (1100, 320, 1),         # more own tiles than the rule allows: 64 rows
    (1056, 129, 33),        # short shares, odd width
])
def test_pairs(B, d, N):
    I, T = clip_pairs(B, d, 51)
    Ib, Tb = f32_to_bf16_bits(I), f32_to_bf16_bits(T)
    I, T = bf16_bits_to_f32(Ib), bf16_bits_to_f32(Tb)
    Id, Td, dt = to_device(I, T, Ib, Tb, "bf16")
    path = dl.DISCO_PATH_NAIVE
    assert dl.disco_describe_plan(B, d, N, dt, path).kernels == dl.DISCO_KERNELS_SMALL
    run = Runner(Id, Td, B, d, N, dt, path)
    for r in sorted({0, N - 1}):
        print(f"case small flat B={B} d={d} N={N} rank={r}", flush=True)
        run.rank(r, S)
        loss, gI, gT, gs = run.results()
        ref = oc.disco_rank(I, T, S, r, N)
        sI, sT, fl = term_scale(oc, I, T, S, r, N)
        check_scalar("loss", loss, ref[0], TOL["f32"]["scalar"])
        check_scalar("gs", gs, ref[3], TOL["f32"]["scalar"] * 10, abs_tol=1e-9)
        check_tensor("gI", gI, ref[1], "f32", sI, fl)
        check_tensor("gT", gT, ref[2], "f32", sT, fl)


@pytest.mark.parametrize("M,d,N", [(97, 40, 2), (300, 130, 3), (834, 128, 4)])
def test_two_views(M, d, N):
    B, r = 2 * M, N - 1
    bits = f32_to_bf16_bits(two_views(M, d, 52))
    Z, Zd = bf16_bits_to_f32(bits), torch.from_numpy(bits.view(np.int16)).cuda()
    assert dl.disco_describe_plan(B, d, N, dl.DISCO_BF16, dl.DISCO_PATH_AUTO, two_view=True).kernels == dl.DISCO_KERNELS_SMALL
    need = dl.ntxent_workspace_bytes(B, d, N, dl.DISCO_BF16, dl.DISCO_PATH_AUTO)
    ws = torch.empty(need, dtype=torch.uint8, device="cuda")
    loss, gs, gZ = torch.zeros(1, device="cuda"), torch.zeros(1, device="cuda"), torch.full((B, d), float("nan"), device="cuda")
    print(f"case small flat two views M={M} d={d} N={N}", flush=True)
    dl.ntxent_loss_fwd_bwd(Zd, B, d, r, N, S, dl.DISCO_BF16, dl.DISCO_PATH_AUTO, 0, loss, gZ, gs, ws, need, torch.cuda.current_stream())
    torch.cuda.synchronize()
    ref, scale = nx.ntxent_rank(Z, S, r, N), nx.ntxent_rank_term_scale(Z, S, r, N)
    check_scalar("loss", float(loss.item()), ref[0], TOL["f32"]["scalar"])
    check_scalar("gs", float(gs.item()), ref[2], TOL["f32"]["scalar"] * 10, abs_tol=1e-9 + 1e-5 * scale[1])
    check_tensor("gZ", gZ.cpu().numpy().astype(np.float64), ref[1], "f32", scale[0], 1e-13 * S / B)
