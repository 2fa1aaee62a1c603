"""The memory-lean path with its rows in chunks: tile counts that no panel width divides, a last chunk that is smaller and
ragged, gradients that are added to, and two-view positives that lie in another chunk.  Against the float64 oracles at the
bf16 bars."""
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


@pytest.mark.parametrize("B,d,N,chunks", [(10100, 64, 4, 2), (10100, 64, 2, 2), (4990, 128, 2, 2), (6500, 64, 1, 2), (1581, 64, 3, 3)])
def test_row_chunks(B, d, N, chunks):
    assert dl.disco_describe_plan(B, d, N, dl.DISCO_BF16, dl.DISCO_PATH_FUSED).row_chunks == chunks
    I, T = clip_pairs(B, d, 61)
    Ib, Tb = f32_to_bf16_bits(I), f32_to_bf16_bits(T)
    I, T = bf16_bits_to_f32(Ib), bf16_bits_to_f32(Tb)
    Id, Td, dt = to_device(I, T, Ib, Tb, "bf16")
    run = Runner(Id, Td, B, d, N, dt, dl.DISCO_PATH_FUSED)
    r = N - 1
    print(f"case row chunks B={B} d={d} N={N}", flush=True)
    run.rank(r, S)
    loss, gI, gT, gs = run.results()
    ref = oc.disco_rank(I, T, S, r, N)
    sI, sT, fl = term_scale(oc, I, T, S, r, N)
    check_scalar("loss", loss, ref[0], TOL["bf16"]["scalar"])
    check_scalar("gs", gs, ref[3], TOL["bf16"]["scalar"] * 10, abs_tol=1e-9)
    check_tensor("gI", gI, ref[1], "bf16", sI, fl)
    check_tensor("gT", gT, ref[2], "bf16", sT, fl)
    run.gI.fill_(0.5); run.gT.fill_(-0.25); run.loss.fill_(2.0); run.gs.fill_(1.0)
    run.rank(r, S, accumulate=True)
    l2, a2, t2, g2 = run.results()
    assert l2 == pytest.approx(2.0 + loss, rel=1e-6) and g2 == pytest.approx(1.0 + gs, rel=1e-6)
    np.testing.assert_allclose(a2, gI + 0.5, rtol=1e-6)
    np.testing.assert_allclose(t2, gT - 0.25, rtol=1e-6)


@pytest.mark.parametrize("M,d,N,chunks", [(2525, 64, 1, 2), (5050, 64, 2, 2), (5050, 64, 4, 2), (825, 64, 3, 3)])
def test_two_view_row_chunks(M, d, N, chunks):
    B, r = 2 * M, N - 1
    assert dl.disco_describe_plan(B, d, N, dl.DISCO_BF16, dl.DISCO_PATH_FUSED, two_view=True).row_chunks == chunks
    Z = two_views(M, d, 7)
    bits = f32_to_bf16_bits(Z)
    Z, Zd = bf16_bits_to_f32(bits), torch.from_numpy(bits.view(np.int16)).cuda()
    need = dl.ntxent_workspace_bytes(B, d, N, dl.DISCO_BF16, dl.DISCO_PATH_FUSED)
    ws = torch.empty(need, dtype=torch.uint8, device="cuda")
    loss, gs, gZ = torch.zeros(1, device="cuda"), torch.zeros(1, device="cuda"), torch.empty(B, d, device="cuda")
    print(f"case row chunks two views M={M} d={d} N={N}", flush=True)
    dl.ntxent_loss_fwd_bwd(Zd, B, d, r, N, S, dl.DISCO_BF16, dl.DISCO_PATH_FUSED, 0, loss, gZ, gs, ws, need, torch.cuda.current_stream())
    torch.cuda.synchronize()
    ref, scale = nx.ntxent_rank(Z, S, r, N), nx.ntxent_rank_term_scale(Z, S, r, N)
    check_scalar("loss", float(loss.item()), ref[0], TOL["bf16"]["scalar"])
    check_scalar("gs", float(gs.item()), ref[2], TOL["bf16"]["scalar"] * 10, abs_tol=1e-9 + 2.0 ** -8 * scale[1])
    check_tensor("gZ", gZ.cpu().numpy().astype(np.float64), ref[1], "bf16", scale[0], 1e-13 * S / B)
