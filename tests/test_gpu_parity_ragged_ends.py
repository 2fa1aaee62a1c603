"""Shares and batches that are not whole tiles: the tile kernels take zeros for the rows past the ends of the matrices instead of what
memory holds there.  The features lie in the middle of larger buffers, once with NaN before and behind them, once with zeros: the same bits, for
one to three rows past a tile and one short of it, both tile sizes, every bf16 path, both losses, and rows that are redone over all keys."""
import numpy as np
import pytest
import torch

import paper_2304_08480_amd as dl
from synth import adversarial_pairs, clip_pairs, f32_to_bf16_bits
from tests.gpu_util import Runner

pytestmark = pytest.mark.gpu
GUARD = 512                                                # rows: more than any tile reaches past an end
S = 14.285714
M, F, Y = dl.DISCO_PATH_MATERIALIZED, dl.DISCO_PATH_FUSED, dl.DISCO_PATH_SYMMETRIC


def _inside(X, fill):
    bits = torch.from_numpy(f32_to_bf16_bits(X).view(np.int16)).cuda()
    all_ = torch.full((X.shape[0] + 2 * GUARD, X.shape[1]), fill, dtype=torch.bfloat16, device="cuda")
    all_[GUARD:-GUARD] = bits.view(torch.bfloat16)
    return all_[GUARD:-GUARD]


@pytest.mark.parametrize("B,d,N,path,kind", [
    (1025, 64, 5, M, None), (1281, 128, 3, M, None), (2306, 256, 2, M, None), (4095, 64, 1, M, None), (6145, 192, 5, M, None),
    (8449, 512, 7, M, None), (9088, 576, 16, M, None), (1154, 192, 2, F, None), (6401, 128, 1, F, None), (9088, 576, 16, F, None),
    (6145, 320, 1, Y, None), (10241, 128, 1, Y, None), (1400, 512, 2, M, "big_norm_low_cos"), (1409, 128, 1, F, "big_norm_low_cos"),
    (6401, 256, 1, Y, "big_norm_low_cos")])
def test_nothing_past_the_ends_takes_part(B, d, N, path, kind):
    I, T = adversarial_pairs(B, d, 31, kind) if kind else clip_pairs(B, d, 31)
    out = []
    for fill in (float("nan"), 0.0):
        run = Runner(_inside(I, fill), _inside(T, fill), B, d, N, dl.DISCO_BF16, path)
        for r in sorted({0, N - 1}):
            print(f"case ends B={B} d={d} N={N} path={path} {kind} rank={r} guard={fill}", flush=True)
            if path == Y:
                run.full(S)
            else:
                run.rank(r, S)
            out.append(run.results())
    for a, b in zip(out[:len(out) // 2], out[len(out) // 2:]):
        assert np.isfinite(a[0]) and a[0] == b[0] and a[3] == b[3] and np.array_equal(a[1], b[1]) and np.array_equal(a[2], b[2])


@pytest.mark.parametrize("B,d,N,path", [(1026, 64, 3, M), (4098, 256, 1, M), (8194, 128, 2, F)])
def test_nothing_past_the_ends_takes_part_two_view(B, d, N, path):
    Z = np.concatenate(clip_pairs(B // 2, d, 33))
    out = []
    for fill in (float("nan"), 0.0):
        Zd = _inside(Z, fill)
        need = dl.ntxent_workspace_bytes(B, d, N, dl.DISCO_BF16, path)
        ws = torch.empty(need, dtype=torch.uint8, device="cuda")
        loss, gs, gZ = torch.zeros(1, device="cuda"), torch.zeros(1, device="cuda"), torch.zeros(B, d, device="cuda")
        print(f"case ends two-view B={B} d={d} N={N} path={path} guard={fill}", flush=True)
        dl.ntxent_loss_fwd_bwd(Zd, B, d, N - 1, N, S, dl.DISCO_BF16, path, 0, loss, gZ, gs, ws, need, torch.cuda.current_stream())
        torch.cuda.synchronize()
        out.append((loss.item(), gs.item(), gZ.cpu().numpy()))
    assert np.isfinite(out[0][0]) and out[0][:2] == out[1][:2] and np.array_equal(out[0][2], out[1][2])
