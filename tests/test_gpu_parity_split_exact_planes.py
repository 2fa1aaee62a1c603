"""The fp32 path's large calls on three bf16 planes: in plans for them, and in plans for fp16 ones that the multiplier or (on the device) the features do not
allow, for both losses and with the rows in chunks.  Against the float64 oracles at the fp32 bars, and which planes a call took."""
import numpy as np
import pytest
import torch

import paper_2304_08480_amd as dl
from oracle import clip_oracle as oc
from oracle import ntxent_oracle as nx
from synth import bf16_bits_to_f32, clip_pairs, f32_to_bf16_bits, two_views
from tests.gpu_util import TOL, Runner, check_scalar, check_tensor, forget_planes, planes_taken, term_scale, to_device

pytestmark = pytest.mark.gpu
S = 14.285714


def _change(X, kind):
    if kind == "long row":
        X[-1] *= 100.0
    if kind == "first row zero":
        X[0] = 0.0
    return X


def _run(B, d, N, dtype, kind, s, path, planes):
    I, T = (_change(X, kind) for X in clip_pairs(B, d, 47))
    Ib = Tb = None
    if dtype == "bf16":
        Ib, Tb = f32_to_bf16_bits(I), f32_to_bf16_bits(T)
        I, T = bf16_bits_to_f32(Ib), bf16_bits_to_f32(Tb)
    s /= max(1.0, float(np.abs((I * T).sum(1)).max()))     # the longest pair keeps CLIP's largest logit
    Id, Td, dt = to_device(I, T, Ib, Tb, dtype)
    assert dl.disco_describe_plan(B, d, N, dt, path).kernels == dl.DISCO_KERNELS_SPLIT
    run, r = Runner(Id, Td, B, d, N, dt, path), N - 1
    print(f"case exact planes {kind} B={B} d={d} N={N} dtype={dtype} path={path} s={s}", flush=True)
    forget_planes(run.ws)
    run.rank(r, s)
    loss, gI, gT, gs = run.results()
    assert planes_taken(run.ws) == planes
    ref, scale = oc.disco_rank(I, T, s, r, N), term_scale(oc, I, T, s, r, N)
    check_scalar("loss", loss, ref[0], TOL["f32"]["scalar"])
    check_scalar("gs", gs, ref[3], TOL["f32"]["scalar"] * 10, abs_tol=1e-9)
    check_tensor("gI", gI, ref[1], "f32", scale[0], scale[2])
    check_tensor("gT", gT, ref[2], "f32", scale[1], scale[2])


@pytest.mark.parametrize("B,d,N,dtype", [(3072, 64, 32, "f32"), (2048, 200, 16, "bf16"), (8192, 32, 32, "bf16")])
def test_planned(B, d, N, dtype):
    _run(B, d, N, dtype, "unit", S, dl.DISCO_PATH_AUTO, "bf16")


# (a multiplier whose gradients' scale would leave fp32's normal numbers in the fp16 form)
@pytest.mark.parametrize("B,d,N,dtype", [(2048, 512, 4, "f32"), (4098, 300, 3, "f32"), (5000, 77, 4, "f32"), (16896, 64, 66, "f32"), (6145, 333, 5, "bf16")])
def test_small_multiplier(B, d, N, dtype):
    _run(B, d, N, dtype, "unit", 1e-6, dl.DISCO_PATH_AUTO, "bf16")


@pytest.mark.parametrize("kind,planes", [("unit", "fp16"), ("long row", "bf16 instead"), ("first row zero", "bf16 instead")])
@pytest.mark.parametrize("B,d,N,dtype,chunks", [(6000, 400, 2, "f32", 6), (4099, 330, 1, "f32", 6), (5001, 500, 1, "bf16", 4)])
def test_rows_in_chunks(B, d, N, dtype, chunks, kind, planes):
    dt = dl.DISCO_F32 if dtype == "f32" else dl.DISCO_BF16
    assert dl.disco_describe_plan(B, d, N, dt, dl.DISCO_PATH_NAIVE).row_chunks == chunks
    _run(B, d, N, dtype, kind, S, dl.DISCO_PATH_NAIVE, planes)


@pytest.mark.parametrize("kind,planes", [("unit", "fp16"), ("long row", "bf16 instead"), ("first row zero", "bf16 instead")])
@pytest.mark.parametrize("M,d,N,dtype", [(2049, 230, 3, "f32"), (4096, 256, 1, "f32"), (4100, 333, 2, "bf16")])
def test_two_views(M, d, N, dtype, kind, planes):
    B, r = 2 * M, N - 1
    Z = _change(two_views(M, d, 48), kind)
    s = S / max(1.0, float((Z * np.roll(Z, M, axis=0)).sum(1).max()))
    if dtype == "bf16":
        bits = f32_to_bf16_bits(Z)
        Z, Zd, dt = bf16_bits_to_f32(bits), torch.from_numpy(bits.view(np.int16)).cuda(), dl.DISCO_BF16
    else:
        Zd, dt = torch.from_numpy(Z).cuda(), dl.DISCO_F32
    assert dl.disco_describe_plan(B, d, N, dt, dl.DISCO_PATH_AUTO, two_view=True).kernels == dl.DISCO_KERNELS_SPLIT
    need = dl.ntxent_workspace_bytes(B, d, N, dt, dl.DISCO_PATH_AUTO)
    ws = torch.empty(need, dtype=torch.uint8, device="cuda")
    loss, gs, gZ = torch.zeros(1, device="cuda"), torch.zeros(1, device="cuda"), torch.full((B, d), float("nan"), device="cuda")
    print(f"case exact planes two views {kind} M={M} d={d} N={N} dtype={dtype}", flush=True)
    forget_planes(ws)
    dl.ntxent_loss_fwd_bwd(Zd, B, d, r, N, s, dt, dl.DISCO_PATH_AUTO, 0, loss, gZ, gs, ws, need, torch.cuda.current_stream())
    torch.cuda.synchronize()
    assert planes_taken(ws) == planes
    ref, scale = nx.ntxent_rank(Z, s, r, N), nx.ntxent_rank_term_scale(Z, s, r, N)
    check_scalar("loss", float(loss.item()), ref[0], TOL["f32"]["scalar"])
    check_scalar("gs", float(gs.item()), ref[2], TOL["f32"]["scalar"] * 10, abs_tol=1e-9 + 1e-5 * scale[1])
    check_tensor("gZ", gZ.cpu().numpy().astype(np.float64), ref[1], "f32", scale[0], 1e-13 * s / B)
