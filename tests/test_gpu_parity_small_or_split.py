"""Calls of narrow fp32 features, tiny shares and odd widths that go to the split kernels, where every operand is mostly padding: one to a
hundred columns in K-steps of 64, shares of 32 rows in tiles of 128, features and gradients off their boundary.  Against the float64
oracles at the fp32 bars, and against the small kernels, which the path takes by name."""
import numpy as np
import pytest
import torch

import paper_2304_08480_amd as dl
from oracle import clip_oracle as oc
from oracle import ntxent_oracle as nx
from synth import clip_pairs, two_views
from tests.gpu_util import TOL, Runner, check_scalar, check_tensor, term_scale, to_device

pytestmark = pytest.mark.gpu
S = 14.285714


def _moved(x, shift):
    return torch.empty(x.numel() + shift, dtype=x.dtype, device="cuda")[shift:].view(x.shape).copy_(x)


@pytest.mark.parametrize("B,d,N,shift", [
    (4096, 2, 128, 0),         # shares of 32 rows, two columns
    (4096, 64, 64, 0),         # shares of 64 rows, one K-step of d
    (6144, 20, 24, 1),         # features off their boundary
    (3072, 77, 1, 0),          # odd width: gradients through partial sums
    (2048, 100, 1, 0),
    (1600, 96, 1, 0),
])
def test_narrow_and_ragged_calls_on_split_kernels(B, d, N, shift):
    I, T = clip_pairs(B, d, 17)
    Id, Td, dt = to_device(I, T, None, None, "f32")
    if shift:
        Id, Td = _moved(Id, shift), _moved(Td, shift)
    assert dl.disco_describe_plan(B, d, N, dt, dl.DISCO_PATH_AUTO).kernels == dl.DISCO_KERNELS_SPLIT
    assert dl.disco_describe_plan(B, d, N, dt, dl.DISCO_PATH_NAIVE).kernels == dl.DISCO_KERNELS_SMALL
    runs = [Runner(Id, Td, B, d, N, dt, p) for p in (dl.DISCO_PATH_AUTO, dl.DISCO_PATH_NAIVE)]
    for r in sorted({0, N - 1}):
        print(f"case small or split B={B} d={d} N={N} rank={r} shift={shift}", flush=True)
        ref, scale = oc.disco_rank(I, T, S, r, N), term_scale(oc, I, T, S, r, N)
        for run in runs:
            run.rank(r, S)
            loss, gI, gT, gs = run.results()
            check_scalar("loss", loss, ref[0], TOL["f32"]["scalar"])
            check_scalar("gs", gs, ref[3], TOL["f32"]["scalar"] * 10, abs_tol=1e-9)
            check_tensor("gI", gI, ref[1], "f32", scale[0], scale[2])
            check_tensor("gT", gT, ref[2], "f32", scale[1], scale[2])
    auto = runs[0]
    auto.gI, auto.gT = _moved(auto.gI, 1), _moved(auto.gT, 1)         # (whole pieces of a row cannot be written: the small kernels, or element by element)
    auto.rank(N - 1, S)
    moved = auto.results()
    np.testing.assert_allclose(moved[1], gI, rtol=1e-3, atol=1e-6 * np.abs(gI).max())
    np.testing.assert_allclose(moved[2], gT, rtol=1e-3, atol=1e-6 * np.abs(gT).max())


@pytest.mark.parametrize("B,d,N", [(2048, 20, 1), (4096, 64, 16), (4096, 77, 8)])
def test_narrow_two_view_calls_on_split_kernels(B, d, N):
    Z = two_views(B // 2, d, 18)
    Zd = torch.from_numpy(Z).cuda()
    assert dl.disco_describe_plan(B, d, N, dl.DISCO_F32, dl.DISCO_PATH_AUTO, two_view=True).kernels == dl.DISCO_KERNELS_SPLIT
    need = dl.ntxent_workspace_bytes(B, d, N, dl.DISCO_F32, dl.DISCO_PATH_AUTO)
    ws = torch.empty(need, dtype=torch.uint8, device="cuda")
    loss, gs, gZ = torch.zeros(1, device="cuda"), torch.zeros(1, device="cuda"), torch.empty(B, d, device="cuda")
    print(f"case small or split two views B={B} d={d} N={N}", flush=True)
    dl.ntxent_loss_fwd_bwd(Zd, B, d, N - 1, N, S, dl.DISCO_F32, dl.DISCO_PATH_AUTO, 0, loss, gZ, gs, ws, need, torch.cuda.current_stream())
    torch.cuda.synchronize()
    ref, scale = nx.ntxent_rank(Z, S, N - 1, N), nx.ntxent_rank_term_scale(Z, S, N - 1, N)
    check_scalar("loss", float(loss.item()), ref[0], TOL["f32"]["scalar"])
    check_scalar("gs", float(gs.item()), ref[2], TOL["f32"]["scalar"] * 10, abs_tol=1e-9 + 1e-5 * scale[1])
    check_tensor("gZ", gZ.cpu().numpy().astype(np.float64), ref[1], "f32", scale[0], 1e-13 * S / B)


@pytest.mark.parametrize("B,d,N,fits", [(2560, 64, 1, False), (4096, 64, 16, True)])     # (the split kernels' workspace in the static array)
def test_less_memory_and_capture(B, d, N, fits):
    I, T = clip_pairs(B, d, 19)
    Id, Td, dt = to_device(I, T, None, None, "f32")
    run, named = Runner(Id, Td, B, d, N, dt, dl.DISCO_PATH_AUTO), Runner(Id, Td, B, d, N, dt, dl.DISCO_PATH_NAIVE)
    assert (run.ws_bytes <= dl.disco_static_scratch_bytes()) == fits and named.ws_bytes < run.ws_bytes
    run.rank(N - 1, S)
    split = run.results()
    named.rank(N - 1, S)
    small = named.results()
    print(f"case less memory B={B} d={d} N={N}", flush=True)
    st = torch.cuda.current_stream()
    dl.disco_loss_fwd_bwd(Id, Td, B, d, N - 1, N, S, dt, dl.DISCO_PATH_AUTO, 0, run.loss, run.gI, run.gT, run.gs, named.ws, named.ws_bytes, st)
    assert all(np.array_equal(a, b) for a, b in zip(run.results(), small))               # what fits the path by name runs as that path
    dl.disco_loss_fwd_bwd_static(Id, Td, B, d, N - 1, N, S, dt, dl.DISCO_PATH_AUTO, 0, run.loss, run.gI, run.gT, run.gs, st)
    assert all(np.array_equal(a, b) for a, b in zip(run.results(), split if fits else small))
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph):
        run.rank(N - 1, S)
    for _ in range(3):
        for o in (run.loss, run.gs, run.gI, run.gT):
            o.fill_(float("nan"))
        graph.replay()
        assert all(np.array_equal(a, b) for a, b in zip(run.results(), split))
        named.rank(0, S)                                   # eager work between the replays
