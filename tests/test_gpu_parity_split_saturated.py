"""The fp32 path's large calls where the softmax has all but decided: off-label masses far below what a gradient entry held to a fixed
number of bits could show, alone or beside rows that are undecided, for both losses, both dtypes and rows in chunks.  Against float64 with
the off-label mass added up directly (the oracle forms P_label - 1 by subtraction), so the bars need no floor: the fp32 one, 1e-4, for each
gradient and for each of its rows.  (What fp32 itself costs: a logit is good to a few 2^-24, s = 70 times that moves an entry by 1e-5.)  A row
may miss the bar by what the key side leaves out of a sum over rows of very different size: an entry of G is held to 2^-51 in rows whose largest is above
2^-16 and to 2^-39 of the row's largest elsewhere, the features of a row to 2^-32 of those of the row with the most mass t_max, so
b rows leave out 2^-31 b t_max c s at most (features of norm 1)."""
import numpy as np
import pytest
import torch

import paper_2304_08480_amd as dl
from synth import bf16_bits_to_f32, clip_pairs, f32_to_bf16_bits
from tests.gpu_util import Runner, forget_planes, planes_taken, to_device

pytestmark = pytest.mark.gpu
BAR = 1e-4


def _gradient_matrix(X, Y, labels, selves, s):
    """softmax - onehot of the rows of s X Y^T, and the rows' cross-entropies."""
    rows = np.arange(len(X))
    E = X @ Y.T
    E = np.exp(s * (E - E[rows, labels][:, None]))
    E[rows, labels] = 0.0
    if selves is not None:
        E[rows, selves] = 0.0
    off = E.sum(1)
    E[rows, labels] = -off
    return E / (1.0 + off)[:, None], np.log1p(off), len(X) * (off / (1.0 + off)).max()


def _reference(I, T, s, r, N):
    I, T = I.astype(np.float64), T.astype(np.float64)
    B, b = len(I), len(I) // N
    own, c = np.arange(r * b, (r + 1) * b), 1.0 / (2 * B)
    Ga, la, ta = _gradient_matrix(I[own], T, own, None, s)
    Gc, lc, tc = _gradient_matrix(T[own], I, own, None, s)
    gI, gT = Gc.T @ T[own], Ga.T @ I[own]
    gI[own] += Ga @ T
    gT[own] += Gc @ I
    return c * (la.sum() + lc.sum()), c * s * gI, c * s * gT, 2.0 ** -31 * c * s * max(ta, tc)


def _check(name, got, ref, left_out):
    rel = np.linalg.norm(got - ref) / np.linalg.norm(ref)
    err, size = np.linalg.norm(got - ref, axis=1), np.linalg.norm(ref, axis=1)
    row = (err / np.maximum(BAR * size + left_out, 1e-300)).max()
    print(f"{name}: {rel:.2e}, worst row {row:.2e} of its bound, {(err / np.maximum(size, 1e-300)).max():.2e} of its norm", flush=True)
    assert rel <= BAR and row <= 1.0, (name, rel, row)


def _pairs(kind, B, d):
    I, T = clip_pairs(B, d, 61)                            # positives of cosine 0.89
    if kind == "mixed":                                    # every third row's positive no nearer than its negatives
        T[::3] = clip_pairs(B, d, 63)[0][::3]
    return I, T


# (2049, 515: rows that are not whole pieces; 1536, 1536 and 2304, 2560: the scaled rows take all the room behind G, and more)
@pytest.mark.parametrize("B,d,N,dtype,path", [(2048, 512, 4, "f32", dl.DISCO_PATH_AUTO), (2049, 515, 3, "f32", dl.DISCO_PATH_AUTO),
                                              (8192, 64, 16, "f32", dl.DISCO_PATH_AUTO), (6000, 400, 2, "f32", dl.DISCO_PATH_NAIVE),
                                              (1536, 1536, 2, "f32", dl.DISCO_PATH_AUTO), (2304, 2560, 3, "f32", dl.DISCO_PATH_AUTO),
                                              (6145, 333, 5, "bf16", dl.DISCO_PATH_AUTO)])
@pytest.mark.parametrize("kind,s", [("near", 30.0), ("near", 40.0), ("near", 50.0), ("near", 70.0), ("mixed", 50.0)])
def test_decided_rows(B, d, N, dtype, path, kind, s):
    _decided(B, d, N, dtype, path, kind, s, "bf16" if dtype == "f32" and (d < 192 or 5 * s > d) else "fp16")


# fp32 features: fp16 planes from d = 192 on while 5 |s| <= d; bf16 features lose nothing in them
@pytest.mark.parametrize("B,d,N,dtype,s,planes", [
    (4096, 191, 4, "f32", 14.0, "bf16"), (4096, 192, 4, "f32", 14.0, "fp16"), (4096, 192, 4, "f32", 38.0, "fp16"), (4096, 192, 4, "f32", -39.0, "bf16"),
    (4098, 320, 3, "f32", 64.0, "fp16"), (4098, 320, 3, "f32", 65.0, "bf16"), (2048, 512, 4, "f32", 100.0, "fp16"), (12288, 100, 8, "bf16", 70.0, "fp16")])
def test_large_multipliers_and_narrow_features(B, d, N, dtype, s, planes):
    _decided(B, d, N, dtype, dl.DISCO_PATH_AUTO, "near", s, planes)


def _decided(B, d, N, dtype, path, kind, s, planes):
    I, T = _pairs(kind, B, d)
    Ib = Tb = None
    if dtype == "bf16":
        Ib, Tb = f32_to_bf16_bits(I), f32_to_bf16_bits(T)
        I, T = bf16_bits_to_f32(Ib), bf16_bits_to_f32(Tb)
    Id, Td, dt = to_device(I, T, Ib, Tb, dtype)
    assert dl.disco_describe_plan(B, d, N, dt, path).kernels == dl.DISCO_KERNELS_SPLIT
    run, r = Runner(Id, Td, B, d, N, dt, path), N - 1
    print(f"case decided {kind} B={B} d={d} N={N} dtype={dtype} path={path} s={s}", flush=True)
    forget_planes(run.ws)
    run.rank(r, s)
    loss, gI, gT, _ = run.results()
    assert planes_taken(run.ws) == planes
    ref = _reference(I, T, s, r, N)
    assert abs(loss - ref[0]) <= BAR * ref[0]
    _check("gI", gI, ref[1], ref[3])
    _check("gT", gT, ref[2], ref[3])
    run.rank(r, s, accumulate=True)
    _, a, t, _ = run.results()
    _check("gI twice", a, 2 * ref[1], 2 * ref[3])
    _check("gT twice", t, 2 * ref[2], 2 * ref[3])


@pytest.mark.parametrize("s", [20.0, 40.0, 80.0])
def test_rows_decided_alike(s):
    # all rows of G have one power of two in common and no row is scaled: pairwise orthogonal features, the positive a copy
    B, N, r = 2048, 4, 1
    I = np.eye(B, dtype=np.float32)
    Id, Td, dt = to_device(I, I, None, None, "f32")
    assert dl.disco_describe_plan(B, B, N, dt, dl.DISCO_PATH_AUTO).kernels == dl.DISCO_KERNELS_SPLIT
    run = Runner(Id, Td, B, B, N, dt, dl.DISCO_PATH_AUTO)
    print(f"case decided alike s={s}", flush=True)
    forget_planes(run.ws)
    run.rank(r, s)
    loss, gI, gT, _ = run.results()
    assert planes_taken(run.ws) == "fp16"
    ref = _reference(I, I, s, r, N)
    assert abs(loss - ref[0]) <= BAR * ref[0]
    _check("gI", gI, ref[1], ref[3])
    _check("gT", gT, ref[2], ref[3])


@pytest.mark.parametrize("M,d,N,s", [(2048, 256, 1, 40.0), (2049, 330, 3, 60.0), (2049, 130, 3, 60.0)])
def test_decided_rows_two_view(M, d, N, s):
    B, r = 2 * M, N - 1
    Z = np.concatenate(clip_pairs(M, d, 62))
    assert dl.disco_describe_plan(B, d, N, dl.DISCO_F32, dl.DISCO_PATH_AUTO, two_view=True).kernels == dl.DISCO_KERNELS_SPLIT
    need = dl.ntxent_workspace_bytes(B, d, N, dl.DISCO_F32, dl.DISCO_PATH_AUTO)
    ws = torch.empty(need, dtype=torch.uint8, device="cuda")
    loss, gs, gZ = torch.zeros(1, device="cuda"), torch.zeros(1, device="cuda"), torch.full((B, d), float("nan"), device="cuda")
    print(f"case decided two views M={M} d={d} N={N} s={s}", flush=True)
    forget_planes(ws)
    dl.ntxent_loss_fwd_bwd(torch.from_numpy(Z).cuda(), B, d, r, N, s, dl.DISCO_F32, dl.DISCO_PATH_AUTO, 0, loss, gZ, gs, ws, need,
                           torch.cuda.current_stream())
    torch.cuda.synchronize()
    assert planes_taken(ws) == ("fp16" if d >= 5 * s else "bf16")
    Z, b = Z.astype(np.float64), B // N
    own = np.arange(r * b, (r + 1) * b)
    G, l, t = _gradient_matrix(Z[own], Z, (own + M) % B, own, s)
    ref = G.T @ Z[own]
    ref[own] += G @ Z
    assert abs(loss.item() - l.sum() / B) <= BAR * l.sum() / B
    _check("gZ", gZ.cpu().numpy().astype(np.float64), s / B * ref, 2.0 ** -31 * s / B * t)
