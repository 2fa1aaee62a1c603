"""GPU parity of the bf16 paths over the instances that the plan of a call chooses between: logit and gradient tiles of
256 or 128, the key-side reduction split or not.  Each shape is there for the instances named beside it; dense
against the float64 oracle, one inner rank overwriting and accumulating."""
import numpy as np
import pytest
import torch

import paper_2304_08480_amd as dl
from oracle import clip_oracle as oc
from oracle import ntxent_oracle as nx
from synth import clip_pairs, two_views, f32_to_bf16_bits, bf16_bits_to_f32
from tests.gpu_util import term_scale, check_scalar, check_tensor, to_device, TOL
from tests.test_gpu_parity_ntxent import Run
from tests.test_gpu_parity_ragged import GuardedRunner

pytestmark = pytest.mark.gpu


def _bits(x):
    b = f32_to_bf16_bits(x)
    return bf16_bits_to_f32(b), b


def _check(got, ref, scale, floor, tag, terms=1.0):
    check_scalar(f"{tag} loss", got[0], terms * ref[0], TOL["bf16"]["scalar"], abs_tol=1e-12)
    check_scalar(f"{tag} gs", got[3], terms * ref[3], TOL["bf16"]["scalar"] * 10, abs_tol=1e-9)
    for n, k in (("gI", 1), ("gT", 2)):
        check_tensor(f"{tag} {n}", got[k], terms * ref[k], "bf16", terms * scale[k - 1], floor)


# (logit tile, gradient tile, key side split, key panels, row chunks) of the plan that the case is there for
@pytest.mark.parametrize("B,d,N,path,plan", [
    (1024, 256, 2, "materialized", (128, 128, False, 1, 1)),     # a workgroup per row in the finalize kernel
    (1000, 64, 1, "materialized", (128, 128, True, 1, 1)),       # the same with the key side split, ragged
    (2176, 64, 17, "materialized", (128, 128, False, 1, 1)),     # shares of exactly one tile
    (2100, 64, 1, "materialized", (128, 128, True, 1, 1)),       # a ragged last split and a ragged tile
    (2304, 320, 3, "materialized", (128, 128, False, 1, 1)),     # the last column tile half full
    (2836, 64, 2, "materialized", (256, 128, True, 1, 1)),
    (4000, 256, 2, "materialized", (256, 128, False, 1, 1)),     # ragged
    (6000, 512, 2, "materialized", (128, 256, False, 1, 1)),     # ragged
    (8192, 1024, 4, "materialized", (256, 256, False, 1, 1)),
    (8100, 1024, 4, "materialized", (256, 256, False, 1, 1)),    # ragged
    (1154, 192, 2, "fused", (128, 128, False, 2, 1)),            # ragged panels
    (9088, 576, 16, "fused", (256, 256, False, 2, 1)),           # panels of large tiles, ragged
    (8320, 192, 5, "fused", (256, 128, False, 3, 1)),            # three panels, ragged shares
    (16384, 320, 4, "fused", (256, 128, False, 1, 2)),           # rows in chunks
    (5000, 320, 1, "symmetric", (128, 128, False, 1, 1)),        # one rank below the size from which the symmetric kernels run
    (5700, 320, 1, "symmetric", (256, 256, False, 1, 1)),        # and above it
])
def test_instances_of_the_tile_kernels(B, d, N, path, plan):
    s = 14.285714
    code = getattr(dl, "DISCO_PATH_" + path.upper())
    got = dl.disco_describe_plan(B, d, N, dl.DISCO_BF16, code)
    assert (got.logit_tile, got.gradient_tile, got.key_splits > 1, got.key_panels, got.row_chunks) == plan
    assert got.kernels == (dl.DISCO_KERNELS_SYMMETRIC if B == 5700 else dl.DISCO_KERNELS_TILES)
    I, T = clip_pairs(B, d, 31, noise=1.0)
    (I, Ib), (T, Tb) = _bits(I), _bits(T)
    Id, Td, dt = to_device(I, T, Ib, Tb, "bf16")
    run = GuardedRunner(Id, Td, B, d, N, dt, code)
    r = N // 2
    print(f"case tile sizes B={B} d={d} N={N} {path} rank={r}", flush=True)
    ref, sc = oc.disco_rank(I, T, s, r, N), term_scale(oc, I, T, s, r, N)
    run.rank(r, s)
    _check(run.results(), ref, sc, sc[2], f"B{B} d{d} N{N} {path}")
    run.rank(r, s, accumulate=True)
    _check(run.results(), ref, sc, 2 * sc[2], f"B{B} d{d} N{N} {path} accumulated", 2.0)
    assert run.guards_intact()


@pytest.mark.parametrize("M,d,N,plan", [
    (1500, 64, 2, (128, 128, True)),      # the positives in the other rank, ragged
    (1500, 192, 1, (256, 128, True)),     # every positive local
    (600, 128, 3, (128, 128, True)),      # a rank that holds rows of both views, positives inside and outside
    (3072, 512, 2, (128, 128, False)),
])
def test_instances_of_the_tile_kernels_two_view(M, d, N, plan):
    s, B = 14.285714, 2 * M
    got = dl.disco_describe_plan(B, d, N, dl.DISCO_BF16, dl.DISCO_PATH_MATERIALIZED, two_view=True)
    assert (got.logit_tile, got.gradient_tile, got.key_splits > 1) == plan
    Z, bits = _bits(two_views(M, d, 32, noise=1.0))
    run = Run(torch.from_numpy(bits.view(np.int16)).cuda(), B, d, N, dl.DISCO_BF16, dl.DISCO_PATH_MATERIALIZED)
    for r in range(N):
        print(f"case tile sizes two-view M={M} d={d} N={N} rank={r}", flush=True)
        ref, (sc, gsc) = nx.ntxent_rank(Z, s, r, N), nx.ntxent_rank_term_scale(Z, s, r, N)
        for terms, acc in ((1.0, False), (2.0, True)):
            run.rank(r, s, accumulate=acc)
            loss, gZ, gs = run.results()
            check_scalar("loss", loss, terms * ref[0], TOL["bf16"]["scalar"])
            check_scalar("gs", gs, terms * ref[2], TOL["bf16"]["scalar"] * 10, abs_tol=terms * (1e-9 + 2.0 ** -8 * gsc))
            check_tensor("gZ", gZ, terms * ref[1], "bf16", terms * sc, terms * 1e-13 * s / B)
