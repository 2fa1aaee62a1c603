"""The plans that calls run under, pinned on the host: no GPU work.  A plan is the fastest of its candidates by the library's
own time model; only a call without a workspace of its own gives speed for staying within the static array."""
import random

import pytest

import paper_2304_08480_amd as dl

BF16, F32 = dl.DISCO_BF16, dl.DISCO_F32
MAT, FUSED, SYM, AUTO, NAIVE = (dl.DISCO_PATH_MATERIALIZED, dl.DISCO_PATH_FUSED, dl.DISCO_PATH_SYMMETRIC, dl.DISCO_PATH_AUTO,
                                dl.DISCO_PATH_NAIVE)
STATIC = dl.disco_static_scratch_bytes()


def _shapes(n, seed):
    rng = random.Random(seed)
    while n:
        b, N = int(2 ** rng.uniform(7, 13)), rng.choice((1, 2, 4, 8, 16, 32, 64))
        if b * N <= 200000:
            n -= 1
            yield b * N, 64 * rng.randint(1, 16), N


@pytest.mark.parametrize("path", [MAT, FUSED], ids=["materialized", "fused"])
def test_a_limit_never_makes_a_plan_faster(path):
    limited = 0
    for B, d, N in _shapes(400, 1):
        free = dl.disco_describe_plan(B, d, N, BF16, path)
        assert free.workspace_bytes == dl.disco_workspace_bytes(B, d, N, BF16, path)
        for limit in (STATIC,) if path == FUSED else (STATIC, 4 * STATIC):       # (a lean plan without a limit has its own budget)
            kept = dl.disco_describe_plan(B, d, N, BF16, path, workspace_limit=limit, check=False)
            if kept.workspace_bytes <= limit:
                assert free.microseconds <= kept.microseconds * 1.0001, (B, d, N, limit)
                limited += kept.workspace_bytes < free.workspace_bytes
    assert limited > 10                                     # (the limit does bind on some of them)


# Shapes whose largest plans lie above the static array (measured with plans of 64 MiB / with these, us: 52550 / 7060,
# 9450 / 556, 12590 / 2476, 1392 / 353, 938 / 545, 659 / 386, 131 / 93).
@pytest.mark.parametrize("B,d,N,path,pieces", [(122880, 1024, 32, FUSED, 8), (39744, 256, 16, FUSED, 3), (61440, 768, 16, FUSED, 4),
                                               (24000, 512, 16, FUSED, 2), (32768, 512, 16, FUSED, 2), (16384, 320, 4, FUSED, 2),
                                               (24448, 256, 64, MAT, 1)])
def test_a_callers_own_workspace_is_not_held_to_the_static_array(B, d, N, path, pieces):
    p = dl.disco_describe_plan(B, d, N, BF16, path)
    assert p.workspace_bytes > STATIC
    assert p.row_chunks * p.key_panels <= pieces


def test_memory_lean_plans_keep_to_their_numerators():
    # 2 b W numerators of 2 bytes for a panel width W of at most half the keys and 16384, in chunks of rows or panels of keys; with
    # what the other parts take (partial products of at most 32 splits, operands and sums) it stays under the stored numerators'
    for B, d, N in _shapes(300, 2):
        p = dl.disco_describe_plan(B, d, N, BF16, FUSED)
        b = (B // N + 255) // 256 * 256
        W = min(16384, ((B + 255) // 256 + 1) // 2 * 256)
        other = 32 * 2 * b * d * 4 + 8 * ((B + 255) // 256 * 256 + b) * (d + 4) + 2 * b * ((B + 255) // 256 * 4) * 4 + (1 << 16)
        assert p.workspace_bytes <= max(2 * b * W * 2 + other, STATIC), (B, d, N)


def test_static_plans_stay_within_the_array():
    for B, d, N in _shapes(300, 3):
        for path in (AUTO, MAT, FUSED, NAIVE) + ((SYM,) if N == 1 else ()):
            p = dl.disco_describe_plan(B, d, N, BF16, path, workspace_limit=STATIC, check=False)
            st = dl.DISCO_OK if p.workspace_bytes <= STATIC else dl.DISCO_ERR_WORKSPACE
            q = dl.DiscoPlan()
            assert dl.binding._lib.disco_describe_plan(B, d, N, BF16, path, 0, STATIC, q) == st
            assert p.workspace_bytes == q.workspace_bytes


# (the sizes that the static entry point took when its plans were the only ones)
@pytest.mark.parametrize("B,d,N,dt,path", [(2048, 256, 4, BF16, AUTO), (4096, 256, 8, BF16, FUSED), (4096, 512, 8, BF16, MAT),
                                           (24448, 256, 64, BF16, MAT), (24000, 512, 16, BF16, FUSED), (39744, 256, 16, BF16, FUSED),
                                           (2560, 64, 1, BF16, SYM), (3072, 512, 1, BF16, SYM), (2048, 512, 4, F32, NAIVE)])
def test_the_static_entry_point_takes_what_it_took(B, d, N, dt, path):
    assert dl.disco_describe_plan(B, d, N, dt, path, workspace_limit=STATIC).workspace_bytes <= STATIC


# fp32 path, large calls: (B, d, N, dtype) and the measured time, us, on the planes that the plan is for.  The model is rough: within a quarter.
@pytest.mark.parametrize("B,d,N,dt,us", [(8192, 512, 8, F32, 201), (12288, 256, 4, F32, 535), (10416, 1024, 8, F32, 691), (12288, 100, 8, BF16, 177)])
def test_the_described_time_is_that_of_the_plan_that_runs(B, d, N, dt, us):
    assert 0.75 * us <= dl.disco_describe_plan(B, d, N, dt, AUTO).microseconds <= 1.25 * us


def test_plan_query_arguments():
    q = dl.DiscoPlan()
    call = dl.binding._lib.disco_describe_plan
    assert call(1024, 64, 2, BF16, MAT, 0, 0, None) == dl.DISCO_ERR_NULL
    assert call(1000, 64, 3, BF16, MAT, 0, 0, q) == dl.DISCO_ERR_SHAPE
    assert call(1024, 65, 2, BF16, MAT, 0, 0, q) == dl.DISCO_ERR_UNSUPPORTED
    assert call(1024, 64, 2, BF16, FUSED, 0, 1, q) == dl.DISCO_ERR_WORKSPACE
    p = dl.disco_describe_plan(32768, 512, 8, F32, AUTO)
    assert p.path == NAIVE and p.kernels == dl.DISCO_KERNELS_SPLIT
    p = dl.disco_describe_plan(512, 64, 2, BF16, AUTO)
    assert p.path == MAT and p.kernels == dl.DISCO_KERNELS_SMALL
    p = dl.disco_describe_plan(32768, 512, 1, BF16, AUTO)
    assert p.path == SYM and p.kernels == dl.DISCO_KERNELS_SYMMETRIC
    assert dl.disco_describe_plan(8192, 128, 1, BF16, AUTO, two_view=True).kernels == dl.DISCO_KERNELS_TILES
