"""Which kernels the fp32 path's calls take, pinned on the host: calls of narrow fp32 features take the split kernels where those were
measured to be faster by a tenth and more (and nearer to 64 bits), and calls that were faster or more accurate on the small kernels keep
them."""
import pytest

import paper_2304_08480_amd as dl

F32, BF16 = dl.DISCO_F32, dl.DISCO_BF16


# us on the small / on the split kernels
@pytest.mark.parametrize("B,d,N,dtype,two_view", [
    (4096, 64, 16, F32, False),       # 66 / 47
    (2560, 64, 1, F32, False),        # 187 / 108
    (2048, 100, 1, F32, False),       # 130 / 88
    (4096, 20, 4, F32, False),        # 88 / 69
    (6144, 20, 24, F32, False),       # 86 / 52
    (2048, 20, 1, F32, True),         # 65 / 54
    (4096, 100, 8, F32, True),        # 66 / 48
])
def test_split_where_it_is_faster(B, d, N, dtype, two_view):
    assert dl.disco_describe_plan(B, d, N, dtype, dl.DISCO_PATH_AUTO, two_view=two_view).kernels == dl.DISCO_KERNELS_SPLIT


@pytest.mark.parametrize("B,d,N,dtype,two_view", [
    (256, 512, 4, F32, False),        # 13.5 / 48
    (1024, 512, 4, F32, False),       # 51 / 59
    (2048, 128, 16, F32, False),      # 40 / 44
    (1024, 64, 4, F32, False),        # 26 / 33
    (1024, 256, 2, F32, False),       # 41 / 46
    (300, 300, 1, BF16, False),       # 23 / 30
    (1024, 1000, 4, BF16, False),     # 39 / 45
    (2048, 1000, 16, BF16, False),    # 48 / 54
    (2048, 896, 64, BF16, True),      # 36 / 50
    (4096, 1024, 512, BF16, True),    # 53 / 67
    (4096, 1024, 512, F32, True),     # 96 / 123
    (1536, 200, 1, F32, False),       # 145 / 84, gradients as accurate or less
    (4096, 128, 16, F32, True),       # 57 / 47, gradients up to 1.9 times as far off at s = 100
    (2560, 100, 1, BF16, False),      # 115 / 88, gradients 1.3 times as far off
])
def test_small_where_it_is_faster_or_more_accurate(B, d, N, dtype, two_view):
    assert dl.disco_describe_plan(B, d, N, dtype, dl.DISCO_PATH_AUTO, two_view=two_view).kernels == dl.DISCO_KERNELS_SMALL


def test_the_kernels_of_the_named_path_fit_its_memory():
    # whatever its kernels, the fp32 path by name takes what its fp32 blocks need and no more
    for B, d, N in ((4098, 64, 1), (8192, 64, 8), (6144, 100, 1), (4096, 20, 4)):
        for dt in (F32, BF16):
            b = B // N
            assert dl.disco_workspace_bytes(B, d, N, dt, dl.DISCO_PATH_NAIVE) <= 2 * b * (B + 3) * 4 + 64 * b + 4096
