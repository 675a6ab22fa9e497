"""Which launch the matrix-core product takes (vbq_kernel_name, descriptors only):
waves per workgroup on both sides of each line of the rule, in the geometry
that the packer chooses and in others."""

import numpy as np
import pytest

from paper_2607_02893_amd import vbq


def _desc(N, K, mixed=True, R=0, C=0):
    bits = np.ones((N, K // 64), dtype=np.uint8)
    if mixed:
        bits[:, ::2] = 4
        bits[0, 0] = 8
    return vbq.pack_size(bits, K, R, C)[1]


def _args(desc, M):
    name = vbq.kernel_name(desc, M)
    assert name.startswith("vbq_mm_kernel<"), name
    return name[len("vbq_mm_kernel<"):-1].split(",")


@pytest.mark.parametrize("M", [3, 4, 16])
@pytest.mark.parametrize("N,K,waves", [
    (4096, 8256, 8), (4097, 8256, 4), (6000, 8256, 4), (5120, 13824, 4), (12288, 8256, 4),  # eight units, 16-row tiles
    (4096, 2048, 8), (4112, 2048, 4), (9000, 576, 4), (12288, 320, 4),                      # four units, three
    (16384, 8256, 8), (20000, 8256, 4), (16384, 4096, 4), (16384, 576, 8), (20000, 576, 4),  # 32-row tiles
    (28672, 4096, 8), (32768, 4096, 8), (32769, 4096, 4), (28672, 2048, 4), (28672, 576, 8),  # 64-row tiles
])
def test_waves_of_mixed_products(N, K, waves, M):
    d = _desc(N, K)
    assert d.tile_rows == (16 if N < 16353 else 32 if N < 28609 else 64)
    assert int(_args(d, M)[0]) == waves


@pytest.mark.parametrize("N,K,waves", [(10240, 2048, 8), (10256, 2048, 4), (10256, 14336, 8), (300, 64, 4)])
def test_waves_of_one_width_products(N, K, waves):
    assert int(_args(_desc(N, K, mixed=False), 4)[0]) == waves


@pytest.mark.parametrize("M", [3, 16])
@pytest.mark.parametrize("N,K,R,C,one_word", [
    (12288, 1024, 0, 0, False), (12289, 1024, 0, 0, True), (14000, 1088, 16, 5, False), (20000, 256, 0, 0, False),
    (28672, 256, 0, 0, True), (28672, 320, 0, 0, True), (28672, 512, 0, 0, False), (300, 256, 64, 1, True),
    (300, 256, 256, 1, False),
])
def test_one_word_variant(N, K, R, C, one_word, M):
    args = _args(_desc(N, K, True, R, C), M)
    assert (args[-1] == "-2") == one_word
    assert args[-1] != "-2" or args[0] == "4" or int(args[1]) == 4


@pytest.mark.parametrize("uniform", [False, True])
@pytest.mark.parametrize("N,K,R,C,ragged", [
    (300, 1024, 0, 0, False), (300, 256, 0, 0, True), (300, 320, 0, 0, True), (300, 64, 0, 0, True), (300, 2048, 0, 0, False),
    (300, 576, 16, 4, True), (300, 8256, 16, 128, True), (20000, 512, 0, 0, False), (20000, 256, 0, 0, True),
    (20000, 576, 32, 2, True), (28672, 64, 0, 0, False), (300, 64, 256, 1, False),
])
def test_ragged_variant(N, K, R, C, ragged, uniform):
    args = _args(_desc(N, K, not uniform, R, C), 4)
    assert args[2] == ("true" if ragged else "false")
