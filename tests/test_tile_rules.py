"""The host rules that choose a kernel's tiles, called in the library (no GPU:
the rules then plan for 256 CUs, as on the card). The functions are C++ ones of
the library's own headers, bound by their mangled names."""
import ctypes

import pytest

from paper_2606_07881_amd import binding


def rule(name, *types, restype=ctypes.c_int):
    f = getattr(binding.lib, name)
    f.argtypes, f.restype = types, restype
    return f


I = ctypes.c_int
NT, NN, TN = 0, 1, 2
f32_tile = rule("_ZN4paci13gemm_f32_tileENS_10GemmLayoutEiiii", I, I, I, I, I)   # (layout, M, N, K, splits)


# Forward (NT) and input-gradient (NN) products in fp32 by how many 128 x 128 tiles they have. Whole
# rounds of the 256 CUs and a last one at least 7/8 full: 128 (4096 x 1024 over 4096: 327 us, 337
# on 64 x 64); less of it: 64 (3072 x 1024: 237 against 327); few: 32.
@pytest.mark.parametrize("lay", [NT, NN])
@pytest.mark.parametrize("M,N,edge", [(4096, 1024, 128), (8192, 512, 128), (16384, 256, 128), (4096, 896, 128),
                                      (4095, 1023, 128), (4096, 864, 128), (4096, 768, 64), (6000, 768, 64),
                                      (4096, 1536, 64), (4096, 1792, 128), (4096, 2048, 128), (4096, 2176, 64),
                                      (8192, 8192, 128), (2048, 1024, 64), (2048, 512, 32), (1, 32, 32)])
def test_f32_tile(lay, M, N, edge):
    assert f32_tile(lay, M, N, 1024, 1) == edge


# a single round over a short K: 64 for the forward products
def test_f32_tile_short_k():
    assert [f32_tile(NT, 8192, 512, K, 1) for K in (64, 255, 256)] == [64, 64, 128]
    assert [f32_tile(NN, 8192, 512, K, 1) for K in (64, 255, 256)] == [128, 128, 128]
    assert f32_tile(NT, 16384, 512, 64, 1) == 128


# Weight gradients: the largest edge with two workgroups per CU, the splits over K counted.
@pytest.mark.parametrize("M,N,splits,edge", [(4096, 1024, 1, 64), (4096, 1024, 2, 128), (4096, 2048, 1, 128),
                                             (512, 512, 8, 64), (64, 64, 16, 32)])
def test_f32_tile_wgrad(M, N, splits, edge):
    assert f32_tile(TN, M, N, 2048, splits) == edge
