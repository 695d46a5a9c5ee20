"""The host rules that choose a kernel's tiles, called in the library (no GPU:
the rules then plan for 256 CUs, as on the card). The functions are C++ ones of
the library's own headers, bound by their mangled names."""
import ctypes

import pytest

from paper_2606_07881_amd import binding
from parity import small_cfg


class Pair(ctypes.Structure):
    _fields_ = [("a", ctypes.c_int), ("b", ctypes.c_int)]


def rule(name, *types, restype=ctypes.c_int):
    f = getattr(binding.lib, name)
    f.argtypes, f.restype = types, restype
    return f


I = ctypes.c_int
P = ctypes.POINTER(I)
f32_tile = rule("_ZN4paci13gemm_f32_tileEiii", I, I, I)                                          # (M, N, splits)

kmajor_plan = rule("_ZN4paci16gemm_kmajor_planEii", I, I, restype=Pair)                          # (M, N)
window_plan = rule("_ZN4paci16gemm_window_planEiil", I, I, ctypes.c_int64, restype=Pair)         # (M, N, K)
group_split = rule("_ZN4paci17wgrad_group_splitEPKiS1_iPNS_9WgradTileE", P, P, I, P)             # (M, N, n, rest)
group_xcd_m = rule("_ZN4paci17wgrad_group_xcd_mEiiiNS_9WgradTileE", I, I, I, I)                  # (M, N, K, tile)
KMAJOR = ["256x128 ring", "256x256", "128x128", "128x64", "64x64"]   # enum KmajorTile
GROUPED = ["256x128", "256x256", "128x128", "64x64"]                 # enum WgradTile


def tokens(c):
    return c["seq"] * c["micro_batch"]


def kmajor(c, N):
    """(tiles, columns of the first of two launches) of a product with N output columns."""
    p = kmajor_plan(tokens(c), N)
    return KMAJOR[p.a], p.b


def weights(c):
    """(out, in) of the weights of a block, in the order of the grouped launch: W_2, W_1, W_o, W_qkv."""
    d, f = c["d_model"], c["d_ff"]
    return [(d, f), (f, d), (d, d), (3 * d, d)] * c["n_layers"]


def grouped(c):
    """Leading problems on 256 x 256 tiles, the tiles of the others, and each one's XCD bands."""
    w, rest = weights(c), I()
    n1 = group_split((I * len(w))(*[m for m, _ in w]), (I * len(w))(*[n for _, n in w]), len(w), ctypes.byref(rest))
    return n1, GROUPED[rest.value], [group_xcd_m(m, n, tokens(c), 1 if i < n1 else rest.value)
                                     for i, (m, n) in enumerate(w)]


def window(c, K=None):
    """(tile columns, splits) of each weight's window product over K micro-batches."""
    return [(p.a, p.b) for p in (window_plan(m, n, tokens(c) * (K or c["K"])) for m, n in weights(c)[:4])]


def cfg(name, d, **kw):
    return small_cfg(name, d_model=d, n_heads=d // 32, head_dim=32, **kw)


# The parity workloads run on the tiles that their descriptions name.
def test_tiles_of_the_parity_workloads():
    assert kmajor(small_cfg("wide_bf16"), 2304) == ("256x256", 0)
    assert kmajor(small_cfg("tall_bf16"), 4064) == ("256x256", 0)
    n1, rest, xcd = grouped(small_cfg("xcd_bf16"))
    assert (n1, rest) == (0, "128x128") and all(xcd)
    n1, rest, xcd = grouped(small_cfg("xcd2_bf16"))
    assert (n1, rest) == (0, "256x128") and all(xcd)
    assert window(small_cfg("win8_bf16")) == [(128, 16)] * 4
    assert window(small_cfg("winsplit_bf16")) == [(128, 4)] * 4
    assert window(small_cfg("winwide_bf16")) == [(128, 2)] * 3 + [(256, 2)]


# So do the cases of the tile tests.
def test_tiles_of_the_tile_tests():
    for d in (32, 64, 128, 160, 288):                                                # test_pingpong_kmajor
        assert kmajor(cfg("tall_bf16", d), 4064) == ("256x256", 0)
    for d in (480, 512):                                                             # test_pingpong_all_products
        c = cfg("dh32_bf16", d, d_ff=64, seq=83, micro_batch=200)
        assert kmajor(c, d) == kmajor(c, 3 * d) == ("256x256", 0)
    c = cfg("dh32_bf16", 640, d_ff=64, seq=85, micro_batch=300)                      # test_ring_rounds
    assert kmajor(c, 640) == kmajor(c, 1920) == ("256x128 ring", 0)
    c = cfg("dh32_bf16", 480, d_ff=1440, seq=81, micro_batch=200)                    # test_column_split
    assert kmajor(c, 1440) == ("256x256", 1024)
    for T in (40, 64, 72, 75, 128, 201):                                             # test_pingpong_grouped
        assert grouped(small_cfg("tall_bf16", d_model=1024, d_ff=4096, seq=T, micro_batch=1))[0] == 4
    for seq, mu in ((33, 1), (33, 3), (101, 5)):                                     # test_grouped_odd_tokens
        assert grouped(small_cfg("ragged_bf16", seq=seq, micro_batch=mu))[:2] == (0, "64x64")
        assert grouped(cfg("dh32_bf16", 544, d_ff=2048, seq=seq, micro_batch=mu))[:2] == (0, "256x128")
    for d, T, sp in ((288, 64, 1), (288, 320, 1), (96, 384, 1), (512, 384, 1), (512, 1088, 2)):   # test_pingpong_window
        assert window(cfg("win_bf16", d, d_ff=416, seq=T // 2), 1) == [(128, sp)] * 4
    for d, T, sp in ((2016, 64, 1), (2016, 192, 1), (1504, 1152, 2)):
        assert window(cfg("win_bf16", d, d_ff=96, seq=T // 2), 1)[3] == (256, sp)
    assert window(small_cfg("winwide_bf16", seq=32, K=18))[3] == (256, 2)            # .._short_segments


# fp32 products: the largest edge with two workgroups per CU, the splits over K counted.
@pytest.mark.parametrize("M,N,splits,edge", [(4096, 2048, 1, 128), (4096, 2047, 1, 128), (4096, 1920, 1, 64),
                                             (4096, 1024, 2, 128), (4096, 1024, 1, 64), (2048, 1024, 1, 64),
                                             (2048, 960, 1, 32), (512, 512, 8, 64), (64, 64, 16, 32), (1, 32, 1, 32)])
def test_f32_tile(M, N, splits, edge):
    assert f32_tile(M, N, splits) == edge
