"""Which calls run another kernel than their pick names: shapes on which the replacement was measured slower keep their own."""
import pytest

from paper_2512_04226_amd import binding as g

BF16, FP8, FP16 = g.GEMM_BF16, g.GEMM_FP8_E4M3, g.GEMM_FP16


def _replaced(M, N, K, dtype, bl, batch=1, beta=0.0):
    c = g.gemm_select_batched(M, N, K, batch, dtype, bl)
    c.beta = beta
    own = c.copy()
    own.own_tile = 1
    return (g.gemm_launched_kernel(c), g.gemm_launched_tile(c)) != (g.gemm_launched_kernel(own), g.gemm_launched_tile(own))


# (the replacement's time over the own kernel's)
@pytest.mark.parametrize("call", [
    (187, 15232, 2816, FP16, 1), (192, 15552, 13952, FP16, 0),            # 1.43, 1.37: three rows of 64x256 tiles for two of 128x128
    (162, 14976, 6144, FP8, 0), (176, 1968, 12464, BF16, 1),              # 1.29, 1.18
    (146, 7648, 6784, FP16, 0), (181, 7552, 7808, FP16, 0),               # 1.39, 1.23: fewer workgroups over the same weights
    (256, 8192, 28672, FP8, 0), (221, 8192, 28672, FP8, 1),               # 1.17
    (1616, 880, 519, BF16, 0, 32, 0.5), (3444, 15503, 527, FP16, 1, 1, 0.5), (2991, 525, 784, BF16, 0, 36, 0.5),   # 1.37, 1.27, 1.20: the old C
    (90, 512, 896, BF16, 1, 25), (73, 240, 960, FP16, 1, 53), (760, 256, 1248, FP16, 0, 23), (265, 784, 3169, BF16, 0, 17),  # 1.28, 1.33, 1.10, 1.23
    (266, 1664, 640, BF16, 0, 13),                                        # 1.14: one full round of two workgroups to a CU
    (226, 57344, 4096, FP16, 0), (142, 57344, 4096, BF16, 0)])            # 1.07, 1.04: two rounds for one
def test_no_other_tile_where_it_was_slower(call):
    assert not _replaced(*call)


@pytest.mark.parametrize("call", [(1152, 2240, 11696, BF16, 0, 1, 0.5), (1501, 3003, 2005, BF16, 0), (64, 8192, 28672, FP8, 0),   # .86, .85, .99
                                  (256, 28672, 8192, BF16, 0), (226, 57344, 4096, FP16, 1),                                      # .90, .97
                                  (329, 2752, 19584, BF16, 0), (342, 2816, 23680, BF16, 0), (121, 2048, 12288, BF16, 1)])        # .67, .64, .92
def test_another_tile_where_it_was_faster(call):
    assert _replaced(*call)
