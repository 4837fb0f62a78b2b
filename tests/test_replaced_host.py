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
                                  (329, 2752, 19584, BF16, 0), (342, 2816, 23680, BF16, 0), (121, 2048, 12288, BF16, 1),         # .67, .64, .92
                                  (576, 14048, 2436, FP8, 1), (944, 8576, 1456, BF16, 1), (315, 736, 3937, FP16, 1, 34)])        # .67, .68, .70
def test_another_tile_where_it_was_faster(call):
    assert _replaced(*call)


@pytest.mark.parametrize("call", [
    (3, 128, 4096, FP8, 0, 7), (46, 224, 7728, FP8, 0), (3, 928, 7936, FP8, 0), (1, 768, 5248, FP8, 0),       # 1.37, 1.38, 1.34, 1.27
    (208, 80, 11920, BF16, 1), (76, 96, 10735, FP16, 1), (160, 288, 9776, BF16, 1), (160, 80, 8688, BF16, 1),  # 1.21, 1.20, 1.18, 1.14
    (66, 49, 10496, FP16, 1, 9), (11, 64, 11119, FP16, 1, 7), (142, 106, 14337, FP8, 1, 2),                   # 1.24, 1.23, 1.20
    (32, 128, 2048, BF16, 0, 12), (62, 70, 3572, BF16, 0, 9), (224, 128, 2592, FP16, 0),                      # 1.13, 1.14, 1.11
    (5, 1280, 4096, BF16, 0)])                                                                                # 1.06
def test_not_sliced_where_it_was_slower(call):
    assert not _replaced(*call)


@pytest.mark.parametrize("call", [(40, 64, 8192, BF16, 1), (1, 1024, 4096, BF16, 1), (2, 2048, 9728, BF16, 1), (19, 32, 8064, BF16, 1),   # .54, .59, .61, .54
                                  (4, 224, 4096, BF16, 0), (5, 1680, 4096, BF16, 0), (2, 128, 4096, FP16, 0),                    # .45, .80, .48
                                  (37, 16, 6784, FP8, 0), (2, 16, 6121, FP8, 0), (55, 70, 4096, FP8, 1)])                       # .67, .70
def test_sliced_where_it_was_faster(call):
    assert _replaced(*call)
