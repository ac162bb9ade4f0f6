"""Columns per workgroup of the windowed explicit-matrix kernel (host rule, no
GPU): widths inside the kernel's range and the LDS budget for every matrix
size, and the widths that the rule's figures name."""
import ctypes

import pytest

LDS = 80 * 1024


@pytest.fixture(scope="module")
def width():
    import paper_2510_17432_amd as csp
    # csp::ellw_columns_per_group(bool, bool, int, long, int, long, long)
    f = ctypes.CDLL(csp._lib._name)["_ZN3csp22ellw_columns_per_groupEbbilill"]
    f.restype = ctypes.c_int
    f.argtypes = [ctypes.c_bool, ctypes.c_bool, ctypes.c_int, ctypes.c_int64, ctypes.c_int,
                  ctypes.c_int64, ctypes.c_int64]
    return f


@pytest.mark.parametrize("fp64", [False, True])
@pytest.mark.parametrize("ring", [False, True])
@pytest.mark.parametrize("nr", [128, 256])
def test_widths_are_in_range(width, fp64, ring, nr):
    for window in (1, 7, 293, 632, 832, 1300, 2048, 5000, 20000):
        fit = max(1, min((7 if nr == 256 else 6) if fp64 else 8, LDS // (window * (16 if fp64 else 8))))
        for slices in (1, 3, 29, 313, 700, 1250, 2048, 3000, 40000):
            for D in (1, 29, 121, 233):
                for Rg in range(1, 33):
                    w = width(fp64, ring, Rg, window, nr, slices, slices * nr * D)
                    assert 1 <= w <= min(fit, Rg), (window, slices, D, Rg)
                    tiles = -(-Rg // w)
                    assert -(-Rg // tiles) == w       # the split that the kernel makes


# (complex128, ring, columns, 97th percentile of the windows, rows of a slice, slices, D) -> width
@pytest.mark.parametrize("case,w", [
    ((False, False, 7, 397, 128, 1253, 61), 7),      # 400^2, D = 61: one round of one tile
    ((False, False, 5, 397, 128, 1253, 61), 5),
    ((False, False, 4, 632, 128, 1253, 121), 2),     # 400^2, D = 121: 2 + 2
    ((False, False, 8, 632, 128, 706, 121), 4),      # 300^2: 4 + 4
    ((False, False, 3, 632, 128, 315, 121), 1),      # 200^2: latency
    ((False, False, 10, 632, 128, 315, 121), 3),
    ((False, False, 5, 832, 256, 1024, 121), 5),     # 512^2
    ((False, False, 7, 832, 256, 1100, 121), 7),     # 530^2
    ((False, False, 6, 832, 256, 1041, 121), 3),     # 516^2, cached
    ((False, False, 6, 828, 256, 1603, 121), 6),     # 640^2, from HBM
    ((False, False, 8, 876, 128, 1583, 233), 8),     # 450^2, D = 233, from HBM
    ((False, False, 7, 876, 128, 1583, 233), 7),
    ((True, False, 5, 632, 128, 706, 121), 5),       # 300^2
    ((True, False, 8, 632, 128, 706, 121), 4),
    ((True, False, 10, 632, 128, 706, 121), 5),
    ((True, False, 4, 632, 128, 315, 121), 2),       # 200^2
    ((True, False, 6, 832, 256, 1100, 121), 6),      # 530^2: 78 KB of LDS
    ((True, False, 7, 632, 128, 1803, 121), 4),      # 480^2, from HBM: 4 + 3
    ((True, False, 7, 603, 256, 2025, 61), 7),       # 720^2, D = 61, from HBM
    ((False, False, 9, 632, 128, 581, 121), 3),      # 272^2: latency
    ((False, False, 9, 632, 128, 660, 121), 3),      # 290^2: four waves per SIMD
    ((False, True, 10, 632, 128, 1253, 121), 5),     # rings: 400^2
    ((False, True, 5, 397, 128, 960, 61), 3),        # 350^2, D = 61
    ((True, True, 9, 397, 128, 615, 61), 5),         # 280^2, D = 61
    ((True, True, 6, 632, 128, 706, 121), 6),        # 300^2
])
def test_widths_of_the_rule(width, case, w):
    fp64, ring, Rg, window, nr, slices, D = case
    assert width(fp64, ring, Rg, window, nr, slices, slices * nr * D) == w
