"""The extraction on both sides of the lines between its two kernels, against
the oracle: small observations by the size of the catalogue and by the number
of pairs, large ones by the size of the catalogue; and chunks of visibilities, whose number is rounded up to a multiple
of eight between 9 and 63, cut by the shortest step and by the fill, and in FP64
on both sides of the smaller table's range of tiles and of waves."""
import pytest

from tests import test_gpu_extract_vp as vp

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("rows,n_src,mixed", [(5200, 800, True), (5200, 801, True), (4000, 1024, False),
                                              (4000, 1025, False), (2000, 2000, True), (2001, 2000, True),
                                              (2000, 2000, False), (2001, 2000, False), (600, 3072, True),
                                              (600, 3073, True), (65, 3072, False), (65, 3073, False),
                                              (24999, 1100, False), (25000, 1100, False), (25000, 1536, True),
                                              (25000, 1537, True), (147968, 1100, True), (147969, 1100, True)])
def test_catalogue_of_a_small_observation(rows, n_src, mixed):
    vp.test_small_extraction_against_oracle(rows, n_src, mixed, "cells")


@pytest.mark.parametrize("mixed", [False, True])
@pytest.mark.parametrize("rows,n_src", [(1024, 2), (1025, 2), (1153, 3), (2049, 5), (8064, 2), (8193, 2), (4097, 501),
                                        (11400, 799)])
def test_chunks_in_multiples_of_eight(rows, n_src, mixed):
    vp.test_small_extraction_against_oracle(rows, n_src, mixed, "cells")


@pytest.mark.parametrize("mixed", [False, True])
@pytest.mark.parametrize("rows,n_src", [(7, 2100), (2048, 2100), (2049, 2100), (2049, 8129), (5003, 2049),
                                        (16129, 2100), (16385, 2049), (90001, 2100), (120001, 4000), (700001, 200),
                                        (400730, 10000), (900001, 10000)])
def test_chunks_of_source_tiles(rows, n_src, mixed):
    vp.test_small_extraction_against_oracle(rows, n_src, mixed, "one" if rows > 20000 else "cells")


@pytest.mark.parametrize("rows,n_src,mixed", [(1612801, 160, False), (1612801, 161, False), (1075201, 192, True),
                                              (1075201, 193, True), (806400, 200, True), (806144, 200, True),
                                              (806400, 200, False), (806144, 200, False)])
def test_catalogue_of_a_large_observation(rows, n_src, mixed):
    vp.test_small_extraction_against_oracle(rows, n_src, mixed, "one")
