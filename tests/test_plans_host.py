"""Choices of the time models, on the host."""
import paper_1212_4137_amd as spca


def test_one_wave_tiles_where_they_are_faster():
    """Shapes 32 to 37 are the one-wave tiles, those below 12 the workgroup
    tiles; each size was measured on both, at the plan's K split."""
    spca.tune_table_clear()
    for size in ((128, 10000, 1000), (256, 10000, 1000), (1024, 1000, 1250), (512, 10000, 1000),
                 (1024, 10000, 1000), (256, 1000, 10000), (77, 7131, 4075), (20, 22453, 3027)):
        assert spca.gemm_plan(*size, 16)[0] < 12, size
    for size in ((16, 1000, 8000), (12, 162, 24937), (339, 653, 10114), (64, 2000, 20000),
                 (181, 649, 1138), (56, 596, 23928), (2, 1325, 33001), (1, 5695, 4128)):
        assert 32 <= spca.gemm_plan(*size, 16)[0] < 38, size
