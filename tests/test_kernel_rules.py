"""Which of two kernels a call takes, at shapes where both were timed (no GPU needed)."""
import pytest

from paper_2312_08656_amd import binding


@pytest.fixture(scope="module")
def lib():
    if not binding.lib_path().exists():
        from paper_2312_08656_amd import build
        build.build()
    return binding.load_library()


@pytest.mark.parametrize("k,dim,value_type,items,entries,units", [
    (17, 256, 0, 60_000, 960_000, 0), (17, 384, 0, 60_000, 960_000, 1), (20, 512, 0, 60_000, 960_000, 1), (21, 384, 0, 1_000_000, 9_000_000, 1),
    (19, 512, 0, 300_000, 9_300_000, 1), (17, 1024, 0, 40_013, 1_240_013, 1), (19, 512, 0, 100_000, 6_100_000, 0), (17, 1024, 0, 100_000, 6_100_000, 1),
    (17, 384, 1, 60_000, 960_000, 0), (17, 512, 1, 60_000, 960_000, 1), (21, 384, 1, 1_000_000, 9_000_000, 0),
    (16, 1024, 0, 60_000, 960_000, 0), (22, 1024, 0, 60_000, 960_000, 0), (9, 64, 0, 60_000, 960_000, 1), (193, 256, 0, 60_000, 960_000, 1)])
def test_forward_row_by_row(lib, k, dim, value_type, items, entries, units):
    assert lib.maxk_fwd_by_units(k, dim, value_type, items, entries) == units
