"""Where the kernels that work by lane groups fetch a work item's entries, up to the largest entry count a graph may have (no GPU needed)."""
import pytest

from paper_2312_08656_amd import binding

MOST = 0x7FFFFFF0  # entries that maxk_graph_create accepts


@pytest.fixture(scope="module")
def lib():
    if not binding.lib_path().exists():
        from paper_2312_08656_amd import build
        build.build()
    return binding.load_library()


@pytest.mark.parametrize("batch", [16, 32, 64])  # entries of a batch
@pytest.mark.parametrize("end", [1, 63, 64, 1000, MOST - 100, MOST - 1, MOST])
def test_batches_fetched_ahead_stay_inside_the_item(lib, batch, end):
    for begin in {max(0, end - n) for n in (1, 2, batch - 1, batch, batch + 1, 2 * batch + 1, 2048)}:
        for base in range(begin, end + batch, batch):  # (the last one is behind the item)
            for ahead in (0, batch, 2 * batch):
                first = lib.maxk_entry_batch(base, ahead, end)
                assert begin <= first < end, (begin, base, ahead)
                assert first == min(base + ahead, end - 1)
