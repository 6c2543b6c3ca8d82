"""Which records of its list a wavefront of the register-tiled backward kernel copies in each step (no GPU needed)."""
import ctypes
import random

import pytest

from paper_2312_08656_amd import binding

RECORDS = 32  # of a list in one step


@pytest.fixture(scope="module")
def lib():
    if not binding.lib_path().exists():
        from paper_2312_08656_amd import build
        build.build()
    return binding.load_library()


def _copied(lib, record0, records, step):
    first, n = ctypes.c_uint32(), ctypes.c_uint32()
    assert lib.maxk_regs_step_list(record0, records, step, ctypes.byref(first), ctypes.byref(n)) == 0
    return first.value, n.value


# lists of eight wavefronts, tile by tile: one far longer than the others at the end and at the beginning, empty tiles, whole steps
_TILES = [[[0] * 7 + [1]], [[600] + [2] * 7], [[4] * 8, [2000, 0, 0, 0, 0, 0, 0, 0]], [[32, 64, 96, 33, 31, 1, 0, 65]], [[0] * 8, [0, 0, 2] + [0] * 5]]


@pytest.mark.parametrize("seed", range(len(_TILES) + 20))
def test_copies_stay_inside_the_records(lib, seed):
    rng = random.Random(seed)
    tiles = _TILES[seed] if seed < len(_TILES) else [[rng.choice([0, 1, 2, rng.randint(0, 90), rng.randint(0, 1500)]) for _ in range(8)]
                                                       for _ in range(rng.randint(1, 6))]
    total, record0 = sum(map(sum, tiles)), 0
    for lists in tiles:
        steps = max(1, max(-(-records // RECORDS) for records in lists))
        for records in lists:
            seen = 0
            for step in range(steps):
                first, n = _copied(lib, record0, records, step)
                assert first + n <= max(total, 1)
                if step * RECORDS < records:
                    assert first == record0 + seen and n == min(records - seen, RECORDS)
                    seen += n
                else:
                    assert n == 1
            assert seen == records
            record0 += records
