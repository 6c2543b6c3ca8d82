"""The tables that the register-tiled backward kernel walks: everything that they make it read or write lies inside its arrays.

The tables are built and read back; the kernel itself is not run here."""
import numpy as np
import pytest
import torch

from test_gpu_bwd_regs import _DTYPE, _SHAPES, _case, _graph

pytestmark = pytest.mark.gpu

if torch.cuda.is_available():
    import paper_2312_08656_amd as maxk

WAVES, RECORDS, BUFFERS, SPARE_STEPS, HOT = 8, 32, 3, 4, 16
_SIZES = ("pitch", "groups", "kr", "n_sets", "spread", "ranges", "run", "longest", "cap", "head", "slots", "rows", "words", "n_steps", "n_records", "n_units",
          "n_parts", "n_sums", "n_split", "n_tail", "part_floats", "hot_parts", "extra_floats")


@pytest.fixture(scope="module", autouse=True)
def _need_gpu():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    maxk.load_library()


def table(gr, which, dtype, i=0):
    lib = maxk.load_library()
    n = lib.maxk_graph_regs_table(gr.handle, i, which, None, 0)
    assert n >= 0
    out = np.zeros(n, np.uint8)
    assert n == 0 or lib.maxk_graph_regs_table(gr.handle, i, which, out.ctypes.data, n) == n
    return out.view(dtype)


def sizes(gr, i=0):
    return dict(zip(_SIZES, table(gr, 0, np.int64, i).tolist(), strict=True))


def longest_sum(gr):
    """Most entries that an accumulator adds up before it is stored, from the records of every step."""
    t = sizes(gr)
    groups, kr, slots, steps = t["groups"], t["kr"], t["slots"], t["n_steps"]
    head = table(gr, 2, np.uint32).reshape(-1, WAVES, t["words"])[:steps].astype(np.int64)
    records = (head[..., 1] & 0xFF) * (1 if kr == 2 else 2 if groups == 1 else 4)
    which = np.repeat(np.arange(steps * WAVES), records.ravel())
    inside = np.arange(len(which)) - np.repeat(np.cumsum(records.ravel()) - records.ravel(), records.ravel())
    acc = (table(gr, 1, np.uint32).reshape(-1, 2, 2)[:, :, 0] & 0xFF)[head[..., 0].ravel()[which] + inside].astype(np.int64)
    group = np.zeros_like(acc) if groups == 1 else (2 * inside[:, None] + np.arange(2)) % groups
    step, wave = np.repeat(which // WAVES, 2), np.repeat(which % WAVES, 2)
    acc, group = acc.ravel(), group.ravel()
    real = acc < slots * kr
    step, wave, acc, group = step[real], wave[real], acc[real], group[real]
    unit, part = table(gr, 5, np.int32).reshape(-1, 5), table(gr, 6, np.int32).reshape(-1, 4)
    worst = 0
    for hot in (False, True):
        ends = np.unique(np.concatenate([unit[:, 2], part[part[:, 1] == slots, 0], part[:, 0] if hot else unit[:, 2]]))
        mine = (acc < HOT * kr) == hot
        sums = np.stack([np.searchsorted(ends, step[mine], side="right"), wave[mine], acc[mine], group[mine]])
        if sums.size:
            worst = max(worst, np.unique(sums, axis=1, return_counts=True)[1].max())
    return worst


def check_sums(gr):
    longest = sizes(gr)["longest"]
    assert longest == 0 or longest_sum(gr) <= longest


def check_steps(gr):
    """The step loop played back: what is copied into a buffer while it may still be read, and where a step's entries look for their rows.

    In step s the rows of step s + 2 are on their way, those of s + 1 may have landed, and other wavefronts still read those of s: each of the
    three has a buffer of its own, or the same rows (a tile with long lists).  Past the end of a unit the steps of the next one follow."""
    t = sizes(gr)
    tile, steps = t["rows"] * WAVES, t["n_steps"]
    head = table(gr, 2, np.uint32).reshape(steps + SPARE_STEPS, WAVES, t["words"])
    buffer, rows = head[..., 1] >> 8, head[..., 2: 2 + t["rows"]]
    assert (buffer == buffer[:, :1]).all()
    for ahead in (1, 2):
        same = buffer[:-ahead, 0] == buffer[ahead:, 0]
        same[max(0, steps - ahead):] = False  # (a buffer that is no longer read)
        at = np.flatnonzero(same)
        assert (rows[at] == rows[at + ahead]).all()
    # the records of a list, in the order of the steps: inside the rows of the step's own buffer
    batch = 1 if t["kr"] == 2 else 2 if t["groups"] == 1 else 4
    first, n = head[:steps, :, 0].astype(np.int64), (head[:steps, :, 1] & 0xFF).astype(np.int64) * batch
    start = first[n > 0]  # (lists do not overlap: check_ranges)
    which = np.broadcast_to(buffer[:steps], n.shape)[n > 0]
    order = np.argsort(start)
    edge = np.repeat(which[order].astype(np.int8), n[n > 0][order])
    record = table(gr, 1, np.uint32).reshape(-1, 4)
    for half in (0, 2):
        real = (record[:, half] & 0xFF) < t["slots"] * t["kr"]  # (padding reads any row, for an accumulator that nobody stores)
        assert (((record[:, half] >> 8) // (t["pitch"] // 256) // tile == edge) | ~real).all()


def check_ranges(gr, N, k):
    t = sizes(gr)
    groups, kr, slots = t["groups"], t["kr"], t["slots"]
    per_wave, steps = slots * groups, t["n_steps"]
    batch = 1 if kr == 2 else 2 if groups == 1 else 4
    assert steps >= 1 and t["n_records"] >= 1

    head = table(gr, 2, np.uint32).reshape(steps + SPARE_STEPS, WAVES, t["words"])
    first, batches, buffer = head[..., 0].astype(np.int64), (head[..., 1] & 0xFF).astype(np.int64), head[..., 1] >> 8
    assert (batches * batch <= RECORDS).all() and (buffer < BUFFERS).all()
    assert (first + np.maximum(batches * batch, 1) <= t["n_records"]).all()
    assert (head[..., 2: 2 + t["rows"]] < N).all()
    assert (batches[steps:] == 0).all()
    # every record belongs to one list
    at, n = first[:steps][batches[:steps] > 0], (batches[:steps] * batch)[batches[:steps] > 0]
    order = np.argsort(at, kind="stable")
    assert n.sum() == t["n_records"] and (np.concatenate([[0], (at + n)[order]])[:-1] == at[order]).all()

    record = table(gr, 1, np.uint32).reshape(-1, 2)[:, 0]
    acc, address = record & 0xFF, record & ~np.uint32(0xFF)
    assert (acc <= slots * kr).all() and (acc % kr == 0).all()
    assert (address % t["pitch"] == 0).all() and (address < BUFFERS * t["rows"] * WAVES * t["pitch"]).all()

    node, row = table(gr, 3, np.int32), table(gr, 4, np.int32)
    assert len(node) == len(row) == t["n_sets"] * WAVES * per_wave
    assert (node >= -1).all() and (node < N).all() and ((node < 0) == (row < 0)).all() and (row >= -1).all()
    assert (row.astype(np.int64) + 1 - N <= t["extra_floats"] // k).all()
    used = np.sort(row[row >= 0])
    assert (np.diff(used) > 0).all() and len(used) == t["head"]  # no two accumulators share a row
    split = table(gr, 8, np.int32).reshape(-1, 3)
    assert (split[:, 0] < N).all() and (split[:, 1:] * k <= t["extra_floats"]).all() and (split[:, 1] < split[:, 2]).all()
    assert (np.sort(row[row >= N] - N) == np.arange(split[:, 2].max(initial=0))).all()

    check_sums(gr)
    check_steps(gr)

    unit, part = table(gr, 5, np.int32).reshape(-1, 5), table(gr, 6, np.int32).reshape(-1, 4)
    at = part.view(np.int64)[:, 1] if len(part) else np.zeros(0, np.int64)
    assert (unit[:, 0] < t["n_sets"]).all() and (0 <= unit[:, 1]).all() and (unit[:, 1] <= unit[:, 2]).all() and (unit[:, 2] <= steps).all()
    assert np.sum(unit[:, 2] - unit[:, 1]) == steps
    assert (np.isin(part[:, 1], [HOT, slots])).all()
    floats = part[:, 1].astype(np.int64) * WAVES * kr * 64
    order = np.argsort(at)
    assert (np.concatenate([[0], (at + floats)[order]])[:-1] == at[order]).all() and floats.sum() == t["part_floats"]
    summed = {int(s) for s in table(gr, 7, np.int32).reshape(-1, 5)[:, 0]}
    for s, begin, end, p0, p1 in unit.tolist():
        assert (p1 > p0) == (s in summed)  # a unit's sums leave as parts, or as results
        if p1 > p0:
            assert (np.diff(np.concatenate([[begin], part[p0:p1, 0]])) > 0).all() and part[p1 - 1, 0] == end and part[p1 - 1, 1] == slots
    for s, w0, w1, h0, h1 in table(gr, 7, np.int32).reshape(-1, 5).tolist():
        whole, hot = WAVES * slots * kr * 64, WAVES * HOT * kr * 64
        assert 0 <= w0 <= w1 and w1 * whole <= t["hot_parts"] and 0 <= h0 <= h1 and t["hot_parts"] + h1 * hot <= t["part_floats"]


@pytest.mark.parametrize("how", ["2", "3"])
@pytest.mark.parametrize("fmt", ["f32", "bf16", "f16"])
@pytest.mark.parametrize("dim,k", _SHAPES)
def test_layouts(monkeypatch, how, fmt, dim, k):
    dim = dim if fmt == "f32" else 2 * dim
    rowptr, col, val, *_ = _case(1501, 60_000, dim, k, fmt, dim + k)
    gr = _graph(monkeypatch, how, rowptr, col, val)
    gr.reserve(dim, k, _DTYPE[fmt])
    assert gr.regs_tables() == 1
    check_ranges(gr, 1501, k)
    gr.destroy()


# few rows and long lists, whole tiles and a row more, one hub beside many short lists, destinations that no set has
@pytest.mark.parametrize("how", ["2", "3"])
@pytest.mark.parametrize("N,nnz,dim,k,hubs", [(1, 5, 64, 8, 1), (2, 3, 256, 32, 1), (9, 4000, 256, 64, 1), (9, 4000, 256, 100, 3), (47, 900, 256, 32, 1),
                                              (48, 9000, 256, 16, 2), (49, 900, 256, 32, 1), (3000, 20_000, 128, 12, 1),
                                              (20_000, 600_000, 256, 64, 1), (300_000, 400_000, 256, 100, 1), (40_000, 3_000_000, 128, 32, 1)])
def test_uneven_lists(monkeypatch, how, N, nnz, dim, k, hubs):
    rowptr, col, val, *_ = _case(N, nnz, dim, k, "f32", N, hubs=hubs)
    gr = _graph(monkeypatch, how, rowptr, col, val)
    gr.reserve(dim, k)
    assert gr.regs_tables() == 1
    check_ranges(gr, N, k)
    gr.destroy()


def _hub(N, d, n):
    """A hub of d in-entries beside n others; its sources crowd into the first tenth of the nodes."""
    gen = torch.Generator(device="cuda").manual_seed(N + d)
    src = torch.cat([torch.randint(N // 10, (d,), generator=gen, device="cuda"), torch.randint(N, (n,), generator=gen, device="cuda")])
    dst = torch.cat([torch.full((d,), 7, device="cuda"), torch.randint(N, (n,), generator=gen, device="cuda")])
    order = torch.argsort(src, stable=True)
    rowptr = torch.zeros(N + 1, dtype=torch.int32, device="cuda")
    rowptr[1:] = torch.cumsum(torch.bincount(src, minlength=N), 0)
    return rowptr, dst[order].to(torch.int32)


# Terms of 1.1 each: what an addition rounds off has the same sign over a whole binade of the sum, so errors add up instead of cancelling
# (3000 of them: 2.7e-5).
# A sum of n equal terms is off by at most (n + 1)/2 units of 2^-24 (half a unit of the running sum an addition); the stored sums are added up in
# 64 bits, and a share and the result are rounded once each.
@pytest.mark.parametrize("how,k", [("2", 64), ("3", 64), ("3", 100), ("3", 24), ("2", 24)])
@pytest.mark.parametrize("N,d,n", [(20_000, 200_000, 200_000), (3000, 40_000, 30_000)])
def test_hub_sums_are_short(monkeypatch, how, k, N, d, n):
    dim = 256
    rowptr, col = _hub(N, d, n)
    gr = _graph(monkeypatch, how, rowptr, col, torch.ones(d + n, device="cuda"))
    dY = torch.full((N, dim), 1.1, device="cuda")
    index = torch.arange(k, device="cuda", dtype=torch.uint8).repeat(N, 1)
    out = torch.empty((N, k), device="cuda")
    maxk.maxk_sspmm_bwd(gr, dY, index, out)
    assert gr.regs_tables() == 1
    exact = torch.bincount(col.long(), minlength=N).double() * float(np.float32(1.1))
    error = ((out.double() - exact[:, None]).abs().amax(1) / exact.clamp_min(1.0)).max().item()
    longest = 128  # the least that any layout is held to
    assert error <= (longest / 2 + 3) * 2.0 ** -24
    check_sums(gr)
    gr.destroy()
