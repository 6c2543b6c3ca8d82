"""The register-tiled backward kernel: every layout of its registers and rows at the edges of its sizes, both ways of dealing
destinations to sets, split destinations, and what happens around it (capture, refused memory, misaligned dY).

Whole numbers below 2^24 throughout, so every order of the sums gives the same bits."""
import pytest
import torch

pytestmark = pytest.mark.gpu

if torch.cuda.is_available():
    import paper_2312_08656_amd as maxk


@pytest.fixture(scope="module", autouse=True)
def _need_gpu():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    maxk.load_library()


_DTYPE = {"f32": torch.float32, "bf16": torch.bfloat16, "f16": torch.float16}


def _case(N, nnz, dim, k, fmt, seed, hubs=3):
    """Random entries (duplicates add), `hubs` destinations and one source with a large share of them, the last tenth of the
    nodes without any."""
    gen = torch.Generator(device="cuda").manual_seed(seed)
    src = torch.randint(N, (nnz,), generator=gen, device="cuda")
    dst = torch.randint(max(1, N - N // 10), (nnz,), generator=gen, device="cuda")
    dst[: nnz // 5] = torch.randint(max(1, min(hubs, N)), (nnz // 5,), generator=gen, device="cuda")
    src[nnz // 5: nnz // 4] = N // 2
    order = torch.argsort(src, stable=True)
    src, dst = src[order], dst[order]
    rowptr = torch.zeros(N + 1, dtype=torch.int32, device="cuda")
    rowptr[1:] = torch.cumsum(torch.bincount(src, minlength=N), 0)
    val = torch.randint(-3, 4, (nnz,), generator=gen, device="cuda").float()
    dY = torch.randint(-5, 6, (N, dim), generator=gen, device="cuda").to(_DTYPE[fmt])
    index = torch.rand(N, dim, generator=gen, device="cuda").topk(k, dim=1).indices.sort(dim=1).values
    want = torch.zeros((N, k), dtype=torch.float64, device="cuda")
    for at in range(0, nnz, 1 << 17):
        s, d = src[at: at + (1 << 17)], dst[at: at + (1 << 17)]
        want.index_add_(0, d, dY[s].double().gather(1, index[d]) * val[at: at + (1 << 17), None].double())
    assert want.abs().max() < 2 ** 24
    return rowptr, dst.to(torch.int32), val, dY, index, want.float()


def _graph(monkeypatch, how, rowptr, col, val):
    monkeypatch.setenv("MAXK_BWD_REGS", how)
    monkeypatch.delenv("MAXK_SLAB_KB", raising=False)
    return maxk.maxk_graph_create(rowptr, col, val)


def _run(gr, dY, index, ib):
    idx = index.to(maxk.index_dtype(ib)) if ib != 2 else index.to(torch.int16)
    out = torch.full((dY.shape[0], index.shape[1]), float("nan"), device="cuda")
    maxk.maxk_sspmm_bwd_narrow(gr, dY, idx, out)
    return out


# rows of 16 bytes to 2 KiB (a copy's quarter, half, whole, one and a half, two), 4 / 2 / 1 destinations a register and two
# registers a destination, whole and partly used lanes
_SHAPES = [(4, 1), (60, 8), (64, 16), (64, 64), (100, 13), (128, 17), (128, 32), (256, 1), (256, 16), (256, 31), (256, 33), (256, 64),
           (256, 65), (256, 128), (300, 20), (384, 96), (388, 40), (512, 12), (512, 128)]


@pytest.mark.parametrize("how", ["2", "3"])
@pytest.mark.parametrize("fmt", ["f32", "bf16", "f16"])
@pytest.mark.parametrize("dim,k", _SHAPES)
def test_every_layout(monkeypatch, how, fmt, dim, k):
    dim = dim if fmt == "f32" else 2 * dim
    rowptr, col, val, dY, index, want = _case(1501, 60_000, dim, k, fmt, dim + k)
    gr = _graph(monkeypatch, how, rowptr, col, val)
    for ib in ([1, 2, 4] if dim <= 256 else [2, 4]):
        out = _run(gr, dY, index, ib)
        assert gr.regs_tables() == 1
        assert torch.equal(out, want)
    gr.destroy()


@pytest.mark.parametrize("how", ["2", "3"])
@pytest.mark.parametrize("N,nnz,dim,k", [(1, 5, 64, 8), (2, 3, 256, 32), (9, 4000, 256, 64),  # lists far beyond one step
                                         (47, 900, 256, 32), (48, 900, 256, 32), (49, 900, 256, 32),  # one tile of rows, and a row more
                                         (300_000, 400_000, 256, 100),  # destinations that no set has: pull takes them
                                         (40_000, 3_000_000, 128, 32)])
def test_edges_of_tiles_and_sets(monkeypatch, how, N, nnz, dim, k):
    rowptr, col, val, dY, index, want = _case(N, nnz, dim, k, "f32", N, hubs=1)
    gr = _graph(monkeypatch, how, rowptr, col, val)
    gr.reserve(dim, k)
    assert gr.regs_tables() == 1
    assert torch.equal(_run(gr, dY, index, 1), want)
    other = index.roll(1, 0)  # other columns on the same tables
    first = _run(gr, dY, other, 4)
    assert torch.equal(first, _run(gr, dY, other, 1)) and gr.regs_tables() == 1
    gr.destroy()


def test_padding_keeps_infinities_in_their_rows(monkeypatch):
    # padding entries read whatever row lies first in a tile: an infinity there must not reach destinations without it
    N, dim, k = 400, 256, 32
    rowptr, col, val, dY, index, want = _case(N, 9000, dim, k, "f32", 3)
    dY[0] = float("inf")
    gr = _graph(monkeypatch, "2", rowptr, col, val.abs() + 1.0)
    hit = torch.zeros(N, dtype=torch.bool, device="cuda")
    hit[col[: int(rowptr[1])].long()] = True
    out = _run(gr, dY, index, 1)
    assert torch.isinf(out[hit]).all() and torch.isfinite(out[~hit]).all() and hit.any() and not hit.all()
    gr.destroy()


@pytest.mark.parametrize("how", ["2", "3"])
def test_captured_and_replayed(monkeypatch, how):
    N, dim, k = 3000, 256, 64
    rowptr, col, val, dY, index, want = _case(N, 90_000, dim, k, "f32", 5)
    gr = _graph(monkeypatch, how, rowptr, col, val)
    gr.reserve(dim, k)
    idx, out, dYs = index.to(torch.uint8), torch.empty((N, k), device="cuda"), torch.empty_like(dY)
    torch.cuda.synchronize()
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph):
        maxk.maxk_sspmm_bwd(gr, dYs, idx, out)
    for rep in range(3):
        dYs.copy_(dY * (rep + 1))
        out.fill_(float("nan"))
        graph.replay()
        torch.cuda.synchronize()
        assert torch.equal(out, want * (rep + 1))
        out.sum().item()  # eager work between replays
    gr.destroy()


def test_refused_memory_and_misaligned_rows_take_the_other_kernels(monkeypatch):
    N, dim, k = 2000, 256, 32
    rowptr, col, val, dY, index, want = _case(N, 50_000, dim, k, "f32", 7)
    gr = _graph(monkeypatch, "2", rowptr, col, val)
    assert gr.bwd_kernel(dim, k) == "register_tiled"
    gr.limit_allocations(0)
    assert torch.equal(_run(gr, dY, index, 1), want)
    assert gr.bwd_kernel(dim, k) == gr.bwd_choice(dim, k)
    gr.limit_allocations(-1)
    assert torch.equal(_run(gr, dY, index, 1), want) and gr.regs_tables() == 0  # asked for again by a reserve only
    gr.reserve(dim, k)
    assert torch.equal(_run(gr, dY, index, 1), want) and gr.regs_tables() == 1
    room = torch.empty(N * dim + 1, device="cuda")
    shifted = room[1:].view(N, dim)
    shifted.copy_(dY)
    assert torch.equal(_run(gr, shifted, index, 1), want)
    for width, kk in ((250, 32), (256, 129), (516, 8)):  # rows that are not whole 16 bytes, k and width beyond its range
        case = _case(N, 50_000, width, kk, "f32", 8)
        assert torch.equal(_run(gr, case[3], case[4], 2), _reference(gr, rowptr, col, val, case)) and gr.regs_tables() == 1
    gr.destroy()


def _reference(gr, rowptr, col, val, case):
    dY, index = case[3], case[4]
    src = torch.repeat_interleave(torch.arange(rowptr.numel() - 1, device="cuda"), (rowptr[1:] - rowptr[:-1]).long())
    want = torch.zeros((dY.shape[0], index.shape[1]), dtype=torch.float64, device="cuda")
    return want.index_add_(0, col.long(), dY[src].double().gather(1, index[col.long()]) * val[:, None].double()).float()
