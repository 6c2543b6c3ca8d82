"""What the choice of the register-tiled backward kernel remembers: tables that were refused memory."""
import pytest
import torch

from test_gpu_bwd_regs import _DTYPE, _case, _graph, _run
from test_gpu_bwd_regs_tables import sizes

pytestmark = pytest.mark.gpu

if torch.cuda.is_available():
    import paper_2312_08656_amd as maxk


@pytest.fixture(scope="module", autouse=True)
def _need_gpu():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    maxk.load_library()


_LAYOUT = ("n_sets", "spread", "ranges", "run", "longest", "cap")
_SAME = ("pitch", "groups", "kr", "head")


def _layout(t):
    return tuple(t[x] for x in _LAYOUT)


def _alike(monkeypatch):
    """Two shapes whose sets hold the same destinations in the same registers, but are laid out differently, for instance because
    they stand in for different kernels (the LDS-tiled one takes fp32 and k % 4 == 0 only)."""
    N, nnz = 4000, 1_500_000
    found = {}
    for fmt, dim, k in (("f32", 256, 64), ("f32", 256, 40), ("f32", 132, 64), ("f32", 132, 33), ("bf16", 512, 64), ("bf16", 264, 64), ("bf16", 512, 40)):
        case = _case(N, nnz, dim, k, fmt, 11)
        gr = _graph(monkeypatch, "2", *case[:3])
        gr.reserve(dim, k, _DTYPE[fmt])
        t = sizes(gr)
        gr.destroy()
        for other in found.setdefault(tuple(t[x] for x in _SAME), []):
            if _layout(other[0]) != _layout(t):
                return other[1:], (case, dim, k, fmt)
        found[tuple(t[x] for x in _SAME)].append((t, case, dim, k, fmt))
    raise AssertionError([[(_layout(x[0]), x[2:]) for x in v] for v in found.values()])


def test_a_refused_layout_denies_no_other(monkeypatch):
    (a, dim_a, k_a, fmt_a), (b, dim_b, k_b, fmt_b) = _alike(monkeypatch)
    gr = _graph(monkeypatch, "2", *a[:3])
    gr.limit_allocations(0)
    assert torch.equal(_run(gr, a[3], a[4], 2), a[5]) and gr.regs_tables() == 0
    gr.limit_allocations(-1)
    assert gr.bwd_kernel(dim_a, k_a, _DTYPE[fmt_a]) != "register_tiled"
    assert gr.bwd_kernel(dim_b, k_b, _DTYPE[fmt_b]) == "register_tiled"
    gr.destroy()
    gr = _graph(monkeypatch, "2", *b[:3])
    gr.limit_allocations(0)
    assert torch.equal(_run(gr, b[3], b[4], 2), b[5])
    _run(gr, a[3], a[4], 2)
    gr.limit_allocations(-1)
    gr.reserve(dim_a, k_a, _DTYPE[fmt_a])  # asks for its own table again, not for the other
    assert gr.regs_tables() == 1 and gr.bwd_kernel(dim_b, k_b, _DTYPE[fmt_b]) != "register_tiled"
    assert torch.equal(_run(gr, b[3], b[4], 2), b[5]) and gr.regs_tables() == 1
    gr.destroy()


def test_a_refusal_leaves_no_mark_on_the_layout(monkeypatch):
    # a slab table refused at one k must not change what another k of that width is compared with once there is memory again
    N, nnz, fmt = 30_000, 6_000_000, "bf16"
    for dim, k in ((256, 64), (512, 64), (512, 128), (1024, 128)):
        case = _case(N, nnz, dim, k, fmt, 12)
        gr = _graph(monkeypatch, "2", *case[:3])
        gr.reserve(dim, k, _DTYPE[fmt])
        fresh = sizes(gr)
        gr.destroy()
        if 16 <= fresh["run"] <= 32:  # it stands in for slab pull
            break
    assert 16 <= fresh["run"] <= 32
    gr = _graph(monkeypatch, "2", *case[:3])
    gr.limit_allocations(0)
    _run(gr, case[3], case[4][:, :k - 8].contiguous(), 2)
    assert torch.equal(_run(gr, case[3], case[4], 2), case[5]) and gr.regs_tables() == 0
    gr.limit_allocations(-1)
    gr.reserve(dim, k, _DTYPE[fmt])
    assert gr.regs_tables() == 1 and sizes(gr) == fresh
    assert torch.equal(_run(gr, case[3], case[4], 2), case[5])
    gr.destroy()


# (graph: a power of a uniform number makes some sources and destinations frequent, 1: none.)  Real numbers; a call gives the same bits every time.
@pytest.mark.parametrize("how", ["2", "3"])
@pytest.mark.parametrize("fmt,dim,k", [("f32", 128, 64), ("f32", 256, 32), ("bf16", 256, 96)])
@pytest.mark.parametrize("N,nnz,power", [(60_000, 6_000_000, 3), (200_000, 3_000_000, 1), (30_000, 4_000_000, 1)])
def test_errors_are_no_larger_than_those_of_the_kernel_before(monkeypatch, how, fmt, dim, k, N, nnz, power):
    gen = torch.Generator(device="cuda").manual_seed(N + k)
    src, dst = ((torch.rand(nnz, generator=gen, device="cuda", dtype=torch.float64) ** power * N).long() for _ in range(2))
    order = torch.argsort(src, stable=True)
    src, dst = src[order], dst[order]
    degree = torch.bincount(src, minlength=N)
    rowptr = torch.zeros(N + 1, dtype=torch.int32, device="cuda")
    rowptr[1:] = torch.cumsum(degree, 0)
    val = (1.0 / degree.double())[src].float()  # mean weights
    dY = torch.randn(N, dim, generator=gen, device="cuda").to(_DTYPE[fmt])
    index = torch.rand(N, dim, generator=gen, device="cuda").topk(k, dim=1).indices.sort(dim=1).values
    exact = torch.zeros((N, k), dtype=torch.float64, device="cuda")
    for at in range(0, nnz, 1 << 18):
        s, d = src[at: at + (1 << 18)], dst[at: at + (1 << 18)]
        exact.index_add_(0, d, dY[s].double().gather(1, index[d]) * val[at: at + (1 << 18), None].double())
    error = {}
    for form in ("1", how):
        gr = _graph(monkeypatch, form, rowptr, dst.to(torch.int32), val)
        out = _run(gr, dY, index, 4)
        assert gr.regs_tables() == (form != "1")
        error[form] = (torch.linalg.vector_norm(out.double() - exact) / torch.linalg.vector_norm(exact)).item()
        gr.destroy()
    # (sums of a few terms are rounded alike by both: a few per cent either way)
    assert error[how] <= 1.05 * error["1"], error
