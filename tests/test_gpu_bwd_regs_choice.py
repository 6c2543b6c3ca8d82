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
        if fresh["run"] == 32:  # it stands in for slab pull
            break
    assert fresh["run"] == 32
    gr = _graph(monkeypatch, "2", *case[:3])
    gr.limit_allocations(0)
    _run(gr, case[3], case[4][:, :k - 8].contiguous(), 2)
    assert torch.equal(_run(gr, case[3], case[4], 2), case[5]) and gr.regs_tables() == 0
    gr.limit_allocations(-1)
    gr.reserve(dim, k, _DTYPE[fmt])
    assert gr.regs_tables() == 1 and sizes(gr) == fresh
    assert torch.equal(_run(gr, case[3], case[4], 2), case[5])
    gr.destroy()
