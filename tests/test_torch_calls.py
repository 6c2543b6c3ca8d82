"""Marshalling in C++ against marshalling in Python: the same bits, the same refusals."""
import pytest
import torch

import paper_2312_08656_amd as maxk
from paper_2312_08656_amd import binding, build


def _both(monkeypatch, call):
    """What `call` gives with either marshalling: a value, or the text of its MaxKError."""
    got = []
    assert binding._FAST is not None, "built with the library"
    for fast in (binding._FAST, None):
        monkeypatch.setattr(binding, "_FAST", fast)
        try:
            got.append(call())
        except maxk.MaxKError as e:
            got.append(str(e))
        monkeypatch.undo()
    return got


def test_the_library_builds_without_a_host_compiler(monkeypatch, tmp_path, capfd):
    # (the module is optional; one of an earlier build does not stay behind)
    old = tmp_path / "_torch_calls.so"
    old.write_bytes(b"of an earlier build")
    monkeypatch.setattr(build, "TORCH_CALLS", old)
    for compiler in ("/nowhere/c++", "false"):
        monkeypatch.setenv("CXX", compiler)
        assert not build.try_torch_calls()
        assert list(tmp_path.iterdir()) == [] and "_torch_calls.so not built" in capfd.readouterr().err


def test_host_tensors_are_refused_alike(monkeypatch):
    binding.load_library()
    H, data, index = torch.zeros(3, 4), torch.zeros(3, 2), torch.zeros(3, 2, dtype=torch.uint8)
    for call in (lambda: maxk.maxk_topk_cbsr(H, 2, data, index), lambda: maxk.maxk_cbsr_scatter(data, index, H),
                 lambda: maxk.maxk_topk_cbsr(H, 3, data, index)):
        fast, slow = _both(monkeypatch, call)
        assert isinstance(fast, str) and fast == slow


class _Counted:
    """The module, and which of its calls were made (True, or a value) and which were left to Python (False or None)."""

    def __init__(self, module):
        self.module, self.made, self.left = module, [], []

    def __getattr__(self, name):
        def call(*args):
            got = getattr(self.module, name)(*args)
            (self.left if got is None or got is False else self.made).append(name)
            return got

        return call


def _counted(monkeypatch, call):
    counted = _Counted(binding._FAST)
    monkeypatch.setattr(binding, "_FAST", counted)
    try:
        call()
    except maxk.MaxKError:
        pass
    finally:
        monkeypatch.undo()
    return counted.made, counted.left


def _case(N=300, dim=40, k=8, seed=1):
    gen = torch.Generator(device="cuda").manual_seed(seed)
    degree = torch.randint(0, 40, (N,), generator=gen, device="cuda")
    rowptr = torch.zeros(N + 1, dtype=torch.int32, device="cuda")
    rowptr[1:] = torch.cumsum(degree, 0)
    nnz = int(rowptr[-1])
    col = torch.randint(N, (nnz,), generator=gen, device="cuda").to(torch.int32)
    g = maxk.maxk_graph_create(rowptr, col, torch.randn(nnz, generator=gen, device="cuda"))
    return g, torch.randn(N, dim, generator=gen, device="cuda"), torch.randn(N, dim, generator=gen, device="cuda")


@pytest.mark.gpu
@pytest.mark.parametrize("dtype", [torch.float32, torch.bfloat16])
@pytest.mark.parametrize("index", [torch.uint8, torch.uint16, torch.int16, torch.int32])
def test_calls_give_the_same_bits(monkeypatch, dtype, index):
    g, H, dY = _case()
    N, dim, k = 300, 40, 8

    def chain():
        data, cols = torch.empty(N, k, dtype=dtype, device="cuda"), torch.empty(N, k, dtype=index, device="cuda")
        Y, dXs, dH = torch.empty(N, dim, device="cuda"), torch.empty(N, k, device="cuda"), torch.empty(N, dim, device="cuda")
        with torch.cuda.stream(torch.cuda.Stream()) as _:
            torch.cuda.synchronize()
            if dtype == torch.float32:
                maxk.maxk_topk_cbsr(H, k, data, cols)
                maxk.maxk_spgemm_fwd(g, data, cols, dim, Y)
                maxk.maxk_spgemm_fwd_noalloc(g, data, cols, dim, Y)
                maxk.maxk_sspmm_bwd(g, dY, cols, dXs)
            else:
                maxk.maxk_topk_cbsr_narrow(H, k, data, cols)
                maxk.maxk_spgemm_fwd_narrow(g, data, cols, dim, Y)
                maxk.maxk_sspmm_bwd_narrow(g, dY.to(dtype), cols, dXs)
            maxk.maxk_cbsr_scatter(dXs, cols, dH)
            torch.cuda.synchronize()
        return data, cols.view(torch.uint8), Y, dXs, dH

    fast, slow = _both(monkeypatch, chain)
    assert all(torch.equal(a, b) for a, b in zip(fast, slow))
    noalloc = ["forward_noalloc"] if dtype == torch.float32 else []
    assert _counted(monkeypatch, chain) == (["topk", "forward", *noalloc, "backward", "scatter"], [])
    g.destroy()


@pytest.mark.gpu
def test_calls_go_to_the_current_stream():
    # some 10 ms of work, then H, on a side stream; nothing waits before the calls
    N, dim, k = 20_000, 256, 16
    g, H, dY = _case(N=N, dim=dim)
    data, cols = torch.empty(N, k, device="cuda"), torch.empty(N, k, dtype=torch.uint8, device="cuda")
    Y, late = torch.empty(N, dim, device="cuda"), torch.zeros(N, dim, device="cuda")
    dXs, dH = torch.empty(N, k, device="cuda"), torch.empty(N, dim, device="cuda")
    busy = torch.randn(8192, 8192, device="cuda")
    side = torch.cuda.Stream()

    def chain():
        maxk.maxk_topk_cbsr(late, k, data, cols)
        maxk.maxk_spgemm_fwd(g, data, cols, dim, Y)
        maxk.maxk_sspmm_bwd(g, late, cols, dXs)
        maxk.maxk_cbsr_scatter(dXs, cols, dH)
        return Y.clone(), dH.clone(), binding.aggregate_forward(g, late, k, 1)[0], binding.aggregate_backward(g, late, cols, dim, k)

    late.copy_(H)
    want = chain()
    torch.cuda.synchronize()
    late.zero_()
    torch.cuda.synchronize()
    with torch.cuda.stream(side):
        for _ in range(2):
            torch.mm(busy, busy)
        late.copy_(H)
        got = chain()
    side.synchronize()
    assert all(torch.equal(a, b) for a, b in zip(got, want))
    g.destroy()


@pytest.mark.gpu
@pytest.mark.parametrize("fast", [True, False])
def test_a_call_that_fails_is_made_once(monkeypatch, fast):
    # a width above the largest is refused by the library itself, and by it alone
    N, dim, k = 30, 1025, 8
    g, _, _ = _case(N=N, dim=40)
    H = torch.zeros(N, dim, device="cuda")
    data, cols = torch.zeros(N, k, device="cuda"), torch.zeros(N, k, dtype=torch.int16, device="cuda")
    dXs, dH = torch.zeros(N, k, device="cuda"), torch.zeros(N, dim, device="cuda")
    calls = [("maxk_topk_cbsr", lambda: maxk.maxk_topk_cbsr(H, k, data, cols)), ("maxk_spgemm_fwd", lambda: maxk.maxk_spgemm_fwd(g, data, cols, dim, H)),
             ("maxk_spgemm_fwd_narrow", lambda: maxk.maxk_spgemm_fwd_narrow(g, data.bfloat16(), cols, dim, H)),
             ("maxk_sspmm_bwd", lambda: maxk.maxk_sspmm_bwd(g, H, cols, dXs)), ("maxk_topk_cbsr", lambda: binding.aggregate_forward(g, H, k, 2)),
             ("maxk_sspmm_bwd", lambda: binding.aggregate_backward(g, H, cols, dim, k))]
    if not fast:
        monkeypatch.setattr(binding, "_FAST", None)
    else:
        monkeypatch.setattr(binding, "_dev", lambda *_: pytest.fail("made again from Python"))
    for name, call in calls:
        with pytest.raises(maxk.MaxKError, match=rf"^{name}: .* \(status -2, hipError -?\d+\)$"):
            call()
    monkeypatch.undo()
    g.destroy()


@pytest.mark.gpu
def test_aggregation_gives_the_same_bits_and_refusals(monkeypatch):
    g, H, dY = _case(dim=300)
    H.requires_grad_(True)

    def step(H, k, grad):
        Y = maxk.maxk_aggregate(H, g, k)
        return Y.detach(), torch.autograd.grad(Y, H, grad)[0]

    for h, grad in ((H, dY), (H.t().contiguous().t(), dY), (H, dY.t().contiguous().t())):  # copies where rows are not together
        fast, slow = _both(monkeypatch, lambda: step(h, 16, grad))
        assert all(torch.equal(a, b) for a, b in zip(fast, slow))
        assert _counted(monkeypatch, lambda: step(h, 16, grad)) == (["aggregate_forward", "aggregate_backward"], [])
    for call in (lambda: step(H, 301, dY), lambda: step(H.double(), 16, dY.double()), lambda: step(H[:299], 16, dY[:299])):
        fast, slow = _both(monkeypatch, call)
        assert isinstance(fast, str) and fast == slow
    g.destroy()
    fast, slow = _both(monkeypatch, lambda: step(H, 16, dY))
    assert fast == slow == "graph handle already destroyed"


@pytest.mark.gpu
def test_calls_refuse_alike(monkeypatch):
    g, H, dY = _case()
    N, dim, k = 300, 40, 8
    data, cols = torch.zeros(N, k, device="cuda"), torch.zeros(N, k, dtype=torch.uint8, device="cuda")
    Y, dXs = torch.zeros(N, dim, device="cuda"), torch.zeros(N, k, device="cuda")
    calls = [lambda: maxk.maxk_topk_cbsr(H, k, data.half(), cols), lambda: maxk.maxk_topk_cbsr(H.t().contiguous().t(), k, data, cols),
             lambda: maxk.maxk_topk_cbsr(H, k, data[:, ::2], cols), lambda: maxk.maxk_spgemm_fwd(g, data, cols, dim + 1, Y),
             lambda: maxk.maxk_spgemm_fwd(g, data.bfloat16(), cols, dim, Y), lambda: maxk.maxk_spgemm_fwd(g, data[:9], cols[:9], dim, Y[:9]),
             lambda: maxk.maxk_spgemm_fwd_noalloc(g, data, cols, dim, Y.double()), lambda: maxk.maxk_sspmm_bwd(g, dY.half(), cols, dXs),
             lambda: maxk.maxk_sspmm_bwd(g, dY, cols, dXs[:, :4]), lambda: maxk.maxk_cbsr_scatter(dXs, cols[:9], Y),
             lambda: maxk.maxk_sspmm_bwd(g, dY[:, ::2], cols, dXs)]
    for call in calls:
        fast, slow = _both(monkeypatch, call)
        assert isinstance(fast, str) and fast == slow
        made, left = _counted(monkeypatch, call)
        assert not made and len(left) == 1
    g.destroy()
