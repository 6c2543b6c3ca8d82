"""GPU parity: the HIP path, called through the C ABI, against the CPU oracle on the
same seeded inputs -- element by element at sizes the oracle finishes in seconds, and on
sampled outputs (plus size-independent properties) at the full benchmark sizes.
Bars: sp_index / sp_data bit-exact; fp32 outputs within 1e-5 * sum|terms| + 1e-6."""
import numpy as np
import pytest
import torch

import oracle
import synth
from helpers import csr_from_coo, read_golden

pytestmark = pytest.mark.gpu

if torch.cuda.is_available():
    import paper_2312_08656_amd as maxk
    from gpu_common import (DeviceGraph, check_backward, check_forward, check_narrow, check_spmm, check_topk, full_pass, gpu_topk,
                            index_to_numpy, say, to_dev)


@pytest.fixture(scope="module", autouse=True)
def _need_gpu():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    maxk.load_library()  # fails loudly if libmaxk.so is missing: there is no fallback
    # small slabs, so that the L2-tiled backward kernel sweeps several slabs even on these small graphs
    import os
    old = os.environ.get("MAXK_SLAB_KB")
    os.environ["MAXK_SLAB_KB"] = "64"
    yield
    if old is None:
        os.environ.pop("MAXK_SLAB_KB", None)
    else:
        os.environ["MAXK_SLAB_KB"] = old


# ------------------------------------------------------------------ small, element by element


def test_golden_example_on_gpu():
    g = read_golden("fig5_fig6_shape_example.txt")
    N, dim, k = (int(r[1]) for r in g["dims"])
    rowptr, col, val = csr_from_coo(N, [(int(a), int(b), float(c)) for a, b, c in g["A_coo"]])
    H = np.array(g["H"], dtype=np.float32)
    dY = np.array(g["dY"], dtype=np.float32)
    for ib in (1, 2, 4):
        sp_data, sp_index = gpu_topk(to_dev(H), k, ib)
        assert np.array_equal(index_to_numpy(sp_index), np.array(g["sp_index"], dtype=np.int32))
        assert np.array_equal(sp_data.cpu().numpy().view(np.uint32), np.array(g["sp_data"], np.float32).view(np.uint32))
        gr = maxk.maxk_graph_create(to_dev(rowptr), to_dev(col), to_dev(val))
        Y = torch.empty((N, dim), device="cuda")
        maxk.maxk_spgemm_fwd(gr, sp_data, sp_index, dim, Y)
        assert np.array_equal(Y.cpu().numpy(), np.array(g["Y"], dtype=np.float32))  # small integers: exact
        for mode in (maxk.BWD_PULL_CSC, maxk.BWD_PUSH_CSR, maxk.BWD_EXPAND_REDUCE, maxk.BWD_SLAB_PULL, maxk.BWD_TILED,
                     maxk.BWD_AUTO):
            gr.set_bwd_mode(mode)
            dXs = torch.empty((N, k), device="cuda")
            maxk.maxk_sspmm_bwd(gr, to_dev(dY), sp_index, dXs)
            assert np.array_equal(dXs.cpu().numpy(), np.array(g["dXs"], dtype=np.float32))
        gr.destroy()


@pytest.mark.parametrize("name", ["tiny", "tiny_directed"])
def test_tiny_configs_full_compare(name):
    cfg = synth.CONFIGS[name]
    dg = DeviceGraph(synth.graph(name))
    H, dY = synth.features(name, "H"), synth.features(name, "dY")
    for k in (8, 1, 3, 64, 20):
        say(f"  {name} k={k}")
        full_pass(dg, H, dY, k, 1, sampled=False)
    full_pass(dg, H, dY, 8, 4, sampled=False)
    dg.close()


@pytest.mark.parametrize("dim,k,ib", [(6, 3, 1), (37, 5, 1), (100, 100, 2), (256, 255, 1), (384, 96, 2), (512, 7, 4),
                                       (1024, 128, 2), (64, 64, 1), (130, 33, 1), (1024, 3, 2), (768, 40, 2), (96, 24, 1), (512, 200, 2), (1024, 300, 2), (260, 100, 2)])
def test_odd_shapes_and_index_widths(dim, k, ib):
    # signed general weights on a directed graph: exercises the transpose and cancellation
    # ((1024, 3): too many private output-row copies for LDS, the forward takes its single-copy fallback)
    g = synth.make_graph(700, 9000, 10, (0.5, 0.2, 0.2), directed=True, self_loops=False, seed=dim + k,
                         weights="normal")
    dg = DeviceGraph(g)
    H, dY = synth.normal_matrix(g.N, dim, 3), synth.normal_matrix(g.N, dim, 4)
    full_pass(dg, H, dY, k, ib, sampled=False)
    dg.close()


@pytest.mark.parametrize("dim,k,ib", [(64, 8, 1), (64, 20, 1), (256, 32, 1), (384, 96, 2), (128, 5, 4)])
def test_small_dense_graph_with_long_slab_visits(dim, k, ib):
    # average degree ~170 on 400 nodes: with the small test slabs many (slab, destination) visits hold more
    # than 32 entries, which the slab kernel hands to whole wavefronts; rows also exceed one 64-entry batch
    g = synth.make_graph(400, 34000, 0, directed=True, self_loops=True, seed=dim + k, weights="normal")
    dg = DeviceGraph(g)
    H, dY = synth.normal_matrix(g.N, dim, 5), synth.normal_matrix(g.N, dim, 6)
    full_pass(dg, H, dY, k, ib, sampled=False)
    dg.close()


@pytest.mark.parametrize("dim,k,last", [(64, 8, 200), (64, 64, 33), (256, 32, 60), (260, 130, 32), (60, 20, 0)])
def test_slab_visits_around_the_long_one(dim, k, last):
    # row-accumulating slab pull: visits of 31 .. 33 and of many more entries, several long ones in a row, slabs that end on
    # one, a slab of long visits only, nodes without any
    N, slab = 601, 64 * 1024 // (dim * 4)
    lengths = [0, 31, 32, 33, 60, 61, 1, 64]
    rng = np.random.default_rng(dim + k)
    rows, cols = [], []
    for s in range(0, N, slab):
        top = min(slab, N - s)
        for j in range(N):
            n = last if j == N - 1 else 40 if s == slab else lengths[(j + s // slab) % 8]
            src = s + rng.permutation(top)[:min(n, top)]
            rows.append(src)
            cols.append(np.full(src.size, j))
    rows, cols = np.concatenate(rows), np.concatenate(cols)
    order = np.lexsort((cols, rows))
    rowptr = np.concatenate([[0], np.cumsum(np.bincount(rows, minlength=N))]).astype(np.int32)
    g = synth.Graph(N, rowptr, cols[order].astype(np.int32), rng.standard_normal(rows.size).astype(np.float32))
    dg = DeviceGraph(g)
    H, dY = synth.normal_matrix(N, dim, 5), synth.normal_matrix(N, dim, 6)
    ref = oracle.topk_cbsr(H, k)
    _, sp_index = gpu_topk(to_dev(H), k, 2)
    check_backward(dg, ref, dY, to_dev(dY), sp_index, maxk.BWD_SLAB_PULL)
    check_narrow(dg, to_dev(H), dY, k, 2, ref, dim)
    dg.close()


@pytest.mark.parametrize("dim,k,fmt", [(16, 8, "f32"), (16, 16, "bf16"), (12, 5, "f32")])
def test_lone_visits_of_slabs_with_one_that_stands_out(dim, k, fmt):
    # lines of 256, 128, 64 and 32 entries in four slabs, visits at each of them and one entry off, the longest's neighbours short
    slab = 64 * 1024 // (dim * (4 if fmt == "f32" else 2))
    longest, N = [860, 430, 214, 40], 3 * slab + 100
    rng = np.random.default_rng(dim + k)
    rows, cols = [], []
    for s, top in enumerate(longest):
        lengths = [n for n in (1, 0, 31, 32, 33, 63, 64, 65, 127, 128, 129, 255, 256, 257, 2) if n <= top]
        for j in range(N):
            n = top if j == 7 else lengths[j % len(lengths)] if j < 97 else j % 3
            src = s * slab + rng.permutation(min(slab, N - s * slab))[:n]
            rows.append(src)
            cols.append(np.full(src.size, j))
        entries = sum(r.size for r in rows[-N:])
        assert maxk.load_library().maxk_lone_visit_line(top, entries) == [256, 128, 64, 32][s]
    rows, cols = np.concatenate(rows), np.concatenate(cols)
    order = np.lexsort((cols, rows))
    rowptr = np.concatenate([[0], np.cumsum(np.bincount(rows, minlength=N))]).astype(np.int32)
    g = synth.Graph(N, rowptr, cols[order].astype(np.int32), rng.standard_normal(rows.size).astype(np.float32))
    dg = DeviceGraph(g)
    H, dY = synth.normal_matrix(N, dim, 5), synth.normal_matrix(N, dim, 6)
    dY_dev = to_dev(dY).to({"f32": torch.float32, "bf16": torch.bfloat16}[fmt])
    ref = oracle.topk_cbsr(H, k)
    _, sp_index = gpu_topk(to_dev(H), k, 1)
    dg.handle.set_bwd_mode(maxk.BWD_SLAB_PULL)
    dXs = torch.full((N, k), float("nan"), device="cuda")
    maxk.maxk_sspmm_bwd_narrow(dg.handle, dY_dev, sp_index, dXs)
    want, size = oracle.sspmm_bwd(g.rowptr, g.col, g.val, dY_dev.float().cpu().numpy(), ref[1])
    assert (np.abs(dXs.cpu().numpy() - want) <= 1e-5 * size + 1e-6).all()
    dg.close()


def test_topk_ties_signed_zero_and_infinities():
    H = synth.normal_matrix(5000, 384, seed=5)
    synth.add_tie_rows(H, seed=5, percent=40, pool=16, const_every=8)
    H[7, :10] = [-0.0, 0.0, -0.0, 0.0, np.inf, -np.inf, np.inf, 0.0, -0.0, 1.0]
    H[8, :] = -np.inf
    H[9, :] = np.float32(-0.0)
    H[9, 5] = 0.0
    Hd = to_dev(H)
    for k in (1, 2, 32, 96, 192, 383, 384):
        sp_data, sp_index = gpu_topk(Hd, k, 2)
        check_topk(H, k, sp_data, sp_index)
    H256 = np.ascontiguousarray(H[:, :256])
    for k in (31, 32, 128, 256):
        sp_data, sp_index = gpu_topk(to_dev(H256), k, 1)
        check_topk(H256, k, sp_data, sp_index)
    # every register layout of the kernel (values per lane x vector width): widths 96..1000
    for dim in (96, 128, 130, 320, 640, 768, 1000):
        Hw = synth.normal_matrix(1500, dim, seed=dim)
        synth.add_tie_rows(Hw, seed=dim, percent=40, pool=16, const_every=8)
        Hw[3, :] = np.float32(0.25)
        for k in (1, dim // 3, dim - 1, dim):
            sp_data, sp_index = gpu_topk(to_dev(Hw), k, 2)
            check_topk(Hw, k, sp_data, sp_index)


@pytest.mark.parametrize("N", [1, 3, 8191, 8192 * 2 + 5, 8192 * 3 + 1, 8192 * 5 - 1, 8192 * 8 + 13, 70001])
def test_topk_row_pipeline_edges_and_value_ranges(N):
    """The top-k kernel gives a wavefront 1..8 consecutive rows (by N) and loads two rows ahead: sizes around every
    rows-per-wavefront step with a ragged last wavefront, and rows whose values make the pivot bisection work hard
    (huge and tiny magnitudes in one row, all-positive and all-negative rows, one outlier, nearly equal values)."""
    rng = np.random.default_rng(N)
    for dim, k, ib in ((256, 32, 1), (100, 7, 1), (384, 96, 2)):
        H = synth.normal_matrix(N, dim, seed=N + dim)
        n = min(N, 64)
        rows = rng.choice(N, size=n, replace=False)
        for i, r in enumerate(rows):
            m = i % 8
            if m == 0:
                H[r] = np.abs(H[r]) + np.float32(1e-3)                 # all positive: the pivot never needs the lower half
            elif m == 1:
                H[r] = -np.abs(H[r]) - np.float32(1e-3)                # all negative
            elif m == 2:
                H[r] *= np.float32(1e-30)                              # tiny magnitudes
                H[r, 0] = np.float32(3e38)                             # ... next to one huge outlier
            elif m == 3:
                H[r] = np.float32(1.0) + H[r] * np.float32(1e-6)       # nearly equal values (few distinct floats: ties)
            elif m == 4:
                H[r] = np.float32(1e-42) * rng.integers(-50, 50, dim).astype(np.float32)  # subnormals with ties
            elif m == 5:
                H[r] = np.float32(-3e38) + np.abs(H[r]) * np.float32(1e31)                # near -FLT_MAX
            elif m == 6:
                H[r] = np.exp(H[r] * np.float32(20.0)).astype(np.float32)                 # 17 orders of magnitude
            else:
                H[r] = np.float32(0.0)
                H[r, dim - 1] = np.float32(-1.0)                       # zeros and one negative
        sp_data, sp_index = gpu_topk(to_dev(H), k, ib)
        check_topk(H, k, sp_data, sp_index)


@pytest.mark.parametrize("dim,k,ib", [(256, 32, 1), (1024, 96, 2), (100, 7, 1)])
def test_topk_neighbouring_rows_far_apart(dim, k, ib):
    """A wavefront starts the pivot search of a row at the pivot of the row before it: here every row has another
    scale and offset than its neighbours (factors of 1e-20..1e20, offsets of either sign, all-zero and constant rows
    in between), so every such start is far from where the row's own pivot lies, in either direction."""
    N = 8192 * 8 + 77
    rng = np.random.default_rng(dim + k)
    H = synth.normal_matrix(N, dim, seed=dim * 7 + k)
    scale = np.float32(10.0) ** rng.integers(-20, 21, size=N).astype(np.float32)
    offset = rng.choice(np.array([0, 0, 1, -1, 50, -50, 1e4, -1e4], np.float32), size=N)
    H *= scale[:, None]
    H += (offset * scale)[:, None]
    H[rng.choice(N, 500, replace=False)] = np.float32(0.0)
    H[rng.choice(N, 500, replace=False)] = np.float32(-7.5)
    assert np.isfinite(H).all()
    sp_data, sp_index = gpu_topk(to_dev(H), k, ib)
    check_topk(H, k, sp_data, sp_index)


def test_empty_graph_empty_rows_duplicates_unsorted_columns():
    # N == 0
    z32 = torch.zeros(1, dtype=torch.int32, device="cuda")
    g0 = maxk.maxk_graph_create(z32, torch.empty(0, dtype=torch.int32, device="cuda"), torch.empty(0, device="cuda"))
    maxk.maxk_spgemm_fwd(g0, torch.empty((0, 4), device="cuda"), torch.empty((0, 4), dtype=torch.uint8, device="cuda"),
                         8, torch.empty((0, 8), device="cuda"))
    g0.destroy()
    maxk.maxk_topk_cbsr(torch.empty((0, 8), device="cuda"), 4, torch.empty((0, 4), device="cuda"),
                        torch.empty((0, 4), dtype=torch.uint8, device="cuda"))
    # a graph with no entries at all: outputs must be overwritten with zeros
    N, dim, k = 50, 16, 4
    H, dY = synth.normal_matrix(N, dim, 1), synth.normal_matrix(N, dim, 2)
    ge = synth.Graph(N, np.zeros(N + 1, np.int32), np.zeros(0, np.int32), np.zeros(0, np.float32))
    dg = DeviceGraph(ge)
    full_pass(dg, H, dY, k, 1, sampled=False)
    dg.close()
    # empty rows, empty columns, duplicate entries, columns in descending order within rows
    rng = np.random.default_rng(3)
    triples = []
    for i in range(N):
        if i % 5 == 0:
            continue  # empty row
        cols = rng.integers(0, N - 7, size=rng.integers(1, 200))  # last columns never referenced; repeats likely
        triples += [(i, int(c), float(rng.standard_normal())) for c in cols]
    rowptr, col, val = csr_from_coo(N, triples)
    for i in range(N):  # reverse each row: unsorted columns
        col[rowptr[i]:rowptr[i + 1]] = col[rowptr[i]:rowptr[i + 1]][::-1].copy()
        val[rowptr[i]:rowptr[i + 1]] = val[rowptr[i]:rowptr[i + 1]][::-1].copy()
    dg = DeviceGraph(synth.Graph(N, rowptr, col, val))
    full_pass(dg, H, dY, k, 1, sampled=False)
    dg.close()


def test_misaligned_views_take_the_scalar_paths():
    g = synth.graph("tiny_directed")
    dim, k = 64, 8
    H, dY = synth.features("tiny_directed", "H"), synth.features("tiny_directed", "dY")
    dg = DeviceGraph(g)
    ref = oracle.topk_cbsr(H, k)
    # H, sp_data and sp_index each start 4 (resp. 1) bytes off a 16-byte boundary
    Hbuf = torch.empty(g.N * dim + 1, device="cuda")
    Hd = Hbuf[1:].view(g.N, dim)
    Hd.copy_(to_dev(H))
    dbuf = torch.empty(g.N * k + 1, device="cuda")
    ibuf = torch.empty(g.N * k + 1, dtype=torch.uint8, device="cuda")
    sp_data, sp_index = dbuf[1:].view(g.N, k), ibuf[1:].view(g.N, k)
    maxk.maxk_topk_cbsr(Hd, k, sp_data, sp_index)
    check_topk(H, k, sp_data, sp_index, ref)
    check_forward(dg, ref, sp_data, sp_index, dim)
    check_backward(dg, ref, dY, to_dev(dY), sp_index, maxk.BWD_PUSH_CSR)
    check_backward(dg, ref, dY, to_dev(dY), sp_index, maxk.BWD_PULL_CSC)
    check_backward(dg, ref, dY, to_dev(dY), sp_index, maxk.BWD_EXPAND_REDUCE)
    check_backward(dg, ref, dY, to_dev(dY), sp_index, maxk.BWD_SLAB_PULL)
    check_backward(dg, ref, dY, to_dev(dY), sp_index, maxk.BWD_TILED)  # sp_index off by one byte: runs slab pull
    dxbuf = torch.empty(g.N * k + 1, device="cuda")  # misaligned dXs: the reduce phase takes its scalar path
    dg.handle.set_bwd_mode(maxk.BWD_EXPAND_REDUCE)
    maxk.maxk_sspmm_bwd(dg.handle, to_dev(dY), sp_index, dxbuf[1:].view(g.N, k))
    dref, dabs = oracle.sspmm_bwd(g.rowptr, g.col, g.val, dY, ref[1])
    assert (np.abs(dxbuf[1:].view(g.N, k).cpu().numpy() - dref) <= 1e-5 * dabs + 1e-6).all()
    dg.handle.set_bwd_mode(maxk.BWD_AUTO)
    check_spmm(dg, H, Hd)
    # Y itself 4 bytes off a 16-byte boundary: forward (two-array, repacked, 16-bit values) and dense SpMM write
    # their rows with 4-byte stores then, whatever the hidden width
    fref, fabs_ = oracle.spgemm_fwd(g.rowptr, g.col, g.val, ref[0], ref[1], dim)
    sref, sabs = oracle.spmm(g.rowptr, g.col, g.val, H)
    ybuf = torch.full((g.N * dim + 1,), float("nan"), device="cuda")
    Yoff = ybuf[1:].view(g.N, dim)
    assert Yoff.data_ptr() % 16 == 4
    al_d, al_i = gpu_topk(to_dev(H), k, 1)
    for sd, si in ((sp_data, sp_index), (al_d, al_i)):
        Yoff.fill_(float("nan"))
        maxk.maxk_spgemm_fwd(dg.handle, sd, si, dim, Yoff)
        assert (np.abs(Yoff.cpu().numpy() - fref) <= 1e-5 * fabs_ + 1e-6).all(), "forward into a misaligned Y"
    Yoff.fill_(float("nan"))
    maxk.maxk_spgemm_fwd_noalloc(dg.handle, al_d, al_i, dim, Yoff)
    assert (np.abs(Yoff.cpu().numpy() - fref) <= 1e-5 * fabs_ + 1e-6).all(), "no-alloc forward into a misaligned Y"
    Yoff.fill_(float("nan"))
    maxk.spmm_baseline(dg.handle, to_dev(H), Yoff)
    assert (np.abs(Yoff.cpu().numpy() - sref) <= 1e-5 * sabs + 1e-6).all(), "dense SpMM into a misaligned Y"
    assert bool(torch.isnan(ybuf[0]))  # the element before the view was not touched
    dg.close()


def test_outputs_are_overwritten_and_calls_repeat():
    g = synth.graph("tiny")
    dg = DeviceGraph(g)
    H, dY = synth.features("tiny", "H"), synth.features("tiny", "dY")
    Hd, dYd = to_dev(H), to_dev(dY)
    sp_data, sp_index = gpu_topk(Hd, 8, 1)
    Y1 = torch.full((g.N, 64), 123.0, device="cuda")
    maxk.maxk_spgemm_fwd(dg.handle, sp_data, sp_index, 64, Y1)
    ref, refabs = oracle.spgemm_fwd(g.rowptr, g.col, g.val, *oracle.topk_cbsr(H, 8), 64)
    assert np.abs(Y1.cpu().numpy() - ref).max() < 1e-4
    for mode in (maxk.BWD_PULL_CSC, maxk.BWD_PUSH_CSR, maxk.BWD_EXPAND_REDUCE, maxk.BWD_SLAB_PULL, maxk.BWD_TILED):
        dg.handle.set_bwd_mode(mode)
        a = torch.full((g.N, 8), 55.0, device="cuda")
        b = torch.full((g.N, 8), -7.0, device="cuda")
        maxk.maxk_sspmm_bwd(dg.handle, dYd, sp_index, a)
        maxk.maxk_sspmm_bwd(dg.handle, dYd, sp_index, b)
        assert (a - b).abs().max().item() < 1e-5
    dg.close()


def test_tables_are_built_once_per_shape_and_reserve_builds_them_ahead():
    """Alternating hidden widths, k and dY formats on one handle never rebuilds a regrouping of A^T; after
    maxk_graph_reserve* the compute call for that shape adds none either."""
    g = synth.make_graph(500, 30000, 0, directed=True, self_loops=True, seed=77, weights="normal")
    dg = DeviceGraph(g)
    h = dg.handle

    def bwd(dim, k, mode, dtype=torch.float32):
        h.set_bwd_mode(mode)
        dY = to_dev(synth.normal_matrix(g.N, dim, dim + k)).to(dtype)
        H = synth.normal_matrix(g.N, dim, 3)
        _, si = gpu_topk(to_dev(H), k, 2)
        out = torch.empty((g.N, k), device="cuda")
        maxk.maxk_sspmm_bwd_narrow(h, dY, si, out)
        torch.cuda.synchronize()
        ref, refabs = oracle.sspmm_bwd(g.rowptr, g.col, g.val, dY.float().cpu().numpy(), oracle.topk_cbsr(H, k)[1])
        assert (np.abs(out.cpu().numpy() - ref) <= 1e-5 * refabs + 1e-6).all()

    assert h.cached_tables() == (0, 0)
    h.set_bwd_mode(maxk.BWD_SLAB_PULL)
    h.reserve(256, 32)
    h.reserve(384, 32)
    h.reserve(256, 32, torch.bfloat16)  # 16-bit rows: a slab height of their own
    n_slab = h.cached_tables()[0]
    assert 2 <= n_slab <= 3 and h.cached_tables()[1] == 0  # (two widths may share a slab height)
    h.set_bwd_mode(maxk.BWD_TILED)
    h.reserve(256, 8)
    h.reserve(256, 32)
    assert h.cached_tables() == (n_slab, 2)
    for _ in range(3):  # alternate shapes, formats and kernels: nothing new is built
        bwd(256, 32, maxk.BWD_SLAB_PULL)
        bwd(384, 32, maxk.BWD_SLAB_PULL)
        bwd(256, 32, maxk.BWD_SLAB_PULL, torch.bfloat16)
        bwd(256, 8, maxk.BWD_TILED)
        bwd(256, 32, maxk.BWD_TILED)
        assert h.cached_tables() == (n_slab, 2)
    bwd(128, 16, maxk.BWD_TILED)  # a shape nobody reserved: built by the call, once
    bwd(128, 16, maxk.BWD_TILED)
    assert h.cached_tables()[1] == 3
    h.set_bwd_mode(maxk.BWD_AUTO)
    dg.close()


# ------------------------------------------------------------------ mid size, element by element


@pytest.mark.parametrize("aggregator", ["mean", "gin_sum"])
def test_other_aggregators_as_edge_weights(aggregator):
    # "A could have different expressions according to aggregator type" (Sec. 3.2): GraphSAGE's mean
    # aggregator is val = 1/d_i (a non-symmetric matrix on a symmetric structure), a GIN-style sum is
    # val = 1 with (1 + eps) on the diagonal (unnormalised magnitudes against the error bound)
    g0 = synth.graph("sparse_mid")
    if aggregator == "mean":
        val = synth.make_weights(g0, "mean")
    else:
        val = np.ones(g0.nnz, dtype=np.float32)
        rows = np.repeat(np.arange(g0.N, dtype=np.int64), np.diff(g0.rowptr))
        val[rows == g0.col] = np.float32(1.0 + 0.1)
    g = synth.Graph(g0.N, g0.rowptr, g0.col, val, dict(g0.meta))
    dg = DeviceGraph(g)
    H, dY = synth.features("sparse_mid", "H"), synth.features("sparse_mid", "dY")
    full_pass(dg, H, dY, 32, 1, sampled=False, spmm=True)
    dg.close()



def test_sparse_mid_full_compare():
    name = "sparse_mid"
    cfg = synth.CONFIGS[name]
    g = synth.graph(name)
    say(f"  {name}: {g.meta}")
    dg = DeviceGraph(g)
    say(f"  handle: {dg.handle.info()}")
    H, dY = synth.features(name, "H"), synth.features(name, "dY")
    for k in cfg.ks:
        say(f"  {name} k={k}")
        full_pass(dg, H, dY, k, cfg.index_bytes, sampled=False, spmm=(k == cfg.ks[0]))
    dg.close()


# ------------------------------------------------------------------ MaxK backward scatter and autograd glue


@pytest.mark.parametrize("dim,k,ib", [(64, 8, 1), (384, 96, 2), (37, 5, 4), (256, 256, 1)])
def test_cbsr_scatter_is_exact(dim, k, ib):
    N = 3001
    H = synth.normal_matrix(N, dim, 12)
    vals = synth.normal_matrix(N, k, 13)
    _, ri = oracle.topk_cbsr(H, k)
    idx_np = ri.astype({1: np.uint8, 2: np.uint16, 4: np.int32}[ib])
    idx_dev = torch.from_numpy(idx_np.view(np.int16) if ib == 2 else idx_np).cuda()
    if ib == 2:
        idx_dev = idx_dev.view(torch.uint16)
    dense = torch.full((N, dim), float("nan"), device="cuda")
    maxk.maxk_cbsr_scatter(to_dev(vals), idx_dev, dense)
    assert np.array_equal(dense.cpu().numpy().view(np.uint32), oracle.cbsr_scatter(vals, ri, dim).view(np.uint32))


# rows per wavefront 1, 2 and 4 with a last wavefront that has fewer; 16-byte and 4-byte stores; k above a wavefront
@pytest.mark.parametrize("N,dim,k,shift", [(1, 4, 4, 0), (5, 33, 32, 0), (16387, 36, 9, 0), (32771, 60, 7, 0), (32771, 60, 7, 1),
                                           (32773, 61, 61, 0), (32770, 260, 130, 0), (9, 1024, 200, 0),
                                           # past L2 by their size, misaligned, just below it
                                           (700_001, 100, 13, 0), (262_147, 272, 9, 0), (262_147, 256, 70, 1), (131_071, 300, 7, 0)])
def test_cbsr_scatter_row_groups(N, dim, k, shift):
    gen = torch.Generator(device="cuda").manual_seed(N + dim)
    values = torch.randn(N, k, generator=gen, device="cuda")
    index = torch.rand(N, dim, generator=gen, device="cuda").topk(k, dim=1).indices.sort(dim=1).values
    buf = torch.full((N * dim + shift,), float("nan"), device="cuda")  # shift: `dense` not 16-byte aligned
    dense = buf[shift:].view(N, dim)
    maxk.maxk_cbsr_scatter(values, index.to(torch.int32), dense)
    assert torch.equal(dense, torch.zeros(N, dim, device="cuda").scatter_(1, index, values))


# products past L2 (everything the pass touches above 256 MiB) and not, whole 64-byte product rows and others
@pytest.mark.parametrize("nnz,dim,k,fmt,past", [(610_000, 130, 128, "f32", 1), (610_000, 130, 128, "bf16", 1), (610_000, 130, 124, "f32", 0),
                                                (310_000, 130, 128, "f16", 0), (1_000_003, 64, 64, "f32", 1)])
def test_expand_reduce_either_side_of_the_infinity_cache(nnz, dim, k, fmt, past):
    N = 20011
    gen = torch.Generator(device="cuda").manual_seed(nnz + k)
    row = torch.randint(N, (nnz,), generator=gen, device="cuda").sort().values
    col = torch.randint(N, (nnz,), generator=gen, device="cuda")
    col[::7] = 3  # one destination of many entries: split over work items
    val = torch.randn(nnz, generator=gen, device="cuda")
    rowptr = torch.zeros(N + 1, dtype=torch.int32, device="cuda")
    rowptr[1:] = torch.bincount(row, minlength=N).cumsum(0)
    gr = maxk.maxk_graph_create(rowptr, col.to(torch.int32), val)
    dY = torch.randn(N, dim, generator=gen, device="cuda").to({"f32": torch.float32, "bf16": torch.bfloat16, "f16": torch.float16}[fmt])
    assert maxk.load_library().maxk_expand_past_l2(N, nnz, dim, k, 4, 0 if fmt == "f32" else 1) == past
    index = torch.rand(N, dim, generator=gen, device="cuda").topk(k, dim=1).indices.sort(dim=1).values
    gr.set_bwd_mode(maxk.BWD_EXPAND_REDUCE)
    dXs = torch.full((N, k), float("nan"), device="cuda")
    maxk.maxk_sspmm_bwd_narrow(gr, dY, index.to(torch.int32), dXs)
    want, size = (torch.zeros(N, dim, dtype=torch.float64, device="cuda") for _ in range(2))
    terms = val.double()[:, None] * dY.double()[row]
    want.index_add_(0, col, terms)
    size.index_add_(0, col, terms.abs())
    assert bool(((dXs - want.gather(1, index)).abs() <= 1e-5 * size.gather(1, index) + 1e-6).all())
    gr.destroy()


def test_autograd_function_matches_the_oracle_chain():
    name = "tiny_directed"
    g = synth.graph(name)
    cfg = synth.CONFIGS[name]
    H, dY = synth.features(name, "H"), synth.features(name, "dY")
    dg = DeviceGraph(g)
    for k in (8, 20):
        Hd = to_dev(H).requires_grad_(True)
        Y = maxk.maxk_aggregate(Hd, dg.handle, k)
        Y.backward(to_dev(dY))
        rd, ri = oracle.topk_cbsr(H, k)
        ref, refabs = oracle.spgemm_fwd(g.rowptr, g.col, g.val, rd, ri, cfg.dim)
        assert (np.abs(Y.detach().cpu().numpy() - ref) <= 1e-5 * refabs + 1e-6).all()
        D, Dabs = oracle.sspmm_bwd(g.rowptr, g.col, g.val, dY, ri)
        want = oracle.cbsr_scatter(D.astype(np.float32), ri, cfg.dim)
        bound = oracle.cbsr_scatter((1e-5 * Dabs + 1e-6).astype(np.float32), ri, cfg.dim) + 1e-7
        got = Hd.grad.cpu().numpy()
        assert (np.abs(got - want) <= bound).all()
        assert ((got != 0).sum(axis=1) <= k).all()
    dg.close()


# ------------------------------------------------------------------ HIP graph capture of a whole step


def test_step_captured_in_a_hip_graph_replays_correctly():
    # a serving / training loop may capture top-k -> forward -> backward once and replay it: after
    # maxk_graph_reserve the calls allocate nothing, synchronise nothing and record no memset nodes.
    # Every replay (fresh inputs in the same buffers, eager work and synchronisations in between) must
    # reproduce the eager result of the same inputs.
    name = "tiny_directed"
    g = synth.graph(name)
    dim, k = synth.CONFIGS[name].dim, 8
    dg = DeviceGraph(g)
    for mode in (maxk.BWD_TILED, maxk.BWD_SLAB_PULL, maxk.BWD_EXPAND_REDUCE, maxk.BWD_PULL_CSC, maxk.BWD_PUSH_CSR):
        dg.handle.set_bwd_mode(mode)
        dg.handle.reserve(dim, k)
        Hs = torch.empty((g.N, dim), device="cuda")
        dYs = torch.empty((g.N, dim), device="cuda")
        sp_data = torch.empty((g.N, k), device="cuda")
        sp_index = torch.empty((g.N, k), dtype=torch.uint8, device="cuda")
        Y = torch.empty((g.N, dim), device="cuda")
        dXs = torch.empty((g.N, k), device="cuda")

        def step():
            maxk.maxk_topk_cbsr(Hs, k, sp_data, sp_index)
            maxk.maxk_spgemm_fwd(dg.handle, sp_data, sp_index, dim, Y)
            maxk.maxk_sspmm_bwd(dg.handle, dYs, sp_index, dXs)

        Hs.copy_(to_dev(synth.normal_matrix(g.N, dim, 100)))
        dYs.copy_(to_dev(synth.normal_matrix(g.N, dim, 200)))
        side = torch.cuda.Stream()
        side.wait_stream(torch.cuda.current_stream())
        with torch.cuda.stream(side):
            step()  # warm-up outside capture
        torch.cuda.current_stream().wait_stream(side)
        torch.cuda.synchronize()
        graph = torch.cuda.CUDAGraph()
        with torch.cuda.graph(graph):
            step()
        for rep in range(4):
            Hn, dYn = synth.normal_matrix(g.N, dim, 300 + rep), synth.normal_matrix(g.N, dim, 400 + rep)
            Hs.copy_(to_dev(Hn))
            dYs.copy_(to_dev(dYn))
            Y.fill_(float("nan"))
            dXs.fill_(float("nan"))
            graph.replay()
            torch.cuda.synchronize()
            rd, ri = oracle.topk_cbsr(Hn, k)
            assert np.array_equal(sp_index.cpu().numpy().astype(np.int32), ri), f"replay {rep}: sp_index"
            ref, refabs = oracle.spgemm_fwd(g.rowptr, g.col, g.val, rd, ri, dim)
            assert (np.abs(Y.cpu().numpy() - ref) <= 1e-5 * refabs + 1e-6).all(), f"replay {rep}: forward"
            ref, refabs = oracle.sspmm_bwd(g.rowptr, g.col, g.val, dYn, ri)
            assert (np.abs(dXs.cpu().numpy() - ref) <= 1e-5 * refabs + 1e-6).all(), f"replay {rep}: backward"
            (Y.sum() + dXs.sum()).item()  # eager work between replays
        del graph
    dg.handle.set_bwd_mode(maxk.BWD_AUTO)
    dg.close()


def test_first_calls_on_a_graph_with_split_rows_may_be_captured():
    # nothing reserved, nothing called before: rows of 129 to 2047 entries are split on a small graph, and their partial
    # sums must not need an allocation under capture (k = 20: no repacked records either)
    N, dim, k = 1500, 64, 20
    rng = np.random.default_rng(91)
    lens = rng.integers(0, 20, N)
    lens[::50], lens[7] = 300, 1400
    cols = [rng.permutation(N)[:n] for n in lens]
    rowptr = np.concatenate([[0], np.cumsum(lens)]).astype(np.int32)
    col = np.concatenate(cols).astype(np.int32)
    val = rng.standard_normal(col.size).astype(np.float32)
    H, dY = to_dev(synth.normal_matrix(N, dim, 92)), to_dev(synth.normal_matrix(N, dim, 93))
    sp_data, sp_index = gpu_topk(H, k, 1)
    gr = maxk.maxk_graph_create(to_dev(rowptr), to_dev(col), to_dev(val))
    gr.set_bwd_mode(maxk.BWD_PULL_CSC)
    Y, Z, dXs = torch.empty((N, dim), device="cuda"), torch.empty((N, dim), device="cuda"), torch.empty((N, k), device="cuda")
    torch.cuda.synchronize()
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph):
        maxk.maxk_spgemm_fwd(gr, sp_data, sp_index, dim, Y)
        maxk.spmm_baseline(gr, H, Z)
        maxk.maxk_sspmm_bwd(gr, dY, sp_index, dXs)
    idx = index_to_numpy(sp_index)
    for rep in range(3):
        dY.mul_(0.5 + rep)
        sp_data.mul_(0.5 + rep)
        for t in (Y, Z, dXs):
            t.fill_(float("nan"))
        graph.replay()
        torch.cuda.synchronize()
        for got, (ref, refabs) in ((Y, oracle.spgemm_fwd(rowptr, col, val, sp_data.cpu().numpy(), idx, dim)),
                                   (Z, oracle.spmm(rowptr, col, val, H.cpu().numpy())),
                                   (dXs, oracle.sspmm_bwd(rowptr, col, val, dY.cpu().numpy(), idx))):
            assert (np.abs(got.cpu().numpy() - ref) <= 1e-5 * refabs + 1e-6).all()
    gr.destroy()


@pytest.mark.parametrize("vt,dtype", [("bf16", "bfloat16"), ("f16", "float16")])
def test_narrow_values_round_like_the_oracle_on_special_values(vt, dtype):
    """Halfway cases, the fp16 subnormal range, overflow to infinity, signed zeros: with k = dim the
    top-k call stores every value of the row, so the stored bits are the rounding of the whole input."""
    rng = np.random.default_rng(11)
    base = np.array([1 + 2.0 ** -8, 1 + 3 * 2.0 ** -8, 1 + 2.0 ** -11, 1 + 3 * 2.0 ** -11, 2049.0, 2051.0, 65504.0,
                     65519.0, 65520.0, 1e6, -1e6, 3.3e38, -3.3e38, 2.0 ** -14, 2.0 ** -15, 2.0 ** -24, 2.0 ** -25,
                     3 * 2.0 ** -25, 2.0 ** -26, 1e-30, -1e-30, 0.0, -0.0, 0.1, -0.1, np.inf, -np.inf], np.float32)
    dim = 64
    rows = [np.resize(base, dim), np.resize(-base, dim)]
    rows += [(rng.standard_normal(dim) * np.exp2(rng.integers(-30, 18, dim))).astype(np.float32) for _ in range(200)]
    bits = rng.integers(0, 2 ** 32, (400, dim), dtype=np.uint64).astype(np.uint32).view(np.float32)
    bits[~np.isfinite(bits)] = 1.0
    H = np.ascontiguousarray(np.vstack(rows + [bits]), dtype=np.float32)
    N = H.shape[0]
    sp_data = torch.empty((N, dim), dtype=getattr(torch, dtype), device="cuda")
    sp_index = torch.empty((N, dim), dtype=torch.uint8, device="cuda")
    maxk.maxk_topk_cbsr_narrow(to_dev(H), dim, sp_data, sp_index)
    torch.cuda.synchronize()
    assert np.array_equal(sp_index.cpu().numpy(), np.tile(np.arange(dim, dtype=np.uint8), (N, 1)))
    got = sp_data.view(torch.int16).cpu().numpy().view(np.uint16)
    assert np.array_equal(got, oracle.narrow(H, vt))


def test_narrow_entry_points_with_fp32_values_are_the_plain_calls():
    cfg = synth.CONFIGS["tiny_directed"]
    g = synth.graph("tiny_directed")
    dg = DeviceGraph(g)
    H = synth.features("tiny_directed", "H")
    k = cfg.ks[0]
    a_d, a_i = gpu_topk(to_dev(H), k, 1)
    b_d = torch.empty_like(a_d)
    b_i = torch.empty_like(a_i)
    maxk.maxk_topk_cbsr_narrow(to_dev(H), k, b_d, b_i)
    assert torch.equal(a_d.view(torch.int32), b_d.view(torch.int32)) and torch.equal(a_i, b_i)
    Y1 = torch.empty((g.N, cfg.dim), device="cuda")
    Y2 = torch.empty_like(Y1)
    maxk.maxk_spgemm_fwd(dg.handle, a_d, a_i, cfg.dim, Y1)
    maxk.maxk_spgemm_fwd_narrow(dg.handle, b_d, b_i, cfg.dim, Y2)
    ref, refabs = oracle.spgemm_fwd(g.rowptr, g.col, g.val, *oracle.topk_cbsr(H, k), cfg.dim)
    for Y in (Y1, Y2):
        assert (np.abs(Y.cpu().numpy() - ref) <= 1e-5 * refabs + 1e-6).all()
    dg.close()


def test_graph_create_rejects_bad_structure():
    """Column ids outside [0, N), a rowptr that does not start at 0 / end at nnz / decreases: the handle is not
    created and nothing is read through the bad ids (the column check is a bounded histogram)."""
    rowptr = np.array([0, 2, 3, 5], np.int32)
    col = np.array([0, 2, 1, 0, 1], np.int32)
    val = np.ones(5, np.float32)
    ok = maxk.maxk_graph_create(to_dev(rowptr), to_dev(col), to_dev(val))
    ok.destroy()
    for bad_col in (3, -1, 2 ** 31 - 1):
        c = col.copy()
        c[3] = bad_col
        with pytest.raises(maxk.MaxKError):
            maxk.maxk_graph_create(to_dev(rowptr), to_dev(c), to_dev(val))
    for bad_ptr in ([1, 2, 3, 5], [0, 2, 3, 4], [0, 3, 2, 5]):
        with pytest.raises(maxk.MaxKError):
            maxk.maxk_graph_create(to_dev(np.array(bad_ptr, np.int32)), to_dev(col), to_dev(val))
    # the library is still usable afterwards
    g2 = maxk.maxk_graph_create(to_dev(rowptr), to_dev(col), to_dev(val))
    Y = torch.empty((3, 4), device="cuda")
    H = to_dev(np.arange(12, dtype=np.float32).reshape(3, 4))
    maxk.spmm_baseline(g2, H, Y)
    want = np.array([[0 + 8, 1 + 9, 2 + 10, 3 + 11], [4, 5, 6, 7], [0 + 4, 1 + 5, 2 + 6, 3 + 7]], np.float32)
    assert np.array_equal(Y.cpu().numpy(), want)
    g2.destroy()


@pytest.mark.parametrize("seed", [1, 2])
def test_random_shapes_sweep(seed):
    """Seeded random (N, density, dim, k, index width) cases through every kernel: catches the shape-dependent paths
    (vector widths, register layouts, packed records, both slab-pull forms, tails) the fixed lists may miss."""
    rng = np.random.default_rng(seed)
    for case in range(16):
        N = int(rng.integers(1, 2500))
        dim = int(rng.choice([4, 8, 20, 64, 100, 128, 256, 260, 384, 512, 768, 1024, int(rng.integers(1, 1025))]))
        k = int(rng.integers(1, dim + 1))
        if rng.random() < 0.3:
            k = max(1, dim // int(rng.choice([2, 4, 8, 16])))
        ib = 1 if dim <= 256 and rng.random() < 0.5 else (2 if rng.random() < 0.7 else 4)
        avg_deg = float(rng.choice([0.5, 2, 8, 40, 150]))
        directed = bool(rng.random() < 0.7)
        M = int(min(0.4 * N * (N - 1) if N > 1 else 0, max(0, N * avg_deg)))
        if not directed:
            M //= 2
        say(f"  case {case}: N={N} M={M} dim={dim} k={k} ib={ib} directed={directed}")
        g = synth.make_graph(N, M, 0, directed=directed, self_loops=bool(rng.random() < 0.5), seed=1000 * seed + case,
                             weights="normal")
        dg = DeviceGraph(g)
        H, dY = synth.normal_matrix(g.N, dim, 7000 + case), synth.normal_matrix(g.N, dim, 8000 + case)
        if rng.random() < 0.3:
            synth.add_tie_rows(H, seed=case, percent=30, pool=8, const_every=4)
        full_pass(dg, H, dY, k, ib, sampled=False, spmm=bool(rng.random() < 0.3))
        dg.close()


@pytest.mark.parametrize("shape", ["one node", "no entries", "one row", "one column", "diagonal"])
@pytest.mark.parametrize("dim,k", [(33, 5), (256, 32), (512, 128)])
def test_auto_choice_at_the_ends_of_the_degree_distribution(shape, dim, k):
    # the cost models behind MAXK_BWD_AUTO read how the entries spread over the rows: the extreme spreads
    N = 1 if shape == "one node" else 257
    pairs = {"one node": [(0, 0)], "no entries": [], "one row": [(3, j) for j in range(N)],
             "one column": [(i, N - 1) for i in range(N)], "diagonal": [(i, i) for i in range(N)]}[shape]
    rowptr, col, val = csr_from_coo(N, [(i, j, 0.5 + 0.001 * i) for i, j in pairs])
    H, dY = synth.normal_matrix(N, dim, 51), synth.normal_matrix(N, dim, 52)
    gr = maxk.maxk_graph_create(to_dev(rowptr), to_dev(col), to_dev(val))
    assert gr.bwd_choice(dim, k) in ("pull", "expand_reduce", "slab_pull", "tiled")
    sp_data, sp_index = gpu_topk(to_dev(H), k, 2)
    dXs = torch.full((N, k), float("nan"), device="cuda")
    maxk.maxk_sspmm_bwd(gr, to_dev(dY), sp_index, dXs)
    torch.cuda.synchronize()
    ref, refabs = oracle.sspmm_bwd(rowptr, col, val, dY, oracle.topk_cbsr(H, k)[1])
    assert (np.abs(dXs.cpu().numpy() - ref) <= 1e-5 * refabs + 1e-6).all()
    gr.destroy()


@pytest.fixture
def _sliced_form(monkeypatch):
    monkeypatch.setenv("MAXK_PULL_FORM", "2")  # column slices wherever the shape allows them


def _mixed_degrees(N, seed):
    """Directed, signed weights: columns (in-degrees) of 0, 1..20, 63, 64, 65, 200 entries and one of N - 1."""
    rng = np.random.default_rng(seed)
    pairs = []
    for j in range(N):
        d = N - 1 if j == 5 else (0, 1, 3, 4, 5, 8, 9, 20, 63, 64, 65, 200)[j % 12]
        pairs += [(int(i), j, float(w)) for i, w in zip(rng.permutation(N)[:d], rng.standard_normal(d))]
    return csr_from_coo(N, pairs)


@pytest.mark.parametrize("dim,k,ib", [(32, 32, 1), (33, 7, 1), (64, 13, 2), (100, 13, 1), (128, 64, 4), (200, 70, 1),
                                      (256, 32, 1), (256, 130, 2), (384, 96, 2), (511, 128, 2), (1024, 4, 4)])
@pytest.mark.parametrize("fmt", ["f32", "bf16", "f16"])
def test_column_sliced_pull(_sliced_form, dim, k, ib, fmt):
    # slices that divide the row or leave a remainder, one to 32 of them, items of 0 entries to split ones, any column order
    N = 700
    rowptr, col, val = _mixed_degrees(N, 61)
    H, dY = synth.normal_matrix(N, dim, 62), synth.normal_matrix(N, dim, 63)
    gr = maxk.maxk_graph_create(to_dev(rowptr), to_dev(col), to_dev(val))
    gr.set_bwd_mode(maxk.BWD_PULL_CSC)
    _, sp_index = gpu_topk(to_dev(H), k, ib)
    idx = oracle.topk_cbsr(H, k)[1]
    shuffle = np.random.default_rng(64).permutation(k)  # the columns of a row may come in any order
    dt = {"f32": torch.float32, "bf16": torch.bfloat16, "f16": torch.float16}[fmt]
    dY_dev = to_dev(dY).to(dt)
    dY_ref = dY_dev.float().cpu().numpy()
    for order in (np.arange(k), shuffle):
        ix = sp_index.view(torch.int16) if ib == 2 else sp_index
        ix = ix[:, torch.from_numpy(order).cuda()].contiguous()
        dXs = torch.full((N, k), float("nan"), device="cuda")
        maxk.maxk_sspmm_bwd_narrow(gr, dY_dev, ix, dXs)
        # dY one element off its alignment: gathers through the copy, or plain pull
        odd = torch.empty(N * dim + 1, dtype=dt, device="cuda")[1:].view(N, dim)
        odd.copy_(dY_dev)
        dXs_odd = torch.full((N, k), float("nan"), device="cuda")
        maxk.maxk_sspmm_bwd_narrow(gr, odd, ix, dXs_odd)
        torch.cuda.synchronize()
        ref, refabs = oracle.sspmm_bwd(rowptr, col, val, dY_ref, np.ascontiguousarray(idx[:, order]))
        for got in (dXs, dXs_odd):
            assert (np.abs(got.cpu().numpy() - ref) <= 1e-5 * refabs + 1e-6).all()
    gr.destroy()


@pytest.mark.parametrize("dim,reserve", [(256, True), (100, True), (100, False)])
def test_column_sliced_pull_in_a_captured_graph(_sliced_form, dim, reserve):
    # not reserved, the copy's buffer may not be allocated under capture: the call falls back to whole rows
    N, k = 700, 20
    rowptr, col, val = _mixed_degrees(N, 71)
    H, dY = to_dev(synth.normal_matrix(N, dim, 72)), to_dev(synth.normal_matrix(N, dim, 73))
    gr = maxk.maxk_graph_create(to_dev(rowptr), to_dev(col), to_dev(val))
    gr.set_bwd_mode(maxk.BWD_PULL_CSC)
    _, sp_index = gpu_topk(H, k, 2)
    dXs = torch.zeros((N, k), device="cuda")
    gr.reserve(dim if reserve else 256, k)  # (dim 256 needs no copy: that builds the partial-sum workspace only)
    torch.cuda.synchronize()
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph):
        maxk.maxk_sspmm_bwd(gr, dY, sp_index, dXs)
    eager = torch.empty_like(dXs)
    for i in range(3):
        dY.mul_(1.5 + i)
        dXs.fill_(float("nan"))
        graph.replay()
        torch.cuda.synchronize()
        maxk.maxk_sspmm_bwd(gr, dY, sp_index, eager)
        torch.cuda.synchronize()
        # the two forms add in a different order: both within n * 2^-24 of sum|terms|, n <= 699 in-entries
        scale = float(dY.abs().max()) * float(np.abs(val).max()) * N
        assert float((dXs - eager).abs().max()) <= 2 * 700 * 2.0 ** -24 * scale
    gr.destroy()


def test_captured_column_sliced_pull_outlives_a_wider_reserve(_sliced_form):
    # the captured pass gathers from the slice-major copy it was captured with; a wider dY needs a larger one
    N, dim, k = 700, 100, 20
    rowptr, col, val = _mixed_degrees(N, 74)
    H, dY = to_dev(synth.normal_matrix(N, dim, 75)), to_dev(synth.normal_matrix(N, dim, 76))
    gr = maxk.maxk_graph_create(to_dev(rowptr), to_dev(col), to_dev(val))
    gr.set_bwd_mode(maxk.BWD_PULL_CSC)
    _, sp_index = gpu_topk(H, k, 2)
    idx = index_to_numpy(sp_index)
    dXs = torch.zeros((N, k), device="cuda")
    gr.reserve(dim, k)
    before = gr.info()["workspace_bytes"]
    torch.cuda.synchronize()
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph):
        maxk.maxk_sspmm_bwd(gr, dY, sp_index, dXs)
    copies = lambda d: N * 128 * -(-4 * d // 128)
    gr.reserve(300, k)
    assert gr.info()["workspace_bytes"] - before >= copies(300), "the narrower copy is meant to stay"
    for i in range(3):
        dY.mul_(1.5 + i)
        dXs.fill_(float("nan"))
        graph.replay()
        torch.cuda.synchronize()
        ref, refabs = oracle.sspmm_bwd(rowptr, col, val, dY.cpu().numpy(), idx)
        assert (np.abs(dXs.cpu().numpy() - ref) <= 1e-5 * refabs + 1e-6).all()
    gr.destroy()


@pytest.mark.parametrize("dim,k,ib", [(8, 8, 1), (100, 8, 1), (255, 16, 1), (256, 16, 2), (64, 32, 1), (256, 32, 4),
                                      (130, 64, 1), (512, 64, 2), (128, 128, 1), (509, 128, 4)])
@pytest.mark.parametrize("fmt", ["f32", "bf16", "f16"])
def test_forward_sweep(monkeypatch, dim, k, ib, fmt):
    # bins of 1, 2 and 4 rows (the last one not full), rows of 0 entries to split ones, any column order, Y misaligned
    monkeypatch.setenv("MAXK_FWD_SWEEP", "2")
    N = 701
    rowptr, col, val = _mixed_degrees(N, 81)  # (column degrees; as rows of the transposed graph)
    order = np.argsort(col, kind="stable")
    rows = np.repeat(np.arange(N), np.diff(rowptr)).astype(np.int32)
    rowptr, col, val = csr_from_coo(N, list(zip(col[order].tolist(), rows[order].tolist(), val[order].tolist())))
    H = synth.normal_matrix(N, dim, 82)
    gr = maxk.maxk_graph_create(to_dev(rowptr), to_dev(col), to_dev(val))
    dt = {"f32": torch.float32, "bf16": torch.bfloat16, "f16": torch.float16}[fmt]
    sp_data = torch.empty((N, k), dtype=dt, device="cuda")
    sp_index = torch.empty((N, k), dtype={1: torch.uint8, 2: torch.int16, 4: torch.int32}[ib], device="cuda")
    maxk.maxk_topk_cbsr_narrow(to_dev(H), k, sp_data, sp_index)
    data, idx = oracle.topk_cbsr(H, k)
    data = sp_data.float().cpu().numpy()
    shuffle = np.random.default_rng(83).permutation(k)
    for perm in (np.arange(k), shuffle):
        at = torch.from_numpy(perm).cuda()
        d, ix = sp_data[:, at].contiguous(), sp_index[:, at].contiguous()
        ref, refabs = oracle.spgemm_fwd(rowptr, col, val, np.ascontiguousarray(data[:, perm]), np.ascontiguousarray(idx[:, perm]), dim)
        for offset in (0, 1):
            Y = torch.full((N * dim + offset,), float("nan"), device="cuda")[offset:].view(N, dim)
            maxk.maxk_spgemm_fwd_narrow(gr, d, ix, dim, Y)
            torch.cuda.synchronize()
            assert (np.abs(Y.cpu().numpy() - ref) <= 1e-5 * refabs + 1e-6).all()
    if fmt == "f32":  # the regrouped graph is there now: the entry point that allocates nothing uses it too
        Y2 = torch.full((N, dim), float("nan"), device="cuda")
        maxk.maxk_spgemm_fwd_noalloc(gr, d, ix, dim, Y2)
        torch.cuda.synchronize()
        assert (np.abs(Y2.cpu().numpy() - ref) <= 1e-5 * refabs + 1e-6).all()
    gr.destroy()


def test_forward_sweep_keeps_infinities_in_their_rows(monkeypatch):
    # padding entries read node 0: a value of infinity there must not reach rows that have no entry of node 0
    monkeypatch.setenv("MAXK_FWD_SWEEP", "2")
    N, dim, k = 40, 64, 32
    rowptr, col, val = csr_from_coo(N, [(i, j, 1.0) for i in range(N) for j in range(1, 1 + i % 5)])
    sp_data = torch.ones((N, k), device="cuda")
    sp_data[0] = float("inf")
    sp_index = torch.arange(k, dtype=torch.uint8, device="cuda").repeat(N, 1).contiguous()
    gr = maxk.maxk_graph_create(to_dev(rowptr), to_dev(col), to_dev(val))
    Y = torch.full((N, dim), float("nan"), device="cuda")
    maxk.maxk_spgemm_fwd(gr, sp_data, sp_index, dim, Y)
    torch.cuda.synchronize()
    want = np.zeros((N, dim), np.float32)
    want[:, :k] = (np.arange(N) % 5)[:, None]
    assert np.array_equal(Y.cpu().numpy(), want)
    gr.destroy()


@pytest.mark.parametrize("sweep", ["1", "2"])
@pytest.mark.parametrize("dim,k", [(256, 64), (300, 16), (255, 32)])
def test_forward_output_past_l2_with_split_rows(monkeypatch, sweep, dim, k):
    # Y above 32 MiB, rows cut into 157 and 24 pieces of uneven length.  Whole numbers below 2^24: any order, the same bits
    monkeypatch.setenv("MAXK_FWD_SWEEP", sweep)
    N = 40_009
    gen = torch.Generator(device="cuda").manual_seed(k)
    rows = torch.cat([torch.arange(N, device="cuda").repeat_interleave(2), torch.full((20_001,), 3, device="cuda"),
                      torch.full((3_000,), N - 1, device="cuda")]).sort().values
    rowptr = torch.zeros(N + 1, dtype=torch.int32, device="cuda")
    rowptr[1:] = torch.cumsum(torch.bincount(rows, minlength=N), 0)
    col = torch.randint(N, rows.shape, generator=gen, device="cuda")
    val = torch.randint(-3, 4, rows.shape, generator=gen, device="cuda").float()
    sp_data = torch.randint(-5, 6, (N, k), generator=gen, device="cuda").float()
    index = torch.rand(N, dim, generator=gen, device="cuda").topk(k, dim=1).indices.sort(dim=1).values
    gr = maxk.maxk_graph_create(rowptr, col.to(torch.int32), val)
    assert gr.info()["n_split_rows"] == 2
    Y = torch.full((N, dim), float("nan"), device="cuda")
    maxk.maxk_spgemm_fwd(gr, sp_data, index.to(torch.int32), dim, Y)
    assert gr.sweep_tables() == (sweep == "2")
    X = torch.zeros(N, dim, device="cuda").scatter_(1, index, sp_data)
    assert torch.equal(Y, torch.zeros(N, dim, device="cuda").index_add_(0, rows, val[:, None] * X[col]))
    gr.destroy()


def test_forward_sweep_of_more_than_2_to_the_24_rows(monkeypatch):
    # the regrouping of A strides over its work items: a workgroup each would be more threads than a launch holds.
    # Whole numbers below 2^24, so every order of the sums gives the same bits
    monkeypatch.setenv("MAXK_FWD_SWEEP", "2")
    N, dim, k = (1 << 24) + 77, 8, 8
    gen = torch.Generator(device="cuda").manual_seed(7)
    rows = torch.sort(torch.randint(N, (N + 5000,), generator=gen, device="cuda")).values
    rows[-3:] = N - 1
    rowptr = torch.zeros(N + 1, dtype=torch.int32, device="cuda")
    rowptr[1:] = torch.cumsum(torch.bincount(rows, minlength=N), 0)
    col = torch.randint(N, rows.shape, generator=gen, device="cuda", dtype=torch.int32)
    val = torch.randint(-3, 4, rows.shape, generator=gen, device="cuda").float()
    sp_data = torch.randint(-5, 6, (N, k), generator=gen, device="cuda").float()
    sp_index = torch.arange(k, dtype=torch.uint8, device="cuda").repeat(N, 1)
    gr = maxk.maxk_graph_create(rowptr, col, val)
    gr.reserve(dim, k)
    assert gr.sweep_tables() == 1
    Y = torch.full((N, dim), float("nan"), device="cuda")
    maxk.maxk_spgemm_fwd(gr, sp_data, sp_index, dim, Y)
    want = torch.zeros_like(Y).index_add_(0, rows, sp_data[col.long()] * val[:, None])
    assert torch.equal(Y, want)
    gr.destroy()


# ------------------------------------------------------------------ what a handle builds, for which shapes, and when not


def _aggregation_case(N, M, dim, k, seed):
    g = synth.make_graph(N, M, 0, directed=True, self_loops=True, seed=seed, weights="normal")
    H, dY = synth.normal_matrix(N, dim, seed + 1), synth.normal_matrix(N, dim, seed + 2)
    gr = maxk.maxk_graph_create(to_dev(g.rowptr), to_dev(g.col), to_dev(g.val))
    sp_data, sp_index = gpu_topk(to_dev(H), k, 2)
    return g, dY, gr, sp_data, sp_index


def _forward(g, gr, sp_data, sp_index, dim):
    Y = torch.full((g.N, dim), float("nan"), device="cuda")
    maxk.maxk_spgemm_fwd(gr, sp_data, sp_index, dim, Y)
    ref, refabs = oracle.spgemm_fwd(g.rowptr, g.col, g.val, sp_data.cpu().numpy(), index_to_numpy(sp_index), dim)
    assert (np.abs(Y.cpu().numpy() - ref) <= 1e-5 * refabs + 1e-6).all()


def test_reserving_one_shape_leaves_the_sweep_to_the_others(monkeypatch):
    monkeypatch.setenv("MAXK_FWD_SWEEP", "2")
    N, dim = 900, 64
    g, _, gr, _, _ = _aggregation_case(N, 9000, dim, 8, 101)
    gr.reserve(dim, 16)
    assert gr.sweep_tables() == 1
    H = to_dev(synth.normal_matrix(N, 96, 104))
    for width, k, tables in ((dim, 16, 1), (32, 16, 1), (dim, 8, 1), (dim, 32, 2), (dim, 32, 2), (96, 8, 3), (dim, 13, 3)):
        # within the reserved shape nothing is built (k = 8 runs row by row); beyond it the first call builds what it needs
        sp_data, sp_index = gpu_topk(H[:, :width].contiguous(), k, 2)
        _forward(g, gr, sp_data, sp_index, width)
        assert gr.sweep_tables() == tables, (width, k)
    gr.destroy()


def test_a_sweep_table_that_does_not_fit_is_tried_once(monkeypatch):
    monkeypatch.setenv("MAXK_FWD_SWEEP", "2")
    N, dim, k = 900, 64, 32
    g, _, gr, sp_data, sp_index = _aggregation_case(N, 9000, dim, k, 111)
    gr.limit_allocations(0)
    for _ in range(3):
        _forward(g, gr, sp_data, sp_index, dim)
    assert gr.limit_allocations(-1) == 1
    _forward(g, gr, sp_data, sp_index, dim)  # memory is there again: a call still builds nothing, a reserve does
    assert gr.sweep_tables() == 0
    gr.reserve(dim, k)
    assert gr.sweep_tables() == 1
    gr.destroy()


_CHOICES = [("expand_reduce", 3001, 300_000, 384, 16), ("tiled", 3001, 900_000, 256, 16), ("slab_pull", 10007, 3_000_000, 256, 13),
            ("pull", 3001, 90_000, 100, 50)]


@pytest.mark.parametrize("reserve", [False, True])
@pytest.mark.parametrize("choice,N,M,dim,k", _CHOICES)
def test_a_backward_kernel_that_does_not_fit_is_given_up_once(monkeypatch, choice, N, M, dim, k, reserve):
    # the library's choice moves on to a kernel that fits, with or without a reserve, and stays there
    monkeypatch.delenv("MAXK_SLAB_KB", raising=False)
    if choice == "pull":
        monkeypatch.setenv("MAXK_PULL_FORM", "2")  # width 100: the column slices need a copy of dY
    g, dY, gr, _, sp_index = _aggregation_case(N, M, dim, k, 121)
    if choice == "pull":
        gr.set_bwd_mode(maxk.BWD_PULL_CSC)
    assert gr.bwd_choice(dim, k) == choice
    gr.limit_allocations(0)
    if reserve:
        gr.reserve(dim, k)
    ref, refabs = oracle.sspmm_bwd(g.rowptr, g.col, g.val, dY, index_to_numpy(sp_index))
    dY_dev, dXs = to_dev(dY), torch.empty((N, k), device="cuda")
    seen = []
    for i in range(3):
        if i == 2:
            gr.limit_allocations(-1)  # memory is there again: the kernel does not change under the caller
        before = torch.cuda.mem_get_info()[0]
        dXs.fill_(float("nan"))
        maxk.maxk_sspmm_bwd(gr, dY_dev, sp_index, dXs)
        torch.cuda.synchronize()
        assert (np.abs(dXs.cpu().numpy() - ref) <= 1e-5 * refabs + 1e-6).all()
        assert gr.cached_tables() == (0, 0)
        assert i == 0 or torch.cuda.mem_get_info()[0] == before
        seen.append((gr.bwd_choice(dim, k), gr.limit_allocations(0 if i < 1 else -1)))
    assert len(set(seen)) == 1 and seen[0][1] >= 1, seen
    assert seen[0][0] == "pull"
    gr.reserve(dim, k)  # asks for the memory again
    assert gr.bwd_choice(dim, k) == choice
    gr.destroy()


def test_the_form_of_the_pull_does_not_move_the_automatic_choice(monkeypatch):
    monkeypatch.delenv("MAXK_SLAB_KB", raising=False)
    for form in ("0", "1", "2"):
        monkeypatch.setenv("MAXK_PULL_FORM", form)
        for choice, N, M, dim, k in _CHOICES[:2]:
            gr = _aggregation_case(N, M, dim, k, 121)[2]
            assert gr.bwd_choice(dim, k) == choice, form
            gr.destroy()


# ------------------------------------------------------------------ how many sums a result is added up in


def _one_large_many_ones(N, large):
    """dY rows of ones, `large` in row 0: node 1 receives from nodes 0..119, node 2 from 0..63, the others from 0 only."""
    ins = [(i, 1) for i in range(120)] + [(i, 2) for i in range(64)] + [(0, j) for j in range(3, N)]
    rowptr, col, val = csr_from_coo(N, [(i, j, 1.0) for i, j in sorted(ins)])
    return rowptr, col, val, {1: 120, 2: 64}


def _large_sum_pass(mode, dim, k, fmt):
    N, large = 130, {"f32": 2.0 ** 24, "bf16": 2.0 ** 24, "f16": 2.0 ** 12}[fmt]
    dt = {"f32": torch.float32, "bf16": torch.bfloat16, "f16": torch.float16}[fmt]
    rowptr, col, val, degree = _one_large_many_ones(N, large)
    gr = maxk.maxk_graph_create(to_dev(rowptr), to_dev(col), to_dev(val * (2.0 ** 24 / large)))  # (f16 ends at 65504)
    gr.set_bwd_mode(mode)
    dY = torch.full((N, dim), large / 2.0 ** 24, dtype=dt, device="cuda")
    dY[0] = large
    sp_index = torch.arange(k, dtype=torch.uint8, device="cuda").repeat(N, 1)
    dXs = torch.empty((N, k), device="cuda")
    maxk.maxk_sspmm_bwd_narrow(gr, dY, sp_index, dXs)
    got = dXs.cpu().numpy()
    gr.destroy()
    return got, degree


@pytest.mark.parametrize("dim,k", [(64, 32), (128, 64), (256, 100)])
@pytest.mark.parametrize("fmt", ["f32", "bf16", "f16"])
@pytest.mark.parametrize("mode", ["expand_reduce", "slab_pull"])
def test_expand_reduce_and_slab_pull_add_up_in_short_sums(mode, dim, k, fmt):
    # as below: expand/reduce adds product rows in pairs of pairs, slab pull adds dY rows in batches of eight
    got, degree = _large_sum_pass(maxk.BWD_EXPAND_REDUCE if mode == "expand_reduce" else maxk.BWD_SLAB_PULL, dim, k, fmt)
    for node, n in degree.items():
        assert np.abs(got[node] - 2.0 ** 24 - (n - 1)).max() <= (3 if mode == "expand_reduce" else 7) + 2, got[node][:4] - 2.0 ** 24


@pytest.mark.parametrize("form", ["1", "2"])
@pytest.mark.parametrize("dim,k", [(64, 8), (64, 13), (128, 32), (128, 64), (256, 100)])
@pytest.mark.parametrize("fmt", ["f32", "bf16", "f16"])
def test_pull_adds_up_in_short_sums(monkeypatch, form, dim, k, fmt):
    # One in-entry adds L, every other adds 1, and L + 1 rounds to L: a running sum that holds L loses all that follow.
    # Products are added four at a time before they reach a running sum, so at most the 3 ones beside L are lost; the
    # sums above L are even numbers, which rounds by 1 at most, twice
    monkeypatch.setenv("MAXK_PULL_FORM", form)
    got, degree = _large_sum_pass(maxk.BWD_PULL_CSC, dim, k, fmt)
    for node, n in degree.items():
        assert np.abs(got[node] - 2.0 ** 24 - (n - 1)).max() <= 3 + 2, got[node][:4] - 2.0 ** 24


@pytest.mark.parametrize("skewed", [False, True])
def test_auto_leaves_close_calls_to_the_kernels_with_short_sums(monkeypatch, skewed):
    # width 256, k = 64, 9 M entries: the tiled kernel is no faster than slab pull or pull, and less exact than both
    monkeypatch.delenv("MAXK_SLAB_KB", raising=False)
    N, nnz, gen = 30011, 9_000_000, torch.Generator(device="cuda").manual_seed(3)
    u = torch.rand((2, nnz), generator=gen, device="cuda", dtype=torch.float64)
    src, col = ((u ** 2 if skewed else u) * N).long()
    rowptr = torch.zeros(N + 1, dtype=torch.int32, device="cuda")
    rowptr[1:] = torch.cumsum(torch.bincount(src, minlength=N), 0)
    gr = maxk.maxk_graph_create(rowptr, col.int(), torch.ones(nnz, device="cuda"))
    assert gr.bwd_choice(256, 64) in ("pull", "slab_pull")
    gr.destroy()


@pytest.mark.parametrize("sweep", ["1", "2"])
@pytest.mark.parametrize("k", [8, 16, 32])
def test_forward_shares_a_row_out_over_its_lane_groups(monkeypatch, sweep, k):
    # Every row has the same neighbours, the first of them with the value L, the others 1, and L + 1 rounds to L: only the
    # entries beside the first one's lane group count.  G = 64 / k groups: at most ceil(n / G) entries are lost.  Adding the
    # G sums up rounds to an even number G - 1 times, by 1 at most
    monkeypatch.setenv("MAXK_FWD_SWEEP", sweep)
    N, n, dim = 120, 100, 64
    rowptr, col, val = csr_from_coo(N, [(i, j, 1.0) for i in range(N) for j in range(n)])
    gr = maxk.maxk_graph_create(to_dev(rowptr), to_dev(col), to_dev(val))
    sp_data = torch.ones((N, k), device="cuda")
    sp_data[0] = 2.0 ** 24
    sp_index = torch.arange(k, dtype=torch.uint8, device="cuda").repeat(N, 1)
    Y = torch.empty((N, dim), device="cuda")
    maxk.maxk_spgemm_fwd(gr, sp_data, sp_index, dim, Y)
    got = Y.cpu().numpy()[:, :k]
    lost, G = 2.0 ** 24 + (n - 1) - got, 64 // k
    assert lost.min() >= -(G - 1) and lost.max() <= -(-n // G) + G - 1, (lost.min(), lost.max())
    gr.destroy()


# ------------------------------------------------------------------ which path a call took


@pytest.mark.parametrize("k", [8, 32, 64])
def test_sweep_tables_are_shared_and_built_once(monkeypatch, k):
    monkeypatch.setenv("MAXK_FWD_SWEEP", "2")
    N, dim = 900, 200
    g, _, gr, sp_data, sp_index = _aggregation_case(N, 9000, dim, k, 131)
    _forward(g, gr, sp_data, sp_index, dim)
    assert gr.sweep_tables() == 1
    Y = torch.full((N, dim), float("nan"), device="cuda")
    maxk.maxk_spgemm_fwd_noalloc(gr, sp_data, sp_index, dim, Y)
    ref, refabs = oracle.spgemm_fwd(g.rowptr, g.col, g.val, sp_data.cpu().numpy(), index_to_numpy(sp_index), dim)
    assert (np.abs(Y.cpu().numpy() - ref) <= 1e-5 * refabs + 1e-6).all()
    gr.reserve(512, k)  # other widths walk the same table
    _forward(g, gr, sp_data, sp_index, dim + 7)
    assert gr.sweep_tables() == 1
    fresh = _aggregation_case(N, 9000, dim, k, 131)[2]
    maxk.maxk_spgemm_fwd_noalloc(fresh, sp_data, sp_index, dim, Y)
    assert fresh.sweep_tables() == 0  # that entry point builds nothing
    monkeypatch.setenv("MAXK_FWD_SWEEP", "1")
    rows = _aggregation_case(N, 9000, dim, k, 131)[2]
    _forward(g, rows, sp_data, sp_index, dim)
    assert rows.sweep_tables() == 0
    for h in (gr, fresh, rows):
        h.destroy()


@pytest.mark.parametrize("k,tables", [(32, 1), (64, 0)])
def test_forward_sweep_in_a_captured_graph(monkeypatch, k, tables):
    # reserved, the captured call walks the table; at a k that nobody reserved it builds nothing and runs row by row
    monkeypatch.setenv("MAXK_FWD_SWEEP", "2")
    N, dim = 900, 128
    g, _, gr, sp_data, sp_index = _aggregation_case(N, 9000, dim, k, 141)
    if tables:
        gr.reserve(dim, k)
    Y = torch.empty((N, dim), device="cuda")
    torch.cuda.synchronize()
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph):
        maxk.maxk_spgemm_fwd(gr, sp_data, sp_index, dim, Y)
    assert gr.sweep_tables() == tables
    idx = index_to_numpy(sp_index)
    for rep in range(3):
        sp_data.mul_(0.5 + rep)
        Y.fill_(float("nan"))
        graph.replay()
        torch.cuda.synchronize()
        ref, refabs = oracle.spgemm_fwd(g.rowptr, g.col, g.val, sp_data.cpu().numpy(), idx, dim)
        assert (np.abs(Y.cpu().numpy() - ref) <= 1e-5 * refabs + 1e-6).all()
    gr.destroy()


@pytest.mark.parametrize("N,dim", [(3_000_000, 256), (17_000_000, 20)])
def test_column_sliced_pull_with_offsets_above_2_gib(_sliced_form, N, dim):
    # dY itself (2.9 GiB, gathered in place) and its slice-major copy (2.0 GiB) through 32-bit offsets.  Whole numbers below
    # 2^24, so every order of the sums gives the same bits
    k, gen = 8, torch.Generator(device="cuda").manual_seed(9)
    rows = torch.sort(torch.randint(N, (N // 2,), generator=gen, device="cuda")).values
    rows[-200_000:] = torch.arange(N - 200_000, N, device="cuda")  # the highest offsets
    rows = torch.sort(rows).values
    rowptr = torch.zeros(N + 1, dtype=torch.int32, device="cuda")
    rowptr[1:] = torch.cumsum(torch.bincount(rows, minlength=N), 0)
    col = torch.randint(N, rows.shape, generator=gen, device="cuda", dtype=torch.int32)
    val = torch.randint(-3, 4, rows.shape, generator=gen, device="cuda").float()
    dY = torch.randint(-5, 6, (N, dim), generator=gen, device="cuda", dtype=torch.int8).float()
    at = torch.arange(k, device="cuda") * (dim // k)
    sp_index = at.to(torch.uint8).repeat(N, 1)
    gr = maxk.maxk_graph_create(rowptr, col, val)
    gr.set_bwd_mode(maxk.BWD_PULL_CSC)
    dXs = torch.full((N, k), float("nan"), device="cuda")
    maxk.maxk_sspmm_bwd(gr, dY, sp_index, dXs)
    want = torch.zeros_like(dXs).index_add_(0, col.long(), dY[:, at][rows] * val[:, None])
    assert torch.equal(dXs, want)
    gr.destroy()
