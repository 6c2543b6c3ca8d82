"""The kernels that work by lane groups: every split of a wavefront; forward every layout of the CBSR and both kernels, backward the pull.

Row lengths at the edges of a batch (8 to 64 entries, whatever the split) and of its steps, k at the edges of every split; each
element within 1e-5 of the sum of the terms' magnitudes of the oracle, the bound of the other parity tests.
"""
import numpy as np
import pytest
import torch

import oracle
import paper_2312_08656_amd as maxk
import synth
from gpu_common import to_dev
from helpers import csr_from_coo

pytestmark = pytest.mark.gpu

_DTYPE = {"f32": torch.float32, "bf16": torch.bfloat16, "f16": torch.float16}
_LENGTHS = (0, 1, 2, 3, 4, 5, 7, 8, 9, 15, 16, 17, 31, 32, 33, 63, 64, 65, 95, 96, 127, 128, 129, 191, 193, 300)


def _graph(seed, shorter=1):
    rng = np.random.default_rng(seed)
    N = 331
    coo = []
    for i in range(N):
        n = _LENGTHS[i % len(_LENGTHS)] // shorter
        coo += [(i, int(j), float(rng.normal())) for j in rng.choice(N, n, replace=False)]
    return N, *csr_from_coo(N, coo)


@pytest.mark.parametrize("k,dim,ib", [(8, 8, 1), (8, 300, 2), (10, 64, 1), (13, 100, 1), (15, 16, 4), (16, 256, 1), (17, 90, 1), (21, 256, 2),
                                      (22, 130, 1), (31, 31, 1), (32, 256, 1), (33, 64, 1), (48, 200, 4), (49, 256, 1), (63, 100, 1), (64, 64, 1),
                                      (65, 256, 1), (96, 384, 2), (97, 256, 1), (127, 130, 4), (128, 256, 1), (192, 255, 1), (9, 256, 1), (130, 256, 1)])
@pytest.mark.parametrize("fmt", ["f32", "bf16", "f16"])
@pytest.mark.parametrize("sweep", ["1", "2"])
def test_forward_by_lane_groups(monkeypatch, k, dim, ib, fmt, sweep):
    monkeypatch.setenv("MAXK_FWD_SWEEP", sweep)
    N, rowptr, col, val = _graph(k)
    H = synth.normal_matrix(N, dim, 5 + k)
    sp_data = torch.empty((N, k), dtype=_DTYPE[fmt], device="cuda")
    sp_index = torch.empty((N, k), dtype={1: torch.uint8, 2: torch.int16, 4: torch.int32}[ib], device="cuda")
    maxk.maxk_topk_cbsr_narrow(to_dev(H), k, sp_data, sp_index)
    index = oracle.topk_cbsr(H, k)[1]
    ref, refabs = oracle.spgemm_fwd(rowptr, col, val, sp_data.float().cpu().numpy(), index, dim)
    for pack in ("0", "192"):  # bytes of the largest row that is repacked: none; those of k <= 32
        monkeypatch.setenv("MAXK_FWD_PACK_MAX", pack)
        gr = maxk.maxk_graph_create(to_dev(rowptr), to_dev(col), to_dev(val))
        Y = torch.full((N, dim), float("nan"), device="cuda")
        maxk.maxk_spgemm_fwd_narrow(gr, sp_data, sp_index, dim, Y)
        torch.cuda.synchronize()
        assert (np.abs(Y.cpu().numpy() - ref) <= 1e-5 * refabs + 1e-6).all(), (k, dim, fmt, sweep, pack)
        gr.destroy()


@pytest.mark.parametrize("sweep", ["1", "2"])
def test_forward_of_a_cbsr_above_4_gib(monkeypatch, sweep):
    # byte offsets of 64 bits: nodes on both sides of the line, each row three entries of weight 1.  Whole numbers: any order, the same bits
    monkeypatch.setenv("MAXK_FWD_SWEEP", sweep)
    N, k, dim = 17_000_000, 64, 64
    gen = torch.Generator(device="cuda").manual_seed(3)
    sp_data = torch.randint(-5, 6, (N, k), generator=gen, device="cuda", dtype=torch.int8).float()
    assert sp_data.numel() * 4 > 2**32
    sp_index = torch.arange(k, dtype=torch.uint8, device="cuda").repeat(N, 1)
    rows = 3000
    rowptr = torch.full((N + 1,), 3 * rows, dtype=torch.int32, device="cuda")
    rowptr[: rows + 1] = torch.arange(0, 3 * rows + 1, 3, dtype=torch.int32, device="cuda")
    col = torch.randint(N, (3 * rows,), generator=gen, device="cuda").to(torch.int32)
    col[:2] = torch.tensor([0, N - 1], dtype=torch.int32)
    gr = maxk.maxk_graph_create(rowptr, col, torch.ones(3 * rows, device="cuda"))
    Y = torch.full((N, dim), float("nan"), device="cuda")
    maxk.maxk_spgemm_fwd(gr, sp_data, sp_index, dim, Y)
    want = sp_data[col.long()].view(rows, 3, dim).sum(1)
    assert torch.equal(Y[:rows], want)
    assert not bool(Y[rows:].any())
    gr.destroy()


@pytest.mark.parametrize("k,dim,ib", [(8, 64, 1), (9, 100, 1), (16, 256, 1), (17, 33, 4), (32, 256, 2), (33, 90, 1), (64, 64, 1), (65, 256, 1),
                                      (128, 130, 1), (129, 256, 1)])
@pytest.mark.parametrize("fmt", ["f32", "bf16", "f16"])
def test_pull_by_lane_groups(monkeypatch, k, dim, ib, fmt):
    monkeypatch.setenv("MAXK_PULL_FORM", "1")  # whole rows
    N, rowptr, col, val = _graph(k + 1)
    order = np.argsort(col, kind="stable")  # the transpose: in-entries of those lengths
    rows = np.repeat(np.arange(N), np.diff(rowptr))
    rowptr, col, val = csr_from_coo(N, list(zip(col[order].tolist(), rows[order].tolist(), val[order].tolist())))
    H = synth.normal_matrix(N, dim, 7 + k)
    index = oracle.topk_cbsr(H, k)[1]
    sp_index = torch.from_numpy(index.astype({1: np.uint8, 2: np.int16, 4: np.int32}[ib])).cuda()
    dY = to_dev(synth.normal_matrix(N, dim, 9)).to(_DTYPE[fmt])
    ref, refabs = oracle.sspmm_bwd(rowptr, col, val, dY.float().cpu().numpy(), index)
    gr = maxk.maxk_graph_create(to_dev(rowptr), to_dev(col), to_dev(val))
    gr.set_bwd_mode(maxk.BWD_PULL_CSC)
    dXs = torch.full((N, k), float("nan"), device="cuda")
    maxk.maxk_sspmm_bwd_narrow(gr, dY, sp_index, dXs)
    torch.cuda.synchronize()
    assert (np.abs(dXs.cpu().numpy() - ref) <= 1e-5 * refabs + 1e-6).all(), (k, dim, fmt)
    gr.destroy()


def test_pull_from_a_gradient_above_4_gib(monkeypatch):
    # byte offsets of 64 bits: sources on both sides of the line.  Whole numbers: any order, the same bits
    monkeypatch.setenv("MAXK_PULL_FORM", "1")
    N, k, dim = 4_300_000, 32, 256
    gen = torch.Generator(device="cuda").manual_seed(4)
    dY = torch.randint(-5, 6, (N, dim), generator=gen, device="cuda", dtype=torch.int8).float()
    assert dY.numel() * 4 > 2**32
    rows = torch.cat([torch.randint(N, (4000,), generator=gen, device="cuda"), torch.tensor([0, N - 1], device="cuda")]).unique()
    rowptr = torch.zeros(N + 1, dtype=torch.int32, device="cuda")
    rowptr[1:] = torch.cumsum(torch.bincount(rows, minlength=N) * 3, 0)
    col = torch.randint(50, (3 * rows.numel(),), generator=gen, device="cuda").to(torch.int32)
    sp_index = torch.arange(200, 200 + k, device="cuda").to(torch.uint8).repeat(N, 1)
    gr = maxk.maxk_graph_create(rowptr, col, torch.ones(col.numel(), device="cuda"))
    gr.set_bwd_mode(maxk.BWD_PULL_CSC)
    dXs = torch.full((N, k), float("nan"), device="cuda")
    maxk.maxk_sspmm_bwd(gr, dY, sp_index, dXs)
    want = torch.zeros(50, k, device="cuda").index_add_(0, col.long(), dY[rows.repeat_interleave(3), 200 : 200 + k])
    assert torch.equal(dXs[:50], want)
    assert not bool(dXs[50:].any())
    gr.destroy()


@pytest.mark.parametrize("N,k", [(5000, 16), (90_000, 8), (90_000, 16), (300_000, 32)])
def test_reserve_holds_the_repacked_records(N, k):
    # a CBSR above 3 MiB is repacked, a smaller one (here that of the smaller k') is not: no forward call at k' <= k allocates
    dim = 64
    rowptr = torch.arange(N + 1, dtype=torch.int32, device="cuda")
    gr = maxk.maxk_graph_create(rowptr, torch.arange(N, dtype=torch.int32, device="cuda"), torch.ones(N, device="cuda"))
    gr.reserve(dim, k)
    held = gr.info()["workspace_bytes"]
    Y = torch.empty((N, dim), device="cuda")
    for kk in range(1, k + 1):
        for fmt in _DTYPE.values():
            for index in (torch.uint8, torch.int16, torch.int32):
                sp_index = torch.arange(kk, device="cuda").to(index).repeat(N, 1)
                maxk.maxk_spgemm_fwd_narrow(gr, torch.ones((N, kk), dtype=fmt, device="cuda"), sp_index, dim, Y)
                assert gr.info()["workspace_bytes"] == held, (N, k, kk, fmt, index)
    torch.cuda.synchronize()
    gr.destroy()


@pytest.mark.parametrize("k,fmt,grows", [(32, "f32", True), (32, "bf16", True), (33, "f32", False), (64, "f32", False), (64, "bf16", False)])
def test_no_buffer_for_records_that_no_kernel_reads(monkeypatch, k, fmt, grows):
    monkeypatch.setenv("MAXK_FWD_PACK_MAX", "1024")
    N, dim = 5000, 64
    rowptr = torch.arange(N + 1, dtype=torch.int32, device="cuda")
    gr = maxk.maxk_graph_create(rowptr, torch.arange(N, dtype=torch.int32, device="cuda"), torch.ones(N, device="cuda"))
    held, Y = gr.info()["workspace_bytes"], torch.empty((N, dim), device="cuda")
    sp_index = torch.arange(k, device="cuda").to(torch.uint8).repeat(N, 1)
    maxk.maxk_spgemm_fwd_narrow(gr, torch.ones((N, k), dtype=_DTYPE[fmt], device="cuda"), sp_index, dim, Y)
    assert (gr.info()["workspace_bytes"] > held) == grows
    assert bool((Y[:, :k] == 1).all()) and not bool(Y[:, k:].any())
    gr.destroy()


@pytest.mark.parametrize("k,tables", [(8, 1), (9, 0), (10, 0), (13, 0), (16, 1), (17, 0), (21, 0), (22, 1), (128, 1), (129, 0), (192, 0)])
def test_widths_that_the_sweep_takes(monkeypatch, k, tables):
    # asked for wherever the shape allows it, it takes k = 8, 16 and 22 to 128, as the header says
    monkeypatch.setenv("MAXK_FWD_SWEEP", "2")
    N, rowptr, col, val = _graph(k)
    gr = maxk.maxk_graph_create(to_dev(rowptr), to_dev(col), to_dev(val))
    gr.reserve(256, k)
    assert gr.sweep_tables() == tables
    gr.destroy()


# k = 17 to 21 on wide rows: by units where the work items are short, by lane groups where they are long
@pytest.mark.parametrize("k,dim,ib,shorter,units", [(17, 256, 1, 1, 0), (17, 257, 2, 1, 0), (17, 1024, 2, 4, 1), (19, 640, 4, 4, 1), (21, 385, 2, 4, 1),
                                                    (20, 300, 2, 1, 0)])
@pytest.mark.parametrize("fmt", ["f32", "bf16", "f16"])
def test_forward_of_wide_rows(monkeypatch, k, dim, ib, shorter, units, fmt):
    monkeypatch.setenv("MAXK_FWD_SWEEP", "1")
    N, rowptr, col, val = _graph(k, shorter)
    gr = maxk.maxk_graph_create(to_dev(rowptr), to_dev(col), to_dev(val))
    value_type = {"f32": maxk.VALUE_F32, "bf16": maxk.VALUE_BF16, "f16": maxk.VALUE_F16}[fmt]
    assert maxk.load_library().maxk_fwd_by_units(k, dim, value_type, gr.info()["n_fwd_items"], len(col)) == units
    H = synth.normal_matrix(N, dim, 5 + k)
    sp_data = torch.empty((N, k), dtype=_DTYPE[fmt], device="cuda")
    sp_index = torch.empty((N, k), dtype={1: torch.uint8, 2: torch.int16, 4: torch.int32}[ib], device="cuda")
    maxk.maxk_topk_cbsr_narrow(to_dev(H), k, sp_data, sp_index)
    ref, refabs = oracle.spgemm_fwd(rowptr, col, val, sp_data.float().cpu().numpy(), oracle.topk_cbsr(H, k)[1], dim)
    gr.destroy()
    for pack in ("0", "192"):
        monkeypatch.setenv("MAXK_FWD_PACK_MAX", pack)
        gr = maxk.maxk_graph_create(to_dev(rowptr), to_dev(col), to_dev(val))
        Y = torch.full((N, dim), float("nan"), device="cuda")
        maxk.maxk_spgemm_fwd_narrow(gr, sp_data, sp_index, dim, Y)
        torch.cuda.synchronize()
        assert (np.abs(Y.cpu().numpy() - ref) <= 1e-5 * refabs + 1e-6).all(), (k, dim, fmt, pack)
        gr.destroy()


# whole rows from beyond L2: by units, every width of a unit and its last k
@pytest.mark.parametrize("k,dim,ib", [(9, 512, 2), (16, 512, 4), (17, 512, 2), (32, 512, 2), (33, 512, 2), (64, 512, 2), (65, 512, 2), (128, 512, 4)])
@pytest.mark.parametrize("fmt", ["f32", "bf16", "f16"])
def test_pull_by_units(monkeypatch, k, dim, ib, fmt):
    monkeypatch.setenv("MAXK_PULL_FORM", "1")
    N, dim, value_type = 14_000, dim if fmt == "f32" else 2 * dim, {"f32": maxk.VALUE_F32, "bf16": maxk.VALUE_BF16, "f16": maxk.VALUE_F16}[fmt]
    g = synth.make_graph(N, 30 * N, 0, directed=True, self_loops=True, seed=k, weights="normal")
    gr = maxk.maxk_graph_create(to_dev(g.rowptr), to_dev(g.col), to_dev(g.val))
    gr.set_bwd_mode(maxk.BWD_PULL_CSC)
    hot = 4_000_000 // (dim * (4 if fmt == "f32" else 2))
    beyond = 1.0 - np.sort(np.diff(g.rowptr))[::-1][:hot].sum() / len(g.col)
    assert maxk.load_library().maxk_pull_by_units(dim, k, value_type, N, len(g.col), beyond) == 1
    index = np.sort(np.random.default_rng(k).permuted(np.tile(np.arange(dim, dtype=np.int32), (N, 1)), axis=1)[:, :k], axis=1)
    sp_index = torch.from_numpy(index.astype({2: np.int16, 4: np.int32}[ib])).cuda()
    dY = to_dev(synth.normal_matrix(N, dim, 9)).to(_DTYPE[fmt])
    ref, refabs = oracle.sspmm_bwd(g.rowptr, g.col, g.val, dY.float().cpu().numpy(), index)
    dXs = torch.full((N, k), float("nan"), device="cuda")
    maxk.maxk_sspmm_bwd_narrow(gr, dY, sp_index, dXs)
    torch.cuda.synchronize()
    assert (np.abs(dXs.cpu().numpy() - ref) <= 1e-5 * refabs + 1e-6).all(), (k, dim, fmt)
    gr.destroy()


# the widest rows a bin is built for are those of the first call; orders in which later widths can share it, and cannot
@pytest.mark.parametrize("widths,most", [((256, 128, 64), 4), ((512, 200, 100, 50), 4), ((64, 128, 256, 512), 8)])
def test_a_handle_holds_few_regrouped_copies(monkeypatch, widths, most):
    monkeypatch.setenv("MAXK_FWD_SWEEP", "2")
    N, rowptr, col, val = _graph(3)
    gr = maxk.maxk_graph_create(to_dev(rowptr), to_dev(col), to_dev(val))
    for dim in widths:
        for k in (8, 16, 24, 32, 33, 64, 96, 128):
            if k > dim:
                continue
            H = synth.normal_matrix(N, dim, k)
            data, index = oracle.topk_cbsr(H, k)
            Y = torch.full((N, dim), float("nan"), device="cuda")
            maxk.maxk_spgemm_fwd(gr, to_dev(data), torch.from_numpy(index.astype(np.int16)).cuda(), dim, Y)
            ref, refabs = oracle.spgemm_fwd(rowptr, col, val, data, index, dim)
            assert (np.abs(Y.cpu().numpy() - ref) <= 1e-5 * refabs + 1e-6).all(), (dim, k)
    assert 4 <= gr.sweep_tables() <= most
    gr.destroy()
