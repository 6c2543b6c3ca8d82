"""The LDS-tiled backward kernel where visits have more than three entries: the rest is added bucket by bucket, eight under way together.

Column j of the adjacency is filled to j / N, so that the buckets (one destination each here) hold every number of entries from none to
45 (tiles of 8 rows, at most nine of them in a range of the sources, five entries each beyond the third), or to 0.15 j / N (tiles of 16).
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


@pytest.mark.parametrize("k,dim,ib", [(4, 64, 1), (8, 256, 1), (16, 256, 1), (16, 300, 2), (20, 40, 4), (32, 256, 4), (64, 256, 1)])
@pytest.mark.parametrize("fill", [1.0, 0.15])
def test_tiled_overflow_buckets(k, dim, ib, fill):
    N = 390
    rng = np.random.default_rng(k + dim)
    coo = []
    for j in range(N):
        coo += [(int(i), j, float(rng.normal())) for i in rng.choice(N, int(j * fill), replace=False)]
    rowptr, col, val = csr_from_coo(N, coo)
    index = oracle.topk_cbsr(synth.normal_matrix(N, dim, 7 + k), k)[1]
    dY = synth.normal_matrix(N, dim, 9)
    ref, refabs = oracle.sspmm_bwd(rowptr, col, val, dY, index)
    sp_index = torch.from_numpy(index.astype({1: np.uint8, 2: np.int16, 4: np.int32}[ib])).cuda()
    gr = maxk.maxk_graph_create(to_dev(rowptr), to_dev(col), to_dev(val))
    gr.set_bwd_mode(maxk.BWD_TILED)
    dXs = torch.full((N, k), float("nan"), device="cuda")
    maxk.maxk_sspmm_bwd(gr, to_dev(dY), sp_index, dXs)
    torch.cuda.synchronize()
    assert (np.abs(dXs.cpu().numpy() - ref) <= 1e-5 * refabs + 1e-6).all(), (k, dim, ib, fill)
    gr.destroy()
