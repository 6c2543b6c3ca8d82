"""Autograd glue for one MaxK aggregation: Y = A * MaxK_k(H)  (training dataflow of Sec. 3.2, Eq. 2).

Forward : maxk_topk_cbsr -> maxk_spgemm_fwd.
Backward: maxk_sspmm_bwd (gradient only at the CBSR support) -> maxk_cbsr_scatter back to dense.
Every step runs in the HIP kernels; torch provides tensors, the stream and the autograd tape.
"""
from __future__ import annotations

import torch

from . import binding as _b


class MaxKAggregate(torch.autograd.Function):
    @staticmethod
    def forward(ctx, H: torch.Tensor, graph: _b.MaxKGraph, k: int, index_bytes: int = 0):
        N, dim = H.shape
        ib = index_bytes or (1 if dim <= 256 else 2 if dim <= 65536 else 4)
        Y, sp_index = _b.aggregate_forward(graph, H.contiguous(), k, ib)
        ctx.graph, ctx.dim, ctx.k = graph, dim, k
        ctx.save_for_backward(sp_index)
        return Y

    @staticmethod
    def backward(ctx, dY: torch.Tensor):
        (sp_index,) = ctx.saved_tensors
        dH = _b.aggregate_backward(ctx.graph, dY.contiguous(), sp_index, ctx.dim, ctx.k)
        return dH, None, None, None


def maxk_aggregate(H: torch.Tensor, graph: _b.MaxKGraph, k: int) -> torch.Tensor:
    """Y = A * MaxK_k(H), differentiable with respect to H."""
    return MaxKAggregate.apply(H, graph, k)
