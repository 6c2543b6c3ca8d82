"""The measured work: aggregation passes of MaxK-GNN as a training or serving program calls them.

Every case is one pass over one graph through the public entry points of ``paper_2312_08656_amd``.  The graphs are
seeded R-MAT (or uniform) graphs generated on the GPU, with the node counts, edge counts, hidden widths and k of the
repository's own benchmark configurations, plus ragged ones; features are N(0,1), optionally with rows of exact ties.

``path`` says what the program does in a pass:

* ``train``   one aggregation layer under autograd: Y = A * MaxK_k(H), then dH for a given dY (fp32);
* ``infer``   the forward half with buffers the program keeps: top-k / CBSR, then the forward SpGEMM (fp32);
* ``serve``   the same through the forward entry point that never allocates (serving loops);
* ``mixed``   a mixed-precision training step through the C-level calls: CBSR values in 16 bits, dY in 16 bits,
              fp32 sums, gradient scattered back to dense rows.
"""
from __future__ import annotations

import math

import torch

import paper_2312_08656_amd as maxk

# name, nodes N, edges M drawn (unordered pairs unless directed), R-MAT corner probabilities a, b, c (a = 0: uniform),
# edge weights "gcn" (1/sqrt(d_i d_j)) or "mean" (1/d_i)
_FIELDS = ("name", "path", "N", "M", "a", "b", "c", "directed", "weights", "dim", "k", "index_bytes", "value", "ties")


def _case(*values):
    return dict(zip(_FIELDS, values))


def listed():
    return [
        # the smallest calls: a graph of a thousand nodes, where launches and host work are all there is.  One forward
        # pass of a serving loop, and one training step
        _case("tiny_serve_k8", "serve", 1024, 8192, 0.0, 0.0, 0.0, False, "gcn", 64, 8, 1, "f32", 0),
        _case("tiny_train_k8", "train", 1024, 8192, 0.0, 0.0, 0.0, False, "gcn", 64, 8, 1, "f32", 0),
        # a few thousand nodes with five hundred neighbours each (the link-prediction graph of the paper's Table 1)
        _case("ddi_train_k16", "train", 4267, 1067911, 0.30, 0.25, 0.25, False, "gcn", 256, 16, 1, "f32", 0),
        # a size nothing was tuned on: odd node count, hidden width 100, odd k, mean aggregation, A^T != A
        _case("ragged_train_k13", "train", 40013, 1200007, 0.45, 0.22, 0.22, True, "mean", 100, 13, 1, "f32", 0),
        # an ordinary citation-graph size, average degree 15, at the k the paper recommends
        _case("sparse_mid_train_k32", "train", 169343, 1166243, 0.57, 0.19, 0.19, False, "gcn", 256, 32, 1, "f32", 0),
        # hidden width 384 with 16-bit indices, skewed directed graph, rows of exact ties
        _case("wide_hidden_train_k96", "train", 716847, 13954819, 0.65, 0.15, 0.15, True, "gcn", 384, 96, 2, "f32", 5),
        # average degree 75 on half a million nodes
        _case("ppa_train_k32", "train", 576289, 21231931, 0.45, 0.22, 0.22, False, "gcn", 256, 32, 1, "f32", 0),
        # dense neighbourhoods at the smallest k of the paper's sweep
        _case("proteins_train_k8", "train", 132534, 39561252, 0.40, 0.22, 0.22, False, "gcn", 256, 8, 1, "f32", 0),
        # the headline graph: inference and a training step at k = 32, a mixed-precision step at k = 64
        _case("dense_infer_k32", "infer", 232965, 57307945, 0.40, 0.22, 0.22, False, "gcn", 256, 32, 1, "f32", 0),
        _case("dense_train_k32", "train", 232965, 57307945, 0.40, 0.22, 0.22, False, "gcn", 256, 32, 1, "f32", 0),
        _case("dense_mixed_k64", "mixed", 232965, 57307945, 0.40, 0.22, 0.22, False, "gcn", 256, 64, 1, "bf16", 0),
        # the largest: 2.4 million nodes, 126 million entries
        _case("large_sparse_train_k64", "train", 2449029, 61859140, 0.57, 0.19, 0.19, False, "gcn", 256, 64, 1, "f32", 0),
    ]


def _nnz(case):
    return case["M"] * (1 if case["directed"] else 2) + case["N"]  # every node also has a self-loop


_MAX_GATHER = 0.8 * 126167309 * 256  # entries x row elements of the largest listed case, with room


def draw(rng):
    """A case of the same ranges: 1 thousand to 2.4 million nodes, average degree 8 to 600, widths 32 to 512, any k."""
    while True:
        N = int(round(math.exp(rng.uniform(math.log(1000), math.log(2449029)))))
        degree = math.exp(rng.uniform(math.log(8), math.log(600)))
        if degree > N / 8:
            continue
        directed = rng.random() < 0.3
        M = int(N * degree / (1 if directed else 2))
        dim = rng.choice([64, 128, 256, 256, 256, 384, 512, rng.randint(32, 512)])
        k = rng.choice([8, 16, 32, 32, 64, 96, 128, rng.randint(2, 128)])
        if k > dim // 2:
            continue
        nnz = M * (1 if directed else 2) + N
        if nnz > 120000000 or nnz * max(dim, 4 * k) > _MAX_GATHER or N * dim > 2449029 * 256:
            continue
        if degree > N / 64:
            a, b, c = rng.choice([(0.0, 0.0, 0.0), (0.30, 0.25, 0.25)])
        else:
            a, b, c = rng.choice([(0.0, 0.0, 0.0), (0.40, 0.22, 0.22), (0.45, 0.22, 0.22), (0.57, 0.19, 0.19)])
        path = rng.choice(["train", "train", "train", "infer", "mixed"])
        value = rng.choice(["bf16", "bf16", "f16"]) if path == "mixed" else "f32"
        index_bytes = 1 if dim <= 256 else 2
        case = _case("", path, N, M, a, b, c, directed, rng.choice(["gcn", "gcn", "mean"]), dim, k, index_bytes, value,
                     rng.choice([0, 0, 0, 5]))
        del case["name"]
        return case


# ------------------------------------------------------------------ inputs


def _generator(seed):
    g = torch.Generator(device="cuda")
    g.manual_seed(int(seed) & 0x7FFFFFFFFFFFFFFF)
    return g


def _pairs(case, n, gen):
    """n candidate pairs (source, target) of the R-MAT recipe; ids >= N and loops are dropped by the caller."""
    N, a, b, c = case["N"], case["a"], case["b"], case["c"]
    if a == 0.0:
        return (torch.randint(N, (n,), generator=gen, device="cuda"), torch.randint(N, (n,), generator=gen, device="cuda"))
    src = torch.zeros(n, dtype=torch.int64, device="cuda")
    dst = torch.zeros(n, dtype=torch.int64, device="cuda")
    for _ in range(max(1, (N - 1).bit_length())):
        u = torch.rand(n, generator=gen, device="cuda")
        src.mul_(2).add_(u >= a + b)
        dst.mul_(2).add_(((u >= a) & (u < a + b)) | (u >= a + b + c))
        del u
    return src, dst


def _csr(case, seed):
    """Exactly M distinct edges (both directions stored unless directed) plus self-loops, as CSR with sorted columns."""
    N, M = case["N"], case["M"]
    gen = _generator(seed)
    keys = torch.empty(0, dtype=torch.int64, device="cuda")
    while keys.numel() < M:
        src, dst = _pairs(case, int((M - keys.numel()) * 1.3) + 1024, gen)
        ok = (src < N) & (dst < N) & (src != dst)
        src, dst = src[ok], dst[ok]
        if not case["directed"]:
            src, dst = torch.minimum(src, dst), torch.maximum(src, dst)
        keys = torch.unique(torch.cat([keys, src * N + dst]))
        del src, dst, ok
    keys = keys[torch.randperm(keys.numel(), generator=gen, device="cuda")[:M]]
    label = torch.randperm(N, generator=gen, device="cuda")  # node ids carry no order
    src, dst = label[keys // N], label[keys % N]
    del keys
    loops = torch.arange(N, device="cuda")
    parts = [src * N + dst, loops * N + loops] + ([] if case["directed"] else [dst * N + src])
    del src, dst
    keys = torch.sort(torch.cat(parts)).values
    del parts
    row = keys // N
    col = (keys - row * N).to(torch.int32)
    degree = torch.bincount(row, minlength=N)
    rowptr = torch.zeros(N + 1, dtype=torch.int32, device="cuda")
    rowptr[1:] = torch.cumsum(degree, 0)
    inv = 1.0 / degree.double()
    if case["weights"] == "gcn":
        root = inv.sqrt()
        val = (root[row] * root[col.long()]).float()
    else:
        val = inv[row].float()
    return rowptr, col, val


def _features(case, seed):
    N, dim = case["N"], case["dim"]
    gen = _generator(seed)
    X = torch.randn(N, dim, generator=gen, device="cuda")
    if case["ties"]:
        rows = torch.randperm(N, generator=gen, device="cuda")[: N * case["ties"] // 100]
        pool = torch.randn(rows.numel(), 64, generator=gen, device="cuda")
        X[rows] = torch.gather(pool, 1, torch.randint(64, (rows.numel(), dim), generator=gen, device="cuda"))
    return X


_DTYPE = {"f32": torch.float32, "bf16": torch.bfloat16, "f16": torch.float16}
_INDEX = {1: torch.uint8, 2: torch.int16, 4: torch.int32}  # 16-bit columns as int16: the patterns are those of uint16


def prepare(case, seed):
    N, dim, k = case["N"], case["dim"], case["k"]
    graph = maxk.maxk_graph_create(*_csr(case, seed * 3 + 1))
    dtype = _DTYPE[case["value"]]
    if case["path"] != "serve":
        graph.reserve(dim, k, dtype)
    state = {"case": case, "graph": graph, "H": _features(case, seed * 3 + 2)}
    if case["path"] == "train":
        state["H"].requires_grad_(True)
    else:
        state["sp_data"] = torch.empty(N, k, dtype=dtype, device="cuda")
        state["sp_index"] = torch.empty(N, k, dtype=_INDEX[case["index_bytes"]], device="cuda")
        state["Y"] = torch.empty(N, dim, device="cuda")
    if case["path"] in ("train", "mixed"):
        state["dY"] = torch.randn(N, dim, generator=_generator(seed * 3 + 3), device="cuda").to(dtype)
    if case["path"] == "mixed":
        state["dXs"] = torch.empty(N, k, device="cuda")
        state["dH"] = torch.empty(N, dim, device="cuda")
    torch.cuda.empty_cache()  # what building the graph needed goes back before the program runs
    return state


def run(state):
    case, graph, H = state["case"], state["graph"], state["H"]
    dim, k, path = case["dim"], case["k"], case["path"]
    if path == "train":
        Y = maxk.maxk_aggregate(H, graph, k)
        (dH,) = torch.autograd.grad(Y, H, state["dY"])
        return {"Y": Y.detach(), "dH": dH}
    sp_data, sp_index, Y = state["sp_data"], state["sp_index"], state["Y"]
    if path == "mixed":
        maxk.maxk_topk_cbsr_narrow(H, k, sp_data, sp_index)
        maxk.maxk_spgemm_fwd_narrow(graph, sp_data, sp_index, dim, Y)
        maxk.maxk_sspmm_bwd_narrow(graph, state["dY"], sp_index, state["dXs"])
        maxk.maxk_cbsr_scatter(state["dXs"], sp_index, state["dH"])
        return {"Y": Y, "dXs": state["dXs"], "dH": state["dH"], "sp_data": sp_data, "sp_index": sp_index}
    maxk.maxk_topk_cbsr(H, k, sp_data, sp_index)
    if path == "serve":
        maxk.maxk_spgemm_fwd_noalloc(graph, sp_data, sp_index, dim, Y)
    else:
        maxk.maxk_spgemm_fwd(graph, sp_data, sp_index, dim, Y)
    return {"Y": Y, "sp_data": sp_data, "sp_index": sp_index}


def work(case):
    """Each input read once, each output written once; one multiply-add per stored entry and kept position."""
    N, dim, k, nnz = case["N"], case["dim"], case["k"], _nnz(case)
    vb = 4 if case["value"] == "f32" else 2
    csr = 4 * (N + 1) + 8 * nnz
    forward = 4 * N * dim + csr + 4 * N * dim  # H, the graph, Y
    if case["path"] in ("infer", "serve"):
        return {"bytes": forward + (4 + case["index_bytes"]) * N * k, "flops": 2 * nnz * k}
    backward = csr + vb * N * dim + 4 * N * dim  # the graph again, dY, dH
    if case["path"] == "mixed":
        backward += (4 + vb + case["index_bytes"]) * N * k  # dXs and the CBSR stay with the program
    return {"bytes": forward + backward, "flops": 4 * nnz * k}


def tolerance(case):
    # fp32 products and sums in every path, in any order; 16-bit values and gradients are inputs that are widened
    # exactly, so they add nothing.  Against the same sums in 64 bits the worst of the cases showed 3.8e-7 (one running
    # sum over thousands of in-entries) and 1.7e-5 for a single element; columns and kept values are the same bits
    return {"rel": 2e-6, "max": 1e-4}
