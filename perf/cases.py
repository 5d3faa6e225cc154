"""The work that programs give this library: sparse matrices of the families it is made for, products at
the feature widths they meet, and GCN training steps, each through the public entry points.

A case is a dict of plain values:

  op       "spmm"       C = A B in fp32 (Plan.spmm)
           "spmm_f16"   binary16(relu(A B + bias)), the fused epilogue (Plan.spmm_f16)
           "gcn_train"  forward and backward of a stack of GCNLayer on one graph: gradients of all
                        weights and biases, and the last layer's output
  matrix   "uniform"      rows x cols, per_row random columns in a row
           "rmat"         normalised adjacency of a power-law graph on 2^scale vertices
           "stencil"      27-point stencil on a grid^3 mesh
           "communities"  n_comm hidden communities of 64 rows, rows and columns permuted
           "pruned"       rows x cols weight with a share `keep` of its entries left
  n        feature width of B and C (spmm, spmm_f16)
  layers, d, symmetric   of a gcn_train: depth and width of the network; whether the program tells the
                         library that the adjacency is symmetric (the backward pass then shares its plan)

Plans are made in ``prepare``: a program plans a matrix once and multiplies with it many times.
"""
import torch

from paper_2603_08734_amd import Plan
from paper_2603_08734_amd.gcn import Adjacency, GCNLayer

DEGREE = 16      # directed edges drawn per vertex of a power-law graph
COMMUNITY = 64   # rows per hidden community


def listed():
    return [
        # smallest call: one small matrix, where latency and launches count
        dict(name="uniform_4096_n32", op="spmm", matrix="uniform", rows=4096, cols=4096, per_row=16, n=32),
        # the headline workload: aggregation over a large power-law graph
        dict(name="rmat_20_n128", op="spmm", matrix="rmat", scale=20, n=128),
        # a medium graph at a width that comes from the data (classes, raw features), not from the kernels
        dict(name="rmat_17_n100", op="spmm", matrix="rmat", scale=17, n=100),
        # a mesh operator on a block of 64 vectors
        dict(name="stencil_96_n64", op="spmm", matrix="stencil", grid=96, n=64),
        # a mesh operator on a few right-hand sides, as an iterative solver applies it
        dict(name="stencil_80_n3", op="spmm", matrix="stencil", grid=80, n=3),
        # hidden locality: the planner's reordering has to find the blocks
        dict(name="communities_8192_n256", op="spmm", matrix="communities", n_comm=8192, n=256),
        # a pruned weight at a batch of 128 tokens, at one token (decode), and at a prefill of 1024
        dict(name="pruned_28672_n128", op="spmm", matrix="pruned", rows=28672, cols=8192, keep=0.2, n=128),
        dict(name="pruned_28672_n1", op="spmm", matrix="pruned", rows=28672, cols=8192, keep=0.2, n=1),
        dict(name="pruned_28672_n1024", op="spmm", matrix="pruned", rows=28672, cols=8192, keep=0.2, n=1024),
        # inference of a graph layer: bias, activation and binary16 output fused into the product
        dict(name="rmat_18_f16_n256", op="spmm_f16", matrix="rmat", scale=18, n=256),
        # a training step of a graph network: forward and backward, large graph
        dict(name="gcn_train_18_d64", op="gcn_train", matrix="rmat", scale=18, symmetric=True, layers=4, d=64),
        # the same on a graph small enough that launches count, at an odd width
        dict(name="gcn_train_12_d50", op="gcn_train", matrix="rmat", scale=12, symmetric=False, layers=2, d=50),
    ]


def _log_int(rng, lo, hi):
    return max(lo, min(hi, round(lo * (hi / lo) ** rng.random())))


def _width(rng, lo, hi):
    """Half of the widths are what the spread gives, odd ones among them; half are multiples of 16."""
    n = _log_int(rng, lo, hi)
    return n if rng.random() < 0.5 or n < 16 else (n + 8) // 16 * 16


def draw(rng):
    op = rng.choice(["spmm", "spmm", "spmm", "spmm", "spmm", "spmm", "spmm_f16", "spmm_f16", "gcn_train"])
    if op == "gcn_train":
        return dict(op=op, matrix="rmat", scale=rng.randint(11, 18), symmetric=rng.random() < 0.5, layers=rng.randint(2, 4), d=_width(rng, 16, 64))
    matrix = rng.choice(["uniform", "rmat", "rmat", "stencil", "communities", "pruned", "pruned", "pruned"])
    if matrix == "pruned":
        c = dict(op=op, matrix=matrix, rows=_log_int(rng, 1024, 28672), cols=_log_int(rng, 1024, 8192),
                 keep=round(rng.uniform(0.1, 0.35), 2), n=_width(rng, 1, 1024))
        return c
    if matrix == "rmat":
        c = dict(op=op, matrix=matrix, scale=rng.randint(12, 20))
    elif matrix == "uniform":
        c = dict(op=op, matrix=matrix, rows=_log_int(rng, 1000, 200000), cols=_log_int(rng, 1000, 200000), per_row=rng.randint(4, 40))
    elif matrix == "stencil":
        c = dict(op=op, matrix=matrix, grid=_log_int(rng, 12, 96))
    else:
        c = dict(op=op, matrix=matrix, n_comm=_log_int(rng, 64, 8192))
    # no more stored entries times features than the headline workload has
    most = int(32.4e6 * 128 / _entries(c))
    return dict(c, n=_width(rng, 1, max(16, min(512, most // 16 * 16))))


# ---- matrices, made on the GPU, handed over as host CSR arrays (what the planner takes) ----
def _shape(case):
    m = case["matrix"]
    if m in ("uniform", "pruned"):
        return case["rows"], case["cols"]
    n = 1 << case["scale"] if m == "rmat" else case["grid"] ** 3 if m == "stencil" else COMMUNITY * case["n_comm"]
    return n, n


def _entries(case):
    """Stored entries, as expected before duplicates are drawn."""
    m = case["matrix"]
    rows, cols = _shape(case)
    if m == "uniform":
        return rows * case["per_row"]
    if m == "rmat":
        return int(rows * (2 * DEGREE + 1) * min(0.94, 0.40 + 0.028 * case["scale"]))
    if m == "stencil":
        return (3 * case["grid"] - 2) ** 3
    if m == "communities":
        return int(rows * (0.3 * COMMUNITY + 4))
    return int(rows * cols * case["keep"])


def _csr(keys, rows, cols, values):
    """Sorted distinct keys row * cols + col -> host (row_ptr, col_idx, values)."""
    r = keys // cols
    row_ptr = torch.zeros(rows + 1, dtype=torch.int64, device=keys.device)
    row_ptr[1:] = torch.cumsum(torch.bincount(r, minlength=rows), 0)
    col = (keys - r * cols).to(torch.int32)
    val = values(r, col, row_ptr).to(torch.float16)
    return row_ptr.cpu().numpy(), col.cpu().numpy(), val.cpu().numpy()


def _matrix(case, g):
    m = case["matrix"]
    rows, cols = _shape(case)
    dev = g.device

    def uniform(*size):
        return torch.rand(*size, device=dev, generator=g)

    def normal(r, c, p):
        return torch.randn(r.numel(), device=dev, generator=g)

    if m == "uniform":
        r = torch.arange(rows, device=dev).repeat_interleave(case["per_row"])
        keys = torch.unique(r * cols + torch.randint(0, cols, (r.numel(),), device=dev, generator=g))
        return _csr(keys, rows, cols, lambda r, c, p: 2 * uniform(r.numel()) - 1)
    if m == "rmat":
        src = torch.zeros(DEGREE * rows, dtype=torch.int64, device=dev)
        dst = torch.zeros_like(src)
        for _ in range(case["scale"]):
            u = uniform(DEGREE * rows)
            src = 2 * src + (u >= 0.76)
            dst = 2 * dst + (((u >= 0.57) & (u < 0.76)) | (u >= 0.95))
        diag = torch.arange(rows, device=dev)
        keys = torch.unique(torch.cat([src * rows + dst, dst * rows + src, diag * rows + diag]))
        del src, dst

        def normalised(r, c, p):
            deg = (p[1:] - p[:-1]).double()
            return (deg[r] * deg[c.long()]).rsqrt()

        return _csr(keys, rows, cols, normalised)
    if m == "stencil":
        k = case["grid"]
        i = torch.arange(rows, device=dev)
        z, y, x = i // (k * k), i // k % k, i % k
        parts = []
        for dz in (-1, 0, 1):
            for dy in (-1, 0, 1):
                for dx in (-1, 0, 1):
                    zz, yy, xx = z + dz, y + dy, x + dx
                    ok = (zz >= 0) & (zz < k) & (yy >= 0) & (yy < k) & (xx >= 0) & (xx < k)
                    parts.append((i * cols + (zz * k + yy) * k + xx)[ok])
        keys = torch.sort(torch.cat(parts))[0]
        del parts
        return _csr(keys, rows, cols, lambda r, c, p: torch.where(r == c, 26.0, -1.1 + 0.2 * uniform(r.numel())))
    if m == "communities":
        blk = torch.nonzero(uniform(case["n_comm"], COMMUNITY, COMMUNITY) < 0.30)
        r = torch.cat([blk[:, 0] * COMMUNITY + blk[:, 1], torch.arange(rows, device=dev).repeat_interleave(4)])
        c = torch.cat([blk[:, 0] * COMMUNITY + blk[:, 2], torch.randint(0, cols, (4 * rows,), device=dev, generator=g)])
        del blk
        perm_r, perm_c = torch.randperm(rows, device=dev, generator=g), torch.randperm(cols, device=dev, generator=g)
        return _csr(torch.unique(perm_r[r] * cols + perm_c[c]), rows, cols, normal)
    # pruned: row r keeps an entry with probability keep * (1 + u_r), u_r ~ U[-0.5, 0.5]
    p = case["keep"] * (0.5 + uniform(rows, 1))
    keys = []
    for r0 in range(0, rows, 4096):
        hit = torch.nonzero(uniform(min(rows, r0 + 4096) - r0, cols) < p[r0:r0 + 4096])
        keys.append((hit[:, 0] + r0) * cols + hit[:, 1])
    return _csr(torch.cat(keys), rows, cols, lambda r, c, p: 0.02 * torch.randn(r.numel(), device=dev, generator=g))


def prepare(case, seed):
    g = torch.Generator(device="cuda").manual_seed(seed)
    rows, cols = _shape(case)
    A = _matrix(case, g)
    state = dict(op=case["op"])
    if case["op"] == "gcn_train":
        d = case["d"]
        adj = Adjacency(*A, cols, symmetric=case["symmetric"])
        state["adj"], state["layers"] = adj, [GCNLayer(adj, d, d) for _ in range(case["layers"])]
        adj.plan(d, transposed=True)
        state["X"] = torch.randn((cols, d), device="cuda", generator=g).to(torch.float16)
        state["target"] = torch.randn((rows, d), device="cuda", generator=g)
        state["W"] = [(torch.randn((d, d), device="cuda", generator=g) / d ** 0.5).requires_grad_(True) for _ in state["layers"]]
        state["bias"] = [(0.1 * torch.randn(d, device="cuda", generator=g)).requires_grad_(True) for _ in state["layers"]]
        return state
    n = case["n"]
    state["plan"] = Plan(*A, cols, n)
    B = torch.randn((cols, n), device="cuda", generator=g) if case["matrix"] in ("rmat", "pruned") else 2 * torch.rand((cols, n), device="cuda", generator=g) - 1
    state["B"] = B.to(torch.float16)
    if case["op"] == "spmm_f16":
        state["bias"] = 0.1 * torch.randn(n, device="cuda", generator=g)
    state["C"] = torch.empty((rows, n), dtype=torch.float16 if case["op"] == "spmm_f16" else torch.float32, device="cuda")
    return state


def run(state):
    if state["op"] == "spmm":
        state["plan"].spmm(state["B"], state["C"])
        return state["C"]
    if state["op"] == "spmm_f16":
        state["plan"].spmm_f16(state["B"], state["C"], state["bias"], relu=True)
        return state["C"]
    for p in state["W"] + state["bias"]:
        p.grad = None
    h = state["X"]
    for i, (layer, w, b) in enumerate(zip(state["layers"], state["W"], state["bias"])):
        h = layer(h, w.to(torch.float16), b, relu=i + 1 < len(state["layers"]))
    loss = ((h.float() - state["target"]) ** 2).sum() / h.shape[0]
    loss.backward()
    return dict(h=h.detach(), dW=[p.grad for p in state["W"]], dbias=[p.grad for p in state["bias"]])


def work(case):
    rows, cols = _shape(case)
    nnz = _entries(case)
    # a value takes 2 bytes; a position 4 bytes, or one bit per cell of the matrix where that is less
    matrix = nnz * 2 + min(nnz * 4, rows * cols / 8)
    if case["op"] == "gcn_train":
        d, layers = case["d"], case["layers"]
        # a layer's product H W (or the gradient dZ) goes into the sparse product and its result comes out;
        # H is read for H W and again for the weight gradient; the last layer's output is compared with the target
        per_layer = 2 * matrix + rows * d * 2 * 8
        return dict(bytes=layers * per_layer + rows * d * 4, flops=layers * (4.0 * nnz * d + 6.0 * rows * d * d))
    out = 2 if case["op"] == "spmm_f16" else 4
    n = case["n"]
    return dict(bytes=matrix + 2 * cols * n + out * rows * n, flops=2.0 * nnz * n)


def tolerance(case):
    # relative 2-norm errors measured against the same path in 64 bits, times about four
    if case["op"] == "gcn_train":
        return {"rel": 1e-2}     # binary16 products, activations and gradients through the layers
    if case["op"] == "spmm_f16":
        return {"rel": 1e-3}     # one rounding to binary16
    return {"rel": 1e-6}         # fp32 sums of exact products
