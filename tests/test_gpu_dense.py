"""The dense half of a GCN layer on the GPU against numpy in 64 bits.

Bounds.  Products of binary16 numbers are exact in fp32; a chain of k fp32 additions is off by at most
k * 2^-23 of the sum of absolute values (2^-23: the matrix units need not round to nearest), and the
result is rounded once to binary16 (2^-11 relative, 2^-25 where it is subnormal).
"""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

GUARD = 64      # halves kept before and behind every output


def _device(x):
    import torch
    return torch.from_numpy(np.ascontiguousarray(x)).cuda()


def _guarded(n, d, dtype, offset=0):
    """An n x d view into a buffer of canaries, `offset` elements off the buffer's alignment."""
    import torch
    buf = torch.full((n * d + 2 * GUARD + offset,), 777.0, dtype=dtype, device="cuda")
    return buf, buf[GUARD + offset:GUARD + offset + n * d].view(n, d)


def _guards_hold(buf, n, d, offset=0):
    b = buf.cpu().numpy()
    return (b[:GUARD + offset] == 777.0).all() and (b[GUARD + offset + n * d:] == 777.0).all()


# one row; edges of the 16- and 32-row groups; one group more than a round of all waves of the backward kernel
# (512 x 4 groups of 32), and of the forward kernel (1024 x 4), two whole rounds of that and a ragged third
@pytest.mark.parametrize("n,d_in,d_out", [(n, *d) for n in (1, 17, 33, 2049, 65537 + 32)
                                          for d in ((8, 64), (9, 31), (16, 16), (32, 33), (33, 8), (50, 50), (63, 57), (64, 64))] +
                         [(n, *d) for n in (131072 + 33, 300001) for d in ((64, 64), (16, 50), (37, 9))])
def test_dense_products(n, d_in, d_out):
    import torch
    from paper_2603_08734_amd import binding
    print(f"case dense n={n} d_in={d_in} d_out={d_out}", flush=True)
    L, rng = binding.lib(), np.random.default_rng(n + 100 * d_in + d_out)
    H, dP = (rng.normal(size=(n, d)).astype(np.float16) for d in (d_in, d_out))
    W = (rng.normal(size=(d_in, d_out)) / np.sqrt(d_in)).astype(np.float16)
    offset = 1 if d_in % 2 else 0       # operands and results at their element's alignment only
    Hd, dPd, Wd = (_guarded(*x.shape, torch.float16, offset)[1].copy_(_device(x)) for x in (H, dP, W))
    (bP, P), (bH, dH), (bW, dW) = (_guarded(a, b, torch.float16, offset) for a, b in ((n, d_out), (n, d_in), (d_in, d_out)))
    work = torch.empty(binding.GRADIENT_PARTS * d_in * d_out, dtype=torch.float32, device="cuda")
    s = torch.cuda.current_stream().cuda_stream
    assert L.rsh_dense_forward(Hd.data_ptr(), Wd.data_ptr(), P.data_ptr(), n, d_in, d_out, s) == 0
    assert L.rsh_dense_backward(Hd.data_ptr(), Wd.data_ptr(), dPd.data_ptr(), dH.data_ptr(), dW.data_ptr(), work.data_ptr(), n, d_in, d_out, s) == 0
    dW_alone = torch.empty_like(Wd)     # no dH wanted
    assert L.rsh_dense_backward(Hd.data_ptr(), None, dPd.data_ptr(), None, dW_alone.data_ptr(), work.data_ptr(), n, d_in, d_out, s) == 0
    torch.cuda.synchronize()
    H, dP, W = (x.astype(np.float64) for x in (H, dP, W))
    # dW: a wave's chain of rows, four waves, 512 / 8 partial sums in a run and three levels above
    chain = 32 * -(-n // (32 * 2048)) + 2 + 64 + 3
    for name, buf, got, ref, total, k in (("P", bP, P, H @ W, abs(H) @ abs(W), d_in), ("dH", bH, dH, dP @ W.T, abs(dP) @ abs(W.T), d_out),
                                          ("dW", bW, dW, H.T @ dP, abs(H.T) @ abs(dP), chain)):
        err = abs(got.cpu().numpy().astype(np.float64) - ref)
        assert (err <= 2.0 ** -11 * abs(ref) + 2.0 ** -25 + (1 + 2.0 ** -11) * k * 2.0 ** -23 * total).all(), f"{name}: {err.max()}"
        assert _guards_hold(buf, *ref.shape, offset), name
    assert torch.equal(dW, dW_alone)


def test_dense_products_keep_infinities_in_their_rows():
    """A row takes its last piece together with features of the piece before: those repeats must not turn an
    infinity there into NaN, and no row sees another's."""
    import torch
    from paper_2603_08734_amd import binding
    H = torch.ones((40, 50), dtype=torch.float16, device="cuda")
    H[7, 45], H[39, 49] = float("inf"), float("inf")
    W = torch.full((50, 50), 0.5, dtype=torch.float16, device="cuda")
    P = binding.dense_forward(H, W)
    dH, _ = binding.dense_backward(W[:40].contiguous(), W, H, True)
    for X in (P, dH):
        assert torch.isinf(X[[7, 39]]).all() and torch.isfinite(X).sum() == 38 * 50


@pytest.mark.parametrize("relu", [True, False])
@pytest.mark.parametrize("n,d,offset", [(1, 1, 0), (5, 7, 0), (300, 50, 0), (2049, 64, 0), (2049, 64, 2), (2049, 64, 1), (70001, 16, 0), (33, 520, 0),
                                        (9, 2050, 0), (40, 4095, 0)])
def test_act_backward(n, d, offset, relu):
    import torch
    from paper_2603_08734_amd import binding
    print(f"case act n={n} d={d} offset={offset} relu={relu}", flush=True)
    L, rng = binding.lib(), np.random.default_rng(n + d)
    dY = _guarded(n, d, torch.float16, offset)[1].copy_(_device(rng.normal(size=(n, d)).astype(np.float16)))
    Y = _guarded(n, d, torch.float16, offset)[1].copy_(torch.relu(_device(rng.normal(size=(n, d)).astype(np.float16))))
    bZ, dZ = _guarded(n, d, torch.float16, offset)
    bb, db = _guarded(1, d, torch.float32)
    work = torch.empty(binding.GRADIENT_PARTS * d, dtype=torch.float32, device="cuda")
    s = torch.cuda.current_stream().cuda_stream
    mask = (Y.data_ptr(), dZ.data_ptr()) if relu else (None, None)
    assert L.rsh_act_backward(dY.data_ptr(), *mask, db.data_ptr(), work.data_ptr(), n, d, s) == 0
    torch.cuda.synchronize()
    want = dY * (Y > 0) if relu else dY
    if relu:
        assert torch.equal(dZ.view(torch.int16), want.contiguous().view(torch.int16)) and _guards_hold(bZ, n, d, offset)
    ref = want.double().sum(0)
    assert ((db[0].double() - ref).abs() <= (-(-n // 512) + 256 + 64 + 8) * 2.0 ** -23 * want.double().abs().sum(0)).all()
    assert _guards_hold(bb, 1, d)
    if relu:      # special values: what a multiplication by 1 or 0 makes of them, and no bias wanted
        dY.view(-1)[::3], Y.view(-1)[::5] = float("inf"), float("nan")
        dY.view(-1)[1::7] = -0.0
        assert L.rsh_act_backward(dY.data_ptr(), *mask, None, None, n, d, s) == 0
        want = (dY * (Y > 0)).contiguous()
        assert torch.equal(dZ.isnan(), want.isnan())
        assert torch.equal(torch.where(want.isnan(), 0, dZ.view(torch.int16)), torch.where(want.isnan(), 0, want.view(torch.int16)))


def test_dense_entry_points_refuse():
    import torch
    from paper_2603_08734_amd import binding
    L = binding.lib()
    p = torch.empty(4096, dtype=torch.float32, device="cuda").data_ptr()
    assert L.rsh_dense_forward(p, None, p, 4, 16, 16, None) == binding.RSH_ERR_NULL
    for n, a, b in ((0, 16, 16), (4, 7, 16), (4, 16, 65)):
        assert L.rsh_dense_forward(p, p, p, n, a, b, None) == binding.RSH_ERR_BAD_OPTION
        assert L.rsh_dense_backward(p, p, p, p, p, p, n, a, b, None) == binding.RSH_ERR_BAD_OPTION
    assert L.rsh_dense_backward(p, None, p, p, p, p, 4, 16, 16, None) == binding.RSH_ERR_NULL
    assert L.rsh_act_backward(p, p, None, p, p, 4, 16, None) == binding.RSH_ERR_NULL
    assert L.rsh_act_backward(p + 1, None, None, p, p, 4, 16, None) == binding.RSH_ERR_BAD_OPTION


@pytest.mark.parametrize("way", ["second derivative", "strided", "wide", "graph"])
def test_layers_around_the_dense_kernels(way):
    """The layer's gradients where the dense kernels stand aside, and replayed from a graph where they do not, equal
    those of its plain call up to binary16 roundings (2^-8 of the largest entry: three roundings chained through
    two products, as in the layer's own tests)."""
    import torch
    from paper_2603_08734_amd.gcn import Adjacency, GCNLayer
    from workloads import make_config
    A, _, _ = make_config(2, small=True)
    d = 72 if way == "wide" else 48
    adj = Adjacency(A.row_ptr, A.col_idx, A.val, A.n_cols, symmetric=True)
    layer, g = GCNLayer(adj, d, d), torch.Generator(device="cuda").manual_seed(4)
    H = torch.randn((A.n_cols, d), device="cuda", generator=g).half()
    W = (torch.randn((d, d), device="cuda", generator=g) / d ** 0.5).half()
    b = torch.randn(d, device="cuda", generator=g)
    G = torch.randn((A.n_rows, d), device="cuda", generator=g).half()

    def gradients(H, W, **kw):
        H, W, bias = (x.detach().requires_grad_(True) for x in (H, W, b))
        return torch.autograd.grad(layer(H, W, bias, True), (H, W, bias), G, **kw)

    want = gradients(H, W)
    if way == "graph":
        torch.cuda.synchronize()
        graph, side = torch.cuda.CUDAGraph(), torch.cuda.Stream()
        with torch.cuda.stream(side):
            gradients(H, W)
        torch.cuda.synchronize()
        with torch.cuda.graph(graph):
            got = gradients(H, W)
        for _ in range(3):
            H.copy_(torch.randn(H.shape, device="cuda", generator=g).half())
            graph.replay()
            want = gradients(H, W)
            torch.cuda.synchronize()
            assert all(torch.equal(x, y) for x, y in zip(got, want))
        return
    if way == "second derivative":
        got = gradients(H, W, create_graph=True)
    elif way == "strided":
        got = gradients(H.t().contiguous().t(), W.t().contiguous().t())
    else:       # the same sums in 64 bits
        Hr, Wr = H.double().cpu(), W.double().cpu()
        M = torch.sparse_csr_tensor(torch.from_numpy(A.row_ptr), torch.from_numpy(A.col_idx.astype(np.int64)),
                                    torch.from_numpy(A.val.astype(np.float64)), size=(A.n_rows, A.n_cols))
        dZ = G.double().cpu() * (layer(H, W, b, True) > 0).cpu()
        dP = M.to_dense().t() @ dZ
        got = [x.cuda() for x in (dP @ Wr.t(), Hr.t() @ dP, dZ.sum(0))]
    for x, y in zip(got, want):
        assert (x.double() - y.double()).abs().max() <= 2.0 ** -8 * y.abs().max()
    adj.destroy()


@pytest.mark.parametrize("way", ["weight", "bias"])
def test_batched_gradients_of_a_layer(way):
    """torch.autograd.grad(..., is_grads_batched=True) hands the layer gradients without memory of their own.  Where no
    sparse product lies behind them -- the weight of a layer whose features need no gradient, a bias alone -- the
    result equals that of one gradient after the other, up to the binary16 roundings of another order of sums."""
    import torch
    from paper_2603_08734_amd.gcn import Adjacency, GCNLayer
    from workloads import make_config
    A, _, _ = make_config(2, small=True)
    d, g = 24, torch.Generator(device="cuda").manual_seed(5)
    adj = Adjacency(A.row_ptr, A.col_idx, A.val, A.n_cols, symmetric=True)
    layer = GCNLayer(adj, d, d, order="AH_W" if way == "weight" else "A_HW")
    H = torch.randn((A.n_cols, d), device="cuda", generator=g).half()
    W = (torch.randn((d, d), device="cuda", generator=g) / d ** 0.5).half().requires_grad_(way == "weight")
    b = torch.randn(d, device="cuda", generator=g).requires_grad_(way == "bias")
    Y, wanted = layer(H, W, b, True), W if way == "weight" else b
    G = torch.randn((3, *Y.shape), device="cuda", generator=g).half()
    got, = torch.autograd.grad(Y, wanted, G, is_grads_batched=True, retain_graph=True)
    for x, one in zip(got, G):
        want, = torch.autograd.grad(Y, wanted, one, retain_graph=True)
        assert (x.double() - want.double()).abs().max() <= 2.0 ** -8 * want.abs().max()
    adj.destroy()
