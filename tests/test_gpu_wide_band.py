"""Layers with many active entries: the ways taken from a device-side count on (dW by columns and as a dense
product, the spike gradient as one), on both sides of it, against float64. Each case states its way."""
import numpy as np
import pytest
import torch

from paper_2105_08810_amd import snn

pytestmark = pytest.mark.gpu

U = 2.0 ** -24


def _csr(rng, T, B, N, share, spare=0, with_g=True):
    """A random active set as the compaction writes it, with `spare` unused slots."""
    on = rng.random((T * B, N)) < share
    rp = np.concatenate([[0], np.cumsum(on.sum(1))]).astype(np.int32)
    col = np.nonzero(on)[1].astype(np.int32)
    n = len(col)
    cap = max(n + spare, 1)
    pad = lambda x, v: np.concatenate([x, np.full(cap - n, v, x.dtype)])
    g = (rng.random(n) + 0.1).astype(np.float32)
    dev = lambda x: torch.from_numpy(x).cuda()
    csr = snn.Csr(dev(rp), dev(pad(col, 10 ** 6)), dev(pad(g, np.float32(np.nan))) if with_g else None,
                  torch.tensor([n], device="cuda"), cap)
    return on, g if with_g else np.ones(n, np.float32), csr, pad


def _dw_way(T, B, n_in, n_out, csr):
    """The way that snn_sparse_dw takes with a full workspace (layers that the matrix-core kernel of narrow bands
    does not take)."""
    cols, dense, _ = snn.snn_sparse_ways(T, B, n_in, n_out)
    n = min(int(csr.row_ptr[-1]), csr.capacity)
    assert csr.capacity >= min(cols, dense)  # the choice is made on the device
    return "product" if n >= dense else "columns" if n >= cols else "entries"


def _grad_in_way(T, B, n_in, n_out, inp):
    least = snn.snn_sparse_ways(T, B, n_in, n_out)[2]
    assert inp.capacity >= least
    return "product" if min(int(inp.row_ptr[-1]), inp.capacity) >= least else "entries"


@pytest.mark.parametrize("T,B,n_in,n_out,share,spare,with_g,way", [
    (60, 10, 700, 400, 0.9, 0, True, "product"),        # slab layer
    (60, 10, 700, 400, 0.3, 150000, True, "entries"),   # with room for the product
    (30, 21, 701, 403, 0.95, 1000, True, "product"),    # rows of no whole 16 bytes
    (30, 37, 900, 130, 0.97, 0, False, "product"),      # rows kernel's layer, no g
    (30, 37, 900, 130, 0.4, 90000, True, "entries"),
    (40, 20, 1300, 300, 0.8, 7, True, "product"),
    (5, 120, 130, 1100, 1.0, 0, True, "product"),
    (64, 100, 2312, 200, 0.15, 0, True, "columns"),     # a last input tile of 8, two column groups, several chunks
    (61, 105, 2309, 203, 0.15, 500, True, "columns"),   # rows of no whole 16 bytes, a last window of five rows
    (64, 100, 2312, 200, 0.05, 300000, True, "entries"),
    (64, 100, 1900, 700, 0.11, 0, False, "columns"),    # six column groups, the last in part, no g
    (10, 160, 4000, 2999, 0.1, 0, True, "columns"),     # one chunk
    (8, 40, 600, 4096, 0.9, 0, True, "product"),        # the widest layer: a block's rows fill 64 KB of LDS
])
def test_dw_wide_band(T, B, n_in, n_out, share, spare, with_g, way):
    rng = np.random.default_rng(n_in + n_out)
    on, g, csr, pad = _csr(rng, T, B, n_out, share, spare, with_g)
    assert _dw_way(T, B, n_in, n_out, csr) == way
    eps = rng.standard_normal(len(g)).astype(np.float32)
    trace = (rng.random((T, B, n_in)) * 2).astype(np.float32)
    dW = snn.sparse_dw(torch.from_numpy(trace).cuda(), csr, torch.from_numpy(pad(eps, np.float32(np.nan))).cuda(), n_out)
    G = np.zeros(on.shape)
    G[on] = (eps * g).astype(np.float64)
    tr = trace.reshape(T * B, n_in).astype(np.float64)
    # float64 sums of float32 products' exact values; partial sums and the result rounded to float32
    assert (np.abs(dW.cpu().numpy() - tr.T @ G) <= 4 * U * (tr.T @ np.abs(G))).all()


@pytest.mark.parametrize("T,B,n_in,n_out,share,way", [(60, 10, 700, 400, 0.95, "product"),
                                                      (64, 100, 2312, 200, 0.18, "columns")])
def test_dw_wide_band_truncated(T, B, n_in, n_out, share, way):
    """A CSR with more entries than slots: the entries below the capacity count, densely and by columns too."""
    rng = np.random.default_rng(3)
    on, g, csr, _ = _csr(rng, T, B, n_out, share)
    cap = len(g) - 20000
    cut = snn.Csr(csr.row_ptr, csr.col_idx[:cap].contiguous(), csr.g[:cap].contiguous(), csr.nnz_dev, cap)
    assert _dw_way(T, B, n_in, n_out, cut) == way
    eps = rng.standard_normal(cap).astype(np.float32)
    trace = (rng.random((T, B, n_in)) * 2).astype(np.float32)
    dW = snn.sparse_dw(torch.from_numpy(trace).cuda(), cut, torch.from_numpy(eps).cuda(), n_out)
    G = np.zeros(on.shape)
    r, c = np.nonzero(on)
    G[r[:cap], c[:cap]] = (eps * g[:cap]).astype(np.float64)
    tr = trace.reshape(T * B, n_in).astype(np.float64)
    assert (np.abs(dW.cpu().numpy() - tr.T @ G) <= 4 * U * (tr.T @ np.abs(G))).all()


def test_dw_wide_band_columns_outside():
    """By columns, an entry with a column outside the layer does not count, as on the other ways."""
    T, B, n_in, n_out = 64, 100, 2312, 200
    rng = np.random.default_rng(4)
    on, g, csr, _ = _csr(rng, T, B, n_out, 0.17)
    eps = rng.standard_normal(len(g)).astype(np.float32)
    trace = (rng.random((T, B, n_in)) * 2).astype(np.float32)
    rp = csr.row_ptr.cpu().numpy()
    first, last = int(rp[5]), int(rp[9]) - 1  # the first entry of row 5, the last of row 8
    csr.col_idx[first], csr.col_idx[last] = -3, n_out + 2
    assert _dw_way(T, B, n_in, n_out, csr) == "columns"
    dW = snn.sparse_dw(torch.from_numpy(trace).cuda(), csr, torch.from_numpy(eps).cuda(), n_out)
    G = np.zeros(on.shape)
    e = (eps * g).astype(np.float64)
    e[[first, last]] = 0.0
    G[on] = e
    tr = trace.reshape(T * B, n_in).astype(np.float64)
    assert (np.abs(dW.cpu().numpy() - tr.T @ G) <= 4 * U * (tr.T @ np.abs(G))).all()
    again = snn.sparse_dw(torch.from_numpy(trace).cuda(), csr, torch.from_numpy(eps).cuda(), n_out)
    assert torch.equal(dW, again)  # the order of the sums is fixed


def test_dw_rows_that_count_past_32_bits():
    """Rows of a malformed CSR that together hold more than 2^31 entries: the offsets of the slab records wrap, and
    no record is read or written outside the workspace."""
    T, B, n_in, n_out, cap = 64, 100, 64, 310, 700000
    rp = torch.zeros(T * B + 1, dtype=torch.int32, device="cuda")
    rp[1::2] = cap  # every second row spans all entries; the count says that there are none
    col = (torch.arange(cap, device="cuda") % n_out).to(torch.int32)
    csr = snn.Csr(rp, col, None, None, cap)
    need = snn.snn_sparse_dw_workspace(T, B, n_in, n_out, cap)
    room = torch.full((need + (1 << 23),), 0x5A, dtype=torch.uint8, device="cuda")
    ws = room[1 << 22:(1 << 22) + need]
    snn.sparse_dw(torch.rand((T, B, n_in), device="cuda"), csr, torch.rand(cap, device="cuda"), n_out, ws=ws)
    assert (room[:1 << 22] == 0x5A).all() and (room[(1 << 22) + need:] == 0x5A).all()


@pytest.mark.parametrize("T,B,n_in,n_out,share", [(30, 37, 900, 130, 0.97), (60, 10, 700, 400, 0.9),
                                                  (64, 100, 2312, 200, 0.15)])
@pytest.mark.parametrize("full", [False, True])
def test_wide_band_workspace_sizes(T, B, n_in, n_out, share, full):
    """The least workspace (for some layers sized without regard to the capacity) and the full one: dW and the spike
    gradient are right, the combined call gives the split calls' bits, and nothing is written behind either."""
    rng = np.random.default_rng(8)
    on, g, out, _ = _csr(rng, T, B, n_out, share)
    on_i, _, inp, _ = _csr(rng, T, B, n_in, 0.95)
    eps = rng.standard_normal(len(g)).astype(np.float32)
    trace = (rng.random((T, B, n_in)) * 2).astype(np.float32)
    W = rng.standard_normal((n_in, n_out)).astype(np.float32)
    alpha = float(np.float32(0.9))
    dev = lambda x: torch.from_numpy(x).cuda()
    q = snn
    cap = 100 if n_out <= 300 and n_in <= 1024 else out.capacity
    sizes = ((q.snn_sparse_dw_workspace_full(T, B, n_in, n_out, out.capacity),
              q.snn_sparse_grad_in_workspace_full(T, B, n_in, n_out, inp.capacity),
              q.snn_sparse_backward_workspace_full(T, B, n_in, n_out, out.capacity, inp.capacity)) if full else
             (q.snn_sparse_dw_workspace(T, B, n_in, n_out, cap), q.snn_sparse_grad_in_workspace(T, B, n_out),
              q.snn_sparse_backward_workspace(T, B, n_in, n_out, cap)))
    rooms = [torch.full((n + (1 << 20),), 0x5A, dtype=torch.uint8, device="cuda") for n in sizes]
    ws = [r[:n] for r, n in zip(rooms, sizes)]
    dW = snn.sparse_dw(dev(trace), out, dev(eps), n_out, ws=ws[0])
    e_in = snn.sparse_grad_in(dev(W), alpha, T, B, out, dev(eps), inp, ws=ws[1])
    dW2, e_in2 = snn.sparse_backward(dev(W), dev(trace), alpha, out, dev(eps), inp, ws=ws[2])
    for r, n in zip(rooms, sizes):
        assert (r[n:] == 0x5A).all()
    assert torch.equal(dW, dW2) and torch.equal(e_in, e_in2)
    G = np.zeros(on.shape)
    G[on] = (eps * g).astype(np.float64)
    tr = trace.reshape(T * B, n_in).astype(np.float64)
    assert (np.abs(dW.cpu().numpy() - tr.T @ G) <= 4 * U * (tr.T @ np.abs(G))).all()
    r, a = (_grad_in_reference(T, B, x, y, alpha)[on_i] for x, y in ((W, G), (np.abs(W), np.abs(G))))
    assert (np.abs(e_in.cpu().numpy() - r) <= 50 * U * a).all()


@pytest.mark.parametrize("T,B,n_in,n_out,share,spare,way", [
    (60, 10, 700, 400, 0.9, 0, "product"), (60, 10, 700, 400, 0.3, 150000, "entries"),
    (30, 37, 900, 130, 0.97, 0, "product"), (64, 100, 2312, 200, 0.15, 0, "columns"),
    (64, 100, 2312, 200, 0.05, 300000, "entries")])
def test_dw_wide_band_layout_then_prepared(T, B, n_in, n_out, share, spare, way):
    """The layout and then the rest, on the full workspace and on the least, give one call's bits; the layout can be
    used again with another eps."""
    rng = np.random.default_rng(n_in)
    _, g, csr, pad = _csr(rng, T, B, n_out, share, spare)
    assert _dw_way(T, B, n_in, n_out, csr) == way
    trace = torch.rand((T, B, n_in), device="cuda")
    eps = torch.from_numpy(pad(rng.standard_normal(len(g)).astype(np.float32), np.float32(0))).cuda()
    for query in (snn.snn_sparse_dw_workspace_full, snn.snn_sparse_dw_workspace):
        n = query(T, B, n_in, n_out, csr.capacity)
        ws, one = torch.full((n,), 0x5A, dtype=torch.uint8, device="cuda"), snn.workspace(n)[:n]
        snn.sparse_dw_layout((T, B, n_in), csr, n_out, ws)
        for e in (eps, 2.0 * eps):
            assert torch.equal(snn.sparse_dw_prepared(trace, csr, e, n_out, ws),
                               snn.sparse_dw(trace, csr, e, n_out, ws=one))


# one chunk (the records are the workspace's last array), several, and the dense product
@pytest.mark.parametrize("T,B,n_in,n_out,share", [(10, 160, 4000, 2999, 0.1), (64, 100, 2312, 200, 0.15),
                                                  (60, 10, 700, 400, 0.9)])
@pytest.mark.parametrize("kind", ["alternating", "falling", "wild"])
def test_dw_wide_band_malformed_row_pointers(T, B, n_in, n_out, share, kind):
    """Row pointers that decrease or lie outside the entry arrays: dW is unspecified, and nothing is written past
    the workspace."""
    TB = T * B
    rng = np.random.default_rng(5)
    cap = int(share * TB * n_out)
    rp = {"alternating": np.where(np.arange(TB + 1) % 2, 0, cap),
          "falling": cap - (np.arange(TB + 1) * cap) // TB,
          "wild": rng.integers(-2 ** 31, 2 ** 31, TB + 1)}[kind].astype(np.int32)
    rp[::128] = cap  # windows that start at the last entry
    rp[TB] = cap     # the entry count by which the way is chosen
    dev = lambda x: torch.from_numpy(x).cuda()
    col = dev(rng.integers(-1, n_out + 1, cap).astype(np.int32))
    csr = snn.Csr(dev(rp), col, None, None, cap)
    assert _dw_way(T, B, n_in, n_out, csr) != "entries"
    need = snn.snn_sparse_dw_workspace_full(T, B, n_in, n_out, cap)
    room = torch.full((need + (1 << 22),), 0x5A, dtype=torch.uint8, device="cuda")
    snn.sparse_dw(torch.rand((T, B, n_in), device="cuda"), csr, torch.rand(cap, device="cuda"), n_out, ws=room[:need])
    assert (room[need:] == 0x5A).all()


@pytest.mark.parametrize("end", [-1, -2 ** 31, 2 ** 31 - 1])
def test_wide_band_malformed_count(end):
    """Whatever the last row pointer holds, dW and the spike gradient are written (their values are unspecified)."""
    T, B, n_in, n_out = 30, 20, 900, 300
    rng = np.random.default_rng(6)
    _, g, out, _ = _csr(rng, T, B, n_out, 0.95)
    _, _, inp, _ = _csr(rng, T, B, n_in, 0.95)
    eps = torch.from_numpy(rng.standard_normal(len(g)).astype(np.float32)).cuda()
    out.row_ptr[T * B], inp.row_ptr[T * B] = end, end
    dW = torch.full((n_in, n_out), np.nan, device="cuda")
    snn.sparse_dw(torch.rand((T, B, n_in), device="cuda"), out, eps, n_out, dW=dW)
    e_in = torch.full((inp.capacity,), np.nan, device="cuda")
    snn.sparse_grad_in(torch.rand((n_in, n_out), device="cuda"), 0.9, T, B, out, eps, inp, eps_in=e_in)
    assert torch.isfinite(dW).all()
    rp = inp.row_ptr.cpu().numpy()
    assert torch.isfinite(e_in[:int(rp[T * B - 1])]).all()  # every row but the last has its bounds


def _grad_in_reference(T, B, W, G, alpha):
    d = np.zeros((T, B, W.shape[1]))
    G = G.reshape(T, B, -1)
    for t in range(T - 1, 0, -1):
        d[t - 1] = alpha * d[t] + G[t]
    return d.reshape(T * B, -1) @ W.astype(np.float64).T


# share_in on both sides of the count from which the product runs; output widths at the ends of a K stage
# and of the folds of two, input widths at a tile's ends, rows that do not fill a tile
@pytest.mark.parametrize("T,B,n_in,n_out,share_out,share_in,spare,way", [
    (30, 20, 900, 300, 0.3, 0.95, 0, "product"), (30, 20, 900, 300, 0.3, 0.1, 500000, "entries"),
    (129, 5, 1025, 257, 0.1, 0.9, 1000, "product"), (3, 427, 640, 256, 0.5, 0.9, 0, "product"),
    (7, 91, 897, 100, 0.9, 1.0, 3, "product"), (64, 20, 700, 35, 0.9, 0.95, 0, "product"),
    (2, 300, 1024, 1024, 0.2, 0.9, 0, "product"), (11, 61, 1000, 770, 0.02, 0.9, 0, "product")])
def test_grad_in_wide_band(T, B, n_in, n_out, share_out, share_in, spare, way):
    rng = np.random.default_rng(n_in * 7 + n_out)
    on_o, g, out, pad_o = _csr(rng, T, B, n_out, share_out)
    on_i, _, inp, _ = _csr(rng, T, B, n_in, share_in, spare)
    assert _grad_in_way(T, B, n_in, n_out, inp) == way
    eps = rng.standard_normal(len(g)).astype(np.float32)
    W = rng.standard_normal((n_in, n_out)).astype(np.float32)
    alpha = float(np.float32(np.exp(-0.1)))
    e_in = torch.full((inp.capacity,), 7.0, device="cuda")
    snn.sparse_grad_in(torch.from_numpy(W).cuda(), alpha, T, B, out, torch.from_numpy(pad_o(eps, np.float32(0))).cuda(),
                       inp, eps_in=e_in)
    G = np.zeros(on_o.shape)
    G[on_o] = (eps * g).astype(np.float64)
    r, a = (_grad_in_reference(T, B, x, y, alpha)[on_i] for x, y in ((W, G), (np.abs(W), np.abs(G))))
    got = e_in.cpu().numpy()
    # float32 recurrence (2 roundings a step, over 1 / (1 - alpha) steps) and sums (8 roundings of the leading
    # sum per 64 terms, 2^-24 left out of each product; a wavefront's dot product below the count: 24 roundings)
    assert (np.abs(got[:len(r)] - r) <= (2 * 11 + 24 + 4) * U * a).all()
    assert (got[len(r):] == 7.0).all()  # slots without an entry stay as they are


@pytest.mark.parametrize("n_out", [1024, 300, 40])
def test_grad_in_wide_band_errors_have_no_mean(n_out):
    """The dense product's rounding errors are as often up as down: a mean would add up over the rows of the next
    dW. Their mean lies within six standard errors."""
    T, B, n_in = 3, 500, 1024
    rng = np.random.default_rng(n_out)
    on_o, g, out, _ = _csr(rng, T, B, n_out, 0.5)
    on_i, _, inp, _ = _csr(rng, T, B, n_in, 0.95)
    eps = rng.standard_normal(len(g)).astype(np.float32)
    W = rng.standard_normal((n_in, n_out)).astype(np.float32)
    assert _grad_in_way(T, B, n_in, n_out, inp) == "product"
    e_in = snn.sparse_grad_in(torch.from_numpy(W).cuda(), 0.5, T, B, out, torch.from_numpy(eps).cuda(), inp)
    G = np.zeros(on_o.shape)
    G[on_o] = (eps * g).astype(np.float64)
    d = e_in.cpu().numpy() - _grad_in_reference(T, B, W, G, 0.5)[on_i]
    assert abs(d.mean()) <= 6 * d.std() / len(d) ** 0.5, (d.mean(), d.std(), len(d))


@pytest.mark.parametrize("big", [3e33, -2e38])  # past the split's range; past it unscaled too
def test_grad_in_wide_band_values_past_the_split(big):
    """A weight too large for the dense product's bf16 parts: its tiles (64 inputs) are formed from float32 operands,
    the other entries in them no less precisely than entry by entry."""
    T, B, n_in, n_out = 2, 700, 256, 1024
    rng = np.random.default_rng(17)
    on_o, g, out, _ = _csr(rng, T, B, n_out, 0.3)
    on_i, _, inp, _ = _csr(rng, T, B, n_in, 1.0)
    eps = (rng.standard_normal(len(g)) * 1e-3).astype(np.float32)
    W = rng.standard_normal((n_in, n_out)).astype(np.float32)
    W[70, 500], W[200, 3] = big, big  # in the second tile and the fourth
    dev = lambda x: torch.from_numpy(x).cuda()
    assert _grad_in_way(T, B, n_in, n_out, inp) == "product"
    run = lambda ws: snn.sparse_grad_in(dev(W), 0.5, T, B, out, dev(eps), inp, ws=ws).cpu().numpy().astype(np.float64)
    got, walk = run(None), run(snn.workspace(snn.snn_sparse_grad_in_workspace(T, B, n_out)))
    G = np.zeros(on_o.shape)
    G[on_o] = (eps * g).astype(np.float64)
    r, a = (_grad_in_reference(T, B, x, y, 0.5)[on_i] for x, y in ((W, G), (np.abs(W), np.abs(G))))
    assert (np.abs(got - r) <= 50 * U * a).all()
    i = np.nonzero(on_i)[1]
    other = (i // 64 % 2 == 1) & (i != 70) & (i != 200) & (a > 0)
    rms = lambda x: np.sqrt(np.mean((x - r)[other] ** 2))
    print("float32 tiles", rms(got), "entry by entry", rms(walk))
    assert rms(got) <= rms(walk)


def test_grad_in_wide_band_past_the_range():
    """Products past float32's range are infinities of the product's sign."""
    T, B, n_in, n_out = 2, 700, 640, 136
    rng = np.random.default_rng(13)
    j = rng.integers(0, n_out, B)  # one entry in every row of the last step; all input entries, enough for the dense product
    rp = np.concatenate([np.zeros(B), np.arange(B + 1)]).astype(np.int32)
    eps = (rng.uniform(0.5, 2, B) * 1e25 * rng.choice([-1, 1], B)).astype(np.float32)
    W = (rng.uniform(0.5, 2, (n_in, n_out)) * 1e20 * rng.choice([-1, 1], (n_in, n_out))).astype(np.float32)
    dev = lambda x: torch.from_numpy(x).cuda()
    out = snn.Csr(dev(rp), dev(j.astype(np.int32)), None, None, B)
    on_i, _, inp, _ = _csr(rng, T, B, n_in, 1.0)
    assert _grad_in_way(T, B, n_in, n_out, inp) == "product"
    e_in = snn.sparse_grad_in(dev(W), 0.5, T, B, out, dev(eps), inp).cpu().numpy().reshape(T, B, n_in)
    assert np.array_equal(e_in[0], np.sign(eps[:, None] * W[:, j].T.astype(np.float64)) * np.inf)
    assert (e_in[1] == 0).all()


def test_grad_in_wide_band_truncated_and_columns_outside():
    """Entries past the input capacity are not written; an entry with a column outside the layer reads 0."""
    T, B, n_in, n_out = 30, 20, 900, 300
    rng = np.random.default_rng(11)
    on_o, g, out, _ = _csr(rng, T, B, n_out, 0.2)
    on_i, _, inp, _ = _csr(rng, T, B, n_in, 0.99)
    eps = rng.standard_normal(len(g)).astype(np.float32)
    W = rng.standard_normal((n_in, n_out)).astype(np.float32)
    col = inp.col_idx.clone()
    rp = inp.row_ptr.cpu().numpy()
    first, last = int(rp[5]), int(rp[9]) - 1  # the first entry of row 5, the last of row 8
    col[first], col[last] = -3, n_in + 2
    cap = inp.capacity - 5000
    cut = snn.Csr(inp.row_ptr, col[:cap].contiguous(), None, None, cap)
    assert _grad_in_way(T, B, n_in, n_out, cut) == "product"
    e_in = snn.sparse_grad_in(torch.from_numpy(W).cuda(), 0.9, T, B, out, torch.from_numpy(eps).cuda(), cut)
    G = np.zeros(on_o.shape)
    G[on_o] = (eps * g).astype(np.float64)
    alpha = float(np.float32(0.9))
    r, a = (_grad_in_reference(T, B, x, y, alpha)[on_i][:cap] for x, y in ((W, G), (np.abs(W), np.abs(G))))
    r[[first, last]] = 0.0
    assert (np.abs(e_in.cpu().numpy() - r) <= 45 * U * a).all()


# many bits per window (placed a lane per column) and few, rows of part windows, of 64 windows and of more,
# tiles that mix both, a capacity in the middle
@pytest.mark.parametrize("T,B,N,share,cut", [
    (7, 5, 33, 0.9, 0), (40, 30, 64, 0.5, 0), (50, 26, 200, 0.3, 0), (20, 33, 300, 0.95, 100), (9, 11, 1024, 1.0, 0),
    (3, 7, 4096, 0.3, 0), (3, 5, 4500, 0.4, 5000), (60, 40, 130, -1.0, 0), (1, 1, 1, 1.0, 0)])
def test_compact_bits_wide_band(T, B, N, share, cut):
    rng = np.random.default_rng(N)
    V = rng.random((T, B, N)).astype(np.float32)
    if share < 0:  # activity that changes along time: tiles of either kind
        on = rng.random((T, B, N)) < np.linspace(0, 1, T)[:, None, None]
    else:
        on = rng.random((T, B, N)) < share
    W64 = (B * N + 63) // 64
    pad = np.zeros((T, W64 * 64), np.uint8)
    pad[:, :B * N] = on.reshape(T, -1)
    words = np.packbits(pad, axis=1, bitorder="little").view(np.int64).reshape(-1)
    n = int(on.sum())
    cap = max(n - cut, 1)
    csr = snn.active_compact_bits(torch.from_numpy(words.copy()).cuda(), torch.from_numpy(V).cuda(), 1.0, 100.0, cap)
    flat = on.reshape(T * B, N)
    assert csr.nnz() == n
    assert np.array_equal(csr.row_ptr.cpu().numpy(), np.concatenate([[0], np.cumsum(flat.sum(1))]))
    m = min(n, cap)
    assert np.array_equal(csr.col_idx.cpu().numpy()[:m], np.nonzero(flat)[1][:m])
    d = np.abs(V[on][:m] - np.float32(1.0))
    x = np.float32(100.0) * d + np.float32(1.0)
    assert (np.abs(csr.g.cpu().numpy()[:m] - 1.0 / (x * x)) <= 4 * U / (x * x)).all()
