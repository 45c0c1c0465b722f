"""Layers with many active entries: the dense products taken from a device-side count on, on both sides
of it, against float64."""
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


# least: the count from which the dense product runs, which shares bracket (600 rows, 700 -> 400: 1.4e5)
@pytest.mark.parametrize("T,B,n_in,n_out,share,spare,with_g", [
    (60, 10, 700, 400, 0.9, 0, True),        # dense product, slab layer
    (60, 10, 700, 400, 0.3, 150000, True),   # room for it, entry by entry
    (30, 21, 701, 403, 0.95, 1000, True),    # rows of no whole 16 bytes
    (30, 37, 900, 130, 0.97, 0, False),      # rows kernel's layer, no g
    (30, 37, 900, 130, 0.4, 90000, True),
    (40, 20, 1300, 300, 0.8, 7, True),
    (5, 120, 130, 1100, 1.0, 0, True),
])
def test_dw_wide_band(T, B, n_in, n_out, share, spare, with_g):
    rng = np.random.default_rng(n_in + n_out)
    on, g, csr, pad = _csr(rng, T, B, n_out, share, spare, with_g)
    eps = rng.standard_normal(len(g)).astype(np.float32)
    trace = (rng.random((T, B, n_in)) * 2).astype(np.float32)
    dW = snn.sparse_dw(torch.from_numpy(trace).cuda(), csr, torch.from_numpy(pad(eps, np.float32(np.nan))).cuda(), n_out)
    G = np.zeros(on.shape)
    G[on] = (eps * g).astype(np.float64)
    tr = trace.reshape(T * B, n_in).astype(np.float64)
    # float64 sums of float32 products' exact values; partial sums and the result rounded to float32
    assert (np.abs(dW.cpu().numpy() - tr.T @ G) <= 4 * U * (tr.T @ np.abs(G))).all()


def test_dw_wide_band_truncated():
    """A CSR with more entries than slots: the entries below the capacity count, on the dense way too."""
    T, B, n_in, n_out = 60, 10, 700, 400
    rng = np.random.default_rng(3)
    on, g, csr, _ = _csr(rng, T, B, n_out, 0.95)
    cap = len(g) - 20000
    cut = snn.Csr(csr.row_ptr, csr.col_idx[:cap].contiguous(), csr.g[:cap].contiguous(), csr.nnz_dev, cap)
    eps = rng.standard_normal(cap).astype(np.float32)
    trace = (rng.random((T, B, n_in)) * 2).astype(np.float32)
    dW = snn.sparse_dw(torch.from_numpy(trace).cuda(), cut, torch.from_numpy(eps).cuda(), n_out)
    G = np.zeros(on.shape)
    r, c = np.nonzero(on)
    G[r[:cap], c[:cap]] = (eps * g[:cap]).astype(np.float64)
    tr = trace.reshape(T * B, n_in).astype(np.float64)
    assert (np.abs(dW.cpu().numpy() - tr.T @ G) <= 4 * U * (tr.T @ np.abs(G))).all()
