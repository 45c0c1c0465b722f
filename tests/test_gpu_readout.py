"""snn_readout_ce against a float64 reference at the edges of its kernels: one class, one step, more
classes than threads, time split over few or many threads per class, ties, infinities, NaN."""
import numpy as np
import pytest
import torch

from paper_2105_08810_amd import snn

pytestmark = pytest.mark.gpu


def _reference(V, labels, mode):
    """(row_ptr, col_idx, eps, loss) of the oracle's definition: strict comparison from step 0 on."""
    T, B, C = V.shape
    if mode == 0:
        best, when = V[0].copy(), np.zeros((B, C), np.int64)
        for t in range(1, T):
            up = V[t] > best
            best[up], when[up] = V[t][up], t
    else:
        best = V.astype(np.float64).sum(0).astype(np.float32)
    a = best.astype(np.float64)
    with np.errstate(invalid="ignore"):
        e = np.exp(a - np.fmax.reduce(a, axis=1, keepdims=True))
        p = e / e.sum(1, keepdims=True)
        loss = np.mean([-np.log(p[b, y]) if 0 <= y < C else np.nan for b, y in enumerate(labels)])
    d = p.copy()
    for b, y in enumerate(labels):
        if 0 <= y < C:
            d[b, y] -= 1.0
    d /= B
    if mode == 1:
        r = np.arange(T * B + 1) * C
        return r, np.tile(np.arange(C), T * B), np.tile(d.reshape(-1), T), loss, p
    rows, cols, eps = [0], [], []
    for t in range(T):
        for b in range(B):
            c = np.nonzero(when[b] == t)[0]
            cols.extend(c)
            eps.extend(d[b, c])
            rows.append(len(cols))
    return np.array(rows), np.array(cols), np.array(eps), loss, p


@pytest.mark.parametrize("mode", [0, 1])
@pytest.mark.parametrize("T,B,C,kind", [
    (1, 1, 1, "normal"), (1, 5, 7, "normal"), (100, 256, 10, "normal"), (37, 300, 4, "ties"), (9, 3, 255, "normal"),
    (33, 2, 257, "ties"), (5, 2, 1025, "normal"), (700, 3, 100, "normal"), (8192, 2, 1, "ties"), (50, 6, 12, "inf"),
    (50, 6, 12, "nan"), (1, 3, 128, "ties"), (1, 300, 130, "normal"), (7, 260, 129, "ties"), (2, 40, 5000, "ties"),
    (3, 2, 16384, "normal"), (300, 3, 300, "ties"), (1, 1, 16384, "normal")])
def test_readout_ce(mode, T, B, C, kind):
    rng = np.random.default_rng(T * 1000 + C)
    V = rng.standard_normal((T, B, C)).astype(np.float32)
    if kind == "ties":
        V = np.round(V)
    if kind == "inf":  # a class that is -inf throughout, one whose first step is
        V[:, :, 3] = -np.inf
        V[0, :, 5] = -np.inf
        if mode == 1:
            V = np.where(np.isinf(V), np.float32(-50.0), V)
    if kind == "nan":  # a NaN after step 0 never wins a strict comparison
        V[1:, :, 2] = np.nan
        if mode == 1:
            pytest.skip("a sum with a NaN is NaN")
    labels = rng.integers(0, C, B).astype(np.int32)
    if kind == "inf":
        labels[:] = 0
    csr, eps, loss, ed = snn.readout_ce(torch.from_numpy(V).cuda(), torch.from_numpy(labels).cuda(), mode, dense=True)
    rp, ci, e, lo, p = _reference(V, labels, mode)
    assert np.array_equal(csr.row_ptr.cpu().numpy(), rp)
    assert np.array_equal(csr.col_idx.cpu().numpy(), ci)
    assert csr.nnz() == len(ci)
    # p: float32 exp and division, each within a few ulp, and a float32 sum of C terms over a tree
    tol = 1e-6 * (4 + np.log2(C)) / B
    assert np.abs(eps.cpu().numpy() - e).max() <= tol
    assert abs(float(loss) - lo) <= 1e-5 * max(1.0, abs(lo))
    dense = np.zeros((T * B, C))
    dense[np.repeat(np.arange(T * B), np.diff(rp)), ci] = e
    assert np.abs(ed.cpu().numpy().reshape(T * B, C) - dense).max() <= tol


def test_readout_ce_label_outside():
    V = torch.randn((6, 3, 5), device="cuda")
    _, eps, loss, _ = snn.readout_ce(V, torch.tensor([1, 9, 0], dtype=torch.int32, device="cuda"), 0)
    assert bool(torch.isnan(loss).all()) and bool(torch.isfinite(eps).all())
