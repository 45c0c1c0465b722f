"""The convolutional forward a pooling window at a time (snn_conv_lif_forward_pool) and the gather of
layers of at most 32 outputs, bit for bit against the oracle at the edges of their tiles."""
import math

import numpy as np
import pytest
import torch

import oracle
from oracle import conv
from paper_2105_08810_amd import snn

pytestmark = pytest.mark.gpu
F32 = np.float32


def _same(x, r, what):
    x = x.cpu().numpy().reshape(-1)
    r = np.ascontiguousarray(r).reshape(-1)
    same = x.view(np.uint32) == r.astype(F32).view(np.uint32) if x.dtype == F32 else x == r
    assert same.all(), f"{what}: {int((~same).sum())} of {same.size} differ"


# steps around a group of eight, one and two filter groups, 1, 2, 4 input channels (one launch), 3 channels and
# 32 filters (pooling and trace behind the layer); spike bytes that are not 1; a full patch; as many wavefronts as
# the layer alone needs to go by windows, one less, and few of them over many steps (pooling behind the layer)
@pytest.mark.parametrize("T,B,H,W,C,Fo,rate,value", [
    (1, 1, 2, 2, 1, 64, 0.5, 1), (2, 3, 4, 2, 1, 64, 0.3, 1), (8, 2, 2, 6, 1, 128, 0.2, 7), (9, 1, 6, 4, 2, 64, 0.2, 1),
    (10, 2, 4, 4, 4, 64, 0.1, 200), (18, 2, 8, 6, 1, 64, 1.0, 1), (11, 2, 4, 4, 3, 64, 0.2, 1), (9, 2, 4, 4, 1, 32, 0.3, 1),
    (3, 512, 2, 4, 1, 64, 0.2, 1), (3, 1023, 2, 2, 2, 64, 0.2, 1), (53, 3, 4, 4, 1, 64, 0.2, 1)])
def test_conv_forward_pool(T, B, H, W, C, Fo, rate, value):
    rng = np.random.default_rng(T * 100 + Fo + C)
    X = (rng.random((T, B, H, W, C)) < rate).astype(np.uint8) * np.uint8(value)
    Wc = (rng.standard_normal((3, 3, C, Fo)) * 0.5 + 0.2).astype(F32)
    a, an, b_th = F32(0.9), F32(0.8), 0.3
    Np = H * W * Fo // 4
    f = conv.conv_network_forward((X != 0).astype(np.uint8), Wc, np.zeros((Np, 1), F32), a, an)
    dev = lambda shape, dt: torch.full(shape, 77, dtype=dt, device="cuda")
    V, S = dev((T, B, H * W * Fo), torch.float32), dev((T, B, H * W * Fo), torch.uint8)
    tr, bits = dev((T, B, H * W * C), torch.float32), dev((snn.snn_active_bits_words(T, B, H * W * Fo),), torch.int64)
    P, arg, trp = dev((T, B, Np), torch.uint8), dev((T, B, Np), torch.uint8), dev((T, B, Np), torch.float32)
    x, w = torch.from_numpy(X).cuda(), torch.from_numpy(Wc).cuda()
    snn.snn_conv_lif_forward_pool(x, w, T, B, H, W, C, Fo, a, 1.0, b_th, V, S, tr, bits, P, arg, trp, an)
    _same(V, f["V"], "V")
    _same(S, f["S"], "S")
    _same(tr, f["trace"], "trace")
    _same(P, f["P"], "P")
    _same(arg, f["arg"], "arg")
    _same(trp, f["trace_out"], "trace of the pooled spikes")
    # the layer alone, and without trace and bitset, gives the same
    V2, S2, bits2 = torch.zeros_like(V), torch.zeros_like(S), torch.zeros_like(bits)
    snn.snn_conv_lif_forward(x, w, T, B, H, W, C, Fo, a, 1.0, b_th, V2, S2, None, bits2)
    assert torch.equal(V, V2) and torch.equal(S, S2) and torch.equal(bits, bits2)
    P2, arg2 = torch.zeros_like(P), torch.zeros_like(arg)
    snn.snn_conv_lif_forward_pool(x, w, T, B, H, W, C, Fo, a, 1.0, b_th, V2, S2, None, None, P2, arg2)
    assert torch.equal(V, V2) and torch.equal(P, P2) and torch.equal(arg, arg2)
    on = np.abs(f["V"].reshape(T, -1) - F32(1.0)) < F32(b_th)
    pad = np.zeros((T, (on.shape[1] + 63) // 64 * 64), np.uint8)
    pad[:, :on.shape[1]] = on
    assert np.array_equal(bits.cpu().numpy(), np.packbits(pad, axis=1, bitorder="little").view(np.int64).reshape(-1))


# inputs a multiple of 16, 8, 4 bytes per row (and odd: the general gather), a row's last piece, lists that fill
# up before the row ends, one to 32 outputs, rows that do not fill a block
@pytest.mark.parametrize("T,B,n_in,n_out,rate", [
    (2, 1, 16, 1, 0.5), (5, 3, 64, 16, 0.2), (4, 7, 1040, 10, 1.0), (3, 5, 200, 10, 0.3), (6, 3, 300, 17, 0.1),
    (3, 2, 4100, 32, 0.9), (3, 2, 12544, 10, 0.02), (4, 3, 520, 31, 1.0), (3, 9, 201, 5, 0.3), (2, 2, 5, 20, 1.0)])
def test_narrow_gather(T, B, n_in, n_out, rate):
    rng = np.random.default_rng(n_in + n_out)
    X = (rng.random((T, B, n_in)) < rate).astype(np.uint8) * np.uint8(9)
    W = (rng.standard_normal((n_in, n_out)) * 0.1).astype(F32)
    f = oracle.lif_forward((X != 0).astype(np.uint8), W, F32(0.9), F32(np.inf))
    V, S, tr = snn.lif_forward(torch.from_numpy(X).cuda(), torch.from_numpy(W).cuda(), F32(0.9), math.inf)
    _same(V, f[0] if isinstance(f, tuple) else f["V"], "V")
    assert not bool(S.any())
