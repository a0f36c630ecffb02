"""Split-product tiles of the statistics and the SwiGLU features at their edges: 128-, 192-
and 256-wide tiles, one contraction chunk and partial ones, more and fewer chunks than LDS
stages, gate and up read as stored and through transposed copies, against numpy in fp64.

Every product sums two- or three-term bf16 splits (operands to about 2^-17) in fp32: 5e-5
of the result's norm, as the statistics' other tests."""
import numpy as np
import pytest
import torch

import paper_2609_39329_amd as pkv
from gpu_util import DEV, host, rel

pytestmark = pytest.mark.gpu
TOL = 5e-5


def normal(seed, *shape, scale=1.0, dtype=torch.float32):
    g = torch.Generator().manual_seed(seed)
    return (torch.randn(shape, generator=g) * scale).to(dtype).to(DEV)


# (M, d_in, d_out): small tiles; one round of 128 x 256; several rounds of 256 x 256
@pytest.mark.parametrize("M,din,dout", [(1, 32, 4), (127, 33, 129), (129, 65, 131), (257, 160, 255),
                                        (130, 4100, 260), (2049, 96, 3970), (4097, 72, 4100)])
@pytest.mark.parametrize("wdt", [torch.bfloat16, torch.float32])
def test_targets_tiles(M, din, dout, wdt):
    print(f"targets M={M} din={din} dout={dout} {wdt}", flush=True)
    Of, Oc, W = normal(1, M, din), normal(2, M, din), normal(3, din, dout, dtype=wdt)
    T = pkv.compute_targets(Of, Oc, W, rho=0)
    ref = (host(Of) - host(Oc)) @ host(W)
    assert rel(host(T), ref) <= TOL


# what the epilogue adds: a residual pair inside the matrix (16-byte loads), at its edges, and
# with rows that are not a multiple of 16 bytes
@pytest.mark.parametrize("M,d", [(31, 32), (256, 256), (300, 260), (260, 261), (1100, 1412)])
def test_targets_residual(M, d):
    print(f"targets with the residual, M={M} d={d}", flush=True)
    Of, Oc = normal(1, M, d), normal(2, M, d)
    W = normal(3, d, d, scale=d ** -0.5, dtype=torch.bfloat16)
    T = pkv.compute_targets(Of, Oc, W, rho=1)
    D = host(Of) - host(Oc)
    assert rel(host(T), D @ host(W) + D) <= TOL


# d_in around 128 and 192 multiples, and past the 128-tiles' limit (2,816)
@pytest.mark.parametrize("rows,din,dout", [(1, 127, 3), (63, 129, 130), (200, 385, 384),
                                           (64, 2817, 33), (97, 2820, 128)])
def test_normal_eq_tiles(rows, din, dout):
    print(f"normal_eq rows={rows} din={din} dout={dout}", flush=True)
    X, Y = normal(4, rows, din), normal(5, rows, dout)
    G, C = pkv.accumulate_normal_eq(X, Y)
    x, y = host(X), host(Y)
    assert rel(host(G), x.T @ x) <= TOL and rel(host(C), x.T @ y) <= TOL
    assert torch.equal(G, G.t().contiguous())
    pkv.accumulate_normal_eq(X, Y, G=G, C=C, accumulate=True)
    assert rel(host(G), 2 * (x.T @ x)) <= TOL and rel(host(C), 2 * (x.T @ y)) <= TOL


# as stored (d_ff a multiple of 8, M <= 1536) and transposed (the others; fp32 weights)
@pytest.mark.parametrize("M,d,d_ff", [(1, 8, 4), (3, 65, 8), (129, 70, 36), (130, 64, 40), (257, 200, 264),
                                      (1536, 130, 136), (1537, 130, 136), (300, 8300, 24),
                                      (40, 128, 33000)])
@pytest.mark.parametrize("wdt", [torch.bfloat16, torch.float32])
def test_features_tiles(M, d, d_ff, wdt):
    print(f"features M={M} d={d} d_ff={d_ff} {wdt}", flush=True)
    Z = normal(6, M, d, scale=0.1)
    Wg, Wu = (normal(s, d, d_ff, scale=d ** -0.5, dtype=wdt) for s in (7, 8))
    H = pkv.mlp_features(Z, Wg, Wu)
    z = host(Z)
    u = z / np.sqrt((z * z).mean(1, keepdims=True) + 1e-5)
    g = u @ host(Wg)
    assert rel(host(H), g / (1 + np.exp(-g)) * (u @ host(Wu))) <= TOL


def test_features_unaligned_rows_of_weights():
    """A weight matrix whose storage starts 8 elements into an allocation still aligns; the
    result does not depend on which copy path is taken."""
    d, d_ff, M = 96, 264, 200
    base = [normal(9 + i, d * d_ff + 8, scale=0.1, dtype=torch.bfloat16) for i in range(2)]
    Wg, Wu = (b[8:].view(d, d_ff) for b in base)
    Z = normal(11, M, d)
    a = pkv.mlp_features(Z, Wg, Wu)
    b = pkv.mlp_features(torch.cat([Z] * 8), Wg, Wu)  # 1,600 rows: transposed copies
    assert torch.equal(a, b[:M])


def test_rounds_split_over_two_shapes():
    """3.1 rounds of 256-tiles: whole rounds and the rest as two launches, residual included."""
    M, din, dout = 4096 * 3 + 300, 40, 4096
    Hf, Hc, W = normal(21, M, din), normal(22, M, din), normal(23, din, dout, dtype=torch.bfloat16)
    Zf, Zc = normal(24, M, dout), normal(25, M, dout)
    T = pkv.compute_block_targets(Hf, Hc, W, Zf, Zc)
    ref = (Hf.double() - Hc.double()) @ W.double() + (Zf.double() - Zc.double())
    assert float((T.double() - ref).norm() / ref.norm()) <= TOL
