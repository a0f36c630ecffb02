"""The reduced-rank patch at the edges of its tall-skinny products (16-row tiles, whole and
partial 16-wide chunks, more and fewer chunks than loads in flight), of the mirrored S
(64- and 128-tiles) and of subspaces narrower than 64, against numpy in fp64 with a planted
gap, where the projected patch is unique.

S = dW^T G dW is FP32-grade (2^-24 per product), the subspace iteration exact fp32 products;
over a gap of a factor above 10 the projector is off by a few 1e-6: bound 2e-5."""
import numpy as np
import pytest
import torch

import paper_2609_39329_amd as pkv
from gpu_util import DEV, host, rel

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("din,dout,r", [(64, 64, 5), (130, 62, 6), (200, 65, 9), (90, 129, 12),
                                        (257, 191, 20), (300, 520, 31), (70, 1025, 16), (129, 656, 40)])
def test_low_rank_edges(din, dout, r):
    print(f"low rank edges din={din} dout={dout} r={r}", flush=True)
    rng = np.random.default_rng(din * dout)
    X = rng.standard_normal((2 * din, din))
    G = (X.T @ X).astype(np.float32)
    dW = (rng.standard_normal((din, r)) @ rng.standard_normal((r, dout))
          + 0.01 * rng.standard_normal((din, dout))).astype(np.float32)
    g, w = G.astype(np.float64), dW.astype(np.float64)
    val, vec = np.linalg.eigh(w.T @ g @ w)
    U = vec[:, -r:]
    dev = lambda a: torch.from_numpy(a).to(DEV)  # noqa: E731
    A, Ur, full = pkv.low_rank_patch(dev(G), dev(dW), r=r)
    Uh = host(Ur)
    assert np.abs(Uh.T @ Uh - np.eye(r)).max() <= 2e-5
    assert rel(host(full), w @ U @ U.T) <= 2e-5
    assert rel(host(A) @ Uh.T, w @ U @ U.T) <= 2e-5
