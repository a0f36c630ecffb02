"""The diagonal-block factorisation at every position of a pivot inside its four-pivot
steps, 16-wide leaves and blocks: the first failing column is reported exactly, and the
factorisation of well-posed systems of any block remainder matches numpy in fp64.

Errors of a solve are bounded by a small multiple of cond * eps: cond below 50 here, so
2e-5 in fp32 (2^-24 * 50 * 4), 2e-3 with three product terms (2^-16 a product) and 1e-6 after
rounding fp64 results to fp32."""
import numpy as np
import pytest
import torch

import paper_2609_39329_amd as pkv
from gpu_util import DEV, host, rel

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("dtype", [torch.float32, torch.float64])
@pytest.mark.parametrize("p", [0, 1, 2, 3, 4, 7, 15, 16, 18, 63, 64, 65, 126, 127, 128, 131, 149])
@pytest.mark.parametrize("pivot", [-1.0, -1e-3, float("nan")])
def test_first_failing_column(dtype, p, pivot):
    print(f"failing column {p} pivot {pivot} {dtype}", flush=True)
    d = 150
    rng = np.random.default_rng(p)
    L = np.tril(rng.standard_normal((d, d)) * 0.05) + np.eye(d)
    G = L @ L.T
    s = L[p, :p] @ L[p, :p]
    lam = 0.25
    G -= lam * np.eye(d)
    G[p, p] = s + pivot - lam  # Schur complement of column p
    G[p + 1:, p + 1:] += 2 * np.eye(d - p - 1)
    if p + 3 < d:
        G[p + 3, p + 3] = -5.0  # a later failure is not reported
    dW, info = pkv.solve_patch(torch.from_numpy(G).to(dtype).to(DEV), torch.ones((d, 4), dtype=dtype, device=DEV), lam)
    assert int(info.item()) == p + 1


@pytest.mark.parametrize("dtype", [torch.float32, torch.float64])
@pytest.mark.parametrize("p", [0, 1, 2, 3, 4, 7, 15, 16, 18, 63, 64, 65, 126, 127, 128, 131, 149])
@pytest.mark.parametrize("coupled", [False, True])
def test_zero_pivot(dtype, p, coupled):
    """A Schur complement of exactly zero: every other pivot is 1 and the entries are small
    whole numbers, so each product and sum of the factorisation is exact."""
    print(f"zero pivot {p} {dtype} coupled {coupled}", flush=True)
    d, lam = 150, 0.25
    L = np.eye(d)
    L[p, p] = 0.0
    if coupled:
        L[p, :p:3] = 1.0   # row p on columns before it: G[p, p] + lam is their number
        L[p + 1:, :p:7] = -1.0
    G = L @ L.T - lam * np.eye(d)
    dW, info = pkv.solve_patch(torch.from_numpy(G).to(dtype).to(DEV), torch.ones((d, 4), dtype=dtype, device=DEV), lam)
    assert int(info.item()) == p + 1


@pytest.mark.parametrize("dtype", [torch.float32, torch.float64])
@pytest.mark.parametrize("p", [0, 1, 2, 3, 4, 7, 14, 15, 16, 30, 31, 63, 64, 127, 128, 131, 149])
@pytest.mark.parametrize("later", [False, True])
def test_infinite_pivot(dtype, p, later):
    """One channel whose diagonal overflowed, its products with the others finite: the
    reciprocal root of the pivot is 0, so the columns after it factor as if it were not there."""
    print(f"infinite pivot {p} {dtype} later failure {later}", flush=True)
    d = 150
    rng = np.random.default_rng(p)
    L = np.tril(rng.standard_normal((d, d)) * 0.05) + np.eye(d)
    G = L @ L.T
    G[p, p] = np.inf
    if later and p + 3 < d:
        G[p + 3, p + 3] = -5.0  # not reported
    dW, info = pkv.solve_patch(torch.from_numpy(G).to(dtype).to(DEV), torch.ones((d, 4), dtype=dtype, device=DEV), 0.25)
    assert int(info.item()) == p + 1


@pytest.mark.parametrize("dtype,tol", [(torch.float32, 2e-5), (torch.float64, 1e-6)])
@pytest.mark.parametrize("d", [1, 2, 3, 4, 5, 15, 16, 17, 33, 63, 64, 65, 100, 127, 128, 129, 145, 260])
def test_block_remainders(dtype, tol, d):
    print(f"remainder d={d} {dtype}", flush=True)
    rng = np.random.default_rng(d)
    X = rng.standard_normal((4 * d, d)) / np.sqrt(4 * d)
    G, C = X.T @ X, rng.standard_normal((d, 9))
    dW, info = pkv.solve_patch(torch.from_numpy(G).to(dtype).to(DEV), torch.from_numpy(C).to(dtype).to(DEV), 0.1)
    assert int(info.item()) == 0
    assert rel(host(dW), np.linalg.solve(G + 0.1 * np.eye(d), C)) <= tol


@pytest.mark.parametrize("mode,tol", [(0, 2e-5), (32, 2e-3)])
def test_wide_right_hand_side(mode, tol):
    """Updates on both sides of the line between one launch with the next factorisation (the
    second block column: 941 tiles of 128) and two (the first: 1413)."""
    d, n = 400, 60000
    print(f"solve {d} x {n} mode {mode}", flush=True)
    rng = np.random.default_rng(7)
    X = rng.standard_normal((4 * d, d)) / np.sqrt(4 * d)
    G, C = X.T @ X, rng.standard_normal((d, n)).astype(np.float32)
    dW, info = pkv.solve_patch(torch.from_numpy(G).float().to(DEV), torch.from_numpy(C).to(DEV), 0.1, mode=mode)
    assert int(info.item()) == 0
    cols = rng.choice(n, 200, replace=False)
    assert rel(host(dW[:, torch.from_numpy(cols).to(DEV)]), np.linalg.solve(G + 0.1 * np.eye(d), C[:, cols].astype(np.float64))) <= tol
