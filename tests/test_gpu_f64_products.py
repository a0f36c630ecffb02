"""fp64 products (statistics with fp64 accumulation, the fp64 solve) at the edges of their
32- and 64-wide tiles and 32-wide K chunks, and the merge of many key ranges, against
numpy in fp64.

An fp64 sum of n products is off by at most n 2^-53 of the sum of magnitudes; for the
random operands here that is below 1e-13 of the result's norm. The solve multiplies it by
the condition number (below 1e3): 1e-10, then rounds to fp32 (6e-8)."""
import numpy as np
import pytest
import torch

import paper_2609_39329_amd as pkv
from gpu_util import DEV, host, rel

pytestmark = pytest.mark.gpu


def dev(a, dtype=torch.float32):
    return torch.from_numpy(np.ascontiguousarray(a)).to(dtype).to(DEV)


@pytest.mark.parametrize("rows,din,dout", [(1, 1, 1), (31, 33, 32), (33, 64, 65), (32, 31, 1),
                                           (97, 130, 63), (70, 1030, 1025)])
@pytest.mark.parametrize("diff", [False, True])
def test_f64_statistics(rows, din, dout, diff):
    print(f"f64 statistics rows={rows} din={din} dout={dout} diff={diff}", flush=True)
    rng = np.random.default_rng(rows + din)
    X, Y, Z = (rng.standard_normal(s).astype(np.float32)
               for s in ((rows, din), (rows, dout), (rows, dout)))
    T = Y.astype(np.float64) - (Z if diff else 0)
    G, C = pkv.accumulate_normal_eq(dev(X), dev(Y), dev(Z) if diff else None, acc=pkv.F64)
    X64 = X.astype(np.float64)
    assert rel(host(G), X64.T @ X64) <= 1e-13
    assert rel(host(C), X64.T @ T) <= 1e-13
    pkv.accumulate_normal_eq(dev(X), dev(Y), dev(Z) if diff else None, G=G, C=C, acc=pkv.F64,
                             accumulate=True)
    assert rel(host(G), 2 * (X64.T @ X64)) <= 1e-13
    assert rel(host(C), 2 * (X64.T @ T)) <= 1e-13


@pytest.mark.parametrize("d,dout", [(1, 3), (63, 65), (64, 31), (130, 33), (515, 70), (1050, 1030)])
def test_f64_solve(d, dout):
    print(f"f64 solve d={d} dout={dout}", flush=True)
    rng = np.random.default_rng(d)
    X = rng.standard_normal((2 * d, d))
    G, C = X.T @ X, rng.standard_normal((d, dout))
    dW, info = pkv.solve_patch(dev(G, torch.float64), dev(C, torch.float64), 0.1)
    assert int(info.item()) == 0
    assert rel(host(dW), np.linalg.solve(G + 0.1 * np.eye(d), C)) <= 1e-7


@pytest.mark.parametrize("dtype,tol", [("f32", 2e-5), ("bf16", 5e-5)])
@pytest.mark.parametrize("dh", [64, 128])
@pytest.mark.parametrize("N,counts", [(2065, None), (2048, (1, 2048)), (40, (33, 2)), (700, (699, 64))])
def test_merge_of_key_ranges(dtype, tol, dh, N, counts):
    """Few queries: the cache is split into up to 64 key ranges, some of them empty for a
    head that keeps few entries."""
    print(f"merge dtype={dtype} dh={dh} N={N} counts={counts}", flush=True)
    rng = np.random.default_rng(N)
    M, Hq, Hkv = 3, 4, 2
    tdt = torch.float32 if dtype == "f32" else torch.bfloat16
    Q, K, V = (dev(rng.standard_normal(s), tdt) for s in ((M, Hq, dh), (Hkv, N, dh), (Hkv, N, dh)))
    cnt = None if counts is None else torch.tensor(counts, dtype=torch.int32, device=DEV)
    idx = torch.from_numpy(rng.permutation(N).astype(np.int32)).to(DEV)
    got = host(pkv.attend_compressed(Q, K, V, idx=idx, counts=cnt)).reshape(M, Hq, dh)
    q, k, v, i = host(Q), host(K), host(V), idx.cpu().numpy()
    ref = np.empty((M, Hq, dh))
    for h in range(Hq):
        g = h // (Hq // Hkv)
        use = i if counts is None else i[:counts[g]]
        s = q[:, h] @ k[g, use].T / np.sqrt(dh)
        w = np.exp(s - s.max(1, keepdims=True))
        ref[:, h] = (w / w.sum(1, keepdims=True)) @ v[g, use]
    assert rel(got, ref) <= tol
