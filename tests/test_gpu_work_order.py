"""Work items handed out longest first (per-head counts; a chunk's own prefix): every row
tile, key range and head is computed exactly once for head counts that are multiples of
the 8 XCDs, divisors of them and neither, against fp64 softmax attention.

Two-term P: 5e-5 of the result's norm, as the compressed pass's other tests."""
import numpy as np
import pytest
import torch

import paper_2609_39329_amd as pkv
from gpu_util import DEV, host, rel

pytestmark = pytest.mark.gpu


def normal(seed, *shape):
    g = torch.Generator().manual_seed(seed)
    return torch.randn(shape, generator=g).bfloat16().to(DEV)


def attend(q, k, v, own=None):
    s = q @ k.T / np.sqrt(q.shape[1])
    if own is not None:
        so = q @ own[0].T / np.sqrt(q.shape[1])
        so[np.triu_indices(len(q), 1)] = -np.inf
        s, v = np.concatenate([s, so], 1), np.concatenate([v, own[1]])
    w = np.exp(s - s.max(1, keepdims=True))
    return (w / w.sum(1, keepdims=True)) @ v


@pytest.mark.parametrize("Hq,Hkv,M", [(16, 16, 300), (8, 8, 513), (8, 4, 700), (6, 2, 200),
                                      (7, 7, 300), (12, 3, 150), (5, 1, 170)])
@pytest.mark.parametrize("counts", [False, True])
@pytest.mark.parametrize("own", [False, True])
def test_every_item_once(Hq, Hkv, M, counts, own):
    print(f"order Hq={Hq} Hkv={Hkv} M={M} counts={counts} own={own}", flush=True)
    dh, N, B = 64, 700, 333
    rng = np.random.default_rng(Hq + M)
    Q, K, V = normal(1, M, Hq, dh), normal(2, Hkv, N, dh), normal(3, Hkv, N, dh)
    Ks, Vs = normal(4, Hkv, M, dh), normal(5, Hkv, M, dh)
    idx = np.stack([rng.permutation(N)[:B] for _ in range(Hkv)]).astype(np.int32)
    cnt = rng.integers(1, B + 1, size=Hkv).astype(np.int32) if counts else np.full(Hkv, B, np.int32)
    kw = dict(idx=torch.from_numpy(idx).to(DEV), counts=torch.from_numpy(cnt).to(DEV) if counts else None)
    if own:
        got = pkv.attend_chunk(Q, K, V, Ks, Vs, p_terms=2, **kw)
    else:
        got = pkv.attend_compressed(Q, K, V, **kw)
    got = host(got).reshape(M, Hq, dh)
    q, k, v, ks, vs = (host(t) for t in (Q, K, V, Ks, Vs))
    for h in range(Hq):
        g = h // (Hq // Hkv)
        use = idx[g, :cnt[g]]
        ref = attend(q[:, h], k[g, use], v[g, use], (ks[g], vs[g]) if own else None)
        assert rel(got[:, h], ref) <= 5e-5, h


@pytest.mark.parametrize("Hq,Hkv,M,B", [(16, 16, 300, 20), (6, 3, 300, 30), (5, 1, 170, 9), (12, 12, 270, 25),
                                        (65, 65, 40, 20), (64, 64, 1100, 90)])
@pytest.mark.parametrize("counts", ["random", "equal", "one long"])
@pytest.mark.parametrize("own", [False, True])
def test_ranked_and_balanced_heads(Hq, Hkv, M, B, counts, own):
    """Per-head counts with one key range or more than one round of items (64 heads): heads
    ranked by the pre-pass, or runs of heads where their counts are balanced."""
    print(f"ranked Hq={Hq} Hkv={Hkv} M={M} counts={counts} own={own}", flush=True)
    dh, N = 64, 200
    rng = np.random.default_rng(Hq + M)
    Q, K, V = normal(1, M, Hq, dh), normal(2, Hkv, N, dh), normal(3, Hkv, N, dh)
    Ks, Vs = normal(4, Hkv, M, dh), normal(5, Hkv, M, dh)
    idx = np.stack([rng.permutation(N)[:B] for _ in range(Hkv)]).astype(np.int32)
    cnt = rng.integers(1, B + 1, size=Hkv).astype(np.int32)
    if counts != "random":
        cnt[:] = B if counts == "equal" else 1
        cnt[Hkv // 2] = B
    kw = dict(idx=torch.from_numpy(idx).to(DEV), counts=torch.from_numpy(cnt).to(DEV))
    if own:
        got = pkv.attend_chunk(Q, K, V, Ks, Vs, p_terms=2, **kw)
    else:
        got = pkv.attend_compressed(Q, K, V, **kw)
    got = host(got).reshape(M, Hq, dh)
    q, k, v, ks, vs = (host(t) for t in (Q, K, V, Ks, Vs))
    for h in range(Hq):
        g = h // (Hq // Hkv)
        use = idx[g, :cnt[g]]
        ref = attend(q[:, h], k[g, use], v[g, use], (ks[g], vs[g]) if own else None)
        assert rel(got[:, h], ref) <= 5e-5, h


def test_chunk_prefix_longer_than_the_cache():
    """A chunk whose own prefix is most of the work: whole own tiles below the diagonal run
    unmasked, the last ones masked; scores outgrowing the first tile at the diagonal."""
    M, dh, N = 1100, 128, 40
    Q, K, V = normal(1, M, 4, dh), normal(2, 1, N, dh), normal(3, 1, N, dh)
    Ks, Vs = normal(4, 1, M, dh), normal(5, 1, M, dh)
    for gain in (1.0, 12.0):
        k_own = (Ks.float() * gain).bfloat16()
        got = host(pkv.attend_chunk(Q, K, V, k_own, Vs, p_terms=2)).reshape(M, 4, dh)
        q, k, v, ks, vs = (host(t) for t in (Q, K, V, k_own, Vs))
        for h in range(4):
            assert rel(got[:, h], attend(q[:, h], k[0], v[0], (ks[0], vs[0]))) <= 5e-5, (gain, h)


@pytest.mark.parametrize("Hq,Hkv,M,N", [(8, 2, 1600, 3000), (2, 1, 2500, 1500), (4, 4, 700, 2000),
                                        (6, 3, 700, 2000), (4, 2, 270, 2600)])
def test_ranges_times_row_tiles_not_a_multiple_of_the_xcds(Hq, Hkv, M, N):
    """A chunk's (key range, row tile) pairs of a head dealt to its XCDs in one sequence that
    ends inside a round, ranges chosen with the own prefix counted (equal or longer than the
    cache's part)."""
    print(f"deal Hq={Hq} Hkv={Hkv} M={M} N={N}", flush=True)
    dh = 64
    Q, K, V = normal(1, M, Hq, dh), normal(2, Hkv, N, dh), normal(3, Hkv, N, dh)
    Ks, Vs = normal(4, Hkv, M, dh), normal(5, Hkv, M, dh)
    got = host(pkv.attend_chunk(Q, K, V, Ks, Vs, p_terms=2)).reshape(M, Hq, dh)
    q, k, v, ks, vs = (host(t) for t in (Q, K, V, Ks, Vs))
    for h in range(Hq):
        g = h // (Hq // Hkv)
        assert rel(got[:, h], attend(q[:, h], k[g], v[g], (ks[g], vs[g]))) <= 5e-5, h


@pytest.mark.parametrize("M", [1023, 1024, 1025])
@pytest.mark.parametrize("dh", [64, 128])
@pytest.mark.parametrize("dtype,tol", [(torch.bfloat16, 5e-5), (torch.float32, 1e-5)])
def test_merge_of_few_and_many_rows(M, dh, dtype, tol):
    """Split key ranges merged by a wave per row below 8,192 rows (M * Hq), by lane groups
    from there on. fp32: sums of 32 bits."""
    print(f"merge M={M} dh={dh} {dtype}", flush=True)
    Q, K, V = (normal(i, *s).to(dtype) for i, s in ((1, (M, 8, dh)), (2, (2, 900, dh)), (3, (2, 900, dh))))
    got = host(pkv.attend_compressed(Q, K, V)).reshape(M, 8, dh)
    q, k, v = (host(t) for t in (Q, K, V))
    for h in range(8):
        assert rel(got[:, h], attend(q[:, h], k[h // 4], v[h // 4])) <= tol, h
