"""The stage lists against the oracle where their ordering takes another way: sizes around a workgroup's
threads, more entries wanted than threads, scores that crowd into a few buckets, equal scores."""
import numpy as np
import pytest
import torch

import oracle
import paper_2502_11494_amd as D

pytestmark = pytest.mark.gpu


def scores(kind, P, n, rng):
    S = 0.02 * rng.standard_normal((P, n))
    if kind == "outliers":       # most scores in a sliver of the range
        S[:, ::97] = 0.95 + 0.01 * rng.standard_normal(S[:, ::97].shape)
        S[:, 1::331] = -0.9
    elif kind == "narrow":       # a range of few representable numbers
        S = 0.75 + 1e-6 * rng.integers(0, 40, (P, n))
    elif kind == "levels":       # more equal scores than a bucket may hold
        S = rng.choice([-0.5, 0.0, -0.0, 0.25, 1.0], (P, n))
    elif kind == "equal":
        S[:] = 0.5
    return np.ascontiguousarray(S.astype(np.float32))


@pytest.mark.parametrize("kind", ["spread", "outliers", "narrow", "levels", "equal"])
@pytest.mark.parametrize("n,P,K", [(5, 2, 5), (63, 3, 20), (511, 4, 300), (512, 16, 60), (513, 8, 513),
                                   (1024, 5, 1024), (1025, 2, 700), (1500, 8, 1050), (2049, 3, 2048),
                                   (3100, 16, 400), (4500, 2, 1900), (16384, 4, 3000)])
def test_lists_against_the_oracle(n, P, K, kind):
    rng = np.random.default_rng(n * 7 + P)
    B = 2
    print(f"[case] n={n} P={P} K={K} {kind}", flush=True)
    S = [scores(kind, P, n, rng) for _ in range(B)]
    piv = np.stack([rng.permutation(n)[:P] for _ in range(B)]).astype(np.int32)
    desc = D.make_desc(B, 64, P, D.DART_F32, N=n, K=K)
    keep = torch.full((B * K,), -1, dtype=torch.int32, device="cuda")
    # no rows: the scores are taken as they are
    D.dart_topk_keep(desc, torch.from_numpy(np.concatenate([s.reshape(-1) for s in S])).cuda(),
                     torch.from_numpy(piv).cuda(), keep, D.alloc_workspace(desc), X=None)
    got = keep.cpu().numpy()
    for b in range(B):
        want = oracle.retain(S[b].astype(np.float64) + 0.0, piv[b], K)
        np.testing.assert_array_equal(got[b * K:(b + 1) * K], want, err_msg=f"sample {b}")


def crowd(kind, P, n, rng):
    S = 0.9 + 0.001 * rng.standard_normal((P, n))
    if kind == "low outliers":            # the rest in the top of the range
        S[:, ::200] = 0.0
    elif kind == "one low":
        S[:, 3] = -0.9
    elif kind == "both ends":
        S[:, ::200], S[:, 7::200] = 0.0, 0.99
    elif kind == "copies":                # a tenth equal, spread over the indices
        S[:, rng.permutation(n)[:n // 10]] = 0.8995
    elif kind == "eight groups":          # as many groups of equal scores as are ranked by bits
        S = 0.1 + 0.1 * rng.integers(0, 8, (P, n))
    elif kind == "nine groups":
        S = 0.1 + 0.05 * rng.integers(0, 9, (P, n))
    elif kind == "neighbours":            # two numbers that no bucket separates, below a spread
        S[:, ::3] = np.float32(0.25)
        S[:, 1::3] = np.nextafter(np.float32(0.25), np.float32(1.0))
        S[:, 2::3] = 0.25 + 1e-3 * rng.random(S[:, 2::3].shape)
    elif kind == "not finite":
        S[:, 2::50] = -np.inf
        S[:, ::40], S[:, 1::60] = np.nan, np.inf
    return np.ascontiguousarray(S.astype(np.float32))


def staged(S, piv, K):
    P = S.shape[0]
    kept = np.zeros(S.shape[1], bool)
    kept[piv] = True
    for i in range(P):
        take = (K - P) // P + (1 if i < (K - P) % P else 0)
        order = np.argsort(np.where(np.isnan(S[i]), np.inf, S[i]), kind="stable")
        kept[order[~kept[order]][:take]] = True
    return np.nonzero(kept)[0]


@pytest.mark.parametrize("kind", ["low outliers", "one low", "both ends", "copies", "eight groups",
                                  "nine groups", "neighbours", "not finite"])
@pytest.mark.parametrize("B,n,P,K", [(2, 300, 4, 60), (2, 1000, 8, 500), (1, 1500, 4, 1000), (20, 2880, 16, 320),
                                     (1, 4096, 8, 3000), (1, 9216, 32, 1024), (1, 16384, 4, 3000)])
def test_lists_of_crowded_scores(B, n, P, K, kind):
    """(B * P > 256 in one of them: several lists to a compute unit.)"""
    rng = np.random.default_rng(n + K)
    print(f"[case] B={B} n={n} P={P} K={K} {kind}", flush=True)
    S = [crowd(kind, P, n, rng) for _ in range(B)]
    piv = np.stack([rng.permutation(n)[:P] for _ in range(B)]).astype(np.int32)
    desc = D.make_desc(B, 64, P, D.DART_F32, N=n, K=K)
    keep = torch.full((B * K,), -1, dtype=torch.int32, device="cuda")
    D.dart_topk_keep(desc, torch.from_numpy(np.concatenate([s.reshape(-1) for s in S])).cuda(),
                     torch.from_numpy(piv).cuda(), keep, D.alloc_workspace(desc), X=None)
    got = keep.cpu().numpy()
    for b in range(B):
        np.testing.assert_array_equal(got[b * K:(b + 1) * K], staged(S[b], piv[b], K), err_msg=f"sample {b}")
