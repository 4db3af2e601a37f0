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
