"""Pivot selection at the edges of its candidate search: samples smaller and larger than the number of
groups, as many pivots as tokens, equal norms, a few norms far above the others, norms that overflow
fp32, both orders."""
import numpy as np
import pytest
import torch

import oracle
import paper_2502_11494_amd as D

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n,P", [(1, 1), (3, 3), (64, 64), (65, 64), (255, 16), (256, 64), (257, 1),
                                 (1023, 8), (1024, 64), (1025, 33), (4096, 16), (9217, 32),
                                 (16384, 64)])
@pytest.mark.parametrize("kind", ["spread", "equal", "heavy", "zero", "overflow"])
@pytest.mark.parametrize("mode", [D.DART_PIVOT_MAX_L1, D.DART_PIVOT_MIN_L1])
def test_pivots_against_the_oracle(n, P, kind, mode):
    rng = np.random.default_rng(n + P)
    X = rng.standard_normal((n, 8)).astype(np.float32)
    if kind == "equal":      # two values of the norm: the index decides
        X = np.sign(X) * np.where(rng.random((n, 1)) < 0.5, 1.0, 2.0)
    elif kind == "heavy":    # some far above, some far below
        X *= np.where(rng.random((n, 1)) < 0.05, 1e6, 1.0) * np.where(rng.random((n, 1)) < 0.05, 1e-6, 1.0)
    elif kind == "zero":
        X[rng.random(n) < 0.9] = 0.0
    elif kind == "overflow":  # norms beyond fp32's range: ranked in fp64 alone
        X *= np.where(rng.random((n, 1)) < 0.5, 3e37, 1.0)
        X = np.clip(X, -1e38, 1e38) * np.where(X > 0, 1.0, 3.0)
    X = X.astype(np.float32)
    desc = D.make_desc(1, 8, P, D.DART_F32, N=n, K=n, pivot_mode=mode)
    piv = torch.full((P,), -1, dtype=torch.int32, device="cuda")
    D.dart_select_pivots(desc, torch.from_numpy(X).cuda(), piv, D.alloc_workspace(desc))
    c = oracle.l1_norms(X, 0)
    want = np.argsort(c if mode == D.DART_PIVOT_MIN_L1 else -c, kind="stable")[:P]
    np.testing.assert_array_equal(piv.cpu().numpy(), want)


@pytest.mark.parametrize("N,P,K", [(700, 2, 699), (1024, 3, 1000), (1025, 4, 1000), (1500, 8, 1050),
                                   (2048, 2, 2047), (2049, 2, 2000), (3500, 3, 3000), (4096, 2, 4095),
                                   (4097, 2, 4000)])
@pytest.mark.parametrize("ties", [False, True])
def test_long_lists_in_order(N, P, K, ties):
    """Lists of nearly all tokens: the ordering kernel's counting sort at its capacity."""
    rng = np.random.default_rng(N)
    S = rng.standard_normal((P, N)).astype(np.float32)
    if ties:
        S = np.round(S, 1)
    piv = rng.permutation(N)[:P].astype(np.int32)
    desc = D.make_desc(1, 64, P, D.DART_BF16, N=N, K=K)
    keep = torch.full((K,), -1, dtype=torch.int32, device="cuda")
    D.dart_topk_keep(desc, torch.from_numpy(S).cuda(), torch.from_numpy(piv).cuda(), keep,
                     D.alloc_workspace(desc))
    np.testing.assert_array_equal(keep.cpu().numpy(), oracle.retain(S, piv, K))
