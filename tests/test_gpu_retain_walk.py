"""The walk of the retained-set kernel at the edges of its variants: quotas on both sides of the run
lengths and of the switch to the walk of all waves, budgets that leave a remainder, lists that do
not fit the staging area, and lists whose heads earlier stages have taken (equal or nearly equal
rows of scores).  Without the hidden states the scores count as exact; with them the boundary of
every stage is decided on fp64 scores (second test)."""
import numpy as np
import pytest
import torch

import oracle
import paper_2502_11494_amd as D
from paper_2502_11494_amd import workloads as W

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("N,P,K", [
    (300, 8, 8), (300, 8, 9), (64, 64, 64), (130, 1, 129), (257, 3, 3 + 3 * 64 - 1),
    (1100, 16, 16 + 16 * 39 + 15), (1500, 16, 16 + 16 * 40), (2300, 16, 16 + 16 * 63),
    (2300, 16, 16 + 16 * 64), (4097, 32, 32 + 32 * 63 + 31), (9000, 33, 33 + 33 * 62),
    (16384, 64, 64 + 64 * 60), (16384, 64, 64 + 64 * 200), (16384, 2, 16000),
])
@pytest.mark.parametrize("kind", ["independent", "alike", "equal"])
def test_walk_against_the_oracle(N, P, K, kind):
    rng = np.random.default_rng(N + P + K)
    print(f"[case] N={N} P={P} K={K} {kind}", flush=True)
    if kind == "independent":
        S = rng.standard_normal((P, N)).astype(np.float32)
    elif kind == "alike":   # every stage begins with what the ones before it took
        S = (rng.standard_normal((1, N)) + 1e-3 * rng.standard_normal((P, N))).astype(np.float32)
    else:                   # the same list for every stage, with ties
        S = np.repeat(np.round(rng.standard_normal((1, N)), 2), P, axis=0).astype(np.float32)
    piv = rng.permutation(N)[:P].astype(np.int32)
    desc = D.make_desc(1, 64, P, D.DART_BF16, N=N, K=K)
    keep = torch.full((K,), -1, dtype=torch.int32, device="cuda")
    D.dart_topk_keep(desc, torch.from_numpy(S).cuda(), torch.from_numpy(piv).cuda(), keep,
                     D.alloc_workspace(desc))
    np.testing.assert_array_equal(keep.cpu().numpy(), oracle.retain(S, piv, K))


def alike_rows(rng, N, P, group, dtype):
    """Groups of nearly equal rows, the scores inside a group a few rounding bounds apart.  The P
    first rows (the pivots) come in two families: the lists inside a family are nearly the same, and
    what the last stage of one wrongly refuses the other does not pick up."""
    Dim = 256 if dtype == D.DART_F32 else 4096
    base = rng.standard_normal((N, Dim)).astype(np.float32)
    X = base[np.concatenate([N - 1 - np.arange(P) * 2 // P, rng.permutation(N - P) // group])]
    if dtype == D.DART_F32:
        return (X * (1 + 5e-6 * rng.standard_normal(X.shape))).astype(np.float32)
    X = (X.view(np.uint32) >> 16).astype(np.uint16)
    X[np.arange(N), rng.integers(0, Dim, N)] ^= 1  # the last bit of an element: 1e-6 each
    return X


BOUNDARIES = [  # (N, P, K, rows per group)
    (300, 1, 70, 40), (600, 8, 8 + 8 * 22, 40), (700, 8, 8 + 8 * 39 + 5, 40),
    (900, 8, 8 + 8 * 41, 50), (1200, 8, 8 + 8 * 63 + 1, 40), (1500, 8, 8 + 8 * 66, 40),
    (4096, 16, 16 + 16 * 30, 200), (4096, 32, 32 + 32 * 50, 60), (5000, 4, 4 + 4 * 300, 2500),
]


def boundary_case(N, P, K, group, dtype):
    """Scores that are wrong by almost as much as the kernel allows for: the order they give differs
    from the exact one where stages end."""
    rng = np.random.default_rng(N + P + K)
    X = alike_rows(rng, N, P, group, dtype)
    piv = np.arange(P, dtype=np.int32)
    exact = oracle.scores(X, W.F32 if dtype == D.DART_F32 else W.BF16, piv)
    tau = D.score_tolerance(dtype)
    S = (exact + 0.7 * tau * rng.uniform(-1, 1, exact.shape)).astype(np.float32)
    assert np.abs(S - exact).max() < tau
    want, _, _, gap = oracle.retain(exact, piv, K, diagnostics=True)
    assert gap[gap > 0].min() > 1e-12  # far above the rounding of an fp64 score (0: equal rows)
    return X, piv, S, want


@pytest.mark.parametrize("N,P,K,group", BOUNDARIES)
@pytest.mark.parametrize("dtype", [D.DART_F32, D.DART_BF16])
def test_boundaries_are_decided_in_fp64(N, P, K, group, dtype):
    """A boundary that is not looked at, or is searched from behind it, gives the set of the scores
    as they are.  Few candidates, more than a look of 64 entries, more than the queue's 1024."""
    print(f"[case] N={N} P={P} K={K} group={group} dtype={dtype}", flush=True)
    X, piv, S, want = boundary_case(N, P, K, group, dtype)
    assert not np.array_equal(want, oracle.retain(S, piv, K))
    Xd = torch.from_numpy(X if dtype == D.DART_F32 else X.view(np.int16))
    Xd = (Xd if dtype == D.DART_F32 else Xd.view(torch.bfloat16)).cuda()
    desc = D.make_desc(1, X.shape[1], P, dtype, N=N, K=K)
    keep = torch.full((K,), -1, dtype=torch.int32, device="cuda")
    D.dart_topk_keep(desc, torch.from_numpy(S).cuda(), torch.from_numpy(piv).cuda(), keep,
                     D.alloc_workspace(desc), X=Xd)
    np.testing.assert_array_equal(keep.cpu().numpy(), want)
