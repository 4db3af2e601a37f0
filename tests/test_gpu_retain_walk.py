"""The walk of the retained-set kernel at the edges of its variants: quotas on both sides of the run
lengths and of the switch to the walk of all waves, budgets that leave a remainder, lists that do
not fit the staging area, and lists whose heads earlier stages have taken (equal or nearly equal
rows of scores)."""
import numpy as np
import pytest
import torch

import oracle
import paper_2502_11494_amd as D

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
