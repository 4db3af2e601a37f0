"""Pivot selection of more samples than there are compute units (two workgroups to a unit) against the
exact norms, beside the same samples in a call of fewer."""
import numpy as np
import pytest
import torch

import paper_2502_11494_amd as D

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("dtype", [D.DART_BF16, D.DART_F32])
@pytest.mark.parametrize("n", [20, 1100, 4096])
def test_pivots_of_many_samples(n, dtype):
    B, P, Dim = 300, 5, 64
    print(f"[case] {B} samples of {n}, dtype {dtype}", flush=True)
    g = torch.Generator(device="cuda").manual_seed(n)
    X = torch.randn((B * n, Dim), generator=g, device="cuda")
    X = X.bfloat16() if dtype == D.DART_BF16 else X
    X[n + 3:2 * n:7] = X[n + 3]  # equal rows: the lowest index first

    def select(samples):
        desc = D.make_desc(samples, Dim, P, dtype, N=n, K=P)
        piv = torch.full((samples * P,), -1, dtype=torch.int32, device="cuda")
        keep = torch.empty(samples * P, dtype=torch.int32, device="cuda")
        S = torch.empty(samples * P * n, device="cuda")
        D.dart_reduce(desc, X[:samples * n], torch.empty((samples * P, Dim), dtype=X.dtype, device="cuda"),
                      keep, D.alloc_workspace(desc), piv_out=piv, S_out=S)
        return piv.cpu().numpy().reshape(samples, P), S

    piv, S = select(B)
    fewer, S_fewer = select(8)
    np.testing.assert_array_equal(piv[:8], fewer)
    # the pivots' norms too: a score's bound is the only difference another tile may make
    tau = D.score_tolerance(dtype)
    assert float((S[:8 * P * n] - S_fewer).abs().max()) <= 2 * tau
    l1 = X.double().abs().sum(1).cpu().numpy().reshape(B, n)
    for b in range(B):
        np.testing.assert_array_equal(piv[b], np.argsort(-l1[b], kind="stable")[:P])
