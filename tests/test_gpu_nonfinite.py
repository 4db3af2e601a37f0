"""Inputs that are not finite: results are unspecified, but nothing is written outside a sample's
part of the outputs, and the other samples' results are what they are without it."""
import dataclasses

import numpy as np
import pytest
import torch

import oracle
import paper_2502_11494_amd as D
from paper_2502_11494_amd import workloads as W

pytestmark = pytest.mark.gpu

GUARD = -77


def check_keep(keep, n, K, others):
    """keep: [B*K] of B samples and guard words; sample 0 is the one that is not finite."""
    assert np.all(keep[K * (1 + len(others)):] == GUARD)
    mine = keep[:K][keep[:K] != GUARD]  # (a slot may stay unwritten)
    assert np.all(mine[1:] > mine[:-1]) and np.all((mine >= 0) & (mine < n))
    for b, want in enumerate(others):
        np.testing.assert_array_equal(keep[K * (b + 1):K * (b + 2)], want)


@pytest.mark.parametrize("bad", [1, 2, 30])          # rows with an infinite element
@pytest.mark.parametrize("per_stage", [1, 2, 17])     # tokens a stage takes (34: all that are left)
@pytest.mark.parametrize("first", [False, True])      # such scores at a list's end, or at its head
@pytest.mark.parametrize("dtype", [D.DART_F32, D.DART_BF16])
def test_undefined_scores_keep_to_their_part(bad, per_stage, first, dtype):
    P, n, Dim = 2, 36, 64
    K = P + P * per_stage - (1 if per_stage == 17 else 0)
    rng = np.random.default_rng(bad * 100 + per_stage)
    print(f"[case] bad={bad} per_stage={per_stage} first={first} dtype={dtype}", flush=True)
    X = rng.standard_normal((2, n, Dim)).astype(np.float32)
    Xt = torch.from_numpy(X).to(torch.float32 if dtype == D.DART_F32 else torch.bfloat16)
    raw = [x.numpy() if dtype == D.DART_F32 else x.view(torch.int16).numpy().view(np.uint16)
           for x in Xt]
    piv = np.array([[0, 1], [0, 1]], dtype=np.int32)
    S = np.stack([oracle.scores(np.ascontiguousarray(r), W.F32 if dtype == D.DART_F32 else W.BF16, p)
                  for r, p in zip(raw, piv)])
    other = oracle.retain(S[1], piv[1], K)
    rows = 2 + rng.permutation(n - 2)[:bad]
    Xt[0, rows, 3] = float("inf")
    S = S.astype(np.float32)
    S[0][:, rows] = -np.float32(np.nan) if first else np.float32(np.nan)
    desc = D.make_desc(2, Dim, P, dtype, N=n, K=K)
    keep = torch.full((2 * K + 64,), GUARD, dtype=torch.int32, device="cuda")
    D.dart_topk_keep(desc, torch.from_numpy(S).cuda(), torch.from_numpy(piv).cuda(), keep,
                     D.alloc_workspace(desc), X=Xt.cuda())
    check_keep(keep.cpu().numpy(), n, K, [other])


@pytest.mark.parametrize("value", [float("inf"), float("nan")])
@pytest.mark.parametrize("bad,K", [(1, 12), (40, 60), (299, 12), (300, 299)])
@pytest.mark.parametrize("dtype", [D.DART_F32, D.DART_BF16])
def test_whole_step_keeps_to_its_part(value, bad, K, dtype):
    w = W.image_batch(seed=bad, B=3, N=300, D=256, P=4, K=K)
    if dtype == D.DART_F32:
        w = dataclasses.replace(w, X=W.bf16_bits_to_f32(w.X), dtype=W.F32)
    refs = [oracle.reduce(w.sample(b), w.dtype, w.P, K) for b in range(3)]
    print(f"[case] {value} bad={bad} K={K} dtype={dtype}", flush=True)
    X = torch.from_numpy(w.X if dtype == D.DART_F32 else w.X.view(np.int16))
    X = (X if dtype == D.DART_F32 else X.view(torch.bfloat16)).cuda()
    X[torch.from_numpy(np.random.default_rng(bad).permutation(300)[:bad]).cuda(), 5] = value
    desc = D.make_desc(3, w.D, w.P, dtype, N=300, K=K)
    keep = torch.full((3 * K + 64,), GUARD, dtype=torch.int32, device="cuda")
    Y = torch.full((3 * K + 4, w.D), 7, dtype=X.dtype, device="cuda")
    D.dart_reduce(desc, X, Y, keep, D.alloc_workspace(desc))
    check_keep(keep.cpu().numpy(), 300, K, [r.keep for r in refs[1:]])
    assert torch.all(Y[3 * K:] == 7)
