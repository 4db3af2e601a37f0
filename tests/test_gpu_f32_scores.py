"""The fp32 score kernels at the edges of their tiles: every kernel and tile height the host can
choose, every number of pivot blocks, rows whose pieces end inside a step, samples that end inside a
tile."""
import numpy as np
import pytest
import torch

import oracle
import paper_2502_11494_amd as D

pytestmark = pytest.mark.gpu

# (lengths, D, P)
CASES = [
    ([1], 4, 1), ([5], 36, 5), ([70], 128, 8), ([67, 3, 258], 1028, 3),        # tiles of 4 rows, 4 pivots
    ([40], 64, 9), ([130], 260, 17), ([1029], 4, 1),
    ([200, 201], 100, 16), ([603], 2052, 8), ([333], 68, 23), ([90], 2052, 64),  # 4 rows, 8 pivots
    ([900], 100, 14), ([901, 2], 1028, 16),                                    # 4 rows, 16 pivots
    ([1100], 36, 8), ([513, 800], 132, 16),                                    # 16 rows
    ([5776], 68, 16), ([700, 2050, 1999, 700], 96, 32), ([5001], 36, 33),      # taller tiles
    ([4500, 33], 40, 48), ([1500], 160, 64),
    ([515, 2, 704], 4100, 5), ([1301], 3076, 8), ([700], 6148, 23), ([33], 8196, 3),  # vector ALU
]


@pytest.mark.parametrize("lengths,Dim,P", CASES)
@pytest.mark.parametrize("pad", [0, 8])
def test_scores_against_the_oracle(lengths, Dim, P, pad):
    rng = np.random.default_rng(sum(lengths) + Dim)
    cu = np.concatenate([[0], np.cumsum(lengths)]).astype(np.int32)
    total, ld = int(cu[-1]), Dim + pad
    X = np.full((total, ld), np.nan, dtype=np.float32)  # whatever lies past a row's end is not used
    X[:, :Dim] = rng.standard_normal((total, Dim)).astype(np.float32)
    X[total // 2, :Dim] = 0.0                           # a zero row scores 0
    piv = np.stack([rng.choice(n, P, replace=n < P) for n in lengths]).astype(np.int32)
    print(f"[case] {lengths} D={Dim} P={P} ld={ld}", flush=True)
    cu_dev = torch.from_numpy(cu).cuda()
    desc = D.make_desc(len(lengths), Dim, P, D.DART_F32, keep_num=1, keep_den=1,
                       cu_seqlens=cu_dev, total_N=total, max_N=max(lengths), ld=ld,
                       pivot_mode=D.DART_PIVOT_MAX_L1)
    Xd = torch.from_numpy(X).cuda()
    S = torch.full((P * total,), -7.0, dtype=torch.float32, device="cuda")
    D.dart_duplication_scores(desc, Xd, torch.from_numpy(piv).cuda(), S, D.alloc_workspace(desc))
    got = S.cpu().numpy().astype(np.float64)
    tau = D.score_tolerance(D.DART_F32)
    for b, n in enumerate(lengths):
        if n < P:  # fewer tokens than pivots: the sample is skipped
            assert np.all(got[P * cu[b]:P * cu[b + 1]] == -7.0)
            continue
        ref = oracle.scores(np.ascontiguousarray(X[cu[b]:cu[b + 1], :Dim]), 0, piv[b])
        err = np.abs(got[P * cu[b]:P * cu[b + 1]].reshape(P, n) - ref)
        assert err.max() <= tau
