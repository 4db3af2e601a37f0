"""The norm pass on its own: short rows (eight to a wave) and long ones with an incomplete last run,
numbers of rows that leave a part of a wave, equal rows, more candidates than the selection keeps in
LDS; and the scores' stores where four of them are not aligned."""
import numpy as np
import pytest
import torch

import paper_2502_11494_amd as D

pytestmark = pytest.mark.gpu
TYPES = {"bf16": (D.DART_BF16, torch.bfloat16), "f32": (D.DART_F32, torch.float32)}


def select(X, crit, code, B, n, P, cu=None):
    more = dict(N=n) if cu is None else dict(cu_seqlens=cu, total_N=X.shape[0], max_N=n)
    desc = D.make_desc(B, X.shape[1], P, code, K=0, keep_num=1, keep_den=1, **more)
    piv = torch.full((B * P,), -1, dtype=torch.int32, device="cuda")
    l1 = torch.full((X.shape[0],), float("nan"), device="cuda")
    kw = {} if crit is None else dict(crit=crit, crit_D=crit.shape[1], crit_ld=crit.stride(0))
    D.dart_select_pivots(desc, X, piv, D.alloc_workspace(desc), l1_out=l1, **kw)
    return piv.cpu().numpy().reshape(B, P), l1.cpu().numpy()


@pytest.mark.parametrize("dtype", ["bf16", "f32"])
@pytest.mark.parametrize("width", [8, 64, 248, 256, 264, 504, 512, 520, 1024, 3584, 4096, 4104, 8200])
@pytest.mark.parametrize("n", [5, 8, 33, 100])
@pytest.mark.parametrize("ragged", [False, True])
def test_norms_and_pivots(dtype, width, n, ragged):
    code, dt = TYPES[dtype]
    print(f"[case] {dtype} width={width} n={n} ragged={ragged}", flush=True)
    g = torch.Generator().manual_seed(width + n)
    C = torch.randn((2 * n, width + 8), generator=g).to(dt)[:, :width]  # (padded rows)
    C[n + 1] = C[n + 4]  # equal rows, in other places of a wave
    X = torch.randn((2 * n, 64), generator=g).to(dt)
    exact = C.double().abs().sum(1).numpy()
    Cd = torch.empty((2 * n, width + 8), dtype=dt, device="cuda")[:, :width]
    Cd.copy_(C)
    cu = torch.tensor([0, n, 2 * n], dtype=torch.int32, device="cuda") if ragged else None
    P = 4
    piv, l1 = select(X.cuda(), Cd, code, 2, n, P, cu)
    # fp64 sums rounded to fp32 once
    assert np.all(np.abs(l1 - exact) <= 2.0 ** -24 * exact * 1.001)
    for b in range(2):
        e = exact[b * n:(b + 1) * n]
        np.testing.assert_array_equal(piv[b], np.argsort(-e, kind="stable")[:P])


@pytest.mark.parametrize("dtype", ["bf16", "f32"])
@pytest.mark.parametrize("n,P", [(129, 3), (513, 5), (3000, 64)])
def test_more_candidates_than_lds_holds(dtype, n, P):
    code, dt = TYPES[dtype]
    X = torch.randn((1, 256), generator=torch.Generator().manual_seed(n)).to(dt).expand(n, 256).contiguous()
    piv, _ = select(X.cuda(), None, code, 1, n, P)
    np.testing.assert_array_equal(piv[0], np.arange(P))


@pytest.mark.parametrize("n", [64, 65, 66, 67, 200])
@pytest.mark.parametrize("P", [3, 16, 20])
def test_scores_stored_at_any_alignment(n, P):
    X = torch.randn((2 * n, 256), generator=torch.Generator().manual_seed(n + P)).bfloat16().cuda()
    desc = D.make_desc(2, 256, P, D.DART_BF16, N=n, K=P)
    piv = torch.arange(P, dtype=torch.int32, device="cuda").repeat(2)
    out = []
    for shift in range(4):
        S = torch.full((2 * n * P + 8,), -7.0, device="cuda")
        D.dart_duplication_scores(desc, X, piv, S[shift:], D.alloc_workspace(desc))
        got = S.cpu().numpy()
        assert np.all(got[:shift] == -7.0) and np.all(got[shift + 2 * n * P:] == -7.0)
        out.append(got[shift:shift + 2 * n * P])
    x = X.double().cpu().numpy().reshape(2, n, 256)
    x /= np.linalg.norm(x, axis=2, keepdims=True)
    exact = np.concatenate([(x[b][:P] @ x[b].T).reshape(-1) for b in range(2)])
    assert np.max(np.abs(out[0] - exact)) <= D.score_tolerance(D.DART_BF16)
    for o in out[1:]:
        np.testing.assert_array_equal(o.view(np.uint32), out[0].view(np.uint32))


@pytest.mark.parametrize("width", [32, 60, 128, 256])
def test_every_entry_ranks_by_the_same_sums(width):
    """fp32 rows that are permutations of one: their sums differ in the last bits of fp64 only, by the
    order of the additions, which is the same whether the samples are packed, spans or come with norms."""
    n, P = 400, 24
    print(f"[case] permuted rows of {width}", flush=True)
    g = torch.Generator().manual_seed(width)
    row = torch.randn(width, generator=g) * torch.exp2(torch.randint(-34, 4, (width,), generator=g).float())
    row[0] = 13.7
    C = torch.stack([row[torch.randperm(width, generator=g)] for _ in range(n)])
    assert len(set(C.double().abs().cumsum(1)[:, -1].tolist())) > 1  # (in whatever order)
    Cd, X = C.cuda(), torch.randn((n, 64), generator=g).cuda()
    kw = dict(crit=Cd, crit_D=width, crit_ld=width)
    zero = torch.zeros(1, dtype=torch.int32, device="cuda")
    cu = torch.tensor([0, n], dtype=torch.int32, device="cuda")
    packed, _ = select(X, Cd, D.DART_F32, 1, n, P)
    ragged, _ = select(X, Cd, D.DART_F32, 1, n, P, cu)
    desc = D.make_desc(1, 64, P, D.DART_F32, K=P, cu_seqlens=cu, total_N=n, max_N=n, span_start=zero, X_rows=n)
    spans = torch.full((P,), -1, dtype=torch.int32, device="cuda")
    D.dart_select_pivots(desc, X, spans, D.alloc_workspace(desc), **kw)
    desc = D.make_desc(1, 64, P, D.DART_F32, N=n, K=P)
    given = torch.full((P,), -1, dtype=torch.int32, device="cuda")
    D.dart_reduce_with_norms(desc, X, torch.empty((P, 64), device="cuda"),
                             torch.empty(P, dtype=torch.int32, device="cuda"), D.alloc_workspace(desc),
                             C.double().abs().sum(1).float().cuda(), 1e-6, piv_out=given, **kw)
    for other in (ragged[0], spans.cpu().numpy(), given.cpu().numpy()):
        np.testing.assert_array_equal(packed[0], other)
