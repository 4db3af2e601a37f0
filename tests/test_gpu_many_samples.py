"""Ragged batches of many small samples: the offsets are filled by a block of the norm pass (256
threads) or by a launch of its own (1024), and the sequence gather finds a row's sample by looks at
64 offsets; no tensors, and more tensors than one launch moves."""
import numpy as np
import pytest
import torch

import oracle
import paper_2502_11494_amd as D
from paper_2502_11494_amd import workloads as W


pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("B,n_tensors,spans", [(1, 1, True), (64, 0, True), (65, 9, True),
                                               (255, 2, False), (257, 1, True), (1030, 1, True),
                                               (1025, 0, False), (2048, 0, False),
                                               (2049, 0, False)])
def test_many_small_samples(B, n_tensors, spans):
    rng = np.random.default_rng(B)
    w = W.ragged_batch(seed=B, B=B, n_lo=5, n_hi=40, D=64, P=3, keep_num=400)
    w.X = np.ascontiguousarray(w.X)
    sq = W.sequences_around(w, seed=2, n_kv=max(n_tensors, 1), kv_width=16)
    print(f"[case] B={B} tensors={n_tensors} spans={spans}", flush=True)
    cu = torch.from_numpy(w.cu).cuda()
    span = torch.from_numpy(sq.span_start).cuda()
    more = dict(span_start=span, X_rows=sq.H.shape[0]) if spans else {}
    Xd = torch.from_numpy((sq.H if spans else w.X).view(np.int16)).view(torch.bfloat16).cuda()
    desc = D.make_desc(B, w.D, w.P, D.DART_BF16, keep_num=w.keep_num, keep_den=w.keep_den,
                       cu_seqlens=cu, total_N=int(w.cu[-1]), max_N=40, **more)
    ws = D.alloc_workspace(desc)
    refs = [oracle.reduce(w.sample(b), w.dtype, w.P, w.budget(b)) if w.budget(b) >= w.P else None
            for b in range(B)]  # (a sample whose budget is below its pivots is skipped)
    keeps = [r.keep if r is not None else np.zeros(0, np.int32) for r in refs]
    total = sum(len(k) for k in keeps)
    keep = torch.full((int(w.cu[-1]),), -1, dtype=torch.int32, device="cuda")
    cu_keep = torch.full((B + 1,), -1, dtype=torch.int32, device="cuda")
    D.dart_reduce(desc, Xd, None, keep, ws, cu_keep=cu_keep)
    skipped = any(r is None for r in refs)
    assert D.dart_device_status(desc, ws) == (D.DART_ERR_DEVICE if skipped else D.DART_OK)
    np.testing.assert_array_equal(keep.cpu().numpy()[:total], np.concatenate(keeps))
    np.testing.assert_array_equal(cu_keep.cpu().numpy(), np.cumsum([0] + [len(k) for k in keeps]))
    if not spans:
        return
    srcs = [torch.from_numpy(t.view(np.int16)).cuda() for t in sq.kv[:n_tensors]]
    row_map_ref, cu_ref = oracle.compact_sequences(sq.seq_cu, sq.span_start, w.lengths, keeps)
    rows = len(row_map_ref)
    dsts = [torch.zeros((rows, t.shape[1]), dtype=t.dtype, device="cuda") for t in srcs]
    row_map = torch.full((rows,), -7, dtype=torch.int32, device="cuda")
    seq_out = torch.full((B + 1,), -1, dtype=torch.int32, device="cuda")
    pos = torch.from_numpy(rng.integers(0, 1 << 40, size=(70, sq.H.shape[0]))).cuda()
    pos_out = torch.full((70, rows), -1, dtype=torch.int64, device="cuda")
    D.dart_compact_sequences(desc, torch.from_numpy(sq.seq_cu).cuda(), keep, list(zip(srcs, dsts)),
                             seq_out, row_map, ws, pos=pos, pos_out=pos_out)
    torch.cuda.synchronize()
    np.testing.assert_array_equal(seq_out.cpu().numpy(), cu_ref)
    np.testing.assert_array_equal(row_map.cpu().numpy(), row_map_ref)
    assert torch.equal(pos_out, pos[:, torch.from_numpy(row_map_ref.astype(np.int64)).cuda()])
    for src, dst in zip(srcs, dsts):
        assert torch.equal(dst, src[torch.from_numpy(row_map_ref.astype(np.int64)).cuda()])


@pytest.mark.parametrize("B,elements,n_hi", [
    (70, 8, 30), (130, 512, 12), (4097, 512, 3), (70000, 8, 2),    # several rows per wave
    (65, 1024, 9), (300, 1024, 3), (64, 520, 40),                  # rows of up to 2 KiB
    (257, 1032, 5), (1, 3000, 50), (64, 2048, 1),                  # a row per wave
    (384, 520, 4), (385, 520, 4), (9000, 1032, 2),                 # the map from a launch of its own
])
def test_sequences_of_few_rows(B, elements, n_hi):
    """Rows of a wave in several sequences, empty sequences (more than 64 in a row), samples that keep
    nothing, one to three looks at the offsets."""
    rng = np.random.default_rng(B + elements)
    print(f"[case] B={B} elements={elements} n_hi={n_hi}", flush=True)
    lens = rng.integers(0, n_hi + 1, B)
    before, after = rng.integers(0, 3, B), rng.integers(0, 3, B)
    gone = rng.integers(0, max(B - 100, 1)) + np.arange(min(100, B // 2))
    lens[gone] = before[gone] = after[gone] = 0
    cu = np.concatenate([[0], np.cumsum(lens)]).astype(np.int32)
    seq = np.concatenate([[0], np.cumsum(before + lens + after)]).astype(np.int32)
    span = (seq[:-1] + before).astype(np.int32)
    keeps = [np.sort(rng.permutation(n)[:n * 2 // 3]).astype(np.int32) for n in lens]  # none of one
    map_ref, cu_ref = oracle.compact_sequences(seq, span, lens, keeps)
    desc = D.make_desc(B, 8, 1, D.DART_BF16, keep_num=2, keep_den=3,
                       cu_seqlens=torch.from_numpy(cu).cuda(), total_N=int(cu[-1]), max_N=n_hi,
                       span_start=torch.from_numpy(span).cuda(), X_rows=int(seq[-1]))
    src = torch.randint(-30000, 30000, (int(seq[-1]), elements), dtype=torch.int16, device="cuda")
    dst = torch.full((len(map_ref) + 3, elements), 7, dtype=torch.int16, device="cuda")
    row_map = torch.full((len(map_ref) + 3,), -7, dtype=torch.int32, device="cuda")
    seq_out = torch.full((B + 1,), -1, dtype=torch.int32, device="cuda")
    pos = torch.arange(2 * int(seq[-1]), device="cuda").reshape(2, -1)
    pos_out = torch.full((2, len(map_ref) + 3), -1, dtype=torch.int64, device="cuda")
    D.dart_compact_sequences(desc, torch.from_numpy(seq).cuda(),
                             torch.from_numpy(np.concatenate(keeps + [np.zeros(1, np.int32)])).cuda(),
                             [(src, dst)], seq_out, row_map, D.alloc_workspace(desc), pos=pos,
                             pos_out=pos_out)
    np.testing.assert_array_equal(seq_out.cpu().numpy(), cu_ref)
    np.testing.assert_array_equal(row_map.cpu().numpy(), np.append(map_ref, [-7] * 3))
    rows = torch.from_numpy(map_ref.astype(np.int64)).cuda()
    assert torch.equal(dst[:-3], src[rows]) and torch.all(dst[-3:] == 7)
    assert torch.equal(pos_out[:, :-3], pos[:, rows]) and torch.all(pos_out[:, -3:] == -1)
