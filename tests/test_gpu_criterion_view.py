"""A criterion that begins where the hidden states do but is another matrix: the first columns of
every row, or every other row.  The pivots are those of the criterion, everything else is the hidden
states'."""
import numpy as np
import pytest
import torch

import oracle
import paper_2502_11494_amd as D
from paper_2502_11494_amd import workloads as W

import gpu_util as G

pytestmark = pytest.mark.gpu


def check(w, Xd, crit, crit_bits, how, monkeypatch, score_mode=D.DART_SCORE_PER_PIVOT):
    kw = {}
    if how == "norms":
        l1 = np.abs(crit_bits if w.dtype == W.F32 else W.bf16_bits_to_f32(crit_bits)).astype(np.float64).sum(1)
        kw = dict(norms=(l1.astype(np.float32), 0.0))
    if how == "one launch":
        monkeypatch.setenv("DART_FUSED", "1")
    assert crit.data_ptr() == Xd.data_ptr()
    got = G.run_reduce(w, Xd=Xd, crit=crit, **kw)
    G.compare(w, got, G.oracle_samples(w, crit=crit_bits))


@pytest.mark.parametrize("how", ["plain", "norms", "one launch"])
@pytest.mark.parametrize("make", [
    lambda: W.image_batch(B=2, N=333, D=520, P=5, K=64, n_centroids=32),
    lambda: W.single_image(N=300, D=512, P=8, K=50, n_centroids=16),
    lambda: W.ragged_batch(B=3, n_lo=200, n_hi=700, D=512, P=16),
], ids=["bf16", "f32", "ragged"])
def test_first_columns(make, how, monkeypatch):
    w = make()
    width = w.D // 2 // 8 * 8
    print(f"[case] first {width} of {w.D} columns, {how}", flush=True)
    Xd = G.to_device(w)
    check(w, Xd, Xd[:, :width], np.ascontiguousarray(w.X[:, :width]), how, monkeypatch)


@pytest.mark.parametrize("how", ["plain", "norms", "one launch"])
@pytest.mark.parametrize("dtype", ["bf16", "f32"])
def test_every_other_row(dtype, how, monkeypatch):
    make = W.image_batch if dtype == "bf16" else W.single_image
    big = make(N=600, D=256, P=6, K=60, n_centroids=32, **(dict(B=1) if dtype == "bf16" else {}))
    w = make(N=300, D=256, P=6, K=60, n_centroids=32, **(dict(B=1) if dtype == "bf16" else {}))
    w.X[:] = big.X[:300]
    print(f"[case] rows 0, 2, 4, ... of twice the rows, {dtype}, {how}", flush=True)
    Xd = G.to_device(big)
    check(w, Xd[:300], Xd[::2], np.ascontiguousarray(big.X[::2]), how, monkeypatch)
