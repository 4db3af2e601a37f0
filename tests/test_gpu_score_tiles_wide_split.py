"""The score tile of eight wave groups (16 rows, an eighth of the chunks per group) against the oracle:
chosen for small batches, and forced on packed samples whose lengths leave partial tiles, with fewer
chunks than groups, a partial last chunk, and the token norms given or from the Gram products."""
import numpy as np
import pytest
import torch

import gpu_util as G
import paper_2502_11494_amd as D
from paper_2502_11494_amd import workloads as W

pytestmark = pytest.mark.gpu


def test_small_batches_take_the_tile():
    desc = D.make_desc(1, 4096, 8, D.DART_BF16, N=256, K=56)
    assert D.dart_score_tile_shape(desc) == (8, 8)


@pytest.mark.parametrize("P,Dh", [(8, 4096), (16, 1096), (3, 392), (16, 64)])
def test_eight_groups_give_the_oracles_result(P, Dh, monkeypatch):
    w = W.ragged_batch(seed=0x8C0 + P + Dh, B=4, D=Dh, P=P, keep_num=400, keep_den=1000,
                       lengths=[401, 64, 333, 17 * 3])
    refs = G.oracle_samples(w)
    crit = W.key_states(w, 256, seed=P)
    crit_dev = torch.from_numpy(crit.view(np.int16)).view(torch.bfloat16).cuda()
    refs_c = G.oracle_samples(w, crit=crit)
    monkeypatch.setenv("DART_SCORE_TILE", "8,8")
    G.compare(w, G.run_reduce(w), refs)                    # norms from the norm pass
    G.compare(w, G.run_reduce(w, crit=crit_dev), refs_c)   # norms from the Gram products
