"""Walks in which one node takes many entries, with holes: claim tiles with a hub whose absent references have no entry, by
segments and by entries, of one step (256 and 1024 references) and of several.

Bar: a row of n references is a sum of n + 1 fp32 terms, taken 8 at a time and 32 or more thereafter: n / 32 + 40 roundings of the
summed magnitudes; n stays below 200 000: sqrt(6250) * 2^-24 = 5e-6 expected, eight times that is 4e-5."""
import numpy as np
import pytest
import torch

import oracle
import paper_2005_13789_amd as ne
from parity_util import rowwise_rel_err
from test_gpu_walks import make, oracle_run

pytestmark = pytest.mark.gpu
DEV = "cuda:0"


@pytest.mark.parametrize("share", [0.03, 0.4])
@pytest.mark.parametrize("d,L,window,K", [(16, 64, 3, 5), (64, 64, 5, 2), (256, 13, 3, 5), (32, 9, 4, 5)])     # by segments; by entries
@pytest.mark.parametrize("refs", [6_000, 120_000, 700_000])
def test_walks_with_a_hub(d, L, window, K, refs, share):
    V, seed, lr = 3000, 12, 1e-3
    R = 1 + window * (K + 1)
    n = -(-refs // (L * R))
    print(f"d={d} L={L} window={window} K={K} walks={n} share={share}", flush=True)
    rng = np.random.default_rng(n + d)
    walks = rng.integers(0, V, (2 * n, L)).astype(np.int32)
    walks[rng.random((2 * n, L)) < share] = 5
    walks[rng.random((2 * n, L)) < 0.1] = -1
    deg = rng.integers(1, 9, V).astype(np.uint32)
    deg[77] = 3000
    t = make(V, d, -(-(n * L * R) // (K + 2)), K, seed)
    alias = ne.ne_build_neg_alias(deg, 0, torch.empty((V, 2), dtype=torch.int32, device=DEV))
    thr, al, _ = oracle.build_alias(deg)
    X, C = t.vertex.cpu().numpy(), t.context.cpu().numpy()
    ne.ne_train_walks(t, alias, torch.from_numpy(walks).to(DEV), n, window, K, [lr, lr], 40)
    torch.cuda.synchronize()
    oracle_run(X, C, walks, n, window, K, [lr, lr], seed, 40, thr, al)
    ex, ec = rowwise_rel_err(t.vertex.cpu().numpy(), X), rowwise_rel_err(t.context.cpu().numpy(), C)
    print(f"  row error X {ex:.2e} C {ec:.2e}", flush=True)
    assert ex <= 4e-5 and ec <= 4e-5
