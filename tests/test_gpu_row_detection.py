"""Detection of rows that several references of a batch name, at the sizes where its parts change: one and several
claim tiles, the smallest and the next numbers of bins, both sizes of a bin's table, and a bin whose rows do not
fit its table (all ids of the batch hash into two bins).  Every row is checked against the oracle.

Bar: a row that n references name is a sum of n + 1 fp32 terms formed by fp32 dot products and an exponential;
n stays below 300 and the products near 1, so 1e-5 of the row's largest element leaves a factor of ten over
sqrt(n) * 2^-24 plus the dot products' own error."""
import numpy as np
import pytest
import torch

import oracle
import paper_2005_13789_amd as ne
from parity_util import rowwise_rel_err
from test_gpu_walks import make

pytestmark = pytest.mark.gpu
DEV = "cuda:0"


def step_and_check(t, alias, thr, al, pairs, K, seed, batches, lr=0.02):
    """The pairs in `batches` batches through ne_train_block, against the oracle batch by batch."""
    n = pairs.shape[0]
    B = -(-n // batches)
    lrs = [lr] * (-(-n // B))
    X, C = t.vertex.cpu().numpy(), t.context.cpu().numpy()
    X0, C0 = X.copy(), C.copy()
    ne.ne_train_block(t, alias, torch.from_numpy(pairs).to(DEV), B, K, lrs, 0)
    torch.cuda.synchronize()
    neg = oracle.sample_negatives(seed, 0, n, K, thr, al, 0) if K else np.zeros((n, 0), np.int32)
    for lo in range(0, n, B):
        oracle.train_batch(X, C, np.ascontiguousarray(pairs[lo:lo + B]), np.ascontiguousarray(neg[lo:lo + B]), lr)
    named_x, named_c = np.unique(pairs[:, 0]), np.unique(np.concatenate([pairs[:, 1], neg.reshape(-1)]))
    Xg, Cg = t.vertex.cpu().numpy(), t.context.cpu().numpy()
    ex, ec = rowwise_rel_err(Xg[named_x], X[named_x]), rowwise_rel_err(Cg[named_c], C[named_c])
    print(f"  row error X {ex:.2e} C {ec:.2e}", flush=True)
    assert ex <= 1e-5 * batches and ec <= 1e-5 * batches
    rest_x, rest_c = np.ones(X.shape[0], bool), np.ones(X.shape[0], bool)
    rest_x[named_x] = False
    rest_c[named_c] = False
    assert np.array_equal(Xg[rest_x].view(np.uint32), X0[rest_x].view(np.uint32))
    assert np.array_equal(Cg[rest_c].view(np.uint32), C0[rest_c].view(np.uint32))


# three references per pair; up to 256 are one bin, then 64, 128 and 256 each up to 32, 64 and 256 bins (2048, 8192 and
# 65 536 references); 1024 references fill a tile, from 262 144 references on the number of bins follows 1024 references each
@pytest.mark.parametrize("B", [1, 2, 85, 86, 170, 171, 341, 342, 682, 683, 1366, 2730, 2731, 21845, 21846, 87381, 87382])
def test_tiles_and_bins(B):
    print(f"B={B}", flush=True)
    V, d, K, seed = 60_000, 8, 1, 11
    rng = np.random.default_rng(B)
    t = make(V, d, B, K, seed)
    deg = rng.integers(1, 9, V).astype(np.uint32)
    alias = ne.ne_build_neg_alias(deg, 0, torch.empty((V, 2), dtype=torch.int32, device=DEV))
    thr, al, _ = oracle.build_alias(deg)
    # a few rows named many times, the rest once or a few times
    pairs = rng.integers(0, V, (3 * B, 2))
    pairs[rng.random(3 * B) < 0.002, 0] = 5
    pairs[rng.random(3 * B) < 0.002, 1] = 7
    step_and_check(t, alias, thr, al, pairs.astype(np.int32), K, seed, 3)


@pytest.mark.parametrize("distinct,more", [(250, 1), (260, 1), (600, 1), (635, 3), (645, 3), (4000, 1)])
def test_rows_of_one_bin_beyond_its_table(distinct, more):
    """All source rows share the top 10 bits of the hash, and so do all context rows: two bins hold everything.
    The tables take 255 distinct rows up to 8192 references, 640 with more: just below, just above, and many times
    as many; each row is named once, twice, 8, 9 or 17 times, or 3 times as often."""
    print(f"distinct={distinct} more={more}", flush=True)
    V, d, seed = 8_000_000, 4, 12
    ids = np.arange(V, dtype=np.uint64)
    same = ids[((ids * 0x9E3779B1) & 0xFFFFFFFF) >> 22 == 321][:distinct]
    assert same.size == distinct
    times = np.array([1, 2, 1, 8, 1, 9, 1, 17])[np.arange(distinct) % 8] * more
    rng = np.random.default_rng(distinct)
    src = rng.permutation(np.repeat(same, times))
    ctx = rng.permutation(np.repeat(same, times))
    pairs = np.stack([src, ctx], axis=1).astype(np.int32)
    t = make(V, d, pairs.shape[0], 0, seed)
    step_and_check(t, None, None, None, pairs, 0, seed, 1)

