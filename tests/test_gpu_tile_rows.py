"""Rows that many references of one claim tile name: the tile then makes one entry of all its references to a row, unless
they lose their slots to other rows, and several entries of one bin, tagged and untagged tiles side by side, share a row's places.

Three references per pair (K = 1).  2730 pairs are 8190 references in 32 tiles of 256, 21 840 pairs 65 520 references in
64 tiles of 1024, 130 000 pairs 390 000 references in 191 tiles of 2048, 200 000 pairs 600 000 references in 147 tiles of 4096, which
are of several steps.  A tile counts as one with many at 4 references of a bin per one of the mean + 2, or 2048 / tiles, or, of several
steps, 3 / 512 of the tile.

Bar: a row of n references is a sum of n + 1 fp32 terms, taken 8 at a time and 32 or more thereafter: n / 32 + 40 roundings of the
summed magnitudes, which stay near the row's (lr 1e-3, scores near 0), 40 of them 2.4e-6; n <= 200 000 references give
6250 * 2^-24 = 3.7e-4 at worst, sqrt(6250) * 2^-24 = 5e-6 as expected; 4e-5 is eight times that."""
import numpy as np
import pytest
import torch

import oracle
import paper_2005_13789_amd as ne
from parity_util import rowwise_rel_err
from test_gpu_walks import make

pytestmark = pytest.mark.gpu
DEV = "cuda:0"


@pytest.mark.parametrize("share", [0.004, 0.02, 0.3, 1.0])
@pytest.mark.parametrize("B", [2730, 21_840, 130_000, 200_000])
def test_rows_of_many_references_per_tile(B, share):
    print(f"B={B} share={share}", flush=True)
    V, d, K, seed, lr = 60_000, 8, 1, 21, 1e-3
    rng = np.random.default_rng(B)
    t = make(V, d, B, K, seed)
    deg = rng.integers(1, 9, V).astype(np.uint32)
    deg[77] = 60_000                                # a hub among the negatives, too
    alias = ne.ne_build_neg_alias(deg, 0, torch.empty((V, 2), dtype=torch.int32, device=DEV))
    thr, al, _ = oracle.build_alias(deg)
    pairs = rng.integers(0, V, (2 * B, 2))
    pairs[rng.random(2 * B) < share, 0] = 5
    pairs[rng.random(2 * B) < share / 2, 1] = 77
    pairs = pairs.astype(np.int32)
    X, C = t.vertex.cpu().numpy(), t.context.cpu().numpy()
    neg_out = torch.empty((2 * B, K), dtype=torch.int32, device=DEV)
    ne.ne_train_block(t, alias, torch.from_numpy(pairs).to(DEV), B, K, [lr, lr], 0, neg_out)
    torch.cuda.synchronize()
    neg = oracle.sample_negatives(seed, 0, 2 * B, K, thr, al, 0)
    assert np.array_equal(neg_out.cpu().numpy(), neg)
    for lo in (0, B):
        oracle.train_batch(X, C, pairs[lo:lo + B], np.ascontiguousarray(neg[lo:lo + B]), lr)
    ex, ec = rowwise_rel_err(t.vertex.cpu().numpy(), X), rowwise_rel_err(t.context.cpu().numpy(), C)
    print(f"  row error X {ex:.2e} C {ec:.2e}", flush=True)
    assert ex <= 4e-5 and ec <= 4e-5


@pytest.mark.parametrize("V,share", [(60_000, 0.02), (60_000, 0.3), (600, 0.0), (3, 0.0)])
@pytest.mark.parametrize("B,K", [(120_000, 5), (25_000, 62), (40_000, 62), (80_000, 62), (160_000, 62)])
def test_rows_of_many_references_in_long_tiles(B, K, V, share):
    """Tiles of 4096, 8192, 16 384 (with 4096 and 8192 bins) and 32 768 references.  600 nodes: more rows in bins with many than
    the tile's table of 512 takes; 3: a few rows take everything.  Up to 160 000 * 64 / 3 = 3.4 M references to a row: bar 4e-5 up to
    200 000 as above, sqrt(3.4 M / 32) * 2^-24 = 2e-5 expected and eight times that otherwise."""
    print(f"B={B} K={K} V={V} share={share}", flush=True)
    d, seed, lr = 8, 22, 1e-4
    rng = np.random.default_rng(B + V)
    t = make(V, d, B, K, seed)
    deg = rng.integers(1, 9, V).astype(np.uint32)
    if share:
        deg[77] = 20_000
    alias = ne.ne_build_neg_alias(deg, 0, torch.empty((V, 2), dtype=torch.int32, device=DEV))
    thr, al, _ = oracle.build_alias(deg)
    pairs = rng.integers(0, V, (2 * B, 2))
    pairs[rng.random(2 * B) < share, 0] = 5
    pairs = pairs.astype(np.int32)
    X, C = t.vertex.cpu().numpy(), t.context.cpu().numpy()
    neg_out = torch.empty((2 * B, K), dtype=torch.int32, device=DEV)
    ne.ne_train_block(t, alias, torch.from_numpy(pairs).to(DEV), B, K, [lr, lr], 0, neg_out)
    torch.cuda.synchronize()
    neg = oracle.sample_negatives(seed, 0, 2 * B, K, thr, al, 0)
    assert np.array_equal(neg_out.cpu().numpy(), neg)
    for lo in (0, B):
        oracle.train_batch(X, C, pairs[lo:lo + B], np.ascontiguousarray(neg[lo:lo + B]), lr)
    ex, ec = rowwise_rel_err(t.vertex.cpu().numpy(), X), rowwise_rel_err(t.context.cpu().numpy(), C)
    print(f"  row error X {ex:.2e} C {ec:.2e}", flush=True)
    bar = 4e-5 if V > 600 else 1.6e-4
    assert ex <= bar and ec <= bar
