"""The smallest batches: batches of one bin, whose two id phases share a launch, and the time that they take next to
larger ones."""
import numpy as np
import pytest
import torch

import oracle
import paper_2005_13789_amd as ne
from parity_util import rowwise_rel_err
from test_gpu_row_detection import step_and_check
from test_gpu_skewed_batches import alias_of, time_of_batch
from test_gpu_walks import make, oracle_run

pytestmark = pytest.mark.gpu
DEV = "cuda:0"


# seven references per pair: 36 pairs are one bin, 37 eight
@pytest.mark.parametrize("star", [0.0, 0.6, 1.0])
@pytest.mark.parametrize("batches", [1, 2, 3])
@pytest.mark.parametrize("B", [1, 9, 36, 37, 73, 147])
def test_small_batches(B, batches, star):
    print(f"B={B} batches={batches} star={star}", flush=True)
    V, K, seed = 700, 5, 8
    rng = np.random.default_rng(B + batches)
    t = make(V, 64, B, K, seed)
    alias, (thr, al) = alias_of(V, rng)
    pairs = rng.integers(0, V, (B * batches, 2))
    pairs[rng.random(B * batches) < star, 0] = 3
    step_and_check(t, alias, thr, al, pairs.astype(np.int32), K, seed, batches)


# references: 1 + window (K + 1) per entry, 200, 208 (one bin) and 416 by entries; 8 + 9 + 16 (K + 1) - 16 = 33 per segment
@pytest.mark.parametrize("wpb,L,window,K", [(1, 25, 1, 6), (2, 13, 1, 6), (4, 13, 1, 6), (4, 16, 2, 1), (9, 16, 2, 1)])
def test_small_batches_of_walks(wpb, L, window, K):
    print(f"walks per batch={wpb} L={L} window={window} K={K}", flush=True)
    V, d, seed = 300, 128, 5
    rng = np.random.default_rng(wpb + L)
    alias, (thr, al) = alias_of(V, rng)
    walks = rng.integers(0, V, (2 * wpb, L)).astype(np.int32)
    t = make(V, d, -(-(wpb * L * (1 + window * (K + 1))) // (K + 2)), K, seed)
    X, C = t.vertex.cpu().numpy(), t.context.cpu().numpy()
    ne.ne_train_walks(t, alias, torch.from_numpy(walks).to(DEV), wpb, window, K, [0.02, 0.01], 3)
    torch.cuda.synchronize()
    oracle_run(X, C, walks, wpb, window, K, [0.02, 0.01], seed, 3, thr, al)
    assert rowwise_rel_err(t.vertex.cpu().numpy(), X) <= 2e-5 and rowwise_rel_err(t.context.cpu().numpy(), C) <= 2e-5


def test_a_small_batch_does_not_take_longer_than_a_large_one():
    """64 pairs against 1024, which name 16 times the rows (17 and 22 us; 43 and 29 while a bin's references were taken
    eight at a time)."""
    pairs = np.random.default_rng(1).integers(0, 10_000, (1024, 2))
    small, large = time_of_batch(10_000, 128, 5, pairs[:64]), time_of_batch(10_000, 128, 5, pairs)
    print(f"64 pairs {small * 1e6:.1f} us, 1024 pairs {large * 1e6:.1f} us", flush=True)
    assert small <= 1.2 * large
