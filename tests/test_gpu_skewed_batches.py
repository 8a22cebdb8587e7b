"""Batches in which one row takes most references, and the time that they take next to ordinary batches."""
import statistics
import time

import numpy as np
import pytest
import torch

import oracle
import paper_2005_13789_amd as ne
from parity_util import rowwise_rel_err
from test_gpu_walks import make

pytestmark = pytest.mark.gpu
DEV = "cuda:0"


def alias_of(V, rng):
    deg = rng.integers(1, 9, V).astype(np.uint32)
    return ne.ne_build_neg_alias(deg, 0, torch.empty((V, 2), dtype=torch.int32, device=DEV)), oracle.build_alias(deg)[:2]


@pytest.mark.parametrize("side", ["source", "context"])
@pytest.mark.parametrize("B,share", [(700, 1.0), (20_000, 0.5), (66_000, 0.3), (66_000, 1.0)])
def test_one_row_takes_many_references(B, share, side):
    """Bar: the row's sum has up to 66 000 fp32 terms, (n / 32 + 40) 2^-24 of them where they agree in sign: 1.3e-4."""
    print(f"B={B} share={share} side={side}", flush=True)
    V, d, K, seed = 40_000, 16, 1, 3
    rng = np.random.default_rng(B)
    t = make(V, d, B, K, seed)
    alias, (thr, al) = alias_of(V, rng)
    pairs = rng.integers(0, V, (B, 2))
    pairs[rng.random(B) < share, 0 if side == "source" else 1] = 11
    pairs = pairs.astype(np.int32)
    X, C = t.vertex.cpu().numpy(), t.context.cpu().numpy()
    ne.ne_train_batch(t, alias, torch.from_numpy(pairs).to(DEV), K, 0.001, 0)
    oracle.train_batch(X, C, pairs, oracle.sample_negatives(seed, 0, B, K, thr, al, 0), 0.001)
    for name, got, want, hub in (("X", t.vertex, X, side == "source"), ("C", t.context, C, side == "context")):
        got = got.cpu().numpy()
        rest = np.arange(V) != 11
        e, eh = rowwise_rel_err(got[rest], want[rest]), rowwise_rel_err(got[11:12], want[11:12])
        print(f"  {name}: rows {e:.2e}, row 11 {eh:.2e}", flush=True)
        assert e <= 1e-5 and eh <= (1.3e-4 if hub else 1e-5)


def seconds(call, rounds=7, calls=20):
    """Time of a call: the median over some rounds of several calls each."""
    for _ in range(2):
        call()
    torch.cuda.synchronize()
    got = []
    for _ in range(rounds):
        t0 = time.perf_counter()
        for _ in range(calls):
            call()
        torch.cuda.synchronize()
        got.append((time.perf_counter() - t0) / calls)
    return statistics.median(got)


def time_of_batch(V, d, K, pairs):
    rng = np.random.default_rng(0)
    t = make(V, d, pairs.shape[0], K, 1)
    alias, _ = alias_of(V, rng) if K else (None, None)
    p = torch.from_numpy(pairs.astype(np.int32)).to(DEV)
    return seconds(lambda: ne.ne_train_batch(t, alias, p, K, 1e-6, 0))


def test_a_dominant_row_does_not_hold_the_batch_up():
    """65 536 pairs with one source row against as many with random ones (about 300 and 45 us; 900 while one lane wrote the
    row's 8192 work items)."""
    pairs = np.random.default_rng(2).integers(0, 500_000, (65_536, 2))
    plain = time_of_batch(500_000, 16, 0, pairs)
    pairs[:, 0] = 9
    star = time_of_batch(500_000, 16, 0, pairs)
    print(f"random sources {plain * 1e6:.1f} us, one source {star * 1e6:.1f} us", flush=True)
    assert star <= 12 * plain


@pytest.mark.parametrize("B,K", [(131_072, 5), (65_536, 10)])
def test_a_hub_does_not_hold_up_a_batch_of_long_tiles(B, K):
    """Beyond 524 288 references a claim tile is of several steps.  30 % of the pairs with one source row against random
    ones: 1.1 times as long (3 and 2 times while such a tile had an entry for each of the row's references)."""
    pairs = np.random.default_rng(4).integers(0, 4_000_000, (B, 2))
    plain = time_of_batch(4_000_000, 16, K, pairs)
    pairs[np.random.default_rng(5).random(B) < 0.3, 0] = 9
    star = time_of_batch(4_000_000, 16, K, pairs)
    print(f"random sources {plain * 1e6:.1f} us, 30 % of one {star * 1e6:.1f} us: {star / plain:.2f}", flush=True)
    assert star <= 1.5 * plain


def test_narrow_rows_with_many_negatives():
    """32 768 pairs with 62 negatives at dim 4 against dim 128, whose rows are 32 times as long: 0.55 of the time
    (0.74 while the apply kernel gave a row 64 lanes there, one for each reference of a pair)."""
    pairs = np.random.default_rng(3).integers(0, 1_000_000, (32_768, 2))
    narrow, wide = time_of_batch(1_000_000, 4, 62, pairs), time_of_batch(1_000_000, 128, 62, pairs)
    print(f"dim 4 {narrow * 1e6:.1f} us, dim 128 {wide * 1e6:.1f} us: {narrow / wide:.3f}", flush=True)
    assert narrow <= 0.65 * wide
