"""Precision of the shared-negative step's parts, on inputs for which the result is known exactly.

Coefficients: a coefficient is -neg_scale * sigmoid(score) in fp32, rounded to bf16.  For a score of -ln(n 2^-23), n < 2^19, the
fp32 sum 1 + exp(-score) is 1 + n 2^-23 whatever the last bits of the exponential are (its relative error of some 2^-22 moves n by
less than an eighth), so the sigmoid is the reciprocal of a known number.  A neg_scale for which the correctly rounded
reciprocal and its neighbour lie on either side of a tie between two bf16 values tells the two apart."""
import numpy as np
import pytest
import torch

import paper_2005_13789_amd as ne

pytestmark = pytest.mark.gpu
DEV = "cuda:0"
F = np.float32
TIE = F(2.0 - 2.0 ** -8)      # halfway between bf16's 1.9921875 and 2, to which it is rounded; products near it have an ulp of 2^-23


def scale_between(low, high):
    """fp32 neg_scale whose product with `low` is below the tie and with `high` is not, or None (a step of the sigmoid is 0.998
    ulp of the product)."""
    s = F(float(TIE) / float(high))
    for _ in range(4):
        s = np.nextafter(s, F(0))
    for _ in range(9):
        if F(s * low) < TIE <= F(s * high):
            return s
        s = np.nextafter(s, F(4))
    return None


def test_coefficients_use_a_correctly_rounded_reciprocal():
    d, N = 64, 128
    X = torch.zeros((2, d), dtype=torch.float32, device=DEV)
    C = torch.zeros((2, d), dtype=torch.float32, device=DEV)
    X[0, :4] = 1.0
    t = ne.ne_create_tables(X, C, 1, init=False)
    alias = ne.ne_build_neg_alias(np.array([1, 0], np.uint32), 0, torch.empty((2, 2), dtype=torch.int32, device=DEV))   # every negative is row 0
    ws = torch.empty(ne.ne_shared_workspace_bytes(d, 1, N), dtype=torch.uint8, device=DEV)
    pair = torch.tensor([[0, 1]], dtype=torch.int32, device=DEV)
    checked, wrong = 0, []
    for n in np.unique(np.geomspace(40, 2 ** 19 - 1, 500).astype(np.int64)):
        z = F(-np.log(float(n) * 2.0 ** -23))
        pieces, rest = [], z                       # the score as three bf16 values, each times 1
        for _ in range(3):
            p = torch.tensor(float(rest)).bfloat16().float().item()
            pieces.append(p)
            rest = F(rest - F(p))
        assert rest == 0
        sigma = F(1.0 / (1.0 + float(n) * 2.0 ** -23))
        for other, want in ((np.nextafter(sigma, F(0)), 2.0), (np.nextafter(sigma, F(2)), 1.9921875)):
            scale = scale_between(min(sigma, other), max(sigma, other))
            if scale is None:
                continue
            X.zero_(); C.zero_()
            X[0, :4] = 1.0
            C[0, 0], C[0, 2], C[0, 3] = pieces
            ne.ne_train_batch_shared(t, alias, pair, N, 1.0, float(scale), 0, ws)
            got = -C[0, 1].item() / N              # N equal deltas, small multiples of 2^-7: exact
            assert got in (2.0, 1.9921875), (n, got)
            checked += 1
            if got != want:
                wrong.append(int(n))
    print(f"{checked} checked, wrong {len(wrong)}", flush=True)
    assert checked >= 800
    assert not wrong, wrong[:10]


def test_coefficients_of_extreme_scores():
    """exp(200) is infinite in fp32: the sigmoid of -200 is 0 and not NaN, that of 200 is 1."""
    d, N = 64, 128
    for score, want in ((-200.0, 0.0), (200.0, 1.0), (0.0, 0.5)):
        X = torch.zeros((2, d), dtype=torch.float32, device=DEV)
        C = torch.zeros((2, d), dtype=torch.float32, device=DEV)
        X[0, :2] = 1.0
        C[0, 0] = score
        t = ne.ne_create_tables(X, C, 1, init=False)
        alias = ne.ne_build_neg_alias(np.array([1, 0], np.uint32), 0, torch.empty((2, 2), dtype=torch.int32, device=DEV))
        ws = torch.empty(ne.ne_shared_workspace_bytes(d, 1, N), dtype=torch.uint8, device=DEV)
        ne.ne_train_batch_shared(t, alias, torch.tensor([[0, 1]], dtype=torch.int32, device=DEV), N, 1.0, 1.0, 0, ws)
        assert C[0, 1].item() == -N * want, (score, C[0, 1].item())


@pytest.mark.parametrize("d", [64, 128, 256])
@pytest.mark.parametrize("B", [1024, 8192])
def test_every_sixteenth_of_a_batch_is_summed_by_itself(d, B):
    """All scores are 0, so every coefficient is -2^-8.  One eighth of the batch has sources of 1 in its first half and of 1/64 of the
    last place of that half's sum in its second, the rest of the batch sources of 0.  Added to the first half's sum, sixteen of the
    small ones are a quarter of its last place and lost; summed by themselves they reach it (B = 1024) or eight times that."""
    N, V, half = 128, 50_000, B // 16
    small = float(np.spacing(np.float32(half))) / 64
    want = -(2.0 ** -8) * (half + half * small)
    assert float(np.float32(want)) == want != -(2.0 ** -8) * half
    X = torch.zeros((V, d), dtype=torch.float32, device=DEV)
    C = torch.zeros((V, d), dtype=torch.float32, device=DEV)
    X[1, 0], X[2, 0] = 1.0, small
    t = ne.ne_create_tables(X, C, 2, init=False)
    alias = ne.ne_build_neg_alias(np.ones(V, np.uint32), 0, torch.empty((V, 2), dtype=torch.int32, device=DEV))
    ws = torch.empty(ne.ne_shared_workspace_bytes(d, B, N), dtype=torch.uint8, device=DEV)
    neg = torch.empty(N, dtype=torch.int32, device=DEV)
    pairs = torch.zeros((B, 2), dtype=torch.int32, device=DEV)
    pairs[10 * half:11 * half, 0] = 1
    pairs[11 * half:12 * half, 0] = 2
    ne.ne_train_batch_shared(t, alias, pairs, N, 1.0, 2.0 ** -7, 1, ws, neg)
    named = torch.bincount(neg.long(), minlength=V)
    named[0] = 0                     # the pairs' context row
    got = C[named == 1, 0]
    assert got.numel() > 100
    print(f"d={d} B={B}: {got.min().item()!r} .. {got.max().item()!r}, wanted {want!r}", flush=True)
    assert (got == want).all()
