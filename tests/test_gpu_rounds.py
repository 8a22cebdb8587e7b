"""Kernels that go through their work in rounds, at the edges of a round: the walk kernel's rows in flight (6, or 16
in small batches), the loss kernel's stride over the pairs, the shared-negative kernels' alternating LDS buffers."""
import numpy as np
import pytest
import torch

import oracle
import paper_2005_13789_amd as ne
from parity_util import rowwise_rel_err
from test_gpu_walks import make, oracle_run

pytestmark = pytest.mark.gpu
DEV = "cuda:0"


@pytest.mark.parametrize("n_walks", [3, 80])      # 42 and 1120 entries, 4 per workgroup: below and above 256 workgroups
@pytest.mark.parametrize("window,K", [(1, 0), (5, 0), (3, 1), (1, 6), (3, 4), (4, 3), (1, 16), (4, 7), (3, 10)])
def test_walk_rows_in_flight(n_walks, window, K):
    """window * (K + 1) rows per entry: 1, 5, 6, 7, 15, 16, 17, 32 and 33.  Bar: fp32 sums of at most a few hundred
    terms per row, 1e-5 of its largest element (as elsewhere for one batch)."""
    print(f"walks n={n_walks} window={window} K={K}", flush=True)
    V, d, L, seed = 4000, 256, 14, 9
    rng = np.random.default_rng(n_walks + window + K)
    deg = rng.integers(1, 9, V).astype(np.uint32)
    walks = rng.integers(0, V, (n_walks, L)).astype(np.int32)
    walks[0, 9:] = -1
    walks[1, 4] = -1
    R = 1 + window * (K + 1)
    t = make(V, d, -(-(n_walks * L * R) // (K + 2)), K, seed)
    alias = ne.ne_build_neg_alias(deg, 0, torch.empty((V, 2), dtype=torch.int32, device=DEV))
    thr, al, _ = oracle.build_alias(deg)
    X, C = t.vertex.cpu().numpy(), t.context.cpu().numpy()
    ne.ne_train_walks(t, alias, torch.from_numpy(walks).to(DEV), n_walks, window, K, [0.02], 40)
    torch.cuda.synchronize()
    oracle_run(X, C, walks, n_walks, window, K, [0.02], seed, 40, thr, al)
    ex, ec = rowwise_rel_err(t.vertex.cpu().numpy(), X), rowwise_rel_err(t.context.cpu().numpy(), C)
    print(f"  row error X {ex:.2e} C {ec:.2e}", flush=True)
    assert ex <= 1e-5 and ec <= 1e-5


@pytest.mark.parametrize("B", [1, 6143, 6144, 6145, 20_000])     # 768 workgroups of 8 pairs: one round, and more
@pytest.mark.parametrize("K", [0, 2, 5])
def test_loss_rounds(B, K):
    """fp32 terms summed in 64 bits: 2^-22 per term, far inside 1e-6 of the sum."""
    print(f"loss B={B} K={K}", flush=True)
    V, d, seed = 5000, 128, 4
    rng = np.random.default_rng(B + K)
    t = make(V, d, 1, K, seed)
    t.context.normal_(0, 0.3)
    deg = rng.integers(1, 9, V).astype(np.uint32)
    alias = ne.ne_build_neg_alias(deg, 0, torch.empty((V, 2), dtype=torch.int32, device=DEV))
    thr, al, _ = oracle.build_alias(deg)
    pairs = rng.integers(0, V, (B, 2)).astype(np.int32)
    loss = torch.zeros((), dtype=torch.float64, device=DEV)
    neg_dev = torch.empty((B, max(K, 1)), dtype=torch.int32, device=DEV)
    ne.ne_eval_loss(t, alias, torch.from_numpy(pairs).to(DEV), K, 7, loss, neg_dev)
    neg = oracle.sample_negatives(seed, 7, B, K, thr, al) if K else np.zeros((B, 0), np.int32)
    if K:
        assert np.array_equal(neg_dev.cpu().numpy(), neg)
    want = oracle.eval_loss(t.vertex.cpu().numpy(), t.context.cpu().numpy(), pairs, neg)
    assert abs(loss.item() - want) <= 1e-6 * want


@pytest.mark.parametrize("d", [64, 128, 256])
@pytest.mark.parametrize("B,N", [(1, 128), (33, 256), (1024, 384), (1025, 512), (2049, 640), (5000, 1152)])
def test_shared_passes(d, B, N):
    """Half a pass of 256 negatives, whole ones and both; one and several stages of the dC product.  Bars: a
    coefficient may flip by one bf16 step, 2^-8 of one of N >= 128 terms, hence 2e-4 of a table's largest delta, and
    a row's own rounding, 2^-24 of values up to 2."""
    print(f"shared d={d} B={B} N={N}", flush=True)
    V, seed, lr = 20_000, 31, 0.05
    scale = 5.0 / N
    rng = np.random.default_rng(B + N)
    gen = torch.Generator(device=DEV)
    gen.manual_seed(seed)
    X = torch.empty((V, d), dtype=torch.float32, device=DEV).normal_(0, 0.2, generator=gen)
    C = torch.empty((V, d), dtype=torch.float32, device=DEV).normal_(0, 0.2, generator=gen)
    X0, C0 = X.clone(), C.clone()
    t = ne.ne_create_tables(X, C, seed, init=False)
    alias = ne.ne_build_neg_alias(np.ones(V, np.uint32), 0, torch.empty((V, 2), dtype=torch.int32, device=DEV))
    ws = torch.full((ne.ne_shared_workspace_bytes(d, B, N),), 0xA5, dtype=torch.uint8, device=DEV)
    neg = torch.empty(N, dtype=torch.int32, device=DEV)
    p = torch.from_numpy(rng.integers(0, V, (B, 2)).astype(np.int32)).to(DEV)
    ne.ne_train_batch_shared(t, alias, p, N, lr, scale, 3, ws, neg)
    src, ctx, ng = p[:, 0].long(), p[:, 1].long(), neg.long()
    x, c = X0[src].double(), C0[ctx].double()
    g0 = lr * (1 - torch.sigmoid((x * c).sum(1, keepdim=True)))
    xq, cq = X0[src].bfloat16().double(), C0[ng].bfloat16().double()
    G = (-scale * torch.sigmoid(xq @ cq.t().contiguous())).float().bfloat16().double()
    dX = torch.zeros((V, d), dtype=torch.float64, device=DEV).index_add_(0, src, g0 * c + lr * (G @ cq))
    dC = torch.zeros((V, d), dtype=torch.float64, device=DEV).index_add_(0, ctx, g0 * x)
    dC.index_add_(0, ng, lr * (G.t().contiguous() @ xq))
    for got, old, want in ((X, X0, dX), (C, C0, dC)):
        err = (got.double() - old.double() - want).abs().max().item()
        top = want.abs().max().item()
        print(f"  delta error {err:.2e} of {top:.2e}", flush=True)
        assert err <= 2e-4 * top + 2 ** -23
        idle = want.abs().sum(1) == 0
        assert torch.equal(got[idle], old[idle])


@pytest.mark.parametrize("n_walks", [3, 80])
@pytest.mark.parametrize("d,L", [(16, 9), (64, 5), (128, 3)])      # 8, 4 and 2 groups to a position, or fewer by K; by entries
@pytest.mark.parametrize("window,K", [(1, 0), (5, 0), (3, 1), (1, 6), (3, 4), (4, 3), (1, 16), (4, 7), (3, 10), (2, 40)])
def test_walk_rows_shared_out(n_walks, d, L, window, K):
    """Positions whose rows several lane groups share: fewer rows than groups, shares that are no multiple of the rows in
    flight, shares that begin inside a pair, holes and ends of walks.  Bar as above."""
    print(f"walks n={n_walks} d={d} window={window} K={K}", flush=True)
    V, seed = 4000, 9
    rng = np.random.default_rng(n_walks + window + K)
    deg = rng.integers(1, 9, V).astype(np.uint32)
    walks = rng.integers(0, V, (n_walks, L)).astype(np.int32)
    walks[0, L - 2:] = -1
    walks[1, L // 2] = -1
    R = 1 + window * (K + 1)
    t = make(V, d, -(-(n_walks * L * R) // (K + 2)), K, seed)
    alias = ne.ne_build_neg_alias(deg, 0, torch.empty((V, 2), dtype=torch.int32, device=DEV))
    thr, al, _ = oracle.build_alias(deg)
    X, C = t.vertex.cpu().numpy(), t.context.cpu().numpy()
    ne.ne_train_walks(t, alias, torch.from_numpy(walks).to(DEV), n_walks, window, K, [0.02], 40)
    torch.cuda.synchronize()
    oracle_run(X, C, walks, n_walks, window, K, [0.02], seed, 40, thr, al)
    ex, ec = rowwise_rel_err(t.vertex.cpu().numpy(), X), rowwise_rel_err(t.context.cpu().numpy(), C)
    print(f"  row error X {ex:.2e} C {ec:.2e}", flush=True)
    assert ex <= 1e-5 and ec <= 1e-5
