"""Rows that many references of a batch name take one rounding at their own size per batch, however small the deltas.

The deltas are chosen so small that eight of them together are below half of a hub element's last place: a sum
that went to the table row eight references at a time would lose all of them."""
import numpy as np
import pytest
import torch

import paper_2005_13789_amd as ne
from test_gpu_walks import make

pytestmark = pytest.mark.gpu
DEV = "cuda:0"
TIMES = [1, 2, 7, 8, 9, 15, 16, 17, 64, 65, 72, 73, 513, 2400, 8000]


@pytest.mark.parametrize("d", [4, 64, 128, 256, 512, 1024])
def test_small_deltas_of_hub_rows_are_not_lost(d):
    """Source row i and context row i are named TIMES[i] times each, against rows that only they name.

    Bar per element, against the same sums in 64 bits: half a last place of the row for the one addition (2^-25, the
    elements lie between 0.5 and 1), (n / 32 + 40) 2^-24 of the summed deltas for the sums before it, and 8 2^-24 of
    them for the coefficient (a dot product of terms below 2^-20, a sigmoid)."""
    print(f"hub rows, d={d}", flush=True)
    H, n = len(TIMES), sum(TIMES)
    V, seed, lr = H + n, 6, 0.01
    gen = torch.Generator().manual_seed(d)
    t = make(V, d, 2 * n, 0, seed)
    # hubs: elements of 0.5 .. 1; the rows they meet: 2e-7 .. 4e-7, so deltas of 1e-9 .. 2e-9
    for table in (t.vertex, t.context):
        table[:H] = (0.5 + 0.49 * torch.rand((H, d), generator=gen)).to(DEV)
        table[H:] = (2e-7 * (1 + torch.rand((n, d), generator=gen))).to(DEV)
    hub = np.repeat(np.arange(H), TIMES)
    other = H + np.arange(n)
    pairs = np.concatenate([np.stack([hub, other], 1), np.stack([other, hub], 1)])
    pairs = np.random.default_rng(d).permutation(pairs).astype(np.int32)
    p = torch.from_numpy(pairs).long()
    times = torch.tensor(TIMES, dtype=torch.float64)[:, None]
    for rep in range(3):       # the later batches find what the first one left behind
        X0, C0 = t.vertex.cpu().double(), t.context.cpu().double()
        x, c = X0[p[:, 0]], C0[p[:, 1]]
        g = float(np.float32(lr)) * (1.0 - torch.sigmoid((x * c).sum(1, keepdim=True)))
        dX = torch.zeros_like(X0).index_add_(0, p[:, 0], g * c)[:H]
        dC = torch.zeros_like(C0).index_add_(0, p[:, 1], g * x)[:H]
        assert float(dX[-1].min()) > 4e-6       # the hottest row's whole update is many last places
        ne.ne_train_batch(t, None, torch.from_numpy(pairs).to(DEV), 0, lr, 0)
        torch.cuda.synchronize()
        for name, got, old, want in (("X", t.vertex, X0, dX), ("C", t.context, C0, dC)):
            err = ((got[:H].cpu().double() - old[:H]) - want).abs()
            bar = 2.0 ** -25 * 1.0001 + (times / 32 + 48) * 2.0 ** -24 * want
            worst = (err / bar).max(dim=1).values
            print(f"  batch {rep} {name}: error / bar by times named: " + " ".join(f"{k}:{w:.2f}" for k, w in zip(TIMES, worst.tolist())), flush=True)
            assert (err <= bar).all()
