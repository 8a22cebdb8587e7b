"""Work items of the shared rows: who writes them (a lane up to 64 references of a row, a wavefront beyond), how the bins'
items are moved together (bins per workgroup), and the entries of a tile in one bin (up to 32 are listed, beyond that searched for).
Every row is checked against the oracle.

Bar: as in test_gpu_row_detection, rows of up to some hundred references."""
import numpy as np
import pytest

from test_gpu_row_detection import step_and_check
from test_gpu_walks import make

pytestmark = pytest.mark.gpu


# two references per pair: 512 bins (4 per workgroup) from 131 073 pairs on, 1024 (8) from 262 145, 2048 from 524 289;
# 32 rows of each multiplicity, the rest of the batch random pairs among many rows
@pytest.mark.parametrize("B", [128, 3000, 131_073, 262_145, 524_289])
def test_multiplicities_and_bins(B):
    print(f"B={B}", flush=True)
    V, d, seed = 500_000, 4, 21
    rng = np.random.default_rng(B)
    times = np.repeat([1, 2, 3, 7, 8, 9, 16, 17, 63, 64, 65, 72, 73, 130], 32 if B > 100_000 else 1)
    rows = rng.permutation(V)[:times.size]
    pairs = rng.integers(0, V, (B, 2))
    for side in range(2):
        named = np.repeat(rng.permutation(rows), times)[:B]
        pairs[rng.permutation(B)[:named.size], side] = named
    t = make(V, d, B, 0, seed)
    step_and_check(t, None, None, None, pairs.astype(np.int32), 0, seed, 1)


# 4096 references: 64 bins, tiles of 256 references with 4 per bin on average and up to 18 before equal rows are looked for
@pytest.mark.parametrize("together", [17, 18, 19, 31, 32, 33, 60])
def test_entries_of_a_tile_in_one_bin(together):
    print(f"together={together}", flush=True)
    V, d, seed = 1_000_000, 4, 22
    rng = np.random.default_rng(together)
    ids = np.arange(V, dtype=np.uint64)
    same = ids[((ids * 0x9E3779B1) & 0xFFFFFFFF) >> 26 == 5]
    pairs = rng.integers(0, V, (2048, 2))
    for tile in (0, 3, 15):          # 128 pairs each
        pairs[tile * 128:tile * 128 + together, 0] = same[tile * 60:tile * 60 + together]
    t = make(V, d, 2048, 0, seed)
    step_and_check(t, None, None, None, pairs.astype(np.int32), 0, seed, 1)
