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


# A chosen number of references of some tiles in one bin.  (tests/test_lds_layout.py has the compiler check these batches' bins and tiles.)
#   2100 pairs     64 bins, tiles of 128 pairs with 4 references per bin on average: segments of up to 32 entries are listed, beyond that searched
#   60 000 pairs  256 bins, tiles of 512 pairs with 4 per bin: up to 18 references of a tile in a bin have an entry each, beyond that
#                 equal rows are looked for; `rows` of them, the others' equals
@pytest.mark.parametrize("B,bits,tile_pairs,tiles,together,rows",
                         [(2100, 6, 128, (0, 3, 15), n, n) for n in (17, 31, 32, 33, 60)]
                         + [(60_000, 8, 512, (0, 50, 116), n, m) for n, m in ((18, 18), (19, 19), (18, 9), (19, 10), (33, 33))])
def test_entries_of_a_tile_in_one_bin(B, bits, tile_pairs, tiles, together, rows):
    print(f"B={B} together={together} rows={rows}", flush=True)
    V, d, seed, bin = 1_000_000, 4, 22, 5
    rng = np.random.default_rng(together)
    ids = np.arange(V, dtype=np.uint64)

    def bin_of(keys):
        return ((keys * 0x9E3779B1) & 0xFFFFFFFF) >> (32 - bits)

    # sources, and contexts, whose key has the top bit, of other bins; then the chosen sources
    sources, contexts = ids[bin_of(ids) != bin], ids[bin_of(ids | 0x80000000) != bin]
    same = rng.permutation(ids[bin_of(ids) == bin])
    pairs = np.stack([rng.choice(sources, B), rng.choice(contexts, B)], axis=1)
    for k, tile in enumerate(tiles):
        named = np.resize(same[k * rows:(k + 1) * rows], together)
        pairs[tile * tile_pairs + rng.permutation(tile_pairs)[:together], 0] = named
    in_bin = (bin_of(pairs[:, 0]) == bin).astype(int) + (bin_of(pairs[:, 1] | 0x80000000) == bin)
    for tile in range(-(-B // tile_pairs)):
        assert in_bin[tile * tile_pairs:(tile + 1) * tile_pairs].sum() == (together if tile in tiles else 0)
    t = make(V, d, B, 0, seed)
    step_and_check(t, None, None, None, pairs.astype(np.int32), 0, seed, 1)
