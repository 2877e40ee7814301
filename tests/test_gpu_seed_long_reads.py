"""Seed candidates of reads with more seeds than a workgroup's lists hold (taken in
turn by every launch shape), and of reads of many hits a bin, which the hash tables
take at once, by their size. Bit-exact against the oracle."""

from __future__ import annotations

import numpy as np
import pytest

from test_gpu_seed_buckets import BASES, check

pytestmark = pytest.mark.gpu


def reads_of(ref, rng, k, counts):
    """A read per number of seeds, from the reference with a few substitutions and N."""
    seqs = []
    for n in counts:
        p = int(rng.integers(0, len(ref) - k * n - k))
        s = ref[p:p + k * n + int(rng.integers(0, k))].copy()
        s[rng.integers(0, len(s), max(1, len(s) // 200))] = BASES[rng.integers(0, 4, max(1, len(s) // 200))]
        if n > 40:
            s[rng.integers(0, len(s), 2)] = ord("N")
        seqs.append(s.tobytes())
    return seqs


@pytest.mark.parametrize("k,G", [(12, 100_003), (8, 400_001), (7, 400_001), (6, 200_003)])
def test_more_seeds_than_the_lists_hold(oracle, k, G):
    """From a hit a seed (64 and 128 threads) to about fifty (cells, in several rounds)."""
    rng = np.random.default_rng(k)
    ref = BASES[rng.integers(0, 4, G)]
    seqs = reads_of(ref, rng, k, [1, 63, 64, 65, 127, 128, 129, 255, 256, 257, 300, 511, 513, 700, 1000, 2049])
    for B in (7, 300, 2048):
        check(oracle, ref, seqs, k, B, (5, 400, 60_000))


@pytest.mark.parametrize("cell_read", [300, 900])
def test_cells_of_many_seeds(oracle, cell_read):
    """More than 24576 hits in more bins than the largest table holds, 256 seeds at a time."""
    rng = np.random.default_rng(cell_read)
    ref = BASES[rng.integers(0, 4, 400_003)]
    seqs = reads_of(ref, rng, 5, [cell_read, 255, 256, 257])
    for B in (1, 12):
        check(oracle, ref, seqs, 5, B, (3, 2000, 30_000))


@pytest.mark.parametrize("hits", [767, 1536, 1537, 6144, 6145, 12288, 12289, 40000])
@pytest.mark.parametrize("vote_bits", [None, "2"])
def test_few_bins(oracle, monkeypatch, hits, vote_bits):
    """One to thirty bins: runs of hits in one bin are put into the table together (votes
    beyond a narrow vote field go to the fallback)."""
    if vote_bits:
        monkeypatch.setenv("GRIM_SEED_VOTE_BITS", vote_bits)
    rng = np.random.default_rng(hits)
    k, G = 12, 24 * 40_100
    ref = BASES[rng.integers(0, 2, G)]
    seed = np.frombuffer(b"GTTGACGTTGCA", np.uint8)
    for cell in rng.choice(G // 24, hits, replace=False):
        ref[24 * cell + 5:24 * cell + 17] = seed
    seqs = [seed.tobytes(), b"TTTTTTTTTTTT" + seed.tobytes() * 2]
    for B in (G, G // 6, G // 29):
        check(oracle, ref, seqs, k, B, (1, 4, 60))
