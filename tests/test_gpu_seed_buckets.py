"""Candidate selection by buckets of bins: hits per read at the edges of each
launch shape, few bins and many, caps that cut among equal votes, buckets that
overflow (a satellite repeat), reads of more seeds than a workgroup's lists hold.
Bit-exact against the oracle."""

from __future__ import annotations

import numpy as np
import pytest

import synth
from gpu_util import dev
from paper_1708_04329_amd import grim
from test_gpu_seeds import gpu_candidates

pytestmark = pytest.mark.gpu
BASES = np.frombuffer(b"ACGT", np.uint8)


def check(oracle, ref, seqs, k, B, caps):
    rd = synth.reads_from_strings(seqs)
    seeds = grim.grim_seeds_build(dev(ref), k)
    for cap in caps:
        co, cb = gpu_candidates(seeds, rd, B, cap)
        want_o, want_b = oracle.seed_candidates(ref, rd.bases, rd.offsets, k, B, cap)
        assert np.array_equal(co, want_o) and np.array_equal(cb, want_b), (B, cap)


@pytest.mark.parametrize("hits", [1, 63, 64, 65, 767, 768, 769, 1536, 1537, 3072, 3073, 6144, 6145, 12288, 12289, 24575,
                                  24576, 24577])
def test_hits_per_read(oracle, hits):
    """A 12-base seed planted `hits` times at random places of its own 12-base grid cells."""
    rng = np.random.default_rng(hits)
    k, G = 12, 24 * 24_600
    ref = BASES[rng.integers(0, 2, G)]  # A and C only: the planted seed's G and T occur nowhere else
    seed = np.frombuffer(b"GTTGACGTTGCA", np.uint8)
    for cell in rng.choice(G // 24, hits, replace=False):
        ref[24 * cell + 5:24 * cell + 17] = seed
    seqs = [seed.tobytes(), b"TTTTTTTTTTTT" + seed.tobytes()]
    for B in (3, 50, 2048):
        check(oracle, ref, seqs, k, B, (1, 300, 30_000))


@pytest.mark.parametrize("n_seeds", [1, 20, 64, 65, 256, 257])
def test_seeds_and_crowded_buckets(oracle, n_seeds):
    """Repeats in one stretch of a long reference: most hits share a few buckets."""
    rng = np.random.default_rng(n_seeds)
    k, G = 6, 200_003
    ref = BASES[rng.integers(0, 4, G)]
    unit = BASES[rng.integers(0, 4, k * n_seeds)]
    for copy in range(1 + 6000 // len(unit)):
        ref[50_000 + copy * len(unit):50_000 + (copy + 1) * len(unit)] = unit
    seqs = [unit.tobytes(), BASES[rng.integers(0, 4, k * n_seeds)].tobytes(), unit[:k].tobytes() * min(n_seeds, 30)]
    for B in (1, 7, 300):
        check(oracle, ref, seqs, k, B, (5, 40, 100_000))


@pytest.mark.parametrize("env", [{}, {"GRIM_SEED_CLASS_MIN": "3"}, {"GRIM_SEED_CLASS_MIN": "6"}, {"GRIM_SEED_CLASS_MIN": "7"}])
def test_shapes_agree(oracle, monkeypatch, env):
    for name, value in env.items():
        monkeypatch.setenv(name, value)
    rng = np.random.default_rng(9)
    ref = BASES[rng.integers(0, 4, 60_000)]
    starts = rng.integers(0, len(ref) - 150, 90)
    seqs = [ref[p:p + int(n)].tobytes() for p, n in zip(starts, rng.integers(3, 150, 90))]
    for B in (1, 64, 999):
        check(oracle, ref, seqs, 5, B, (3, 64, 5000))


@pytest.mark.parametrize("hits,cap", [(24_577, 8), (24_577, 20_000), (70_000, 1), (70_000, 100), (70_000, 60_000)])
def test_more_hits_than_fit(oracle, hits, cap):
    """Reads whose hits are first counted by cell: thresholds above and below what the cells leave."""
    rng = np.random.default_rng(hits + cap)
    k, cells = 5, 80_000
    ref = BASES[rng.integers(0, 2, 12 * cells)]
    a, b = b"GTTGG", b"TGGTT"
    for n, cell in enumerate(rng.choice(cells, hits, replace=False)):  # one hit, two or three per 12 bases
        ref[12 * cell:12 * cell + 5] = np.frombuffer(a, np.uint8)
        if n % 5 == 0:
            ref[12 * cell + 5:12 * cell + 10] = np.frombuffer(b, np.uint8)
    seqs = [a, a + b, a + b + a + b, b, a * 30]
    for B in (12, 40, 6000):
        check(oracle, ref, seqs, k, B, (cap,))
