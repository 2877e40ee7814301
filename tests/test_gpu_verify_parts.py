"""Bounded verification of lists whose workgroups take several pairs for each lane,
of reads that the sift can look through and others. Against the oracle's dynamic
program, on a sample of the pairs."""

from __future__ import annotations

import numpy as np
import pytest

import synth
from gpu_util import dev
from paper_1708_04329_amd import grim
from test_gpu_verify import run_verify

pytestmark = pytest.mark.gpu


def listed(cand):
    co = np.zeros(len(cand) + 1, np.int64)
    co[1:] = np.cumsum([len(c) for c in cand])
    return co, np.concatenate([np.array(c, np.int32) for c in cand])


@pytest.mark.parametrize("n_pairs", [8192 * 256 + 1, 3 * 8192 * 256 + 513])
def test_several_pairs_per_lane(oracle, n_pairs):
    """More than 256 pairs per workgroup, sifted and not, short reads and bins."""
    rng = np.random.default_rng(n_pairs)
    B, O, q, G, n = 64, 64, 5, 40_007, 3_000
    ref = np.frombuffer(b"ACGT", np.uint8)[rng.integers(0, 4, G)]
    nb = -(-G // B)
    starts = rng.integers(0, G - 60, n)
    lens = rng.choice([20, 27, 33, 60], n)
    seqs = [ref[p:p + m].tobytes() for p, m in zip(starts, lens)]
    budget = rng.choice([0, 1, 4], n).astype(np.uint16)  # pieces of 13 bases and more, and shorter ones
    rd = synth.reads_from_strings(seqs)
    co = (np.arange(n + 1, dtype=np.int64) * n_pairs) // n
    cb = rng.integers(0, nb, n_pairs).astype(np.int32)
    cb[co[:-1]] = starts // B
    idx = grim.grim_build_index(dev(ref), B, O, q, grim.LAYOUT_REF)
    got_d, got_m = run_verify(idx, rd, co, cb, bounded=True, max_edits=budget)
    assert (got_m[co[:-1]] == 1).all() and (got_d[co[:-1]] == 0).all()
    some = np.sort(rng.choice(n, 60, replace=False))
    sub = rd.subset(some)
    sco, scb = listed([cb[co[r]:co[r + 1]] for r in some])
    want_d, want_m = oracle.verify_bounded(ref, B, O, q, sub.bases, sub.offsets, sco, scb, max_edits=budget[some])
    keep = np.concatenate([np.arange(co[r], co[r + 1]) for r in some])
    assert np.array_equal(got_d[keep], want_d) and np.array_equal(got_m[keep], want_m)
