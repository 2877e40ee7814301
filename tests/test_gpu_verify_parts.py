"""Bounded verification of long bins: texts cut into up to 64 parts, more parts in a
workgroup than its table holds (texts are then taken as they are), and lists whose
workgroups take several pairs for each lane. Against the oracle's dynamic program,
on every pair or a sample of them."""

from __future__ import annotations

import random

import numpy as np
import pytest

import synth
from gpu_util import dev
from paper_1708_04329_amd import grim
from test_gpu_verify import run_verify
from test_gpu_verify_sift import edited

pytestmark = pytest.mark.gpu


def listed(cand):
    co = np.zeros(len(cand) + 1, np.int64)
    co[1:] = np.cumsum([len(c) for c in cand])
    return co, np.concatenate([np.array(c, np.int32) for c in cand])


@pytest.mark.parametrize("B,step,n_reads", [(4_000, 700, 12), (9_000, 1_500, 60), (20_000, 3_000, 60)])
def test_texts_of_many_parts(oracle, B, step, n_reads):
    """Copies of one unit all along the reference, reads of it: every bin is left by
    the sift and its pieces lie from end to end (9 and 20 kbp: 48 and 64 parts, so
    256 pairs make three and four times the 4096 parts of a workgroup's table)."""
    rng = random.Random(B)
    G, O, q = 12 * B + 77, 300, 5
    unit = rng.choices(b"ACGT", k=300)
    ref = bytearray(rng.choices(b"ACGT", k=G))
    for p in range(0, G - 300, step):
        ref[p:p + 300] = bytes(unit)
        ref[p + rng.randrange(300)] = rng.choice(b"ACGT")
    nb = -(-G // B)
    seqs, budget, cand = [], [], []
    for i in range(n_reads):
        L = rng.choice([30, 100, 190, 193, 250])
        E = rng.choice([0, 1, L // 30, L // 20])
        s = edited(rng, bytes(unit[7:7 + L]), E, rng.randrange(E + 1))
        seqs.append(s + b"ACGTA"[:max(0, 5 - len(s))])
        budget.append(E)
        cand.append(list(range(nb)))
    ref = np.frombuffer(bytes(ref), np.uint8).copy()
    rd = synth.reads_from_strings(seqs)
    co, cb = listed(cand)
    budget = np.array(budget, np.uint16)
    idx = grim.grim_build_index(dev(ref), B, O, q, grim.LAYOUT_REF)
    got_d, got_m = run_verify(idx, rd, co, cb, bounded=True, max_edits=budget)
    want_d, want_m = oracle.verify_bounded(ref, B, O, q, rd.bases, rd.offsets, co, cb, max_edits=budget)
    assert np.array_equal(got_d, want_d) and np.array_equal(got_m, want_m)
    assert want_m.any()


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
