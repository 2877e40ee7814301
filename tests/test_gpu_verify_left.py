"""Bounded verification with reads of one to sixteen 32-base words in one call:
all classes, classes left out at either end, single ones; more listed pairs per
class than a workgroup takes; texts around found pieces that are cut into parts.
Bit-exact against the oracle's dynamic program."""

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


@pytest.mark.parametrize("words", [range(1, 17), range(1, 9), range(9, 17), [8, 9], [1], [16], [2, 5, 12]])
def test_classes_in_one_call(oracle, words):
    rng = random.Random(sum(words))
    G, B, O, q = 20_011, 900, 600, 5
    unit = rng.choices(b"ACGT", k=700)
    ref = bytearray(rng.choices(b"ACGT", k=G))
    for p in range(0, G - 700, 1400):  # copies of one text: pieces found far apart in a bin
        ref[p:p + 700] = bytes(unit)
    nb = -(-G // B)
    seqs, cand, budget = [], [], []
    for w in words:
        for i in range(26):
            L = 32 * w - rng.choice([0, 0, 1, 31 if w > 1 else 20])
            E = rng.choice([0, 1, L // 30, L // 20])
            p = rng.randrange(0, G - L)
            s = edited(rng, bytes(ref[p:p + L]), E, rng.randrange(E + 1))[:32 * w]
            seqs.append(s + b"ACGTA"[:max(0, 5 - len(s))])
            budget.append(E)
            cand.append(sorted({p // B, *(rng.randrange(nb) for _ in range(24))}))
    ref = np.frombuffer(bytes(ref), np.uint8).copy()
    rd = synth.reads_from_strings(seqs)
    co = np.zeros(rd.n + 1, np.int64)
    co[1:] = np.cumsum([len(c) for c in cand])
    cb = np.concatenate([np.array(c, np.int32) for c in cand])
    budget = np.array(budget, np.uint16)
    idx = grim.grim_build_index(dev(ref), B, O, q, grim.LAYOUT_REF)
    got_d, got_m = run_verify(idx, rd, co, cb, bounded=True, max_edits=budget)
    want_d, want_m = oracle.verify_bounded(ref, B, O, q, rd.bases, rd.offsets, co, cb, max_edits=budget)
    assert np.array_equal(got_d, want_d) and np.array_equal(got_m, want_m)
    assert want_m.any() and not want_m.all()
