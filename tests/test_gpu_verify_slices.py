"""The sift of bounded verification in several launches (a launch holds fewer than
2^32 threads, one per listed pair): slices that end inside and between the
workgroups' pairs give the oracle's distances."""

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


@pytest.mark.parametrize("most", [1, 63, 256, 257, 100000])
def test_slices_agree(oracle, monkeypatch, most):
    monkeypatch.setenv("GRIM_VERIFY_SLICE", str(most))
    rng = random.Random(most)
    G, B, O, q = 9_011, 300, 300, 5
    ref = bytearray(rng.choices(b"ACGT", k=G))
    seqs, cand, budget = [], [], []
    nb = -(-G // B)
    for i in range(40):
        L = rng.choice([30, 100, 250])
        E = rng.choice([0, L // 50, L // 20, L // 8])
        p = rng.randrange(0, G - L)
        seqs.append(edited(rng, bytes(ref[p:p + L]), E, rng.randrange(E + 1)) + b"ACGTA")
        budget.append(E + 5)
        cand.append(sorted({p // B, *(rng.randrange(nb) for _ in range(12))}))
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
