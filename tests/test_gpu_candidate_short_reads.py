"""Candidate checks around 64 tokens, up to which every lane takes one token of a
read: counts and pass flags against the oracle."""

from __future__ import annotations

import random

import numpy as np
import pytest

import synth
from gpu_util import dev, empty, host
from paper_1708_04329_amd import grim

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("q,layout", [(1, 0), (4, 0), (5, 0), (5, 1), (5, 2), (6, 1), (7, 1), (8, 0)])
def test_around_a_token_per_lane(oracle, monkeypatch, q, layout):
    import torch
    monkeypatch.setenv("GRIM_CAND_COOP", str(layout))
    rng = random.Random(q)
    B, O, nb = 64, 200, 30
    ref = np.frombuffer(bytes(rng.choices(b"ACGTN", weights=[5, 3, 3, 5, .1], k=B * nb - 5)), np.uint8).copy()
    seqs = []
    for L in (q, q + 1, q + 2, q + 3, q + 62, q + 63, q + 64, q + 65):
        for kind in range(4):
            p = rng.randrange(0, len(ref) - L)
            s = bytearray(ref[p:p + L].tobytes())
            if kind == 1:
                s[rng.randrange(L)] = ord("n")
            if kind == 2:
                s = bytearray(b"A" * L)
            seqs.append(bytes(s))
    rng.shuffle(seqs)
    rd = synth.reads_from_strings(seqs)
    co = np.arange(rd.n + 1, dtype=np.int64) * 7
    cb = np.concatenate([np.array(sorted(rng.sample(range(nb), 7)), np.int32) for _ in range(rd.n)])
    budget = np.array([rng.choice([0, 1, 3]) for _ in range(rd.n)], np.uint16)
    idx = grim.grim_build_index(dev(ref), B, O, q, grim.LAYOUT_BM)
    want_c, want_p = oracle.scan_candidates(oracle.bits(ref, B, O, q), q, rd.bases, rd.offsets, co, cb, max_edits=budget)
    cnt, pas = empty((len(cb),), torch.uint16), empty((len(cb),), torch.uint8)
    reads = grim.ReadSet(dev(rd.bases), dev(rd.offsets), max_edits=dev(budget), allow_short_overlap=True)
    grim.grim_filter_candidates(idx, reads, dev(co), dev(cb), cnt, pas)
    assert np.array_equal(host(cnt.view(torch.int16)).view(np.uint16), want_c)
    assert np.array_equal(host(pas), want_p)
