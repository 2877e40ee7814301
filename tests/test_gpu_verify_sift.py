"""Bounded verification where the search for unedited pieces decides: budgets
around the shortest piece it uses (13 bases), the most pieces (16) and the
steps of its comparison counts; edits placed one in each piece but one, so that
a single piece (at every place and text phase) is left; reads at the ends of
their bins and of the reference; N in reads and reference; lists from one pair
to several workgroups. Bit-exact against the oracle's dynamic program."""

from __future__ import annotations

import random

import numpy as np
import pytest

import synth
from gpu_util import dev
from paper_1708_04329_amd import grim
from test_gpu_verify import run_verify

pytestmark = pytest.mark.gpu


def other(rng, b):
    return rng.choice([c for c in b"ACGT" if c != b])


def edited(rng, s: bytes, E: int, keep: int) -> bytes:
    """One edit inside every one of the E + 1 pieces of s but piece `keep` (a length-keeping
    pair of edits now and then, so that the pieces after it shift)."""
    n = len(s) // (E + 1)
    b = bytearray(s)
    for i in reversed(range(E + 1)):
        if i == keep:
            continue
        p = i * n + rng.randrange(n)
        op = rng.random()
        if op < 0.7:
            b[p] = other(rng, b[p])
        elif op < 0.85:
            b.insert(p, rng.choice(b"ACGT"))
        else:
            del b[p]
    return bytes(b)


@pytest.mark.parametrize("L,E", [(13, 0), (12, 0), (16, 0), (26, 1), (25, 1), (64, 3), (66, 4), (100, 5), (100, 6),
                                 (104, 7), (103, 7), (150, 8), (160, 10), (250, 13), (208, 15), (256, 15), (512, 15),
                                 (512, 16), (250, 18), (300, 11)])
def test_one_piece_left(oracle, L, E):
    rng = random.Random(31 * L + E)
    G, B, O, q = 9_003, 700, L + E, 5
    ref = bytearray(rng.choices(b"ACGT", k=G))
    ref[4000:4040] = b"N" * 40
    seqs, cand = [], []
    nb = -(-G // B)
    for i in range(96):
        # anywhere, at a bin's first base, at the last base a bin covers, at the reference's end
        p = [rng.randrange(0, G - L), B * rng.randrange(0, nb - 2), G - L, max(0, 3970 - L + rng.randrange(60))][i % 4]
        s = bytearray(edited(rng, bytes(ref[p:p + L]), E, rng.randrange(E + 1)))
        if i % 8 == 5 and len(s) > 4:
            s[rng.randrange(len(s))] = ord("N")
        s = bytes(s)[:512]
        s = s + b"A" * max(0, 6 - len(s))
        seqs.append(s.lower() if i % 16 == 3 else s)
        x = p // B
        cand.append(sorted({x, max(0, x - 1), min(nb - 1, x + 1), rng.randrange(nb), nb - 1}))
    ref = np.frombuffer(bytes(ref), np.uint8).copy()
    rd = synth.reads_from_strings(seqs)
    co = np.zeros(rd.n + 1, np.int64)
    co[1:] = np.cumsum([len(c) for c in cand])
    cb = np.concatenate([np.array(c, np.int32) for c in cand])
    idx = grim.grim_build_index(dev(ref), B, O, q, grim.LAYOUT_REF)
    budget = np.full(rd.n, E, np.uint16)
    got_d, got_m = run_verify(idx, rd, co, cb, bounded=True, max_edits=budget)
    want_d, want_m = oracle.verify_bounded(ref, B, O, q, rd.bases, rd.offsets, co, cb, max_edits=budget)
    bad = np.nonzero(got_d != want_d)[0]
    assert len(bad) == 0, [(int(k), int(got_d[k]), int(want_d[k])) for k in bad[:8]]
    assert np.array_equal(got_m, want_m)
    assert want_m.any() and not want_m.all()


@pytest.mark.parametrize("n", [1, 3, 63, 65, 700])
def test_list_sizes(oracle, n):
    """Mixed lengths and budgets (some past the pieces' limits), masks, several list chunks."""
    rng = random.Random(n)
    G, B, O, q = 30_011, 100, 300, 5
    ref = bytearray(rng.choices(b"ACGT", k=G))
    seqs, cand, budget = [], [], []
    nb = -(-G // B)
    for i in range(n):
        L = rng.choice([20, 100, 150, 250, 300])
        E = rng.choice([0, L // 50, L // 20, L // 8])
        p = rng.randrange(0, G - L)
        seqs.append(edited(rng, bytes(ref[p:p + L]), E, rng.randrange(E + 1)) + b"ACGTA")
        budget.append(E + 5)
        cand.append(sorted({p // B, *(rng.randrange(nb) for _ in range(rng.choice([0, 2, 9, 70, 400])))}))
    ref = np.frombuffer(bytes(ref), np.uint8).copy()
    rd = synth.reads_from_strings(seqs)
    co = np.zeros(rd.n + 1, np.int64)
    co[1:] = np.cumsum([len(c) for c in cand])
    cb = np.concatenate([np.array(c, np.int32) for c in cand])
    budget = np.array(budget, np.uint16)
    idx = grim.grim_build_index(dev(ref), B, O, q, grim.LAYOUT_REF)
    mask = (np.random.default_rng(n).random(len(cb)) < 0.6).astype(np.uint8)
    sparse = np.where(np.random.default_rng(n + 1).random(len(cb)) < 0.04, 128, 0).astype(np.uint8)
    sparse[-1] = 2  # the last pair of a list, whatever its place among 16
    for m in (None, mask, sparse):
        for bounded in (True, False):
            got_d, got_m = run_verify(idx, rd, co, cb, mask=m, bounded=bounded, max_edits=budget)
            fn = oracle.verify_bounded if bounded else oracle.verify
            want_d, want_m = fn(ref, B, O, q, rd.bases, rd.offsets, co, cb, verify_mask=m, max_edits=budget)
            assert np.array_equal(got_d, want_d) and np.array_equal(got_m, want_m)
